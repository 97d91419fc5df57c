// Index arithmetic of the global reductions (diagnostics, projection), apart
// from their kernels: no device code and no HIP types, and constexpr, so that a
// host compiler can evaluate it at the largest lattices that lbm_create takes
// (an overflow is an error in a constant expression).  Lattices have nx, ny >= 1
// and pitch * ny < 2^31 with pitch >= nx a multiple of 64.
#pragma once

#include <stdint.h>

namespace lbm {

// k mod n in [0, n).  The remainder is corrected where it is negative: (k % n +
// n) % n passes 2^31 for n above 2^30.
constexpr int32_t wrap_mode(int32_t k, int32_t n)
{
    const int32_t r = k % n;
    return r < 0 ? r + n : r;
}

// (m v) mod n for a mode 0 <= m < n and a coordinate -1 <= v < n.  Up to 65535
// the product fits 32 unsigned bits (not 31: 65534 * 65534), and the remainder
// costs a 32-bit division instead of a 64-bit one.
constexpr uint32_t phase_index(int32_t m, int32_t v, int32_t n)
{
    const uint32_t w = (uint32_t)(v < 0 ? v + n : v);
    if (n <= 0xffff) return (uint32_t)m * w % (uint32_t)n;
    return (uint32_t)((uint64_t)m * w % (uint32_t)n);
}

// Cells of the lattice that a block of a reduction takes: block b has the
// columns [cols (b mod bx), ...) and every by-th band of h rows, h = threads >>
// shift, from band b / bx on.  Its threads lie in rows of 2^shift (at least the
// lattice's width where that is less than the block's), so that a thread
// keeps its column.  Neighbouring bands go to neighbouring blocks, so that the
// device sweeps through memory as one front: with a stretch of rows of its own
// for each block, 4096^2 FP32 diagnostics took 166 us instead of 110.
struct RedShape {
    int32_t bx, by, cols, shift;
    constexpr int blocks() const { return bx * by; }
};

// (In unsigned 32 bits, which hold nx and a stretch of columns beside it: 64-bit
// divisions cost a host-bound projection 0.1 us of 8.)
constexpr RedShape red_shape(int32_t nx, int32_t ny, int threads, int max_blocks)
{
    RedShape g{};
    while ((1 << g.shift) < threads && (1 << g.shift) < nx) ++g.shift;
    const uint32_t w = 1u << g.shift, h = (uint32_t)threads >> g.shift, most = (uint32_t)max_blocks;
    const uint32_t tx = ((uint32_t)nx + w - 1) >> g.shift;
    const uint32_t cols = w * ((tx + most - 1) / most), bx = ((uint32_t)nx + cols - 1) / cols;
    // at least two cells per thread
    const uint32_t want = ((uint32_t)ny + 2 * h - 1) / (2 * h), by = most / bx < want ? most / bx : want;
    g.cols = (int32_t)cols;
    g.bx = (int32_t)bx;
    g.by = by > 1 ? (int32_t)by : 1;
    return g;
}

// Columns [from, to) of the blocks of column number bx: unsigned, since a
// thread's next column, up to 1023 beyond the last, can pass 2^31.
struct RedCols {
    uint32_t from, to;
};

constexpr RedCols red_cols(const RedShape &g, int bx, int32_t nx)
{
    const uint32_t from = (uint32_t)bx * (uint32_t)g.cols, to = from + (uint32_t)g.cols;
    return {from, to < (uint32_t)nx ? to : (uint32_t)nx};
}

}  // namespace lbm

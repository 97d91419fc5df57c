// Kernels of the D2Q9 MRT lattice Boltzmann library (gfx950, wave64): one
// step per launch, the pool's one-step kernel, initialisation, readback,
// reductions, and the launch dispatch (the several-steps kernels live in
// lbm_step_common.hpp and are instantiated in lbm_multi_<type>.hip).
//
// Layout.  Structure of arrays: population i of row y at x lives at
// buf[i * plane + y * pitch + x], pitch = nx rounded up to 64 elements, two
// buffers (ping-pong).  The stored field is the post-collision deviation of
// the previous step, not yet streamed:  P_i(y) = g*_i(y, t-1), so that the
// pre-collision deviation at time t is g_i(x, t) = P_i(x - v_i)
// (pull streaming, Sec. 2.2, Eq. l-mrt-lbs).  One step therefore reads the
// nine pulled values of a cell, collides them and writes the nine results
// to the same cell of the other buffer: every HBM access of the step is a
// row-contiguous, coalesced stream; only the x-shift of populations with
// v_x != 0 is misaligned by one element.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "lbm_reduce.hpp"
#include "lbm_step_common.hpp"

namespace lbm {

namespace {

// One cell per lane: nine direct (possibly misaligned) loads.
// FLAGS bit 0: non-temporal loads; bit 1: the nine loads of the lane's next
// row are issued before the current row is collided and stored.
template <typename S, typename C, int FLAGS>
__global__ void __launch_bounds__(1024) k_step_v1(StepArgs<C> a)
{
    using R = typename Store<S>::raw;
    using W = typename Store<S>::wide;
    constexpr bool NT = (FLAGS & 1) != 0;
    constexpr bool PIPE = (FLAGS & 2) != 0;
    constexpr uint32_t E = sizeof(R);
    int bid = blockIdx.x;
    if (a.xcd_remap) bid = remap_xcd(bid, a.nblocks);
    const int tile_x = bid % a.tiles_x, tile_y = bid / a.tiles_x;
    const int x = tile_x * blockDim.x + threadIdx.x;
    if (x >= a.nx) return;
    const uint32_t c0 = (uint32_t)x * E;
    const uint32_t cm = (uint32_t)((x == 0 ? a.nx : x) - 1) * E;
    const uint32_t cp = (uint32_t)((x + 1 == a.nx) ? 0 : x + 1) * E;
    const char *__restrict__ src = (const char *)a.src;
    char *__restrict__ dst = (char *)a.dst;
    const uint64_t pb = (uint64_t)a.plane * E;
    const uint32_t rb = (uint32_t)a.pitch * E;
    auto gather = [&](int y, W w[9]) {
        const int ym = (y == 0 ? a.ny : y) - 1;
        const int yp = (y + 1 == a.ny) ? 0 : y + 1;
        gather9<S, NT>(src, pb, (uint32_t)y * rb, (uint32_t)ym * rb, (uint32_t)yp * rb, c0, cm, cp, w);
    };
    int y = tile_y * a.tile_h + threadIdx.y;
    if (y >= a.ny) return;
    W w[9];
    gather(y, w);
    for (int rr = 0; rr < a.rows; ++rr) {
        const int yn = y + blockDim.y;
        const bool more = rr + 1 < a.rows && yn < a.ny;
        W nxt[9];
        if constexpr (PIPE) {
            if (more) gather(yn, nxt);
        }
        cell_update<S, C>(w, a.r, a.scale, a.inv_scale);
        store9<S>(dst, pb, (uint32_t)y * rb + c0, w);
        if (!more) return;
        if constexpr (PIPE) {
#pragma unroll
            for (int i = 0; i < 9; ++i) w[i] = nxt[i];
        } else {
            gather(yn, w);
        }
        y = yn;
    }
}

// Row strips: a workgroup owns whole rows and walks each one in chunks of
// blockDim.x cells.  The cache line that two neighbouring chunks of an
// x-shifted population share is then read twice by the same workgroup in
// quick succession (an L2 hit) instead of by two workgroups that may sit on
// different XCDs.  FLAGS as for k_step_v1 (bit 1 prefetches the next chunk).
template <typename S, typename C, int FLAGS>
__global__ void __launch_bounds__(1024) k_step_strip(StepArgs<C> a)
{
    using R = typename Store<S>::raw;
    using W = typename Store<S>::wide;
    constexpr bool NT = (FLAGS & 1) != 0;
    constexpr bool PIPE = (FLAGS & 2) != 0;
    constexpr uint32_t E = sizeof(R);
    int bid = blockIdx.x;
    if (a.xcd_remap) bid = remap_xcd(bid, a.nblocks);
    const char *__restrict__ src = (const char *)a.src;
    char *__restrict__ dst = (char *)a.dst;
    const uint64_t pb = (uint64_t)a.plane * E;
    const uint32_t rb = (uint32_t)a.pitch * E;
    const int y0 = bid * a.tile_h + threadIdx.y;
    for (int rr = 0; rr < a.rows; ++rr) {
        const int y = y0 + rr * blockDim.y;
        if (y >= a.ny) return;
        const int ym = (y == 0 ? a.ny : y) - 1;
        const int yp = (y + 1 == a.ny) ? 0 : y + 1;
        const uint32_t r0 = (uint32_t)y * rb, rm = (uint32_t)ym * rb, rp = (uint32_t)yp * rb;
        auto gather = [&](int x, W w[9]) {
            const uint32_t cm = (uint32_t)((x == 0 ? a.nx : x) - 1) * E;
            const uint32_t cp = (uint32_t)((x + 1 == a.nx) ? 0 : x + 1) * E;
            gather9<S, NT>(src, pb, r0, rm, rp, (uint32_t)x * E, cm, cp, w);
        };
        int x = threadIdx.x;
        if (x >= a.nx) continue;
        W w[9];
        gather(x, w);
        while (true) {
            const int xn = x + blockDim.x;
            const bool more = xn < a.nx;
            W nxt[9];
            if constexpr (PIPE) {
                if (more) gather(xn, nxt);
            }
            cell_update<S, C>(w, a.r, a.scale, a.inv_scale);
            store9<S>(dst, pb, r0 + (uint32_t)x * E, w);
            if (!more) break;
            if constexpr (PIPE) {
#pragma unroll
                for (int i = 0; i < 9; ++i) w[i] = nxt[i];
            } else {
                gather(xn, w);
            }
            x = xn;
        }
    }
}

// VX consecutive cells per lane: aligned vector loads; the one-element
// x-shift of populations with v_x = +-1 is taken from the neighbouring lane
// (cross-lane shuffle), and only the first / last lane of a wave loads its
// edge element directly.  Needs nx % VX == 0 and blockDim.x % 64 == 0.
template <typename S, typename C, int VX, int FLAGS>
__global__ void __launch_bounds__(1024) k_step_vec(StepArgs<C> a)
{
    constexpr bool NT = (FLAGS & 1) != 0;
    using R = typename Store<S>::raw;
    using W = typename Store<S>::wide;
    using V = typename VecOf<R, VX>::type;
    int bid = blockIdx.x;
    if (a.xcd_remap) bid = remap_xcd(bid, a.nblocks);
    const int tile_x = bid % a.tiles_x, tile_y = bid / a.tiles_x;
    const int lane = threadIdx.x & 63;
    const int xl = (tile_x * (int)blockDim.x + (int)threadIdx.x) * VX;
    if (xl - lane * VX >= a.nx) return;            // the whole wave is past the row end
    const bool active = xl < a.nx;
    const int x0 = active ? xl : 0;
    const int xleft = (x0 == 0 ? a.nx : x0) - 1;
    const int xright = (x0 + VX >= a.nx) ? 0 : x0 + VX;
    const bool edge_l = lane == 0;
    const bool edge_r = lane == 63 || xl + VX >= a.nx;
    const R *__restrict__ src = (const R *)a.src;
    R *__restrict__ dst = (R *)a.dst;
    const int64_t P = a.plane;
    int y = tile_y * a.tile_h + threadIdx.y;
    for (int rr = 0; rr < a.rows; ++rr, y += blockDim.y) {
        if (y >= a.ny) return;
        const int ym = (y == 0 ? a.ny : y) - 1;
        const int yp = (y + 1 == a.ny) ? 0 : y + 1;
        const int64_t rowoff[3] = {(int64_t)y * a.pitch, (int64_t)ym * a.pitch, (int64_t)yp * a.pitch};
        // source row of each population: 0 = own row, 1 = y-1 (v_y = +1), 2 = y+1 (v_y = -1)
        constexpr int ROW[9] = {0, 0, 1, 0, 2, 1, 1, 2, 2};
        W w[9][VX];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const R *row = src + i * P + rowoff[ROW[i]];
            V raw;
            if constexpr (NT) raw = __builtin_nontemporal_load((const V *)(row + x0));
            else raw = *(const V *)(row + x0);
            W vals[VX];
#pragma unroll
            for (int k = 0; k < VX; ++k) {
                if constexpr (VX == 1) vals[k] = Store<S>::widen(raw);
                else vals[k] = Store<S>::widen(raw[k]);
            }
            if (VX_[i] == 0) {
#pragma unroll
                for (int k = 0; k < VX; ++k) w[i][k] = vals[k];
            } else if (VX_[i] == 1) {                  // needs x0-1 .. x0+VX-2
                W left = __shfl_up(vals[VX - 1], 1, 64);
                if (edge_l) left = Store<S>::widen(row[xleft]);
                w[i][0] = left;
#pragma unroll
                for (int k = 1; k < VX; ++k) w[i][k] = vals[k - 1];
            } else {                                   // needs x0+1 .. x0+VX
                W right = __shfl_down(vals[0], 1, 64);
                if (edge_r) right = Store<S>::widen(row[xright]);
#pragma unroll
                for (int k = 0; k < VX - 1; ++k) w[i][k] = vals[k + 1];
                w[i][VX - 1] = right;
            }
        }
#pragma unroll
        for (int k = 0; k < VX; ++k) {
            W c[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) c[i] = w[i][k];
            cell_update<S, C>(c, a.r, a.scale, a.inv_scale);
#pragma unroll
            for (int i = 0; i < 9; ++i) w[i][k] = c[i];
        }
        if (active) {
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                V out;
#pragma unroll
                for (int k = 0; k < VX; ++k) {
                    if constexpr (VX == 1) out = Store<S>::narrow(w[i][k]);
                    else out[k] = Store<S>::narrow(w[i][k]);
                }
                __builtin_nontemporal_store(out, (V *)(dst + i * P + rowoff[0] + x0));
            }
        }
    }
}

// VX consecutive cells per lane from overlapping aligned vector loads: a
// population with v_x = +1 needs x0-1 .. x0+VX-2, taken from the aligned
// vectors at x0-VX and x0; one with v_x = -1 needs x0+1 .. x0+VX, from the
// vectors at x0 and x0+VX (both wrap periodically).  The neighbouring
// vectors are the adjacent lanes' own vectors, so the extra loads are
// served by the cache; there is no cross-lane exchange and no divergent
// edge load.  Needs nx % VX == 0.
template <typename S, typename C, int VX, int FLAGS>
__global__ void __launch_bounds__(1024) k_step_wide(StepArgs<C> a)
{
    constexpr bool NT = (FLAGS & 1) != 0;
    using R = typename Store<S>::raw;
    using W = typename Store<S>::wide;
    using V = typename VecOf<R, VX>::type;
    int bid = blockIdx.x;
    if (a.xcd_remap) bid = remap_xcd(bid, a.nblocks);
    const int tile_x = bid % a.tiles_x, tile_y = bid / a.tiles_x;
    const int x0 = (tile_x * (int)blockDim.x + (int)threadIdx.x) * VX;
    if (x0 >= a.nx) return;
    const int xl = (x0 == 0 ? a.nx : x0) - VX;           // previous vector (wrapped)
    const int xr = (x0 + VX == a.nx) ? 0 : x0 + VX;       // next vector (wrapped)
    const R *__restrict__ src = (const R *)a.src;
    R *__restrict__ dst = (R *)a.dst;
    const int64_t P = a.plane;
    auto vload = [&](const R *p) -> V {
        if constexpr (NT) return __builtin_nontemporal_load((const V *)p);
        else return *(const V *)p;
    };
    auto el = [](const V &v, int k) -> R {
        if constexpr (VX == 1) return v;
        else return v[k];
    };
    int y = tile_y * a.tile_h + threadIdx.y;
    for (int rr = 0; rr < a.rows; ++rr, y += blockDim.y) {
        if (y >= a.ny) return;
        const int ym = (y == 0 ? a.ny : y) - 1;
        const int yp = (y + 1 == a.ny) ? 0 : y + 1;
        const int64_t rowoff[3] = {(int64_t)y * a.pitch, (int64_t)ym * a.pitch, (int64_t)yp * a.pitch};
        constexpr int ROW[9] = {0, 0, 1, 0, 2, 1, 1, 2, 2};
        W w[9][VX];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const R *row = src + i * P + rowoff[ROW[i]];
            const V cur = vload(row + x0);
            if (VX_[i] == 0) {
#pragma unroll
                for (int k = 0; k < VX; ++k) w[i][k] = Store<S>::widen(el(cur, k));
            } else if (VX_[i] == 1) {
                const V prev = vload(row + xl);
                w[i][0] = Store<S>::widen(el(prev, VX - 1));
#pragma unroll
                for (int k = 1; k < VX; ++k) w[i][k] = Store<S>::widen(el(cur, k - 1));
            } else {
                const V next = vload(row + xr);
#pragma unroll
                for (int k = 0; k < VX - 1; ++k) w[i][k] = Store<S>::widen(el(cur, k + 1));
                w[i][VX - 1] = Store<S>::widen(el(next, 0));
            }
        }
#pragma unroll
        for (int k = 0; k < VX; ++k) {
            W c[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) c[i] = w[i][k];
            cell_update<S, C>(c, a.r, a.scale, a.inv_scale);
#pragma unroll
            for (int i = 0; i < 9; ++i) w[i][k] = c[i];
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            V out;
#pragma unroll
            for (int k = 0; k < VX; ++k) {
                if constexpr (VX == 1) out = Store<S>::narrow(w[i][k]);
                else out[k] = Store<S>::narrow(w[i][k]);
            }
            __builtin_nontemporal_store(out, (V *)(dst + i * P + rowoff[0] + x0));
        }
    }
}

// ---- batched step over a pool of lattices ----------------------------------------
//
// A one-step launch advances every active member of one storage class by
// one step, a T-step launch by T steps.  The grid is persistent (a fixed
// number of workgroups strides over the tile table), so the same launch
// serves any membership.  A one-step tile is a rectangle of one member
// (whole rows of a narrow lattice, a row segment of a wide one) whose cells
// are walked as a flattened (row, column) index so narrow lattices still
// fill whole waves; a T-step task is one strip segment of one member, taken
// by one wave.  Which launches of a recorded chunk a member takes, and hence
// which of its buffers is the source, follows from its remaining step count
// (chunk schedule in lbm_internal.hpp).  The per-cell work is the same
// gather9 / cell_update / store9 and strip_pass as the single-lattice
// kernels, so a lattice gives bit-identical results alone or in a pool.

template <typename S, typename C>
__global__ void __launch_bounds__(1024) k_pool_step(const PoolHeader *hdr, const PoolMember *mem,
                                                     const PoolTile *tiles, int range, int i, int kk, int T)
{
    using R = typename Store<S>::raw;
    using W = typename Store<S>::wide;
    const int begin = hdr->begin[range], end = hdr->end[range];
    for (int ti = begin + (int)blockIdx.x; ti < end; ti += (int)gridDim.x) {
        const PoolTile tile = tiles[ti];
        const PoolMember *m = mem + tile.member;
        const int64_t rem = m->t_target - m->t_done;
        const int64_t span = rem < kk ? rem : kk;
        const int64_t q = member_multi(rem, kk, T);
        if (i >= span - q * T) continue;                 // not one of its one-step launches
        const int par = (int)((m->cur0 + m->flips + q + i) & 1);
        const char *__restrict__ src = (const char *)m->buf[par];
        char *__restrict__ dst = (char *)m->buf[par ^ 1];
        const int nx = m->nx, ny = m->ny;
        constexpr uint32_t E = sizeof(R);
        const uint64_t pb = (uint64_t)m->plane * E;
        const uint32_t rb = (uint32_t)m->pitch * E;
        const Relax<C> r = member_relax<C>(m);
        const float scale = m->scale, inv_scale = m->inv_scale;
        const int ncols = tile.ncols;
        const int ncell = tile.nrows * ncols;
        for (int c = threadIdx.x; c < ncell; c += blockDim.x) {
            const int dy = c / ncols;
            const int x = tile.x0 + (c - dy * ncols);
            const int y = tile.y0 + dy;
            const uint32_t cm = (uint32_t)((x == 0 ? nx : x) - 1) * E;
            const uint32_t cp = (uint32_t)((x + 1 == nx) ? 0 : x + 1) * E;
            const int ym = (y == 0 ? ny : y) - 1;
            const int yp = (y + 1 == ny) ? 0 : y + 1;
            const uint32_t r0 = (uint32_t)y * rb;
            W w[9];
            gather9<S, false>(src, pb, r0, (uint32_t)ym * rb, (uint32_t)yp * rb, (uint32_t)x * E, cm, cp, w);
            cell_update<S, C>(w, r, scale, inv_scale);
            store9<S>(dst, pb, r0 + (uint32_t)x * E, w);
        }
    }
}

__global__ void k_pool_commit(PoolMember *mem, int nmem, int kk, int T)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nmem) return;
    const int64_t rem = mem[i].t_target - mem[i].t_done;
    if (rem > 0) {
        const int64_t span = rem < kk ? rem : (int64_t)kk;
        const int64_t q = member_multi(rem, kk, T);
        mem[i].t_done += span;
        mem[i].flips += q + span - q * T;
    }
}

// ---- block reductions (fixed order, deterministic) ---------------------------

// v plus the value that a DPP control moves into the lane (0 where none does).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v)
{
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, false);
    return v + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Sum over the wave, in lane 63: shifts within the rows of 16 lanes, then the
// rows' totals broadcast onward.  18 sums take 324 vector instructions, about
// 0.7 us; LDS shuffles (__shfl_xor) took 216 LDS instructions and 2 us.
__device__ __forceinline__ double wave_sum63(double v)
{
    v = dpp_add<0x111, 0xf>(v);                         // row_shr:1
    v = dpp_add<0x112, 0xf>(v);                         // row_shr:2
    v = dpp_add<0x114, 0xf>(v);                         // row_shr:4
    v = dpp_add<0x118, 0xf>(v);                         // row_shr:8
    v = dpp_add<0x142, 0xa>(v);                         // row_bcast:15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v);                      // row_bcast:31 into rows 2 and 3
}

// Block sums of N accumulators: red[k] for the whole block after the call.
template <int N, int BT>
__device__ __forceinline__ void block_sums(const double (&acc)[N], double (&red)[N])
{
    __shared__ double part[BT / 64][N];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const double v = wave_sum63(acc[k]);
        if (lane == 63) part[wave][k] = v;
    }
    __syncthreads();
    if ((int)threadIdx.x < N) {
        double s = 0.0;
        for (int wv = 0; wv < BT / 64; ++wv) s += part[wv][threadIdx.x];
        red[threadIdx.x] = s;
    }
    __syncthreads();
}

__device__ __forceinline__ void block_max_to(double v, double *out)
{
    __shared__ double red[16];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int nw = (blockDim.x + 63) >> 6;
        double s = 0.0;
        for (int wv = 0; wv < nw; ++wv) s = fmax(s, red[wv]);
        *out = s;
    }
}

// Sums `width` columns of nb partial rows in a fixed order: one wave per
// column (one block, 16 waves).  mode 0: sums into out; 1: maxima into out;
// 2: sums, then the projection's phases (project_finish).  The columns one
// after another in one block of 256 took 18.5 us for 18 of them.
struct Mode {
    int32_t mx, my, nx, ny;
    double inv_scale;
};

__device__ __forceinline__ void project_finish(const double *sums, const Mode &m, double *out);

__global__ void __launch_bounds__(1024) k_final(const double *partials, int nb, int width, int mode, Mode pm, double *out)
{
    __shared__ double red[32];
    const int lane = threadIdx.x & 63;
    for (int k = threadIdx.x >> 6; k < width; k += 16) {
        double s = 0.0;
        for (int j = lane; j < nb; j += 64) {
            const double v = partials[(size_t)j * width + k];
            s = mode == 1 ? fmax(s, v) : s + v;
        }
        if (mode == 1) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s = fmax(s, __shfl_xor(s, off, 64));
        } else {
            s = wave_sum63(s);
        }
        if (lane == 63) red[k] = s;
    }
    __syncthreads();
    if (mode == 2) project_finish(red, pm, out);
    else if ((int)threadIdx.x < width) out[threadIdx.x] = red[threadIdx.x];
}

// ---- initialisation, readback, diagnostics ------------------------------------

struct CellArgs {
    int32_t nx, ny, pitch;
    int32_t div_shift;        // cell / nx = cell * div_mul >> div_shift
    uint32_t div_mul;
    int64_t plane;
    double scale, inv_scale;
    Relax<double> r;
    double fbase[9];
};

CellArgs make_cell_args(const View &v)
{
    CellArgs c;
    c.nx = v.nx;
    c.ny = v.ny;
    c.pitch = v.pitch;
    // exact for cell numbers below 2^31, which nx * ny <= pitch * ny keeps to:
    // mul = ceil(2^(31 + l) / nx) < 2^32 with 2^l >= nx
    int l = 0;
    while (((int64_t)1 << l) < v.nx) ++l;
    c.div_shift = 31 + l;
    c.div_mul = (uint32_t)((((uint64_t)1 << c.div_shift) + v.nx - 1) / v.nx);
    c.plane = v.plane;
    c.scale = v.scale;
    c.inv_scale = v.inv_scale;
    c.r = make_relax<double>(v);
    for (int i = 0; i < 9; ++i) c.fbase[i] = v.fbase[i];
    return c;
}

// Row and column of cell c of the row-major fields.
__device__ __forceinline__ void cell_xy(const CellArgs &a, int64_t c, int &x, int &y)
{
    y = (int)((uint64_t)(uint32_t)c * a.div_mul >> a.div_shift);
    x = (int)c - y * a.nx;
}

__device__ __forceinline__ int wrap(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// x / B, correctly rounded, for B = 6 or 9: the rounded reciprocal is half a
// unit roundoff off, so x times it is within one unit in the last place of
// the quotient, and one residual step rounds correctly (Markstein, "Computation
// of elementary functions on the IBM RISC System/6000", 1990, theorem on
// division by fused multiply-add).  Infinities and NaN pass through.
template <int B>
__device__ __forceinline__ double div_by(double x)
{
    constexpr double r = 1.0 / B;
    const double q = x * r;
    const double c = fmad(fmad(-(double)B, q, x), r, q);
    return isfinite(q) ? c : q;
}

// back_transform of an equilibrium deviation, whose dm[5] = -dm[1] and dm[6] =
// -dm[2], with five divisions in place of eleven (the quotients by 18 and 36 are
// the one by 9 halved, which is exact, those by 12 the one by 6), each of them
// by its constant: the same values.  General divisions took as long as the
// memory traffic of the whole kernel (4096^2 FP32: 280 us with a 64-bit division
// for the cell's row, now 216; the pass that only measures 232, now 126).
__device__ __forceinline__ void back_transform_eq(const double dm[9], double f[9])
{
    const double r = div_by<9>(dm[0]);
    const double ex = div_by<6>(dm[1]), ey = div_by<6>(dm[2]);
    const double e9 = div_by<9>(dm[3]), s9 = div_by<9>(dm[4]);
    const double ea = -(0.25 * e9) - 0.5 * s9;
    const double ed = 0.5 * e9 + 0.25 * s9;
    const double qx = -ex, qy = -ey;
    const double qxd = 0.5 * qx, qyd = 0.5 * qy;
    const double pxx = 0.25 * dm[7], pxy = 0.25 * dm[8];
    f[0] = r - e9 + s9;
    f[1] = r + ex + ea - qx + pxx;
    f[2] = r + ey + ea - qy - pxx;
    f[3] = r - ex + ea + qx + pxx;
    f[4] = r - ey + ea + qy - pxx;
    f[5] = r + ex + ey + ed + qxd + qyd + pxy;
    f[6] = r - ex + ey + ed - qxd + qyd - pxy;
    f[7] = r - ex - ey + ed - qxd - qyd + pxy;
    f[8] = r + ex - ey + ed + qxd - qyd - pxy;
}

// g(x) = M^{-1} dmeq(rho - rho0, rho u - j0), FP64; stored at P_i(x - v_i).
template <typename S>
__global__ void __launch_bounds__(1024) k_init(CellArgs a, const double *rho, const double *ux,
                                              const double *uy, typename Store<S>::raw *dst,
                                              double *partials, int measure_only)
{
    using W = typename Store<S>::wide;
    const int64_t n = (int64_t)a.nx * a.ny;
    double mx = 0.0;
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
         c += (int64_t)gridDim.x * blockDim.x) {
        int x, y;
        cell_xy(a, c, x, y);
        const double r = rho[c];
        double dm[9], g[9];
        delta_meq<double>(r - a.r.rho0, r * ux[c] - a.r.j0x, r * uy[c] - a.r.j0y, a.r, dm);
        back_transform_eq(dm, g);
#pragma unroll
        for (int i = 0; i < 9; ++i) mx = fmax(mx, fabs(g[i]));
        if (!measure_only) {
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int xs = wrap(x - VX_[i], a.nx), ys = wrap(y - VY_[i], a.ny);
                dst[i * a.plane + (int64_t)ys * a.pitch + xs] = Store<S>::narrow((W)(g[i] * a.scale));
            }
        }
    }
    if (measure_only) block_max_to(mx, partials + blockIdx.x);
}

// rho, u of the pre-collision state, FP64.
template <typename S>
__global__ void __launch_bounds__(256) k_moments(CellArgs a, const typename Store<S>::raw *src,
                                                 double *rho, double *ux, double *uy)
{
    const int64_t n = (int64_t)a.nx * a.ny;
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
         c += (int64_t)gridDim.x * blockDim.x) {
        int x, y;
        cell_xy(a, c, x, y);
        double r = 0.0, jx = 0.0, jy = 0.0;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int xs = wrap(x - VX_[i], a.nx), ys = wrap(y - VY_[i], a.ny);
            const double g = (double)Store<S>::widen(src[i * a.plane + (int64_t)ys * a.pitch + xs]) * a.inv_scale;
            r += g;
            jx += VX_[i] * g;
            jy += VY_[i] * g;
        }
        const double rr = a.r.rho0 + r;
        rho[c] = rr;
        ux[c] = (a.r.j0x + jx) / rr;
        uy[c] = (a.r.j0y + jy) / rr;
    }
}

template <typename S>
__global__ void __launch_bounds__(256) k_read_pop(CellArgs a, const typename Store<S>::raw *src, double *f)
{
    const int64_t n = (int64_t)a.nx * a.ny;
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
         c += (int64_t)gridDim.x * blockDim.x) {
        int x, y;
        cell_xy(a, c, x, y);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int xs = wrap(x - VX_[i], a.nx), ys = wrap(y - VY_[i], a.ny);
            const double g = (double)Store<S>::widen(src[i * a.plane + (int64_t)ys * a.pitch + xs]) * a.inv_scale;
            f[i * n + c] = a.fbase[i] + g;
        }
    }
}

template <typename S>
__global__ void __launch_bounds__(256) k_write_pop(CellArgs a, const double *f, typename Store<S>::raw *dst)
{
    using W = typename Store<S>::wide;
    const int64_t n = (int64_t)a.nx * a.ny;
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n;
         c += (int64_t)gridDim.x * blockDim.x) {
        int x, y;
        cell_xy(a, c, x, y);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int xs = wrap(x - VX_[i], a.nx), ys = wrap(y - VY_[i], a.ny);
            dst[i * a.plane + (int64_t)ys * a.pitch + xs] = Store<S>::narrow((W)((f[i * n + c] - a.fbase[i]) * a.scale));
        }
    }
}

// Threads per block of a reduction: 1024 where 512 blocks of 256 would leave
// a thread more than eight cells.
bool red_wide(const View &v) { return (int64_t)v.nx * v.ny > (int64_t)kRedBlocks * 256 * 8; }

RedShape red_split(const View &v, bool wide) { return red_shape(v.nx, v.ny, wide ? 1024 : 256, kRedBlocks); }

// Global sums of the collision invariants (aligned reads: a global sum does
// not need the pull shift) and the count of non-finite stored values.
template <typename S, int BT>
__global__ void __launch_bounds__(BT) k_diag(CellArgs a, RedShape g, const typename Store<S>::raw *src, double *partials)
{
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    __shared__ double red[4];
    const int by = (int)blockIdx.x / g.bx, bx = (int)blockIdx.x - by * g.bx;
    const RedCols cols = red_cols(g, bx, a.nx);
    const uint32_t w = 1u << g.shift;
    const int h = BT >> g.shift;
    for (uint32_t x = cols.from + (threadIdx.x & (w - 1)); x < cols.to; x += w)
#pragma unroll 2
        for (int y = by * h + ((int)threadIdx.x >> g.shift); y < a.ny; y += g.by * h) {
            const typename Store<S>::raw *p = src + ((int64_t)y * a.pitch + x);
            double r = 0.0, jx = 0.0, jy = 0.0;
            int bad = 0;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const double v = (double)Store<S>::widen(p[i * a.plane]);
                bad += !isfinite(v);
                r += v;
                jx += VX_[i] * v;
                jy += VY_[i] * v;
            }
            acc[0] += r;
            acc[1] += jx;
            acc[2] += jy;
            acc[3] += bad;
        }
    block_sums<4, BT>(acc, red);
    if (threadIdx.x < 4) partials[(size_t)blockIdx.x * 4 + threadIdx.x] = red[threadIdx.x];
}

// e^{-2 pi i m v / n} as (cos, sin) of the exact phase fraction ((m v) mod n) / n,
// 0 <= m < n, -1 <= v < n.
__device__ __forceinline__ void phase(int m, int v, int n, double *cs, double *sn)
{
    const double p = (double)phase_index(m, v, n);
    sincospi(2.0 * (p / n), sn, cs);
}

// out = sums * inv_scale * e^{-i k.v_i} (the pull shift), 9 complex values.
__device__ __forceinline__ void project_finish(const double *sums, const Mode &m, double *out)
{
    const int i = threadIdx.x;
    if (i >= 9) return;
    double cx, sx, cy, sy;
    phase(m.mx, VX_[i], m.nx, &cx, &sx);
    phase(m.my, VY_[i], m.ny, &cy, &sy);
    const double cs = cx * cy - sx * sy, sn = sx * cy + cx * sy;
    const double re = sums[2 * i] * m.inv_scale, im = sums[2 * i + 1] * m.inv_scale;
    out[2 * i] = re * cs + im * sn;          // (re + i im)(cs - i sn)
    out[2 * i + 1] = im * cs - re * sn;
}

// sum_y P_i(y) e^{-i k.y}; the pull shift e^{-i k.v_i} is applied afterwards
// (project_finish).  The phase separates into a column's and a row's factor:
// a thread keeps its column's, the rows' are made once per block (256 at a
// time) and read from LDS, so a cell costs four multiply-adds for its phase
// instead of two 64-bit divisions and a sincospi.  With the final sums by one
// wave per column and the phases of the shift in the same launch, a small
// lattice's projection takes 7.4 us (two launches' latency) instead of 30, and
// 4096^2 FP32 117 us (5.2 TB/s) instead of 229.
template <typename S, int BT>
__global__ void __launch_bounds__(BT) k_project(CellArgs a, RedShape g, const typename Store<S>::raw *src, Mode m,
                                                double *partials, double *out)
{
    double acc[18];
#pragma unroll
    for (int k = 0; k < 18; ++k) acc[k] = 0.0;
    __shared__ double ec[256], es[256], red[18];
    const int by = (int)blockIdx.x / g.bx, bx = (int)blockIdx.x - by * g.bx;
    const RedCols cols = red_cols(g, bx, a.nx);
    const uint32_t w = 1u << g.shift;
    const int hs = __ffs(BT >> g.shift) - 1, h = 1 << hs;
    // the block's rows by their order in it
    const int first = by << hs, band = g.by << hs;
    const int bands = first < a.ny ? (a.ny - first + band - 1) / band : 0;
    for (int q0 = 0; q0 < bands << hs; q0 += 256) {
        const int n = min(256, (bands << hs) - q0);
        const auto row = [&](int q) { return first + ((q0 + q) >> hs) * band + ((q0 + q) & (h - 1)); };
        if ((int)threadIdx.x < n) phase(m.my, min(row((int)threadIdx.x), a.ny - 1), a.ny, &ec[threadIdx.x], &es[threadIdx.x]);
        __syncthreads();
        for (uint32_t x = cols.from + (threadIdx.x & (w - 1)); x < cols.to; x += w) {
            double cx, sx;
            phase(m.mx, (int)x, a.nx, &cx, &sx);
#pragma unroll 2
            for (int q = (int)threadIdx.x >> g.shift; q < n; q += h) {
                const int y = row(q);
                if (y >= a.ny) break;
                const typename Store<S>::raw *p = src + ((int64_t)y * a.pitch + x);
                const double cy = ec[q], sy = es[q];
                const double cs = cx * cy - sx * sy, sn = sx * cy + cx * sy;
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const double v = (double)Store<S>::widen(p[i * a.plane]);
                    acc[2 * i] = fmad(v, cs, acc[2 * i]);
                    acc[2 * i + 1] = fmad(-v, sn, acc[2 * i + 1]);
                }
            }
        }
        __syncthreads();
    }
    block_sums<18, BT>(acc, red);
    if (gridDim.x == 1) project_finish(red, m, out);
    else if (threadIdx.x < 18) partials[(size_t)blockIdx.x * 18 + threadIdx.x] = red[threadIdx.x];
}

int grid_for(int64_t n, int block, int cap)
{
    int64_t b = (n + block - 1) / block;
    if (b > cap) b = cap;
    if (b < 1) b = 1;
    return (int)b;
}

template <template <typename> class F, typename... Args>
hipError_t dispatch_storage(int storage, Args &&...args)
{
    switch (storage) {
    case LBM_STORE_F64: return F<double>::run(args...);
    case LBM_STORE_F32: return F<float>::run(args...);
    case LBM_STORE_F16: return F<f16_tag>::run(args...);
    case LBM_STORE_BF16: return F<bf16_tag>::run(args...);
    default: return hipErrorInvalidValue;
    }
}

template <typename S, typename C>
hipError_t launch_step_typed(const View &v, const void *src, void *dst, const lbm_launch &cfg, hipStream_t st)
{
    StepArgs<C> a;
    a.src = src;
    a.dst = dst;
    a.nx = v.nx;
    a.ny = v.ny;
    a.pitch = v.pitch;
    const int vx = cfg.variant <= 3 ? 1 << cfg.variant : (cfg.variant >= 5 ? 1 << (cfg.variant - 4) : 1);
    const int tile_w = cfg.block_x * vx;
    a.tiles_x = cfg.variant == 4 ? 1 : (v.nx + tile_w - 1) / tile_w;
    a.tile_h = cfg.block_y * cfg.rows;
    a.rows = cfg.rows;
    const int tiles_y = (v.ny + a.tile_h - 1) / a.tile_h;
    a.nblocks = a.tiles_x * tiles_y;
    a.xcd_remap = cfg.xcd_remap;
    a.plane = v.plane;
    a.r = make_relax<C>(v);
    a.scale = (float)v.scale;
    a.inv_scale = (float)v.inv_scale;
    a.nwaves = 0;
    a.out_cols = 0;
    if (cfg.variant >= 8) {
        // strips of multi_strip_cols output columns, segments of `rows` rows,
        // one wave each (with the shared halo: one workgroup of block_y
        // waves each, strips as wide as its lanes allow)
        const int T = cfg.variant - 6;
        const bool wg = (cfg.flags & kWgHalo) != 0;
        a.out_cols = multi_strip_cols(T, (int)sizeof(typename Store<S>::raw), wg ? 64 * cfg.block_y : 64);
        a.tiles_x = (v.nx + a.out_cols - 1) / a.out_cols;
        a.tile_h = cfg.rows;
        const int segs = (v.ny + cfg.rows - 1) / cfg.rows;
        a.nwaves = a.tiles_x * segs;
        a.nblocks = wg ? a.nwaves : (a.nwaves + cfg.block_y - 1) / cfg.block_y;
    }
    const dim3 grid(a.nblocks), block(cfg.block_x, cfg.block_y);
    if (cfg.variant >= 8) return launch_multi<S, C>(a, grid, block, cfg.variant - 6, cfg.flags, st);
    const bool nt = cfg.flags & 1, pipe = cfg.flags & 2;
    switch (cfg.variant * 4 + (pipe ? 2 : 0) + (nt ? 1 : 0)) {
    case 0: hipLaunchKernelGGL((k_step_v1<S, C, 0>), grid, block, 0, st, a); break;
    case 1: hipLaunchKernelGGL((k_step_v1<S, C, 1>), grid, block, 0, st, a); break;
    case 2: hipLaunchKernelGGL((k_step_v1<S, C, 2>), grid, block, 0, st, a); break;
    case 3: hipLaunchKernelGGL((k_step_v1<S, C, 3>), grid, block, 0, st, a); break;
    case 4: hipLaunchKernelGGL((k_step_vec<S, C, 2, 0>), grid, block, 0, st, a); break;
    case 5: hipLaunchKernelGGL((k_step_vec<S, C, 2, 1>), grid, block, 0, st, a); break;
    case 8: hipLaunchKernelGGL((k_step_vec<S, C, 4, 0>), grid, block, 0, st, a); break;
    case 9: hipLaunchKernelGGL((k_step_vec<S, C, 4, 1>), grid, block, 0, st, a); break;
    case 12: hipLaunchKernelGGL((k_step_vec<S, C, 8, 0>), grid, block, 0, st, a); break;
    case 13: hipLaunchKernelGGL((k_step_vec<S, C, 8, 1>), grid, block, 0, st, a); break;
    case 16: hipLaunchKernelGGL((k_step_strip<S, C, 0>), grid, block, 0, st, a); break;
    case 17: hipLaunchKernelGGL((k_step_strip<S, C, 1>), grid, block, 0, st, a); break;
    case 18: hipLaunchKernelGGL((k_step_strip<S, C, 2>), grid, block, 0, st, a); break;
    case 19: hipLaunchKernelGGL((k_step_strip<S, C, 3>), grid, block, 0, st, a); break;
    case 20: hipLaunchKernelGGL((k_step_wide<S, C, 2, 0>), grid, block, 0, st, a); break;
    case 21: hipLaunchKernelGGL((k_step_wide<S, C, 2, 1>), grid, block, 0, st, a); break;
    case 24: hipLaunchKernelGGL((k_step_wide<S, C, 4, 0>), grid, block, 0, st, a); break;
    case 25: hipLaunchKernelGGL((k_step_wide<S, C, 4, 1>), grid, block, 0, st, a); break;
    case 28: hipLaunchKernelGGL((k_step_wide<S, C, 8, 0>), grid, block, 0, st, a); break;
    case 29: hipLaunchKernelGGL((k_step_wide<S, C, 8, 1>), grid, block, 0, st, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <typename S>
struct InitF {
    static hipError_t run(const View &v, const double *rho, const double *ux, const double *uy, void *dst,
                          double *partials, double *result, bool measure, hipStream_t st)
    {
        const CellArgs a = make_cell_args(v);
        const int64_t n = (int64_t)v.nx * v.ny;
        const int g = measure ? kRedBlocks : grid_for(n, 256, 65536);
        hipLaunchKernelGGL(k_init<S>, dim3(g), dim3(measure && n > kRedBlocks * 256 ? 1024 : 256), 0, st, a, rho, ux, uy,
                           (typename Store<S>::raw *)dst, partials, (int)measure);
        if (measure) hipLaunchKernelGGL(k_final, dim3(1), dim3(1024), 0, st, partials, g, 1, 1, Mode{}, result);
        return hipGetLastError();
    }
};

template <typename S>
struct MomentsF {
    static hipError_t run(const View &v, const void *src, double *rho, double *ux, double *uy, hipStream_t st)
    {
        const CellArgs a = make_cell_args(v);
        const int g = grid_for((int64_t)v.nx * v.ny, 256, 65536);
        hipLaunchKernelGGL(k_moments<S>, dim3(g), dim3(256), 0, st, a,
                           (const typename Store<S>::raw *)src, rho, ux, uy);
        return hipGetLastError();
    }
};

template <typename S>
struct ReadPopF {
    static hipError_t run(const View &v, const void *src, double *f, hipStream_t st)
    {
        const CellArgs a = make_cell_args(v);
        const int g = grid_for((int64_t)v.nx * v.ny, 256, 65536);
        hipLaunchKernelGGL(k_read_pop<S>, dim3(g), dim3(256), 0, st, a, (const typename Store<S>::raw *)src, f);
        return hipGetLastError();
    }
};

template <typename S>
struct WritePopF {
    static hipError_t run(const View &v, const double *f, void *dst, hipStream_t st)
    {
        const CellArgs a = make_cell_args(v);
        const int g = grid_for((int64_t)v.nx * v.ny, 256, 65536);
        hipLaunchKernelGGL(k_write_pop<S>, dim3(g), dim3(256), 0, st, a, f, (typename Store<S>::raw *)dst);
        return hipGetLastError();
    }
};

template <typename S>
struct DiagF {
    static hipError_t run(const View &v, const void *src, double *partials, double *result, hipStream_t st)
    {
        const CellArgs a = make_cell_args(v);
        const bool wide = red_wide(v);
        const RedShape g = red_split(v, wide);
        const typename Store<S>::raw *p = (const typename Store<S>::raw *)src;
        if (wide) hipLaunchKernelGGL((k_diag<S, 1024>), dim3(g.blocks()), dim3(1024), 0, st, a, g, p, partials);
        else hipLaunchKernelGGL((k_diag<S, 256>), dim3(g.blocks()), dim3(256), 0, st, a, g, p, partials);
        hipLaunchKernelGGL(k_final, dim3(1), dim3(1024), 0, st, partials, g.blocks(), 4, 0, Mode{}, result);
        return hipGetLastError();
    }
};

template <typename S>
struct ProjectF {
    static hipError_t run(const View &v, const void *src, int32_t mx, int32_t my, double *partials,
                          double *out, hipStream_t st)
    {
        const CellArgs a = make_cell_args(v);
        const typename Store<S>::raw *p = (const typename Store<S>::raw *)src;
        const Mode m{wrap_mode(mx, v.nx), wrap_mode(my, v.ny), v.nx, v.ny, v.inv_scale};
        const bool wide = red_wide(v);
        const RedShape g = red_split(v, wide);
        if (wide) hipLaunchKernelGGL((k_project<S, 1024>), dim3(g.blocks()), dim3(1024), 0, st, a, g, p, m, partials, out);
        else hipLaunchKernelGGL((k_project<S, 256>), dim3(g.blocks()), dim3(256), 0, st, a, g, p, m, partials, out);
        // a lattice of one block has its result already
        if (g.blocks() > 1)
            hipLaunchKernelGGL(k_final, dim3(1), dim3(1024), 0, st, partials, g.blocks(), 18, 2, m, out);
        return hipGetLastError();
    }
};

}  // namespace

size_t storage_bytes(int32_t storage)
{
    switch (storage) {
    case LBM_STORE_F64: return 8;
    case LBM_STORE_F32: return 4;
    case LBM_STORE_F16:
    case LBM_STORE_BF16: return 2;
    default: return 0;
    }
}

int steps_per_launch(const lbm_launch &cfg) { return cfg.variant >= 8 && cfg.variant <= 13 ? cfg.variant - 6 : 1; }

// Output columns of a strip: 64 - 2(T-1) lanes see all their neighbours for
// T stages.  The count is rounded down to a whole number of 32-byte (else
// 16-byte) pieces of a stored row when that costs at most two columns, so
// that neighbouring strips' row stores meet on sector boundaries (measured:
// 58 -> 56 columns at T = 4 is +17 % for FP32 and FP64 storage; larger cuts
// cost more lanes than they gain).
int multi_strip_cols(int T, int elem_bytes, int lanes)
{
    const int raw = lanes - 2 * (T - 1);
    for (int bytes : {32, 16}) {
        const int a = elem_bytes >= bytes ? 1 : bytes / elem_bytes;
        const int aligned = raw - raw % a;
        if (raw - aligned <= 2) return aligned;
    }
    return raw;
}

bool step_shape_supported(const View &v, const lbm_launch &cfg)
{
    if (cfg.variant >= 8 && cfg.variant <= 13) {
        // several steps per pass: one wave per strip and segment
        if (cfg.variant >= 11 && (cfg.flags & 1)) return false;   // T = 5, 6, 7: no non-temporal loads
        // T = 7 with one wave per strip: plain pipeline only
        if (cfg.variant == 13 && (cfg.flags & 16) && !(cfg.flags & kWgHalo)) return false;
        if (cfg.flags & kWgHalo) {
            // shared halo: T = 4 .. 7, flags 32, 34 or 40 (no shuffles,
            // loads one or two rows ahead or none), plain or skewed
            // pipeline (+16); FP64 storage only T = 6, 7, plain
            if (cfg.variant < 10) return false;
            const int f = cfg.flags & ~16;      // bit 4: the skewed pipeline, one exchange per row
            if (f != kWgHalo && f != (kWgHalo | 2) && f != (kWgHalo | 8)) return false;
            // FP64 storage: T = 6 and 7, plain pipeline
            if (v.storage == LBM_STORE_F64 && (cfg.variant < 12 || (cfg.flags & 16))) return false;
            return cfg.block_x == 64 && cfg.block_y >= 1 && cfg.block_y <= kWgMaxWaves && cfg.rows >= 1 &&
                   cfg.rows <= 4096 && (cfg.xcd_remap == 0 || cfg.xcd_remap == 1);
        }
        return cfg.block_x == 64 && cfg.block_y >= 1 && cfg.block_y <= 4 && cfg.rows >= 1 &&
               cfg.rows <= 4096 && (cfg.xcd_remap == 0 || cfg.xcd_remap == 1) && cfg.flags >= 0 &&
               cfg.flags <= 29 && !((cfg.flags & 8) && (cfg.flags & 2)) &&
               // skewed pipeline: T = 3 and 4, no non-temporal loads
               (!(cfg.flags & 16) || (cfg.variant >= 9 && !(cfg.flags & 1)));
    }
    if (cfg.variant < 0 || cfg.variant > 7) return false;
    if (cfg.block_x < 1 || cfg.block_y < 1 || cfg.rows < 1 || cfg.rows > 64) return false;
    if (cfg.block_x * cfg.block_y > 1024 || cfg.block_x * cfg.block_y < 64) return false;
    if (cfg.block_x % 64 != 0 && cfg.block_x * cfg.block_y % 64 != 0) return false;
    if (cfg.xcd_remap != 0 && cfg.xcd_remap != 1) return false;
    if (cfg.flags < 0 || cfg.flags > 3) return false;
    if ((cfg.flags & 2) && cfg.variant != 0 && cfg.variant != 4) return false;   // pipelining: one-cell kernels
    if (cfg.variant >= 1 && cfg.variant <= 3) {
        const int vx = 1 << cfg.variant;
        if (cfg.block_x % 64 != 0 || v.nx % vx != 0) return false;
    }
    if (cfg.variant >= 5 && v.nx % (1 << (cfg.variant - 4)) != 0) return false;
    return true;
}

hipError_t launch_step(const View &v, const void *src, void *dst, const lbm_launch &cfg, hipStream_t st)
{
    if (v.compute == LBM_COMPUTE_F64) {
        if (v.storage == LBM_STORE_F64) return launch_step_typed<double, double>(v, src, dst, cfg, st);
        return hipErrorInvalidValue;
    }
    switch (v.storage) {
    case LBM_STORE_F64: return launch_step_typed<double, float>(v, src, dst, cfg, st);
    case LBM_STORE_F32: return launch_step_typed<float, float>(v, src, dst, cfg, st);
    case LBM_STORE_F16: return launch_step_typed<f16_tag, float>(v, src, dst, cfg, st);
    case LBM_STORE_BF16: return launch_step_typed<bf16_tag, float>(v, src, dst, cfg, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_init(const View &v, const double *rho, const double *ux, const double *uy, void *dst,
                       double *partials, double *result, bool measure_only, hipStream_t st)
{
    return dispatch_storage<InitF>(v.storage, v, rho, ux, uy, dst, partials, result, measure_only, st);
}

hipError_t launch_moments(const View &v, const void *src, double *rho, double *ux, double *uy, hipStream_t st)
{
    return dispatch_storage<MomentsF>(v.storage, v, src, rho, ux, uy, st);
}

hipError_t launch_read_populations(const View &v, const void *src, double *f, hipStream_t st)
{
    return dispatch_storage<ReadPopF>(v.storage, v, src, f, st);
}

hipError_t launch_write_populations(const View &v, const double *f, void *dst, hipStream_t st)
{
    return dispatch_storage<WritePopF>(v.storage, v, f, dst, st);
}

hipError_t launch_diagnostics(const View &v, const void *src, double *partials, double *result, hipStream_t st)
{
    return dispatch_storage<DiagF>(v.storage, v, src, partials, result, st);
}

hipError_t launch_project(const View &v, const void *src, int32_t mx, int32_t my, double *partials, double *out,
                          hipStream_t st)
{
    return dispatch_storage<ProjectF>(v.storage, v, src, mx, my, partials, out, st);
}

Relax<float> relax_f32(const View &v) { return make_relax<float>(v); }
Relax<double> relax_f64(const View &v) { return make_relax<double>(v); }

void *pool_step_kernel(int cls)
{
    switch (cls) {
    case LBM_STORE_F64 * 2 + LBM_COMPUTE_F64: return reinterpret_cast<void *>(&k_pool_step<double, double>);
    case LBM_STORE_F64 * 2 + LBM_COMPUTE_F32: return reinterpret_cast<void *>(&k_pool_step<double, float>);
    case LBM_STORE_F32 * 2 + LBM_COMPUTE_F32: return reinterpret_cast<void *>(&k_pool_step<float, float>);
    case LBM_STORE_F16 * 2 + LBM_COMPUTE_F32: return reinterpret_cast<void *>(&k_pool_step<f16_tag, float>);
    case LBM_STORE_BF16 * 2 + LBM_COMPUTE_F32: return reinterpret_cast<void *>(&k_pool_step<bf16_tag, float>);
    default: return nullptr;
    }
}

void *pool_commit_kernel() { return reinterpret_cast<void *>(&k_pool_commit); }

void *pool_multi_kernel(int cls, int T, int flags)
{
    switch (cls) {
    case LBM_STORE_F64 * 2 + LBM_COMPUTE_F64: return pool_multi_fn<double, double>(T, flags);
    case LBM_STORE_F64 * 2 + LBM_COMPUTE_F32: return pool_multi_fn<double, float>(T, flags);
    case LBM_STORE_F32 * 2 + LBM_COMPUTE_F32: return pool_multi_fn<float, float>(T, flags);
    case LBM_STORE_F16 * 2 + LBM_COMPUTE_F32: return pool_multi_fn<f16_tag, float>(T, flags);
    case LBM_STORE_BF16 * 2 + LBM_COMPUTE_F32: return pool_multi_fn<bf16_tag, float>(T, flags);
    default: return nullptr;
    }
}

hipError_t launch_pool_step(int range, const PoolHeader *hdr, const PoolMember *mem, const PoolTile *tiles, int i,
                            int kk, int T, int grid, int block, hipStream_t st)
{
    void *f = pool_step_kernel(range / kChains);
    if (!f) return hipErrorInvalidValue;
    void *args[] = {(void *)&hdr, (void *)&mem, (void *)&tiles, (void *)&range, (void *)&i, (void *)&kk, (void *)&T};
    return hipLaunchKernel(f, dim3(grid), dim3(block), args, 0, st);
}

hipError_t launch_pool_multi(int range, int T, int flags, const PoolHeader *hdr, const PoolMember *mem,
                             const PoolTile *tiles, int j, int grid, int waves, hipStream_t st)
{
    void *f = pool_multi_kernel(range / kChains, T, flags);
    if (!f) return hipErrorInvalidValue;
    void *args[] = {(void *)&hdr, (void *)&mem, (void *)&tiles, (void *)&range, (void *)&j};
    return hipLaunchKernel(f, dim3(grid), dim3(64, waves), args, 0, st);
}

hipError_t launch_pool_commit(PoolMember *mem, int nmem, int kk, int T, hipStream_t st)
{
    hipLaunchKernelGGL(k_pool_commit, dim3((nmem + 255) / 256), dim3(256), 0, st, mem, nmem, kk, T);
    return hipGetLastError();
}

}  // namespace lbm

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

}  // namespace lbm

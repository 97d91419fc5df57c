// Several steps per launch on register tiles: the step kernel of small and
// medium lattices.
//
// A workgroup of W waves holds a tile of 64 columns by W R rows in registers
// (lane = column, wave = R consecutive rows), advances it T steps and writes
// the cells that T steps leave valid: the tile without T - 1 rows and columns
// on each side.  Populations move along x by DPP whole-wave shifts and along
// y by register renaming; only the rows at a wave's edge go through LDS (six
// values per lane and step, two buffers in turn, one barrier per step).  A
// wave skips the steps in which none of its rows is needed any more, so half
// of the halo rows' work is saved.
//
// Why tiles: below about 2^22 cells the strips of k_step_multi are too few to
// fill the device with segments tall enough to pay for their 2 (T-1) start-up
// rows, and one-step launches spend most of their 2-4 us on launch and memory
// latency.  A tile launch costs about 3.3 us plus 0.3 us per step until the
// vector ALUs fill; from there on it issues close to the ALU's rate, and what
// bounds it is the share of the tile that is halo: a 64 x 48 tile
// writes 52 x 36 cells after T = 7 steps.  Measured against what these sizes
// took before (us per step of step(n), a pulse on a field at rest;
// profiles/k_step_tile_shapes.csv): FP32 64^2 3.7 -> 0.70, 181 x 147 3.7 -> 0.79,
// 600 x 430 4.3 -> 1.5 (one-step launches), 1000 x 760 5.4 -> 3.0, 2048^2 14.5 ->
// 13.4 (strips); FP64 64^2 3.7 -> 0.89, 1500 x 1001 11.5 -> 9.5; BF16 600 x 430
// 3.9 -> 1.6.
#include <algorithm>
#include <cmath>
#include <vector>

#include "lbm_step_common.hpp"

namespace lbm {

namespace {

template <typename C>
struct TileArgs {
    const void *src;
    void *dst;
    int32_t nx, ny, pitch, tiles_x;
    int32_t out_cols, out_rows, nblocks, T;
    uint32_t inv_tiles_x;     // ceil(2^32 / tiles_x) where that divides exactly, else 0
    int64_t plane;
    Relax<C> r;
    float scale, inv_scale;
};

constexpr int kTileWaves = 16;    // most waves of a workgroup (a lane then has 128 registers)
constexpr int kTileCols = 64;     // columns of a tile: one per lane
constexpr int kTileXch = kTileCols + 2;   // columns of an exchange row

// Waves that a tile of t needs: fewer than its shape's where the lattice has
// fewer rows.
int tile_waves(const TileShape &t, int ny, int steps)
{
    const int need = std::min(t.rows * t.waves, ny + 2 * (steps - 1));
    return (need + t.rows - 1) / t.rows;
}

size_t tile_lds(int waves, size_t wide) { return (size_t)waves * 2 * 6 * kTileXch * wide; }

// v mod n for v in [-64, n + 64): no division unless n is small.
__device__ __forceinline__ int wrap_near(int v, int n)
{
    if (n < 64) return wrap_mod(v, n);
    return v < 0 ? v + n : (v >= n ? v - n : v);
}

// Value of the lane to the left / right; lane 0 / 63 of the wave gets zero
// (bound_ctrl: the result needs no copy of an old value, so the shift can
// write any register; those lanes' cells are not used).
template <int CTRL, typename V>
__device__ __forceinline__ V shift0(V v)
{
    if constexpr (sizeof(V) == 4) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
    } else {
        const uint64_t u = (uint64_t)__double_as_longlong(v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
        return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    }
}
template <typename V>
__device__ __forceinline__ V left(V v) { return shift0<kDppWaveShr1>(v); }
template <typename V>
__device__ __forceinline__ V right(V v) { return shift0<kDppWaveShl1>(v); }

// T steps of the tile whose `rows` x `cols` output cells start at (x0, y0), by
// the calling workgroup (every wave with the same arguments).
template <typename S, typename C, int R>
__device__ __forceinline__ void tile_pass(const void *src_, void *dst_, int nx, int ny, int pitch, int64_t plane,
                                          const Relax<C> &relax, float scale, float inv_scale, int T, int x0, int y0,
                                          int rows, int cols, char *lds)
{
    using Raw = typename Store<S>::raw;
    using W = typename Store<S>::wide;
    constexpr uint32_t E = sizeof(Raw);
    const int lane = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.y), nw = (int)blockDim.y;
    const int need = rows + 2 * (T - 1);                  // tile rows they depend on
    const int lo = wv * R;                                // first tile row of the wave
    const int xl = x0 + lane - (T - 1);
    const int c = wrap_near(xl, nx);
    const uint32_t c0 = (uint32_t)c * E;
    const uint32_t cm = (uint32_t)((c == 0 ? nx : c) - 1) * E;
    const uint32_t cp = (uint32_t)((c + 1 == nx) ? 0 : c + 1) * E;
    const uint32_t pb = (uint32_t)plane * E, rb = (uint32_t)pitch * E;
    const __amdgpu_buffer_rsrc_t src = whole_rsrc((const char *)src_), dst = whole_rsrc((const char *)dst_);
    W w[R][9];
    if (lo < need) {
        int y = y0 - (T - 1) + lo;
        y = ny < 64 ? __builtin_amdgcn_readfirstlane(wrap_mod(y, ny)) : y < 0 ? y + ny : y >= ny ? y - ny : y;
        int ym = (y == 0 ? ny : y) - 1;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int yp = (y + 1 == ny) ? 0 : y + 1;
            const uint32_t r0 = (uint32_t)y * rb, rm = (uint32_t)ym * rb, rp = (uint32_t)yp * rb;
            w[j][0] = ld_buf<S, false>(src, c0, r0);
            w[j][1] = ld_buf<S, false>(src, cm, 1 * pb + r0);
            w[j][2] = ld_buf<S, false>(src, c0, 2 * pb + rm);
            w[j][3] = ld_buf<S, false>(src, cp, 3 * pb + r0);
            w[j][4] = ld_buf<S, false>(src, c0, 4 * pb + rp);
            w[j][5] = ld_buf<S, false>(src, cm, 5 * pb + rm);
            w[j][6] = ld_buf<S, false>(src, cp, 6 * pb + rm);
            w[j][7] = ld_buf<S, false>(src, cp, 7 * pb + rp);
            w[j][8] = ld_buf<S, false>(src, cm, 8 * pb + rp);
            ym = y;
            y = yp;
        }
    }
    // rows that cross a wave's edge go through LDS: [wave][step parity][value
    // (populations 2, 5, 6 of the wave's last row, 4, 7, 8 of its first)]
    // [column + 1] (the pad makes the neighbouring columns constant offsets)
    W *const mine = (W *)lds + wv * (2 * 6 * kTileXch) + lane + 1;
    const W *const below = (W *)lds + (wv > 0 ? wv - 1 : 0) * (2 * 6 * kTileXch) + lane + 1;
    const W *const above = (W *)lds + (wv + 1 < nw ? wv + 1 : wv) * (2 * 6 * kTileXch) + lane + 1;
    // With more than two rows per lane, or two in 16-bit storage, a wave at
    // the tile's edge also skips the single rows that a step does not need, and
    // the branch around each row keeps the compiler from interleaving the
    // rows, whose conversions it otherwise holds in registers.  Us per step,
    // all rows of a live wave | this: BF16 600 x 430 1.79 | 1.63, FP16 400 x 300
    // 1.25 | 1.14, 1500 x 1400 7.81 | 7.24, FP32 1536 x 1024 5.50 | 5.37, FP64 600
    // x 430 2.50 | 2.44.  Otherwise, with one or two rows, the branches cost a
    // wave's chain more than they save (64^2 FP32 0.69 | 0.73).
    constexpr bool ROWWISE = R > 2 || (R == 2 && Store<S>::scaled);
    auto update = [&](int j) {
        cell_update<S, C>(w[j], relax, scale, inv_scale);
        round_trip9<S>(w[j]);
    };
    auto step = [&](int k, auto par) {
        constexpr int B = decltype(par)::value * 6 * kTileXch;
        // step k is needed on tile rows k .. need - 1 - k
        const bool live = lo + R > k && lo < need - k;    // wave-uniform
        if (live) {
            const int from = ROWWISE ? k - lo : 0, to = ROWWISE ? need - k - lo : R;
            if (from <= 0 && to > 0) update(0);
            if constexpr (R > 1)
                if (from < R && to >= R) update(R - 1);
            mine[B + 0 * kTileXch] = w[R - 1][2];
            mine[B + 1 * kTileXch] = w[R - 1][5];
            mine[B + 2 * kTileXch] = w[R - 1][6];
            mine[B + 3 * kTileXch] = w[0][4];
            mine[B + 4 * kTileXch] = w[0][7];
            mine[B + 5 * kTileXch] = w[0][8];
#pragma unroll
            for (int j = 1; j < R - 1; ++j)
                if (j >= from && j < to) update(j);
        }
        __syncthreads();
        if (live) {
            // new row j: populations 0, 1, 3 of old row j, 2, 5, 6 of old row
            // j - 1, 4, 7, 8 of old row j + 1, shifted along x
            W n2 = below[B], n5 = below[B + 1 * kTileXch - 1], n6 = below[B + 2 * kTileXch + 1];
            const W u4 = above[B + 3 * kTileXch], u7 = above[B + 4 * kTileXch + 1], u8 = above[B + 5 * kTileXch - 1];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const W k2 = w[j][2], k5 = w[j][5], k6 = w[j][6];
                w[j][1] = left(w[j][1]);
                w[j][3] = right(w[j][3]);
                w[j][2] = n2;
                w[j][5] = n5;
                w[j][6] = n6;
                if (j + 1 < R) {
                    w[j][4] = w[j + 1 < R ? j + 1 : j][4];
                    w[j][7] = right(w[j + 1 < R ? j + 1 : j][7]);
                    w[j][8] = left(w[j + 1 < R ? j + 1 : j][8]);
                    n2 = k2;
                    n5 = left(k5);
                    n6 = right(k6);
                } else {
                    w[j][4] = u4;
                    w[j][7] = u7;
                    w[j][8] = u8;
                }
            }
        }
    };
    int k = 0;
    for (; k + 2 < T; k += 2) {
        step(k, std::integral_constant<int, 0>{});
        step(k + 1, std::integral_constant<int, 1>{});
    }
    if (k + 1 < T) step(k, std::integral_constant<int, 0>{});
    if (lo + R <= T - 1 || lo >= T - 1 + rows) return;
    const bool col = lane >= T - 1 && lane < T - 1 + cols && xl < nx;
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int tr = lo + j - (T - 1);                  // row of the tile's output
        if (tr < 0 || tr >= rows) continue;               // wave-uniform
        cell_update<S, C>(w[j], relax, scale, inv_scale);
        const uint32_t ro = (uint32_t)(y0 + tr) * rb;
        if (col) {
#pragma unroll
            for (int i = 0; i < 9; ++i) st_buf<S>(dst, c0, (uint32_t)i * pb + ro, w[j][i]);
        }
    }
}

template <typename S, typename C, int R>
__global__ void __launch_bounds__(64 * kTileWaves) k_step_tile(TileArgs<C> a)
{
    extern __shared__ char lds[];
    const int bid = remap_xcd((int)blockIdx.x, a.nblocks);
    const int ty = a.inv_tiles_x ? (int)__umulhi((uint32_t)bid, a.inv_tiles_x) : bid / a.tiles_x;
    const int x0 = (bid - ty * a.tiles_x) * a.out_cols, y0 = ty * a.out_rows;
    tile_pass<S, C, R>(a.src, a.dst, a.nx, a.ny, a.pitch, a.plane, a.r, a.scale, a.inv_scale, a.T, x0, y0,
                       min(a.out_rows, a.ny - y0), a.out_cols, lds);
}

// k_pool_multi's launch j on tile tasks: a workgroup per tile, in contiguous
// ranges per XCD, so that neighbouring tiles' halos meet in one L2 (FP64, 60
// members of 8.5M cells: 57.8 -> 53.8 us per step against tiles dealt out in turn
// to 4096 workgroups; FP32, 256 of 30M: 122 -> 102).  The grid covers the
// largest range; the workgroups beyond a range's own tiles end at once.
template <typename S, typename C, int R>
__global__ void __launch_bounds__(64 * kTileWaves)
k_pool_tile(const PoolHeader *__restrict__ hdr, const PoolMember *__restrict__ mem, const PoolTile *__restrict__ tiles,
            int range, int j, int T)
{
    extern __shared__ char lds[];
    const int begin = hdr->mbegin[range], n = hdr->mend[range] - begin;
    if ((int)blockIdx.x >= n) return;
    const PoolTile tile = tiles[begin + remap_xcd((int)blockIdx.x, n)];   // workgroup-uniform
    const PoolMember *m = mem + tile.member;
    if ((int64_t)(j + 1) * T > m->t_target - m->t_done) return;
    const int par = (int)((m->cur0 + m->flips + j) & 1);
    tile_pass<S, C, R>(m->buf[par], (void *)m->buf[par ^ 1], m->nx, m->ny, m->pitch, m->plane, member_relax<C>(m),
                       m->scale, m->inv_scale, T, tile.x0, tile.y0, tile.nrows, tile.ncols, lds);
}

template <typename S, typename C>
void *pool_tile_fn(int rows)
{
    switch (rows) {
    case 1: return reinterpret_cast<void *>(&k_pool_tile<S, C, 1>);
    case 2: return reinterpret_cast<void *>(&k_pool_tile<S, C, 2>);
    case 3: return reinterpret_cast<void *>(&k_pool_tile<S, C, 3>);
    case 4: return reinterpret_cast<void *>(&k_pool_tile<S, C, 4>);
    default: return nullptr;
    }
}

template <typename S, typename C>
hipError_t launch_tile_typed(const View &v, const void *src, void *dst, const TileShape &t, int steps, hipStream_t st)
{
    TileArgs<C> a;
    a.src = src;
    a.dst = dst;
    a.nx = v.nx;
    a.ny = v.ny;
    a.pitch = v.pitch;
    a.plane = v.plane;
    a.r = make_relax<C>(v);
    a.scale = (float)v.scale;
    a.inv_scale = (float)v.inv_scale;
    a.T = steps;
    tile_output({t.rows, t.waves, steps}, &a.out_cols, &a.out_rows);
    if (steps < 1 || a.out_cols < 1 || a.out_rows < 1 || t.waves > kTileWaves || !tile_fits(v)) return hipErrorInvalidValue;
    a.tiles_x = (v.nx + a.out_cols - 1) / a.out_cols;
    a.nblocks = a.tiles_x * ((v.ny + a.out_rows - 1) / a.out_rows);
    const uint64_t inv = (((uint64_t)1 << 32) + a.tiles_x - 1) / a.tiles_x;
    a.inv_tiles_x = a.tiles_x > 1 && (uint64_t)a.nblocks * a.tiles_x < ((uint64_t)1 << 32) ? (uint32_t)inv : 0;
    const int waves = tile_waves(t, v.ny, steps);
    const dim3 grid(a.nblocks), block(64, waves);
    const size_t lds = tile_lds(waves, sizeof(typename Store<S>::wide));
#define LBM_TILE(R_)                                                                                      \
    case R_:                                                                                              \
        hipLaunchKernelGGL((k_step_tile<S, C, R_>), grid, block, lds, st, a);                             \
        break;
    switch (t.rows) {
        LBM_TILE(1) LBM_TILE(2) LBM_TILE(3) LBM_TILE(4)
    default: return hipErrorInvalidValue;
    }
#undef LBM_TILE
    return hipGetLastError();
}

// Launch time of a tile shape: a model fitted by storage type to a sweep of
// sizes and shapes; the 16-bit rows are then set 16 % below their fit, by what
// skipping single rows saves.  Against profiles/k_step_tile_shapes.csv (20 sizes
// per storage type, every shape and T) the time of the shape that it picks is
// 5 % (FP64), 6 % (FP32), 8 % (FP16, 6 % of it too low) and 13 % (BF16, 11 % too
// low) off in the root mean square, and the pick takes 7, 3, 2 and 4 % longer than
// the best shape on average, at most 23 % (FP64 2200 x 2150: six steps for eight),
// 16, 12 and 13 %.
// t0: launch and memory latency; row: one row of one wave, one step, on a SIMD
// of its own; wg: load and store of one workgroup; bw: bytes per us to and from
// memory.
struct TileCost {
    double t0, row, wg, bw;
};
constexpr TileCost kTileCost[4] = {{1.99, 0.205, 1.70, 6.1e6},    // FP64
                                   {1.89, 0.110, 1.69, 5.1e6},    // FP32
                                   {1.43, 0.118, 2.11, 3.75e6},   // FP16
                                   {2.02, 0.112, 1.50, 3.75e6}};  // BF16

// What a launch of shape t on a lattice consists of: tiles, the wave-steps of
// all of them, cells moved to and from memory.
struct TileLoad {
    double tiles = 0, live = 0, cells = 0;
    bool add(const View &v, const TileShape &t)
    {
        const int h = t.steps - 1, R = t.rows;
        const int oc = kTileCols - 2 * h, orow = R * t.waves - 2 * h;
        if (oc < 8 || orow < 1) return false;
        const double n = (double)((v.nx + oc - 1) / oc) * ((v.ny + orow - 1) / orow);
        const int need = std::min(orow, v.ny) + 2 * h;
        int w_live = 0;
        for (int w = 0; w * R < need; ++w) w_live += std::min(t.steps, std::min(w * R + R, need - w * R));
        tiles += n;
        live += n * w_live;
        cells += n * kTileCols * R * t.waves + (double)v.nx * v.ny;
        return true;
    }
};

double tile_us(int storage, const TileShape &t, const TileLoad &l)
{
    const TileCost &c = kTileCost[storage];
    const int R = t.rows;
    // workgroups resident per compute unit (512 registers per SIMD lane, 160 KB of LDS)
    const size_t wide = storage == LBM_STORE_F64 ? 8 : 4;
    const int regs = ((wide == 8 ? 44 + 18 * R : 27 + 9 * R) + 7) / 8 * 8;
    const double m = std::max(1, std::min(std::min(8, 512 / regs) * 4 / t.waves,
                                          (int)(160 * 1024 / tile_lds(t.waves, wide))));
    const double per_cu = l.tiles / device_cus();
    const bool many = per_cu > 4 * m;                     // rounds blur into one another
    const double n = many ? per_cu + 0.5 * m : std::ceil(per_cu);
    const double rounds = many ? n / m : std::ceil(n / m);
    const double issue = n * (l.live / l.tiles) * R * c.row / 4;
    const double latency = rounds * (t.steps * (0.03 * R + 0.1) + c.wg);
    const double mem = l.cells * 9 * storage_bytes(storage) / c.bw;
    return c.t0 + std::max(std::max(issue + c.wg, latency), mem) +
           (m < 2 && n > 1 ? 0.5 * mem : 0.15 * std::min(issue, mem));
}

// The tile shapes in use.  More than four rows per lane leave too few waves in
// flight, fewer than twelve waves too little tile for its halo.  Four rows: FP64
// with eight waves (with sixteen, one workgroup per compute unit is left), 16-bit
// with sixteen (61-63 registers: two workgroups per compute unit; a pool of eight
// FP16 lattices of 128^2 to 1024^2 11.2 -> 9.0 us per step against three rows).  FP32
// not: sixteen waves of four rows against three take 3.76 | 3.01 us per step at
// 1000 x 760, 5.47 | 5.38 at 1536 x 1024, 12.59 | 12.69 at 2048^2.
constexpr int32_t kTileShapes[][2] = {{1, 12}, {1, 16}, {2, 12}, {2, 16}, {3, 12}, {3, 16}, {4, 8}, {4, 16}};
bool tile_shape_used(int storage, const int32_t s[2])
{
    if (s[0] < 4) return true;
    return s[1] == 8 ? storage == LBM_STORE_F64 : storage >= LBM_STORE_F16;
}

}  // namespace

// Lattices whose nine planes one buffer resource reaches.
bool tile_fits(const View &v) { return (uint64_t)v.plane * storage_bytes(v.storage) * 9 <= 0xFFFFFFFFull; }

// The tile shape with the least time per step by tile_us; T up to 9 (beyond,
// the halo outgrows what a launch costs at every size measured).
TileShape tile_shape(const View &v)
{
    TileShape best{0, 0, 0};
    double best_us = INFINITY;
    if (!tile_fits(v)) return best;
    for (const auto &s : kTileShapes) {
        if (!tile_shape_used(v.storage, s)) continue;
        for (int T = 2; T <= 9; ++T) {
            const TileShape t{s[0], s[1], T};
            TileLoad l;
            if (!l.add(v, t)) continue;
            const double us = tile_us(v.storage, t, l) / T;
            if (us < best_us) {
                best_us = us;
                best = t;
            }
        }
    }
    return best;
}

// The same for T-step launches of several lattices together, at the T given;
// *us: the launch's time by the model, infinite where there is no shape (a
// lattice beyond the reach of a buffer resource among them).
TileShape tile_shape(const std::vector<const View *> &vs, int T, double *us_out)
{
    TileShape best{0, 0, 0};
    double best_us = *us_out = INFINITY;
    int storage = LBM_STORE_BF16;                         // the widest present
    for (const View *v : vs) {
        if (!tile_fits(*v)) return best;
        storage = std::min(storage, v->storage);
    }
    for (const auto &s : kTileShapes) {
        if (!tile_shape_used(storage, s)) continue;
        const TileShape t{s[0], s[1], T};
        TileLoad l;
        bool ok = !vs.empty();
        for (const View *v : vs) ok = ok && l.add(*v, t);
        const double us = ok ? tile_us(storage, t, l) : INFINITY;
        if (us < best_us) {
            best_us = us;
            best = t;
        }
    }
    *us_out = best_us;
    return best;
}

// Output columns and rows of a tile.
void tile_output(const TileShape &t, int *cols, int *rows)
{
    *cols = kTileCols - 2 * (t.steps - 1);
    *rows = t.rows * t.waves - 2 * (t.steps - 1);
}

void *pool_tile_kernel(int cls, int rows)
{
    switch (cls) {
    case LBM_STORE_F64 * 2 + LBM_COMPUTE_F64: return pool_tile_fn<double, double>(rows);
    case LBM_STORE_F64 * 2 + LBM_COMPUTE_F32: return pool_tile_fn<double, float>(rows);
    case LBM_STORE_F32 * 2 + LBM_COMPUTE_F32: return pool_tile_fn<float, float>(rows);
    case LBM_STORE_F16 * 2 + LBM_COMPUTE_F32: return pool_tile_fn<f16_tag, float>(rows);
    case LBM_STORE_BF16 * 2 + LBM_COMPUTE_F32: return pool_tile_fn<bf16_tag, float>(rows);
    default: return nullptr;
    }
}

hipError_t launch_pool_tile(int range, const TileShape &t, const PoolHeader *hdr, const PoolMember *mem,
                            const PoolTile *tiles, int j, int grid, hipStream_t st)
{
    const int cls = range / kChains;
    void *f = pool_tile_kernel(cls, t.rows);
    if (!f) return hipErrorInvalidValue;
    int T = t.steps;
    void *args[] = {(void *)&hdr, (void *)&mem, (void *)&tiles, (void *)&range, (void *)&j, (void *)&T};
    return hipLaunchKernel(f, dim3(grid), dim3(64, t.waves), args, pool_tile_lds(cls, t.waves), st);
}

size_t pool_tile_lds(int cls, int waves) { return tile_lds(waves, cls / 2 == LBM_STORE_F64 ? 8 : 4); }

hipError_t launch_tile(const View &v, const void *src, void *dst, const TileShape &t, int steps, hipStream_t st)
{
    if (v.compute == LBM_COMPUTE_F64) return launch_tile_typed<double, double>(v, src, dst, t, steps, st);
    switch (v.storage) {
    case LBM_STORE_F64: return launch_tile_typed<double, float>(v, src, dst, t, steps, st);
    case LBM_STORE_F32: return launch_tile_typed<float, float>(v, src, dst, t, steps, st);
    case LBM_STORE_F16: return launch_tile_typed<f16_tag, float>(v, src, dst, t, steps, st);
    case LBM_STORE_BF16: return launch_tile_typed<bf16_tag, float>(v, src, dst, t, steps, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm

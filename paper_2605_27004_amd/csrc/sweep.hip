// sweep.hip -- two steps of the periodic update in one pass over HBM (D3Q19 and D3Q27, FP32 and
// FP64 storage, no walls, gray cells or body force).
//
// A single step reads and writes every population once, which is what bounds it (2 q sizeof(S)
// bytes per cell and step). A sweep reads and writes them once per TWO steps: a work-group owns a
// tile of columns in x and y and walks up in z. On each plane it makes the first step on the tile
// and one cell around it (from the state in HBM, by the pull of k_step), passes the post-collision
// values to its neighbours through LDS, and makes the second step one plane below, which it stores.
// The arithmetic is collide_cell on the same values in the same order, rounded to the storage type
// in between, so the result is bit for bit that of two single steps.
//
// What bounds it: the first step is made again on the tile's rim (11 rows of lanes for 8 rows of
// cells at the D3Q19 256^3 tile below), so FP32 is bound by its VALU work (753 instructions per
// two steps and cell, VALU 70% busy, the clock down to 1.95 GHz) and FP64 by HBM and LDS space (one
// work-group of 10 waves per compute unit; 5.4 TB/s, VALU 30% busy). Us per step, two single steps ->
// sweep: D3Q19 FP32 256^3 387.6 -> 262.7, 128^3 48.3 -> 37.0; FP64 256^3 801.7 -> 508.5,
//   250 x 190 x 130 356.2 -> 190.2; D3Q27 FP32 256^3 556.0 -> 428.6, FP64 256^3 1175 -> 898.
//
//  * Lanes: wave w of the tile is one row of 64 cells (two of 32), so the stores of a wave are
//    whole cache lines, and the columns left and right of the tile sit in the last waves. One flat
//    lane order over the rim-included rows split each stored row between two waves: 1.28 x the
//    bytes written and 346 instead of 288 us.
//  * The next plane's pulls are issued before the first collision and waited for after the second
//    one, so a plane's whole arithmetic covers them.
//  * Every work-group of a segment walks z in step with its neighbours, whose pulls share its rim
//    lines in the XCD's L2 (consecutive tiles on one XCD): FETCH_SIZE 1.28 x one read of the state
//    against 2.1 x, and 275 against 385 us, when each work-group took an equal run of planes that
//    starts anywhere.
#include <algorithm>

#include <hip/hip_runtime.h>

#include "cell.hpp"
#include "common.hpp"
#include "sweep.hpp"

#pragma clang fp contract(off)

namespace lbm {
namespace {

using namespace cell;

// Two steps over the tile (tx, ty) of TX columns by ty_cells rows (at most TYM) and the z-planes of
// one of `segs` segments. AUX: cache policy of the stores. Rows of whole cache lines are written
// non-temporally (256^3 FP32 266 against 275 us cached); other rows leave parts of lines at both ends of a
// tile's rows, which cached stores let the L2 put together (250 x 190 x 130 FP32 135.6 -> 120.6, FP64
// 218.9 -> 193.1, D3Q27 FP64 170 x 160 x 150 295.5 -> 257.1).
template <int LAT, typename S, int ORDER, int TX, int TYM, bool REGS, int AUX>
__global__ __launch_bounds__(((TX + 2) * (TYM + 2) + 63) / 64 * 64) void k_sweep(
    const S *__restrict__ src, S *__restrict__ dst, const Grid g, const StepConsts<typename Conv<S>::C> k,
    const int ty_cells, const uint32_t tiles_x, const uint32_t tiles, const uint32_t segs)
{
    using L = Lattice<LAT>;
    using C = typename Conv<S>::C;
    constexpr int NP = L::NP, W = TX + 2, COLS = W * (TYM + 2);
    constexpr PullOrder<LAT> kPull{};
    __shared__ S lds[sweep::ring_values<LAT, REGS>() * COLS];

    // lanes 0 .. TX H - 1: the tile's own x, row by row; then the columns left and right of it
    const int H = ty_cells + 2, IN = TX * H;
    const int t = threadIdx.x;
    const bool column = t < W * H;
    int hx, hy;
    if (t < IN) {
        hx = 1 + t % TX;
        hy = t / TX;
    } else {
        const int h = column ? t - IN : 0;
        hx = (h & 1) ? W - 1 : 0;
        hy = h >> 1;
    }
    const uint32_t step = g.bc * (uint32_t)sizeof(S);

    // consecutive tiles of a segment on one XCD
    const uint32_t n8 = gridDim.x / 8u, r8 = gridDim.x % 8u, xcd = blockIdx.x % 8u, loc = blockIdx.x / 8u;
    const uint32_t b = xcd < r8 ? xcd * (n8 + 1u) + loc : r8 * (n8 + 1u) + (xcd - r8) * n8 + loc;
    const uint32_t tile = b % tiles, seg = b / tiles;
    const int z_begin = (int)((uint64_t)g.nz * seg / segs), z_end = (int)((uint64_t)g.nz * (seg + 1u) / segs);
    const int xo = (int)(tile % tiles_x) * TX + hx - 1, yo = (int)(tile / tiles_x) * ty_cells + hy - 1;
    const bool inner = t < IN && hy >= 1 && hy <= ty_cells && xo < g.nx && yo < g.ny;
    const Cell c = cell_of(g, (xo + g.nx) % g.nx, (yo + g.ny) % g.ny, 0);
    // in-plane byte offsets of the nine columns a pull reads
    uint32_t off[3][3];
#pragma unroll
    for (int cy = -1; cy <= 1; ++cy)
#pragma unroll
        for (int cx = -1; cx <= 1; ++cx)
            off[cy + 1][cx + 1] = (c.at + back(c.ox, cx) + back(c.oy, cy)) * (uint32_t)sizeof(S);
    // plane `it` of the walk: z_begin - 1 + it, periodic
    const auto plane_at = [&](int it) {
        const int z = z_begin - 1 + it;
        return z < 0 ? z + g.nz : (z >= g.nz ? z - g.nz : z);
    };
    const auto load = [&](int it, S *pre) {
        const int z = plane_at(it);
        const __amdgpu_buffer_rsrc_t r0 = sweep::plane_rsrc(src + (uint64_t)z * g.zs);
        const __amdgpu_buffer_rsrc_t rm = sweep::plane_rsrc(src + (uint64_t)(z == 0 ? g.nz - 1 : z - 1) * g.zs);
        const __amdgpu_buffer_rsrc_t rp = sweep::plane_rsrc(src + (uint64_t)(z == g.nz - 1 ? 0 : z + 1) * g.zs);
#pragma unroll
        for (int j = 0; j < L::Q; ++j) {
            const int i = kPull.dir[j];
            const PairRow v = i == 0 ? PairRow{0, 0, 0} : L::pair((i - 1) / 2);
            const int sg = (i & 1) ? 1 : -1, cz = sg * v.cz;
            pre[i] = sweep::ld_buf<S>(cz > 0 ? rm : (cz < 0 ? rp : r0), off[sg * v.cy + 1][sg * v.cx + 1],
                                      (uint32_t)i * step);
        }
    };
    const auto store = [&](int it, const C *gp, const C *gm) {
        const PlaneStores ps = plane_stores(dst, g, Ref{(uint64_t)plane_at(it - 1) * g.zs, c.at});
        st_plane_aux<AUX>(ps, 0, Conv<S>::st(gp[0]));
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            st_plane_aux<AUX>(ps, 2 * p + 1, Conv<S>::st(gp[p + 1]));
            st_plane_aux<AUX>(ps, 2 * p + 2, Conv<S>::st(gm[p + 1]));
        }
    };
    sweep::planes<LAT, S, ORDER, REGS, COLS>(
        lds, hy * W + hx, column, inner, z_end - z_begin + 2, k, load, [](int cx, int cy) { return cx + cy * W; }, store);
}

}  // namespace

namespace {

constexpr uint32_t kCus = 256;  // compute units of the MI355X; one work-group of a sweep runs on each

// Tile widths and largest heights of the compiled sweeps (the LDS of a tile and its rim, and 1,024
// lanes), and the measured time of one row of `tx` cells of one plane (us); a plane of a tile of h
// rows takes the time of h + 1, but low_us + h low_row_us at least: with few waves its latencies count.
struct SweepTile {
    int lattice, storage, tx, tym;
    double row_us, low_us, low_row_us;
};
constexpr SweepTile kTiles[] = {
    {kD3Q19, kF32, 64, 13, 0.46, 2.0, 0.0},
    {kD3Q19, kF64, 32, 16, 0.46, 1.65, 0.27},
    {kD3Q19, kF64, 64, 7, 0.87, 0.0, 0.0},
    {kD3Q27, kF32, 64, 9, 0.78, 0.0, 0.0},
    {kD3Q27, kF64, 32, 10, 0.72, 2.7, 0.40},
};

// Bytes per us of single steps over grids of `both` bytes of populations: rows of 64 n cells 5.8 TB/s up to 90 MB
// (6.0 to 6.3 at 40 MB, by where the buffers lie), other rows 5.4 TB/s where they are no whole cache lines and
// the caches no longer hold the state.
double single_rate(const Grid &g, int bytes, double both)
{
    if (g.nx % 64 == 0 && both <= 300e6) return both <= 90e6 ? 5.8e6 : 6.1e6;
    return both > 300e6 && g.nx * bytes % 128 != 0 ? 5.4e6 : 6.3e6;
}

}  // namespace

// The cut of a grid into tiles and segments, from the time that a cut takes: rounds of one
// work-group per compute unit x planes (two more than the segment's, for the rim) x rows. Measured
// over grids of 40 x 40 x 500 to 256^3, even and odd, it is right to 10% or so. Against it, with the
// latencies of low tiles, stands the time of two single steps: 2 us a launch and the bytes. The line so
// lies between 40 and 100 MB of populations in FP32 and near 80 MB in FP64 (D3Q19) or 200 MB (D3Q27): below, the
// work-groups are too few and their rims too large (us per step, single against sweep, D3Q19 FP32: 48^3
// 5.7 / 6.1, 64^3 7.2 to 8.3 / 7.2, 64 x 69 x 83 12.2 / 9.7, 100^3 24.3 / 28.4, 150 x 101 x 75 28.5 / 29.8, 128 x 96 x 80
// 24.7 / 20.8, 200 x 150 x 100 80.7 / 68.7, 250 x 190 x 130 175.3 / 120.6; D3Q27 FP32: 100^3 34.0 / 46.3, 128^3
// 73.6 / 63.0; D3Q19 FP64: 64 x 48 x 54 10.5 / 12.0, 64 x 64 x 52 12.4 / 13.6, 64^3 15.8 / 15.0, 77 x 85 x 60
// 22.2 / 23.9, 110 x 120 x 100 78.7 / 56.6; D3Q27 FP64: 64^3 21.0 / 22.6, 64 x 99 x 60 29.0 / 31.1, 64 x 108 x 81
// 43.5 / 38.9).
SweepPlan plan_sweep(int lattice, int storage, const Grid &g)
{
    SweepPlan best{0, 0, 0};
    const int bytes = storage == kF64 ? 8 : 4;
    const double q = lattice == kD3Q19 ? 19.0 : 27.0;
    const double both = 2.0 * q * bytes * g.n;  // bytes of a step
    double best_us = 1e300, low_us = 1e300;
    for (const SweepTile &t : kTiles) {
        if (t.lattice != lattice || t.storage != storage) continue;
        // D3Q19 FP64: rows of 32 cells where they are whole cache lines (256^3: 505 against 532 us),
        // else of 64 cells, which leave half the partial lines (250 x 190 x 130: 249 against 214 us)
        if (lattice == kD3Q19 && storage == kF64 && (t.tx == 32) != (g.nx % 16 == 0)) continue;
        const int64_t tx = (g.nx + t.tx - 1) / t.tx;
        for (int ty = t.tym; ty >= 3; --ty) {
            const int64_t tiles = tx * ((g.ny + ty - 1) / ty);
            for (int segs = 1; segs <= std::max(1, g.nz / 2) && segs <= 64; ++segs) {
                const int64_t rounds = (tiles * segs + kCus - 1) / kCus;
                const double planes = (double)rounds * ((g.nz + segs - 1) / segs + 2);
                const double us = 2.0 + planes * (ty + 1) * t.row_us;
                if (us < best_us) {
                    best_us = us;
                    low_us = 2.0 + planes * std::max((ty + 1) * t.row_us, t.low_us + ty * t.low_row_us);
                    best = SweepPlan{t.tx, ty, segs};
                }
            }
        }
    }
    const double single_us = 2.0 * (2.0 + both / single_rate(g, bytes, both));
    return low_us < single_us / 1.05 ? best : SweepPlan{0, 0, 0};
}

hipError_t launch_sweep(int lattice, int storage, int order, const Grid &g, const StepConsts<double> &k64,
                        const StepConsts<float> &k32, const SweepPlan &p, const void *src, void *dst,
                        hipStream_t stream)
{
    const uint32_t tiles_x = (uint32_t)((g.nx + p.tx - 1) / p.tx), tiles_y = (uint32_t)((g.ny + p.ty - 1) / p.ty);
    const uint32_t tiles = tiles_x * tiles_y;
    const dim3 grid(tiles * (uint32_t)p.segs);
    const dim3 block((uint32_t)((p.tx + 2) * (p.ty + 2) + 63) / 64 * 64);
    const bool whole_lines = g.nx * (storage == kF64 ? 8 : 4) % 128 == 0;
#define LBM_SWEEP_A(LAT, S, O, TX, TYM, REGS, AUX, KC)                                                           \
    hipLaunchKernelGGL((k_sweep<LAT, S, O, TX, TYM, REGS, AUX>), grid, block, 0, stream, (const S *)src, (S *)dst, g, \
                       KC, p.ty, tiles_x, tiles, (uint32_t)p.segs)
#define LBM_SWEEP(LAT, S, TX, TYM, REGS, KC)                                                                     \
    do {                                                                                                         \
        if (order == 2) {                                                                                        \
            if (whole_lines) LBM_SWEEP_A(LAT, S, 2, TX, TYM, REGS, 2, KC);                                       \
            else LBM_SWEEP_A(LAT, S, 2, TX, TYM, REGS, 0, KC);                                                   \
        } else {                                                                                                 \
            if (whole_lines) LBM_SWEEP_A(LAT, S, 3, TX, TYM, REGS, 2, KC);                                       \
            else LBM_SWEEP_A(LAT, S, 3, TX, TYM, REGS, 0, KC);                                                   \
        }                                                                                                        \
        return hipGetLastError();                                                                                \
    } while (0)
    if (lattice == kD3Q19 && storage == kF32) LBM_SWEEP(kD3Q19, float, 64, 13, true, k32);
    if (lattice == kD3Q19 && storage == kF64 && p.tx == 32) LBM_SWEEP(kD3Q19, double, 32, 16, false, k64);
    if (lattice == kD3Q19 && storage == kF64) LBM_SWEEP(kD3Q19, double, 64, 7, false, k64);
    if (lattice == kD3Q27 && storage == kF32) LBM_SWEEP(kD3Q27, float, 64, 9, true, k32);
    if (lattice == kD3Q27 && storage == kF64) LBM_SWEEP(kD3Q27, double, 32, 10, false, k64);
#undef LBM_SWEEP
#undef LBM_SWEEP_A
    return hipErrorInvalidValue;
}

}  // namespace lbm

// tile.hip -- several steps of a two-dimensional grid in one launch (D2Q9, every storage type, wall
// model and force but one: see tile_serves).
//
// A D2Q9 step is short: on small grids its launch and its latencies bound it (64 x 64: 3.6 us a
// step, whatever it computes), on large ones HBM. Here a work-group takes a tile of cells with a rim
// of steps - 1 cells around it through `steps` steps: the cells live in registers, their
// post-collision values pass to the neighbours through LDS between the steps, and only the first
// step reads the state and only the last one writes it (every one where the caller wants each
// state). The rim's outermost cells go wrong step by step, one cell deep each, and are never stored.
// The arithmetic of a cell is the single step's (collide_cell on the same values in the same order,
// rounded to the storage type in between), so the result is bit for bit the single steps'.
//
// What bounds it then: large grids the VALU work (rim included 1.2 x the single steps'), small ones
// the latency of a step in LDS (0.65 us). Us per step, single -> tiles: 64^2 FP64 3.9 -> 1.0, 512^2
// FP32 with gray cells 6.2 -> 3.5, 1000 x 700 FP64 16.5 -> 8.3, 3000 x 2000 FP32 76.5 -> 33.2,
// 4096^2 FP32 193.7 -> 90.0, 2816 x 2746 FP16 46.6 -> 34.2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "cell.hpp"
#include "common.hpp"

#pragma clang fp contract(off)

namespace lbm {
namespace {

using namespace cell;

enum TileMode : int { kTilePlain = 0, kTileLinks = 1, kTileGray = 2 };  // as the step kernel's modes

// T lanes, R cells each, in rows of TW cells; row r of a lane is row ly + r T / TW of the tile. One
// LDS buffer and two barriers per step: two buffers would need one, but halve the work-groups that
// share a compute unit (4096^2 FP32: 90.6 against 121 us).
// every: with 0 the last state goes to dst; else state s (after s + 1 steps) to dst + s every.
template <typename S, int ORDER, int MODE, int T, int R, int TW>
__global__ __launch_bounds__(T) void k_tile(const S *__restrict__ src, S *__restrict__ dst, const uint64_t every,
                                            const Grid g, const StepConsts<typename Conv<S>::C> k,
                                            const uint32_t *__restrict__ links, const float *__restrict__ gray,
                                            const int steps, const uint32_t tiles_x)
{
    using L = Lattice<kD2Q9>;
    using C = typename Conv<S>::C;
    constexpr int NP = L::NP, RG = T / TW, H = RG * R, N = TW * H, PAD = 1;
    constexpr int PL = N + 2 * PAD;  // a direction's plane; the rim's corners reach one cell past it
    __shared__ S buf[L::Q - 1][PL];
    const int t = threadIdx.x, lx = t % TW, ly = t / TW, rim = steps - 1;
    const int ow = TW - 2 * rim, oh = H - 2 * rim;
    const int xo = (int)(blockIdx.x % tiles_x) * ow - rim + lx, y0 = (int)(blockIdx.x / tiles_x) * oh - rim;
    int x = xo % g.nx;
    if (x < 0) x += g.nx;

    C gp[R][NP + 1], gm[R][NP + 1];
    uint32_t at[R], lk[R];
    C mg[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int y = (y0 + ly + r * RG) % g.ny;
        if (y < 0) y += g.ny;
        const Cell c = cell_of(g, x, y, 0);
        at[r] = c.at;
        lk[r] = MODE == kTileLinks && links ? links[c.own] : 0u;
        mg[r] = MODE == kTileGray ? (C)gray[c.own] : C(0);
        if (lk[r] & 1u) {
#pragma unroll
            for (int p = 0; p <= NP; ++p) gp[r][p] = gm[r][p] = C(0);
        } else {
            gp[r][0] = Conv<S>::ld(ld_pop(src, g, 0, own_ref(c)));
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                if constexpr (MODE == kTileLinks) {
                    gp[r][p + 1] = Conv<S>::ld(ld_slot(src, g, slot_plus<kD2Q9>(c, p, lk[r])));
                    gm[r][p + 1] = Conv<S>::ld(ld_slot(src, g, slot_minus<kD2Q9>(c, p, lk[r])));
                } else {
                    gp[r][p + 1] = Conv<S>::ld(ld_pop(src, g, 2 * p + 1, src_plus<kD2Q9>(c, p)));
                    gm[r][p + 1] = Conv<S>::ld(ld_pop(src, g, 2 * p + 2, src_minus<kD2Q9>(c, p)));
                }
            }
        }
    }
    for (int s = 0; s < steps; ++s) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int row = ly + r * RG;
            // rows that the last step's cells no longer depend on drop out one by one
            if (row < s || row >= H - s) continue;
            if (!(lk[r] & 1u)) {
                C pp[NP + 1], pm[NP + 1];
                if constexpr (MODE == kTileGray) {
#pragma unroll
                    for (int p = 0; p <= NP; ++p) {
                        pp[p] = gp[r][p];
                        pm[p] = gm[r][p];
                    }
                }
                collide_cell<kD2Q9, ORDER, MODE != kTilePlain, C, kClose<S>>(k, gp[r], gm[r]);
                if constexpr (MODE == kTileGray) {
                    gp[r][0] = fmad(mg[r], pp[0] - gp[r][0], gp[r][0]);
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        const C a = gp[r][p + 1];
                        gp[r][p + 1] = fmad(mg[r], pm[p + 1] - a, a);
                        gm[r][p + 1] = fmad(mg[r], pp[p + 1] - gm[r][p + 1], gm[r][p + 1]);
                    }
                }
            }
            S v[L::Q];
            v[0] = Conv<S>::st(gp[r][0]);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                v[2 * p + 1] = Conv<S>::st(gp[r][p + 1]);
                v[2 * p + 2] = Conv<S>::st(gm[r][p + 1]);
            }
            const int yo = y0 + row;
            if ((s == steps - 1 || every != 0u) && row >= rim && row < H - rim && lx >= rim && lx < TW - rim &&
                xo < g.nx && yo < g.ny) {
                S *out = dst + (uint64_t)s * every;
                const PlaneStores ps = plane_stores(out, g, Ref{0u, at[r]});
#pragma unroll
                for (int i = 0; i < L::Q; ++i) st_plane_aux<0>(ps, i, v[i]);
            }
            if (s < steps - 1) {
                gp[r][0] = Conv<S>::ld(v[0]);
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    gp[r][p + 1] = Conv<S>::ld(v[2 * p + 1]);
                    gm[r][p + 1] = Conv<S>::ld(v[2 * p + 2]);
                }
#pragma unroll
                for (int i = 1; i < L::Q; ++i) buf[i - 1][PAD + row * TW + lx] = v[i];
            }
        }
        if (s == steps - 1) break;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int row = ly + r * RG;
            if (row < s + 1 || row >= H - s - 1 || (lk[r] & 1u)) continue;
            const S *here = &buf[0][PAD + row * TW + lx];
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const PairRow c = L::pair(p);
                const int d = c.cy * TW + c.cx;
                C a = Conv<S>::ld(here[2 * p * PL - d]), b = Conv<S>::ld(here[(2 * p + 1) * PL + d]);
                if constexpr (MODE == kTileLinks) {  // halfway bounce-back: the cell's own opposite value
                    const C ob = gm[r][p + 1], oa = gp[r][p + 1];
                    if (lk[r] >> (2 * p + 1) & 1u) a = ob;
                    if (lk[r] >> (2 * p + 2) & 1u) b = oa;
                }
                gp[r][p + 1] = a;
                gm[r][p + 1] = b;
            }
        }
        __syncthreads();
    }
}

}  // namespace

namespace {

// The compiled tiles: lanes, cells per lane and row length (TilePlan::shape is the index).
struct TileShape {
    int t, r, tw;
    int height() const { return t / tw * r; }
};
constexpr TileShape kShapes[] = {{512, 1, 32}, {512, 2, 64}, {1024, 2, 64}};  // 32 x 16, 64 x 16, 64 x 32

template <typename S, int ORDER, int MODE>
hipError_t run_tile(const Grid &g, const StepConsts<typename Conv<S>::C> &k, const uint32_t *links, const float *gray,
                    const void *src, void *dst, uint64_t every, const TilePlan &p, int steps, hipStream_t stream)
{
    const TileShape &sh = kShapes[p.shape];
    const int ow = sh.tw - 2 * (steps - 1), oh = sh.height() - 2 * (steps - 1);
    if (steps < 1 || ow < 1 || oh < 1) return hipErrorInvalidValue;
    const uint32_t tx = (uint32_t)((g.nx + ow - 1) / ow), ty = (uint32_t)((g.ny + oh - 1) / oh);
#define LBM_TILE(I)                                                                                               \
    hipLaunchKernelGGL((k_tile<S, ORDER, MODE, kShapes[I].t, kShapes[I].r, kShapes[I].tw>), dim3(tx * ty), dim3(sh.t), \
                       0, stream, (const S *)src, (S *)dst, every, g, k, links, gray, steps, tx)
    if (p.shape == 0) LBM_TILE(0);
    else if (p.shape == 1) LBM_TILE(1);
    else LBM_TILE(2);
#undef LBM_TILE
    return hipGetLastError();
}

}  // namespace

// FP16 with a solid mask or a force (and no gray cells) stays with single steps. The compiler turns
// a multiply-add and its conversion to FP16 into one instruction that rounds once (v_fma_mixlo_f16)
// where no branch lies between the two; in that mode the single-step kernel gets it for some of the
// directions and this one for none, so their results differ in the last bit now and then. Without walls
// and with gray cells both kernels get it for all nine, in every tile, pull and order; whether a compiler
// does so is read from the built code in tests/test_host_fp16_rounding.py. Nothing of the kind exists for BF16.
bool tile_serves(int storage, bool gray, bool links_or_force)
{
    return storage != kF16 || gray || !links_or_force;
}

// The tile and the steps per launch (shape -1: single steps), from sweeps over both (us per step; k =
// steps per launch):
//  * small grids: the fewest cells per work-group, and many steps, since latency bounds a step
//    whatever the rim costs (64^2 FP64: 32 x 16 k 8 1.00, k 5 1.28, 64 x 16 k 8 1.40; 200 x 150 FP32:
//    32 x 16 k 6 1.33, k 8 1.64, 64 x 16 k 7 1.48);
//  * up to 400,000 cells: one large tile per compute unit (512^2: 64 x 32 k 6 FP64 3.59, FP32 3.01,
//    FP16 2.95; k 4 3.98, 3.32, 3.35; 64 x 16 k 4 3.99, 3.5, 3.5);
//  * above, the VALU bounds and the rim counts: 64 x 32, k 5 (3001 x 1999 FP32 k 4 35.5, k 5 34.6, k 6
//    35.2; 64 x 16 k 4 38.1), k 4 with the two equilibria of the force (2816 x 2746 FP32 gray k 4 52.2,
//    k 5 54.0). FP64 takes 64 x 16, k 4, two of which share a compute unit's LDS (2816 x 2746: 75.5
//    against 81.3 with 64 x 32), and so do 16-bit storage and a force with k 3 (FP16 gray 50.5 against
//    59.9: its conversions take the VALU, and the larger tile's registers the waves).
//
// Against that plan stands the single step: a tile that the grid does not fill computes its idle columns and
// rows all the same, so strips and rows a little longer than a tile may lose (us per step, single -> tiles:
// 4,000,000 x 1 FP32 51 -> 422, 100,000 x 4 FP16 5.4 -> 11.5, 8 x 125,000 FP32 12 -> 33, 64 x 6000 BF16 with
// a force 5.5 -> 8.7; but 24 x 40,000 FP64 22 -> 21, 20,000 x 30 FP32 8.7 -> 6.4). The times of both over
// 55 grids of 1 x 8192 to 300,000 x 20 cells, plain, with gray cells and with a force, are within 20%
// (80% of them) of
//  * a launch of tiles: 6.5 us (32 x 16), 9 us (64 x 16) or, of the tile that has a compute unit to itself,
//    5 us and most of a turn, and a turn of one tile per compute unit: steps x cells (the rows that
//    drop out left out) x the time of a cell;
//  * a single step: 3.9 us at least, or 2.8 us and the time of its cells.
TilePlan plan_tile(int storage, const Grid &g, bool general, bool gray)
{
    const bool f64 = storage == kF64, f32 = storage == kF32;
    const double cell_us = 1e-6 * g.n;
    TilePlan p;
    if (g.n <= 8192) p = TilePlan{0, 8, 2};
    else if (g.n <= 100000) p = TilePlan{0, 6, 2};
    else if (g.n <= 400000) p = TilePlan{2, 6, 2};
    else if (f64) p = TilePlan{1, 4, 2};
    else if (f32) p = TilePlan{2, general ? 4 : 5, 2};
    else p = general ? TilePlan{1, 3, 2} : TilePlan{2, 5, 2};
    if (p.shape == 2) {
        // a launch of the large tile takes 8 to 12 us whatever its steps, so two steps alone may lose (us per step,
        // single against tile: FP32 400 x 300 3.6 / 4.3, with a force 3.8 / 4.8, 512^2 5.9 / 4.6; BF16 512^2 4.0 / 5.0,
        // 1000 x 700 7.4 / 6.4; FP64 400 x 300 with a force 5.0 / 6.4, 576 x 664 12.3 / 7.8)
        const double t2 = (double)((g.nx + 61) / 62) * (double)((g.ny + 29) / 30);
        const double two_us = f64   ? (general ? 11.3 : 9.0) + 0.02 * t2
                              : f32 ? (general ? 8.2 : 7.5) + 0.015 * t2 + (t2 > 256.0 ? 4.0 : 0.0)
                                    : (general ? 9.6 + 0.017 * t2 : 8.2 + 0.0125 * t2);
        // (long rows of 64 n cells have slower single steps: boxes)
        const double ps = (f64 ? 20.0 : (f32 ? (general ? 11.0 : 10.0) : (general ? 7.3 : 5.8))) *
                          (g.nx > 256 && g.nx % 64 == 0 ? 1.2 : 1.0);
        if (two_us >= 2.0 * std::max(3.7, 2.8 + ps * cell_us)) p.least = 3;
    }
    if (p.steps == 3 && g.n < 1000000) p.least = 3;  // (BF16 448 x 1017 with a force 6.1 / 7.4)

    const TileShape &sh = kShapes[p.shape];
    const int ow = sh.tw - 2 * (p.steps - 1), oh = sh.height() - 2 * (p.steps - 1);
    const double tiles = (double)((g.nx + ow - 1) / ow) * (double)((g.ny + oh - 1) / oh), turns = tiles / 256.0;
    const double cell_ns = f64   ? (gray ? 1.8 : (general ? 1.9 : 1.27))
                           : f32 ? (gray ? 1.1 : (general ? 1.4 : 0.85))
                                 : (gray ? 1.25 : (general ? (p.shape == 2 ? 1.6 : 1.35) : 0.78));
    const double turn_us = 1e-3 * cell_ns * p.steps * sh.tw * (sh.height() - p.steps + 1);
    // (with links or a force in 16-bit storage the large tile's registers leave room for one: whole turns count)
    const double large_turns = !f64 && !f32 && general && !gray ? std::ceil(turns) : std::max(1.0, turns + 0.75);
    const double launch_us = p.shape == 2 ? 5.0 + turn_us * large_turns
                                          : (p.shape == 0 ? 6.5 : 9.0) + turn_us * turns;
    // (past the Infinity Cache a quarter more in FP64, a fifth in FP32)
    const bool large = 18.0 * (f64 ? 8 : (f32 ? 4 : 2)) * g.n > 300e6;
    const double cell_ps = f64 ? (large ? 25.0 : 20.0) : (f32 ? (large ? 12.0 : 10.0) : (general ? 7.3 : 5.8));
    // (rows that the lane exchange serves are at the model's lower side, others at its upper side)
    const double factor = g.nx % 64 == 0 && g.nx <= 256 ? (f64 || f32 ? 1.0 : 0.95) : 1.1;
    const double single_us = std::max(3.9, factor * (2.8 + cell_ps * cell_us));
    return launch_us / p.steps < single_us ? p : TilePlan{-1, 1, 1};
}

hipError_t launch_tile(int storage, int order, const Grid &g, const StepConsts<double> &k64,
                       const StepConsts<float> &k32, const uint32_t *links, const float *gray, const void *src,
                       void *dst, uint64_t every, const TilePlan &p, int steps, hipStream_t stream)
{
    const auto go = [&](auto sv, const auto &k) {
        using S = decltype(sv);
#define LBM_MODE(M)                                                                                                \
    (order == 2 ? run_tile<S, 2, M>(g, k, links, gray, src, dst, every, p, steps, stream)                            \
                : run_tile<S, 3, M>(g, k, links, gray, src, dst, every, p, steps, stream))
        if (gray) return LBM_MODE(kTileGray);
        if constexpr (!std::is_same<S, _Float16>::value)
            if (links || k.forced) return LBM_MODE(kTileLinks);
        return LBM_MODE(kTilePlain);
#undef LBM_MODE
    };
    switch (storage) {
    case kF64: return go(double{}, k64);
    case kF32: return go(float{}, k32);
    case kF16: return go(_Float16{}, k32);
    case kBF16: return go(__bf16{}, k32);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm

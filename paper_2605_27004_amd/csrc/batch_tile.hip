// batch_tile.hip -- several steps of every two-dimensional domain of a batch in one launch (D2Q9, FP32 and
// FP64 storage).
//
// A step of a batch of planes is short: its launch and its latencies bound it (3.4 us for 64 planes of 10
// to 64 cells a side). As in the single grid's tiles, a work-group takes cells through several steps,
// one cell per lane in registers, and the post-collision values pass to the neighbours through LDS in
// between. A work-group's cells are whole rows of one domain, which wrap in x: the whole domain where that
// fits, which then wraps in y too and needs no rim, or else some rows and a rim of `rim` rows above
// and below, of which the outermost go wrong step by step and are never stored. The arithmetic of a cell is
// the single step's, rounded to the storage type in between, so the result is bit for bit the same.
//
// What bounds it then: the latency of a step in LDS (0.70 us with 512 lanes, 0.93 with 1,024) for few
// domains, the VALU with the rim for many. Us per step: 8 planes of 10 to 30 cells a side FP32 2.76 -> 0.97,
// 128 of 16 to 64 4.4 -> 2.9, 512 of them FP64 22.8 -> 9.9.
#include <hip/hip_runtime.h>

#include "batch.hpp"
#include "cell.hpp"
#include "common.hpp"

#pragma clang fp contract(off)

namespace lbm {
namespace {

using namespace cell;

template <typename S, int ORDER, int T>
__global__ __launch_bounds__(T) void k_batch_tile(const S *__restrict__ src, S *__restrict__ dst,
                                                  const BatchSweepRec *__restrict__ recs,
                                                  const BatchDomain *__restrict__ doms,
                                                  const StepConsts<typename Conv<S>::C> *__restrict__ kc, const int steps,
                                                  const int rim)
{
    using L = Lattice<kD2Q9>;
    using C = typename Conv<S>::C;
    constexpr int NP = L::NP;
    __shared__ S buf[L::Q - 1][T];

    const BatchSweepRec r = recs[blockIdx.x];
    const BatchDomain dm = doms[r.dom];
    const StepConsts<C> k = kc[r.dom];
    const Grid g = dm.g;
    const bool whole = r.rows == g.ny;
    const int H = whole ? g.ny : r.rows + 2 * rim;
    const int t = threadIdx.x;
    const bool cell = t < g.nx * H;  // (the records keep nx H <= T)
    uint32_t hx;
    const int hy = (int)div_by(cell ? (uint32_t)t : 0u, dm.mx, (uint32_t)g.nx, hx);
    int y = whole ? hy : (r.y0 + hy - rim) % g.ny;
    if (y < 0) y += g.ny;
    const bool inner = cell && (whole || (hy >= rim && hy < rim + r.rows && r.y0 + hy - rim < g.ny));
    const FlatCell c = flat_cell_of(g, hx, (uint32_t)y, 0u);

    C gp[NP + 1], gm[NP + 1];
    gp[0] = Conv<S>::ld(ld_pop(src + dm.base, g, 0, own_ref(c)));
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        gp[p + 1] = Conv<S>::ld(ld_pop(src + dm.base, g, 2 * p + 1, src_plus<kD2Q9>(c, p)));
        gm[p + 1] = Conv<S>::ld(ld_pop(src + dm.base, g, 2 * p + 2, src_minus<kD2Q9>(c, p)));
    }
    // neighbours in the tile: rows wrap in x, and in y where the tile holds the whole domain
    const int xm = hx == 0u ? g.nx - 1 : -1, xp = (int)hx == g.nx - 1 ? 1 - g.nx : 1;
    const int ym = whole && hy == 0 ? (g.ny - 1) * g.nx : -g.nx;
    const int yp = whole && hy == g.ny - 1 ? -(g.ny - 1) * g.nx : g.nx;
    const auto at = [&](int cx, int cy) {
        return t + (cx < 0 ? xm : (cx > 0 ? xp : 0)) + (cy < 0 ? ym : (cy > 0 ? yp : 0));
    };
    for (int s = 0; s < steps; ++s) {
        // rows of the rim that the last step's cells no longer depend on drop out one by one
        if (cell && (whole || (hy >= s && hy < H - s))) {
            collide_cell<kD2Q9, ORDER, false, C, kClose<S>>(k, gp, gm);
            if (s < steps - 1) {
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    buf[2 * p][t] = Conv<S>::st(gp[p + 1]);
                    buf[2 * p + 1][t] = Conv<S>::st(gm[p + 1]);
                }
                gp[0] = Conv<S>::ld(Conv<S>::st(gp[0]));
            }
        }
        if (s == steps - 1) break;
        __syncthreads();
        if (cell && (whole || (hy >= s + 1 && hy < H - s - 1))) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const PairRow v = L::pair(p);
                gp[p + 1] = Conv<S>::ld(buf[2 * p][at(-v.cx, -v.cy)]);
                gm[p + 1] = Conv<S>::ld(buf[2 * p + 1][at(v.cx, v.cy)]);
            }
        }
        __syncthreads();
    }
    if (!inner) return;
    const PlaneStores ps = plane_stores(dst + dm.base, g, own_ref(c));
    st_plane_aux<0>(ps, 0, Conv<S>::st(gp[0]));
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        st_plane_aux<0>(ps, 2 * p + 1, Conv<S>::st(gp[p + 1]));
        st_plane_aux<0>(ps, 2 * p + 2, Conv<S>::st(gm[p + 1]));
    }
}

}  // namespace

hipError_t launch_batch_tile(int storage, int order, uint32_t nrecs, const BatchSweepRec *recs, const BatchDomain *doms,
                             const StepConsts<double> *k64, const StepConsts<float> *k32, const void *src, void *dst,
                             int steps, const BatchTilePlan &p, hipStream_t stream)
{
    if (nrecs == 0) return hipSuccess;
    if (steps < 1 || steps > p.steps) return hipErrorInvalidValue;
    const auto go = [&](auto sv, const auto *kc) {
        using S = decltype(sv);
#define LBM_TILE(O, T)                                                                                            \
    hipLaunchKernelGGL((k_batch_tile<S, O, T>), dim3(nrecs), dim3(T), 0, stream, (const S *)src, (S *)dst, recs, doms, \
                       kc, steps, p.steps - 1)
        if (p.lanes == 512) {
            if (order == 2) LBM_TILE(2, 512); else LBM_TILE(3, 512);
        } else {
            if (order == 2) LBM_TILE(2, 1024); else LBM_TILE(3, 1024);
        }
#undef LBM_TILE
        return hipGetLastError();
    };
    return storage == kF64 ? go(double{}, k64) : go(float{}, k32);
}

}  // namespace lbm

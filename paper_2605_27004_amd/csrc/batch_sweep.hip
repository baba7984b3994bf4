// batch_sweep.hip -- two steps of every domain of a batch in one pass over HBM (D3Q19 and D3Q27, FP32 and
// FP64 storage): the plane loop of sweep.hpp on batched domains.
//
// A work-group takes whole rows of one domain -- `rows` of them and one on either side, or the whole
// cross-section where that fits -- through the z-planes of its record, with the domain's own
// constants. Whole rows need no rim in x (their periodic neighbours are in the tile), pack the lanes
// whatever the row's length, and give stores that run on from row to row, which leaves a part of
// a cache line only at a tile's two ends. So less work is made twice here than in a sweep over one
// large grid (8% in y and 5% in z for 40^3), but four more VALU instructions per pull address the
// linear blocks. Bit for bit the result of two single steps.
//
// us per step, single steps -> sweep (domains of 16 to 64 cells a side): D3Q19 FP32 512 domains 803.2 ->
// 620.3, 128 domains 210.1 -> 173.1, FP64 128 domains 464.5 -> 293.3; D3Q27 FP32 128 domains 303.6 -> 258.0,
// FP64 64 domains 301.8 -> 266.2.
#include <hip/hip_runtime.h>

#include "batch.hpp"
#include "cell.hpp"
#include "sweep.hpp"

#pragma clang fp contract(off)

namespace lbm {
namespace {

using namespace cell;

// Columns of a tile: what LDS holds (ring_values per column), in whole waves, and at most 1,024 lanes.
template <int LAT, typename S> constexpr bool kRegs = sizeof(S) == 4;
template <int LAT, typename S> constexpr int sweep_cols()
{
    constexpr int fit = 160 * 1024 / (sweep::ring_values<LAT, kRegs<LAT, S>>() * (int)sizeof(S));
    // D3Q27 FP32 needs 150 registers: 12 waves
    constexpr int most = LAT == kD3Q27 && sizeof(S) == 4 ? 768 : 1024;
    return fit < most ? fit : most;
}

template <int LAT, typename S, int ORDER>
__global__ __launch_bounds__((sweep_cols<LAT, S>() + 63) / 64 * 64) void k_batch_sweep(
    const S *__restrict__ src, S *__restrict__ dst, const BatchSweepRec *__restrict__ recs,
    const BatchDomain *__restrict__ doms, const StepConsts<typename Conv<S>::C> *__restrict__ kc)
{
    using L = Lattice<LAT>;
    using C = typename Conv<S>::C;
    constexpr int NP = L::NP, COLS = sweep_cols<LAT, S>();
    constexpr PullOrder<LAT> kPull{};
    __shared__ S lds[sweep::ring_values<LAT, kRegs<LAT, S>>() * COLS];

    const BatchSweepRec r = recs[blockIdx.x];
    const BatchDomain dm = doms[r.dom];
    const StepConsts<C> k = kc[r.dom];
    const Grid g = dm.g;
    const bool whole = r.rows == g.ny;  // the tile holds every row: no rim in y either
    const int H = whole ? r.rows : r.rows + 2;
    const bool column = (int)threadIdx.x < g.nx * H;
    const uint32_t t = column ? threadIdx.x : 0u;
    uint32_t hx;
    const int hy = (int)div_by(t, dm.mx, (uint32_t)g.nx, hx);
    int y = whole ? hy : r.y0 + hy - 1;
    if (y < 0) y += g.ny;
    // the rim rows of a ragged last tile may lie past the grid's first rows more than once
    while (y >= g.ny) y -= g.ny;
    const bool inner = column && (whole || (hy >= 1 && hy <= r.rows && r.y0 + hy - 1 < g.ny));

    const AxisOff ox = axis_off(hx, (uint32_t)g.nx, 1u), oy = axis_off((uint32_t)y, (uint32_t)g.ny, (uint32_t)g.nx);
    const uint32_t plane = (uint32_t)g.nx * (uint32_t)g.ny;
    const uint32_t n0 = (uint32_t)y * (uint32_t)g.nx + hx;
    uint32_t own[3][3];  // in-plane cell of the nine columns a pull reads
#pragma unroll
    for (int cy = -1; cy <= 1; ++cy)
#pragma unroll
        for (int cx = -1; cx <= 1; ++cx) own[cy + 1][cx + 1] = n0 + back(ox, cx) + back(oy, cy);
    // storage index of canonical cell m: (m >> lb) q B + (m mod B) = m + (m >> lb) (q - 1) B
    const uint32_t gap = (uint32_t)(L::Q - 1) << g.lb;
    const auto plane_at = [&](int it) {
        const int z = r.z0 - 1 + it;
        return z < 0 ? z + g.nz : (z >= g.nz ? z - g.nz : z);
    };
    const __amdgpu_buffer_rsrc_t in = sweep::plane_rsrc(src + dm.base);
    const auto load = [&](int it, S *pre) {
        const int z = plane_at(it);
        const uint32_t p0 = (uint32_t)z * plane, pm = (uint32_t)(z == 0 ? g.nz - 1 : z - 1) * plane,
                       pp = (uint32_t)(z == g.nz - 1 ? 0 : z + 1) * plane;
#pragma unroll
        for (int j = 0; j < L::Q; ++j) {
            const int i = kPull.dir[j];
            const PairRow v = i == 0 ? PairRow{0, 0, 0} : L::pair((i - 1) / 2);
            const int sg = (i & 1) ? 1 : -1, cz = sg * v.cz;
            const uint32_t m = own[sg * v.cy + 1][sg * v.cx + 1] + (cz > 0 ? pm : (cz < 0 ? pp : p0));
            const uint32_t at = __umul24(m >> g.lb, gap) + m;
            pre[i] = sweep::ld_buf<S>(in, at * (uint32_t)sizeof(S), (uint32_t)(i << g.lb) * (uint32_t)sizeof(S));
        }
    };
    const auto store = [&](int it, const C *gp, const C *gm) {
        // a wave's cells start and end inside cache lines: cached stores in FP32 (512 domains 664 ->
        // 620 us per step), while FP64 is bound by the bytes (128 domains 293 us, 303 cached)
        constexpr int AUX = sizeof(S) == 4 ? 0 : 2;
        const uint32_t m = n0 + (uint32_t)plane_at(it - 1) * plane;
        const PlaneStores ps = plane_stores(dst + dm.base, g, Ref{0u, __umul24(m >> g.lb, gap) + m});
        st_plane_aux<AUX>(ps, 0, Conv<S>::st(gp[0]));
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            st_plane_aux<AUX>(ps, 2 * p + 1, Conv<S>::st(gp[p + 1]));
            st_plane_aux<AUX>(ps, 2 * p + 2, Conv<S>::st(gm[p + 1]));
        }
    };
    // neighbours in the tile: rows wrap in x, and in y where the tile holds all of them
    const int xm = hx == 0u ? g.nx - 1 : -1, xp = (int)hx == g.nx - 1 ? 1 - g.nx : 1;
    const int ym = whole && hy == 0 ? (g.ny - 1) * g.nx : -g.nx;
    const int yp = whole && hy == g.ny - 1 ? -(g.ny - 1) * g.nx : g.nx;
    const auto nbr = [&](int cx, int cy) { return (cx < 0 ? xm : (cx > 0 ? xp : 0)) + (cy < 0 ? ym : (cy > 0 ? yp : 0)); };
    sweep::planes<LAT, S, ORDER, kRegs<LAT, S>, COLS>(lds, (int)t, column, inner, r.z1 - r.z0 + 2, k, load, nbr, store);
}

template <typename F> auto by_kind(int lattice, int storage, F &&f)
{
    using D19 = std::integral_constant<int, kD3Q19>;
    using D27 = std::integral_constant<int, kD3Q27>;
    if (lattice == kD3Q19) return storage == kF64 ? f(D19{}, double{}) : f(D19{}, float{});
    return storage == kF64 ? f(D27{}, double{}) : f(D27{}, float{});
}

}  // namespace

int batch_sweep_columns(int lattice, int storage)
{
    if (lattice == kD2Q9 || (storage != kF32 && storage != kF64)) return 0;
    return by_kind(lattice, storage, [](auto lat, auto sv) { return sweep_cols<decltype(lat)::value, decltype(sv)>(); });
}

hipError_t launch_batch_sweep(int lattice, int storage, int order, uint32_t nrecs, const BatchSweepRec *recs,
                              const BatchDomain *doms, const StepConsts<double> *k64, const StepConsts<float> *k32,
                              const void *src, void *dst, hipStream_t stream)
{
    if (nrecs == 0) return hipSuccess;
    return by_kind(lattice, storage, [&](auto lat, auto sv) {
        using S = decltype(sv);
        constexpr int LAT = decltype(lat)::value;
        const StepConsts<typename Conv<S>::C> *kc;
        if constexpr (sizeof(S) == 8) kc = k64; else kc = k32;
        const dim3 block((sweep_cols<LAT, S>() + 63) / 64 * 64);
        if (order == 2)
            hipLaunchKernelGGL((k_batch_sweep<LAT, S, 2>), dim3(nrecs), block, 0, stream, (const S *)src, (S *)dst, recs,
                               doms, kc);
        else
            hipLaunchKernelGGL((k_batch_sweep<LAT, S, 3>), dim3(nrecs), block, 0, stream, (const S *)src, (S *)dst, recs,
                               doms, kc);
        return hipGetLastError();
    });
}

}  // namespace lbm

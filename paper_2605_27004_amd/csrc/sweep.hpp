// sweep.hpp -- the plane loop of the two-step sweeps (sweep.hip: one grid; batch_sweep.hip: a batch of
// domains): two steps of the periodic update on a tile of columns, walking up in z. What bounds it and
// why it is built so stands in sweep.hip.
#pragma once

#include <hip/hip_runtime.h>

#include "cell.hpp"
#include "common.hpp"

#pragma clang fp contract(off)

namespace lbm {
namespace sweep {

using namespace cell;

// Place in LDS of direction i among the directions with the same c_z; -1 for those that stay in
// their column (c_x = c_y = 0: rest, +z, -z), which their lane keeps.
template <int LAT> struct Ring {
    int slot[Lattice<LAT>::Q];
    int count[3];  // by c_z + 1
    constexpr Ring() : slot(), count()
    {
        for (int i = 0; i < Lattice<LAT>::Q; ++i) {
            const PairRow v = i == 0 ? PairRow{0, 0, 0} : Lattice<LAT>::pair((i - 1) / 2);
            slot[i] = (v.cx == 0 && v.cy == 0) ? -1 : count[((i & 1) ? v.cz : -v.cz) + 1]++;
        }
    }
};

constexpr int cz_of(PairRow v, int i) { return (i & 1) ? v.cz : -v.cz; }

// Raw buffer resource on a z-plane (the same for the whole work-group, see plane_stores): the q
// pulls of a cell then take nine lane offsets and a scalar offset per direction, with no address
// arithmetic per load.
template <typename S> __device__ inline __amdgpu_buffer_rsrc_t plane_rsrc(const S *p)
{
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint64_t u = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)) << 32) |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<S *>(u), (short)0, -1, 0x00020000);
}

template <typename S> __device__ inline S ld_buf(__amdgpu_buffer_rsrc_t r, uint32_t off, uint32_t soff)
{
    if constexpr (sizeof(S) == 4)
        return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, (int)soff, 0));
    else
        return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, (int)soff, 0));
}

// v[0] goes to the end, the others move down.
template <typename P, int N> __device__ inline void rotate(P *(&v)[N])
{
    P *f = v[0];
#pragma unroll
    for (int j = 0; j + 1 < N; ++j) v[j] = v[j + 1];
    v[N - 1] = f;
}

// Barrier that orders LDS only: the work-group's global loads and stores stay in flight across it.
__device__ inline void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS values per column of a tile: the planes of c_z = +1, 0 and -1 values that are kept.
template <int LAT, bool REGS> constexpr int ring_values()
{
    constexpr Ring<LAT> R{};
    return (REGS ? 2 : 3) * R.count[2] + 2 * R.count[1] + (REGS ? 2 : 1) * R.count[0];
}

// `count` planes, each once: the first step on every column of the tile, handed on through LDS, then
// the second step on the plane below where `inner` is set (from the third plane on).
//   lds: ring_values COLS elements; col: this lane's place among the COLS; column: it has one.
//   load(it, pre): issues the q pulls of plane `it` of this lane's column.
//   nbr(cx, cy): distance in LDS from this lane's column to the one at (+cx, +cy) (inner lanes only).
//   store(it, gp, gm): stores the second step's values, of plane it - 1.
// The second step of plane z needs the first step's values of planes z - 1 (c_z = +1), z (c_z = 0)
// and z + 1 (c_z = -1). REGS: each lane reads its neighbours' values as soon as a plane is there and
// keeps them in registers until their turn, so LDS holds one plane, twice (one barrier per plane);
// else LDS holds the planes until their turn (three, two and one of them, two barriers per plane),
// for FP64, whose registers would spill (505 against 570 us at D3Q19 256^3; FP32 the other way
// round, 265 against 285 us).
template <int LAT, typename S, int ORDER, bool REGS, int COLS, typename Load, typename Nbr, typename Store>
__device__ inline void planes(S *lds, const int col, const bool column, const bool inner, const int count,
                              const StepConsts<typename Conv<S>::C> &k, Load &&load, Nbr &&nbr, Store &&store)
{
    using L = Lattice<LAT>;
    using C = typename Conv<S>::C;
    constexpr int NP = L::NP;
    constexpr Ring<LAT> R{};
    constexpr int NU = REGS ? 2 : 3, NF = 2, ND = REGS ? 2 : 1;
    // LDS places of this column, [0] the plane read, the last one the plane written
    S *up[NU], *flat[NF], *down[ND];
    {
        S *p = lds + col;
#pragma unroll
        for (int j = 0; j < NU; ++j, p += R.count[2] * COLS) up[j] = p;
#pragma unroll
        for (int j = 0; j < NF; ++j, p += R.count[1] * COLS) flat[j] = p;
#pragma unroll
        for (int j = 0; j < ND; ++j, p += R.count[0] * COLS) down[j] = p;
    }
    S pre[L::Q];
    load(0, pre);
    // values waiting for their plane's second step: w1 one plane old (c_z = 0 and +1), w2 two (+1)
    C w1[L::Q], w2[L::Q];
#pragma unroll
    for (int i = 0; i < L::Q; ++i) w1[i] = w2[i] = C(0);
    for (int it = 0; it < count; ++it) {
        C gp[NP + 1], gm[NP + 1];
        gp[0] = Conv<S>::ld(pre[0]);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            gp[p + 1] = Conv<S>::ld(pre[2 * p + 1]);
            gm[p + 1] = Conv<S>::ld(pre[2 * p + 2]);
        }
        if (it + 1 < count) load(it + 1, pre);
        __builtin_amdgcn_sched_barrier(0);
        collide_cell<LAT, ORDER, false, C, kClose<S>>(k, gp, gm);
        C now[L::Q];
#pragma unroll
        for (int i = 0; i < L::Q; ++i) {
            const S val = Conv<S>::st(i == 0 ? gp[0] : ((i & 1) ? gp[(i - 1) / 2 + 1] : gm[(i - 1) / 2 + 1]));
            const int cz = i == 0 ? 0 : cz_of(L::pair((i - 1) / 2), i);
            if (R.slot[i] < 0)
                now[i] = Conv<S>::ld(val);
            else if (column)
                (cz > 0 ? up[NU - 1] : (cz == 0 ? flat[NF - 1] : down[ND - 1]))[R.slot[i] * COLS] = val;
        }
        lds_barrier();
        if (inner) {
            constexpr int RU = REGS ? NU - 1 : 0, RF = REGS ? NF - 1 : 0, RD = ND - 1;
#pragma unroll
            for (int i = 0; i < L::Q; ++i) {
                const PairRow v = i == 0 ? PairRow{0, 0, 0} : L::pair((i - 1) / 2);
                const int sg = (i & 1) ? 1 : -1, cz = sg * v.cz;
                if (R.slot[i] >= 0)
                    now[i] = Conv<S>::ld((cz > 0 ? up[RU] : (cz == 0 ? flat[RF] : down[RD]))
                                             [R.slot[i] * COLS + nbr(-sg * v.cx, -sg * v.cy)]);
            }
#pragma unroll
            for (int i = 0; i < L::Q; ++i) {
                const int cz = i == 0 ? 0 : cz_of(L::pair((i - 1) / 2), i);
                const bool wait = REGS || R.slot[i] < 0;
                const C val = !wait || cz < 0 ? now[i] : (cz == 0 ? w1[i] : w2[i]);
                if (wait && cz > 0) w2[i] = w1[i];
                if (wait && cz >= 0) w1[i] = now[i];
                if (i == 0) gp[0] = val;
                else if (i & 1) gp[(i - 1) / 2 + 1] = val;
                else gm[(i - 1) / 2 + 1] = val;
            }
            collide_cell<LAT, ORDER, false, C, kClose<S>>(k, gp, gm);
        }
        // the next plane's loads end here, before this plane's stores are issued
#pragma unroll
        for (int i = 0; i < L::Q; ++i) asm volatile("" : "+v"(pre[i]));
        if (it >= 2 && inner) store(it, gp, gm);
        if (!REGS) lds_barrier();
        rotate(up);
        rotate(flat);
        rotate(down);
    }
}

}  // namespace sweep
}  // namespace lbm

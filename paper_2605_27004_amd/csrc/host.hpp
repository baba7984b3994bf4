// host.hpp -- host-side helpers shared by the single-grid (capi.cpp) and batched (batch.cpp)
// parts of the C ABI: error reporting, parameter preparation and per-step constants.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <string>

#include "../../include/lbm.h"
#include "common.hpp"

namespace lbm {
namespace host {

constexpr double kCs2 = 1.0 / 3.0;

// Velocity set in the library's canonical order (rest, then +c / -c of each pair).
struct LatticeTable {
    int q, d, np;
    int c[kMaxQ][3];
    double w[kMaxQ];
    int opp[kMaxQ];
};

// Validated parameters with everything derived from them on the host.
struct Prepared {
    lbm_derived dv;
    LatticeTable lat;
    int d, q, bytes;
    uint32_t n;
};

// Message of the last failing call on this thread (lbm_last_error).
extern thread_local std::string g_last_error;

// Record a message for lbm_last_error and return `code`.
int fail(int code, const char *fmt, ...);
int fail_hip(hipError_t e, const char *what);

bool table_of(int lattice, LatticeTable &t);
int storage_bytes(int storage);

// Validate p and derive A^-1, K, omega, r_i and the shift; LBM_OK or a negative code.
int prepare(const lbm_params *p, Prepared &out);

// Kernel constants of one parameter set in arithmetic precision C.
template <typename C> StepConsts<C> consts_for(const lbm_params &p, const Prepared &pr);

// Target bytes of one direction plane of one block in the population layout (Grid): rows per
// block is the largest divisor of ny with rows * nx * bytes <= block_bytes(bytes), at least 1.
// Blocks of about this size keep a work-group's 2q population streams within one compact
// stretch of memory; measured on the D3Q19 256^3 step, 8 KiB was best for FP32 and FP16,
// 32 KiB for FP64.
constexpr int64_t block_bytes(int bytes) { return bytes == 8 ? 32768 : 8192; }

// Extents and population layout of an nx x ny x nz grid of q directions in `bytes`-byte
// storage (the caller has validated the sizes).
Grid grid_of(int64_t nx, int64_t ny, int64_t nz, int q, int bytes);

int64_t align256(int64_t b);
bool aligned256(const void *ptr);

// Whether the stream is being recorded into a graph.
bool recording(hipStream_t stream);

// Launches for n steps of at most `most` each: the fewest. While the stream is being recorded into a graph
// (and most > 1), as many as leave the state in the buffer that n launches of one step would, at most one
// more: a graph of an even number of steps can then be replayed, each replay going on from the state that the
// last one left.
int64_t launches_for(int64_t n, int64_t most, hipStream_t stream);
// Steps of the next launch when `left` steps are to be taken in `launches` of them.
inline int64_t steps_of_launch(int64_t left, int64_t launches) { return (left + launches - 1) / launches; }

// A place in pinned host memory, for the few totals that a call's last kernel writes and the call
// then waits for: a read-out takes one synchronisation that way, where a copy to pageable memory
// costs another 9 us (lbm_moments of a 64^2 grid 27.0 -> 18.7 us). The places come from one block for the
// whole process, allocated at the first use and kept: 16 of 32 KiB. Each belongs to one call at a
// time, from its construction to its end, so calls on other threads, streams and devices never
// share one. p is null when none is free or the totals are larger; the caller then copies.
// A place is given back only once the stream has been waited for: by wait(), or, where a call ends
// early because something failed, by the destructor, since a kernel enqueued before the failure may still
// write to it. If that wait fails too, the place stays taken.
class HostSlot {
public:
    HostSlot(size_t bytes, hipStream_t stream);
    ~HostSlot();
    HostSlot(const HostSlot &) = delete;
    HostSlot &operator=(const HostSlot &) = delete;
    hipError_t wait();  // for the stream, whether there is a place or not
    double *p;

private:
    hipStream_t stream_;
    int at_;
    bool waited_;
};

}  // namespace host
}  // namespace lbm

// The context behind the opaque lbm_ctx handle (host memory only; the device buffers belong to
// the caller).
struct lbm_ctx {
    lbm_params p;
    lbm::host::Prepared pr;
    lbm::Grid grid;
    lbm::StepConsts<double> k64;
    lbm::StepConsts<float> k32;
    void *pop[2];
    int cur;                 // index of the buffer that holds the current state
    double *partials;        // reduction partials, then the totals (in the caller's scratch)
    uint32_t *links;         // link words or row index (grid.nrec); null without a solid mask
    float *gray;             // null without a gray field
    hipStream_t stream;
    int64_t t;
    int block_x, block_y;    // of a launch of one step
    int launch_flags;        // kLaunchDefault until lbm_set_launch
    lbm::SweepPlan sweep;    // how steps are taken two at a time (tx = 0: they are not)
    lbm::TilePlan tile;      // how several steps of a D2Q9 grid go into one launch (shape -1: none do)
};

namespace lbm {
namespace host {

// lbm_moments with the reduction partials (kPartials * moments_groups doubles) and the totals
// (kPartials doubles) at the given device addresses. pinned: totals may come through a HostSlot.
int moments_with(lbm_ctx *c, double *rho, double *s, double *totals, double *partials, double *dtot, bool pinned);

}  // namespace host
}  // namespace lbm

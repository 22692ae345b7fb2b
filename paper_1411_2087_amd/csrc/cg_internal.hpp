// Solver state and helpers shared by the CG sources.
#pragma once

#include "dslash_core.hpp"

namespace hisq {

enum { CG_RUNNING = 0, CG_CONVERGED = 1, CG_BREAKDOWN = 2, CG_STALLED = 3 };

// Gate of the kernels of a solver iteration: closed when the solve is done
// or a reliable update is pending.  The iteration pauses there; the host
// runs the update outside the captured graph at its next state check and
// the iterations resume.
enum { GATE_PAUSE = 3 };
__device__ __forceinline__ bool paused(const SolverFlags &f) { return f.done || f.reliable; }
__device__ __forceinline__ bool solver_gate_closed(const SolverFlags *f, int gate)
{
    return gate == GATE_PAUSE ? paused(*f) : gate_closed(f, gate);
}
// Device-resident scalars of one solve.  `flags` comes first: kernels gate on it.
struct CGState {
    SolverFlags flags;
    int iter;        // iterations completed
    int nupdates;    // reliable updates done
    double tol2;     // tol^2
    double bb;       // |b|^2
    double stop2;    // tol^2 |b|^2
    double m4;       // 4 m^2
    double delta2;   // reliable-update threshold delta^2
    double rr;       // |r|^2 of the current iterate (inner residual in mixed modes)
    double rr_new;   // |r|^2 after the last update
    double rr_true;  // last FP64 true residual |b - A x|^2
    double maxrr;    // max |r_inner|^2 since the last reliable update
    double alpha, beta, pAp;
    // stagnation watch of the mixed solver (reliable updates that do not
    // reduce the true residual, or an inner solve that stops triggering them)
    double rr_upd;   // true |r|^2 at the last reliable update (or the start)
    int last_upd;    // iteration of the last reliable update
    int first_gap;   // iterations from the start to the first reliable update
    int poor;        // consecutive reliable updates that did not halve |r|
    int pending;     // the last iteration's |r|^2 partials are not in the state yet
};

// What a finished reduction, of value v, does to the state.
enum {
    FIN_BB = 0,           // bb = v ; stop2 = tol2 * bb
    FIN_PAP = 1,          // pAp = v ; alpha or breakdown
    FIN_UPD_PLAIN = 2,    // rr_new = v ; iter++ ; converged? ; beta ; rr
    FIN_UPD_MIXED = 3,    // as above, deciding reliable updates
    FIN_INIT_PLAIN = 4,   // rr = rr_true = v ; done = v <= stop2
    FIN_TRUE = 5,         // rr_true = v
    FIN_RELIABLE = 6,     // rr_true = v ; beta = v / rr ; rr = maxrr = v ; reliable = 0 ; done?
    FIN_INIT_MIXED = 7,   // rr = maxrr = rr_true = v ; done = v <= stop2
};

__device__ __forceinline__ void finalize(CGState *st, int mode, double v)
{
    switch (mode) {
    case FIN_BB:
        st->bb = v;
        st->stop2 = st->tol2 * v;
        break;
    case FIN_PAP:
        st->pAp = v;
        if (!(v > 0.0) || !isfinite(v)) {
            st->flags.done = CG_BREAKDOWN;
        } else {
            st->alpha = st->rr / v;
        }
        break;
    case FIN_UPD_PLAIN:
        st->rr_new = v;
        st->iter += 1;
        if (!isfinite(v)) {
            st->flags.done = CG_BREAKDOWN;
        } else if (v <= st->stop2) {
            st->flags.done = CG_CONVERGED;
            st->rr = v;
        } else {
            st->beta = v / st->rr;
            st->rr = v;
        }
        break;
    case FIN_UPD_MIXED:
        st->rr_new = v;
        st->iter += 1;
        if (!isfinite(v)) {
            st->flags.done = CG_BREAKDOWN;
        } else if (v <= st->stop2 || v < st->delta2 * st->maxrr) {
            st->flags.reliable = 1;
        } else {
            st->maxrr = fmax(st->maxrr, v);
            st->beta = v / st->rr;
            st->rr = v;
            // the inner solve has gone ten times as long as its first cycle without a reliable update
            if (st->first_gap > 0 && st->iter - st->last_upd > 10 * st->first_gap + 1000) st->flags.done = CG_STALLED;
        }
        break;
    case FIN_INIT_PLAIN:
        st->beta = 0.0;  // the first direction is p = r
        st->rr = v;
        st->rr_true = v;
        st->flags.done = (v <= st->stop2) ? CG_CONVERGED : 0;
        break;
    case FIN_TRUE:
        st->rr_true = v;
        break;
    case FIN_RELIABLE: {
        const int gap = st->iter - st->last_upd;
        if (st->first_gap == 0) st->first_gap = gap > 0 ? gap : 1;
        // poor: the true residual fell by less than sqrt(delta) since the last
        // update (an update fires after a fall by delta in the iterated residual),
        // or did not halve when delta is small
        st->poor = (v > fmax(0.25, sqrt(st->delta2)) * st->rr_upd) ? st->poor + 1 : 0;
        st->rr_upd = v;
        st->last_upd = st->iter;
        st->rr_true = v;
        st->nupdates += 1;
        st->beta = v / st->rr;
        st->rr = v;
        st->maxrr = v;
        st->flags.reliable = 0;
        if (!isfinite(v)) st->flags.done = CG_BREAKDOWN;
        else if (v <= st->stop2) st->flags.done = CG_CONVERGED;
        else if (st->poor >= 2) st->flags.done = CG_STALLED;  // the inner operator is too far from A
        break;
    }
    case FIN_INIT_MIXED:
        st->beta = 0.0;
        st->rr = v;
        st->maxrr = v;
        st->rr_true = v;
        st->rr_upd = v;
        st->last_upd = 0;
        st->first_gap = 0;
        st->poor = 0;
        st->flags.reliable = 0;
        st->flags.done = (v <= st->stop2) ? CG_CONVERGED : 0;
        break;
    }
}

// Scratch of the standalone dot product: the per-workgroup partials of the
// first stage (at most BLAS_MAX_BLOCKS workgroups, striding over the vectors)
// and the result.  dot_on launches the two stages on `s` and copies the
// result to out_host (synchronises `s`).
constexpr int BLAS_MAX_BLOCKS = 1024;
constexpr size_t DOT_PART_BYTES = 2 * sizeof(double) * BLAS_MAX_BLOCKS;
constexpr size_t DOT_WS_BYTES = DOT_PART_BYTES + 256;
int dot_on(const void *x, const void *y, long long n, int prec, double out_host[2], char *ws, hipStream_t s);

int blas_blocks(long long n);
size_t cg_partials_count(const Geom &g);
size_t cg_multi_workspace_bytes(const Geom &g, int nrhs, int mode);
size_t fcg_ws_bytes(const Geom &g, int channels);
size_t fat_paths_ws_bytes(const int dims[4]);  // links.hip
// Pinned host mirrors of the solvers' device states: one block per thread,
// allocated by the first solve on the thread and kept, so no solve allocates
// or frees pinned memory (hipHostFree would synchronise the device).  Slots:
// fcg_solve keeps its state live while its plain-CG fallback uses PIN_CG.
enum { PIN_CG = 0, PIN_MULTI = 1, PIN_FCG = 2, PIN_SLOTS = 3 };
constexpr size_t PIN_SLOT_BYTES = 16384;
void *pinned_slot(int slot);
inline CGState *pinned_state() { return (CGState *)pinned_slot(PIN_CG); }
hipStream_t capture_stream();
hisq_cg_opts resolve_opts(const hisq_cg_opts *opts, const Geom &g);

}  // namespace hisq

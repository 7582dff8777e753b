// State of the valid-ratio search (section 3.5.2).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace spamm {

// Thresholds tried per round: the next 15 multiples of the mean product while
// the upper bound grows, then the 15 midpoints that the next four bisection
// steps can reach.  A round costs its launch whatever it counts (one
// bisection per pair of norms and threshold), so more steps per round mean
// fewer rounds.
constexpr int kProbeDepth = 4;
constexpr int kProbeCands = (1 << kProbeDepth) - 1;
constexpr int kProbeStride = kProbeCands + 1;  // counts of one k, padded
constexpr int kMaxExpand = 1024;

struct SearchState {
    double ave, lo, hi, tau, ratio, target, tol, triples;
    int64_t kept;
    int32_t k, iters, max_iters, bisect, done;
};

// Threshold v = 1 .. kProbeCands of the round that follows state st: k ave for
// the next k, or the midpoint at node v of the bisection tree below [lo, hi]
// (node v's children are 2v, with hi, and 2v + 1, with lo, moved to v's midpoint).
__device__ inline double probe_tau(const SearchState& st, int v) {
    if (!st.bisect) return double(st.k + v) * st.ave;
    double lo = st.lo, hi = st.hi;
    for (int b = 30 - __builtin_clz(unsigned(v)); b >= 0; --b) {
        const double mid = 0.5 * (lo + hi);
        if ((v >> b) & 1)
            lo = mid;
        else
            hi = mid;
    }
    return 0.5 * (lo + hi);
}

// tau starts at ave; the upper bound k ave grows by ave while the ratio there
// is still above the target; then bisection in [0, k ave] until the ratio is
// within tol of the target or max_iters steps ran.
__device__ inline void search_advance(SearchState* st, const int32_t* counts) {
    if (st->done) return;
    if (!st->bisect) {
        for (int c = 0; c < kProbeCands && !st->bisect; ++c) {
            ++st->k;
            st->hi = double(st->k) * st->ave;
            st->kept = int64_t(counts[c]);
            st->ratio = double(st->kept) / st->triples;
            if (!(st->ratio > st->target + st->tol && st->k < kMaxExpand)) {
                st->bisect = 1;
                st->tau = st->hi;
                st->lo = 0.0;
                st->iters = 0;
            }
        }
        if (!st->bisect) return;
    } else {
        for (int v = 1; v <= kProbeCands;) {
            const double off = st->ratio - st->target;
            if (!((off < 0.0 ? -off : off) > st->tol && st->iters < st->max_iters)) break;
            const double mid = 0.5 * (st->lo + st->hi);
            st->kept = int64_t(counts[v - 1]);
            st->ratio = double(st->kept) / st->triples;
            st->tau = mid;
            ++st->iters;
            if (st->ratio > st->target) {
                st->lo = mid;
                v = 2 * v + 1;
            } else {
                st->hi = mid;
                v = 2 * v;
            }
        }
    }
    const double off = st->ratio - st->target;
    st->done = !((off < 0.0 ? -off : off) > st->tol && st->iters < st->max_iters);
}

// rows_b [bdim*bdim]: B's leaf norms, every row ascending; cols_a [bdim*bdim]:
// A's, transposed; ksums [bdim]: per k the sum of its products.  state (may be
// null): receives init.
hipError_t launch_norms_sort(const double* pyr_a, const double* pyr_b, int64_t bdim, int lv, double* rows_b,
                             double* cols_a, double* ksums, SearchState* state, const SearchState& init,
                             hipStream_t s);
// Round `round` (0, 1, ...) of the search after launch_norms_sort: states [2]
// and counts[2] (bdim * kProbeStride each) hold the state and the per-k counts
// of the even and odd rounds.
hipError_t launch_ratio_probe(const double* rows_b, const double* cols_a, const double* ksums, int64_t bdim,
                              SearchState* states, int32_t* const* counts, int round, hipStream_t s);
// The state after `rounds` rounds, into states[rounds & 1].
hipError_t launch_ratio_finish(int64_t bdim, SearchState* states, int32_t* const* counts, int rounds, hipStream_t s);

// One question and its answer per step of the search for an error target.
constexpr int kQueries = 3;
struct StepAnswer {
    double sumsq;               // of E at the threshold evaluated
    double least[kQueries];     // smallest norm product >= x[q], +inf if none
    double most;                // largest norm product, at least 0
    int64_t dropped;            // products added to E
    int64_t kept[kQueries];     // norm products >= x[q]
};
struct StepQuery {
    double x[kQueries];  // each > 0
    int count;
};
// partials: bdim entries of kQueryPartial doubles (launch_norms_sort's arrays
// as input); the sums and counts of launch_block_dropped over `blocks` blocks
// (0: none).  The answer is one StepAnswer in device memory.
constexpr int kQueryPartial = 2 * kQueries + 1;
hipError_t launch_norm_query(const double* rows_b, const double* cols_a, int64_t bdim, const StepQuery& q,
                             double* partials, hipStream_t s);
hipError_t launch_step_answer(const double* partials, int64_t bdim, int queries, const double* sums,
                              const int32_t* counts, int64_t blocks, StepAnswer* out, hipStream_t s);

}  // namespace spamm

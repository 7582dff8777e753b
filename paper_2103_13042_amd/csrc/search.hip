// Counting norm products against thresholds, for the threshold searches.
//
// The number of leaf triples with fl64(nA[i,k] * nB[k,j]) >= tau is wanted for
// one tau after another.  For a fixed nA[i,k] the rounded product does not
// fall when nB[k,j] grows, so with row k of B's norms sorted once the kept j of
// (i, k) are a suffix of the row, found by bisection with the very same
// comparison: bdim^2 log2(bdim) products per threshold instead of bdim^3, and
// the count is the same whole number.  norms_sort_kernel sorts the rows (and
// transposes A's norms, so that a block reads its column in one piece).
//
// Norms of infinity and NaN (inputs with infinities) keep the plan's meaning:
// a NaN product is not kept.  NaN norms of B are sorted as -1, below every
// norm, where the product is negative and never kept; a zero norm of A meets
// infinity only at the top of a row, where its product is NaN, and is counted
// on its own.
#include <hip/hip_runtime.h>

#include <cmath>

#include "internal.h"
#include "search.h"

namespace spamm {

namespace {
constexpr int kSortThreads = 256;
constexpr int kSortMax = 1024;  // tiles per side at most (SPAMM_MAX_BDIM)
constexpr int kProbeThreads = 256;

// sum over the block in a fixed order (every thread gets it)
__device__ __forceinline__ double block_total(double v, double* red) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double tot = 0.0;
    for (unsigned w = 0; w < blockDim.x / 64; ++w) tot += red[w];
    __syncthreads();
    return tot;
}

// The state of round `round` (into *st, shared): the state of the round before
// it advanced by that round's counts.  Every thread of the block calls it.
__device__ __forceinline__ void advance_state(const SearchState* states, const int32_t* before, int round, int bdim,
                                              SearchState* st) {
    __shared__ int32_t tally[kProbeStride][kProbeThreads / kProbeStride + 1];
    __shared__ int32_t counts[kProbeStride];
    const int tid = threadIdx.x;
    static_assert(sizeof(SearchState) % 8 == 0 && sizeof(SearchState) / 8 <= 64, "copied by one wave");
    if (tid < int(sizeof(SearchState) / 8))
        reinterpret_cast<uint64_t*>(st)[tid] =
            reinterpret_cast<const uint64_t*>(states + (round == 0 ? 0 : (round - 1) & 1))[tid];
    if (round > 0) {
        int32_t v = 0;
        for (int e = tid; e < bdim * kProbeStride; e += kProbeThreads) v += before[e];  // one threshold per thread
        tally[tid % kProbeStride][tid / kProbeStride] = v;
    }
    __syncthreads();
    if (round > 0 && tid < kProbeStride) {
        int32_t v = 0;
#pragma unroll
        for (int u = 0; u < kProbeThreads / kProbeStride; ++u) v += tally[tid][u];
        counts[tid] = v;
    }
    __syncthreads();
    if (round > 0 && tid == 0) search_advance(st, counts);
    __syncthreads();
}

// first index of the ascending row s[0 .. len) whose product with a is kept
// (len if none); step0 is the largest power of two <= len
__device__ __forceinline__ int first_kept(const double* s, int len, int step0, double a, double tau) {
    int idx = 0;
    for (int step = step0; step > 0; step >>= 1)
        if (idx + step <= len && !(a * s[idx + step - 1] >= tau)) idx += step;
    return idx;
}
}  // namespace

// Block k: row k of B's leaf norms in ascending order, column k of A's as a
// row, and the product of their sums (the sum of every product of this k).
__global__ __launch_bounds__(kSortThreads) void norms_sort_kernel(const double* __restrict__ la,
                                                                  const double* __restrict__ lb, int64_t side,
                                                                  int64_t bdim, double* __restrict__ rows_b,
                                                                  double* __restrict__ cols_a,
                                                                  double* __restrict__ ksums,
                                                                  SearchState* __restrict__ state, SearchState init) {
    __shared__ double s[kSortMax];
    __shared__ double red[kSortThreads / 64];
    const int64_t k = blockIdx.x;
    const int tid = threadIdx.x;
    if (k == 0 && state && tid == 0) *state = init;
    int p = 1;
    while (p < bdim) p <<= 1;
    double rb = 0.0, ca = 0.0;
    for (int j = tid; j < p; j += kSortThreads) {
        double v = -1.0;
        if (j < bdim) {
            const double x = lb[k * side + j];
            rb += x;
            v = x >= 0.0 ? x : -1.0;  // NaN sorts below every norm
        }
        s[j] = v;
    }
    for (int64_t i = tid; i < bdim; i += kSortThreads) {
        const double x = la[i * side + k];
        cols_a[k * bdim + i] = x;
        ca += x;
    }
    rb = block_total(rb, red);
    ca = block_total(ca, red);
    if (tid == 0) ksums[k] = ca * rb;
    // bitonic sort of p values
    for (int size = 2; size <= p; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int e = tid; e < p / 2; e += kSortThreads) {
                const int lo = 2 * e - (e & (stride - 1)), hi = lo + stride;
                const double x = s[lo], y = s[hi];
                if ((x > y) == ((lo & size) == 0)) {
                    s[lo] = y;
                    s[hi] = x;
                }
            }
            __syncthreads();
        }
    for (int j = tid; j < bdim; j += kSortThreads) rows_b[k * bdim + j] = s[p - int(bdim) + j];
}

// One round of the valid-ratio search: the counts at every threshold of the
// current state (probe_tau), per k.  Each block first brings the state up to
// date with the previous round's counts, the same steps in every block, so
// rounds follow each other on the stream with no host read in between, and a
// round after the search has ended returns at once.  The counts go to memory
// per k and are added by the readers (13 us a round at 256 tiles per side, 16
// with 15 counters that every block added to atomically).  N = 8192, leaf 32:
// nine thresholds took nine count and scan launches of 19 us with a host read
// after each, and 138 us for the mean; the search is now 450 -> 80 us.
__global__ __launch_bounds__(kProbeThreads) void ratio_probe_kernel(const double* __restrict__ rows_b,
                                                                    const double* __restrict__ cols_a,
                                                                    const double* __restrict__ ksums, int bdim,
                                                                    SearchState* __restrict__ states,
                                                                    const int32_t* __restrict__ before,
                                                                    int32_t* __restrict__ counts, int round) {
    __shared__ double s[kSortMax];
    __shared__ double red[kProbeThreads / 64];
    __shared__ SearchState st;
    __shared__ int tally[kProbeCands][kProbeThreads + 16];
    const int tid = threadIdx.x;
    const int64_t k = blockIdx.x;
    for (int j = tid; j < bdim; j += kProbeThreads) s[j] = rows_b[k * bdim + j];
    double ave = 0.0;
    if (round == 0) {  // mean product: the sums of every k in a fixed order
        double part = 0.0;
        for (int e = tid; e < bdim; e += kProbeThreads) part += ksums[e];
        ave = block_total(part, red) / (double(bdim) * double(bdim) * double(bdim));
    }
    advance_state(states, before, round, bdim, &st);
    if (round == 0) {
        if (tid == 0) st.ave = ave;
        __syncthreads();
    }
    // round 0 finds its state in states[0] and leaves the mean there; later
    // rounds write the slot that the round before last used
    if (k == 0 && tid == 0) {
        if (round == 0)
            states[0].ave = ave;
        else
            states[round & 1] = st;
    }
    if (st.done) return;
    double taus[kProbeCands];
#pragma unroll
    for (int c = 0; c < kProbeCands; ++c) taus[c] = probe_tau(st, c + 1);
    int step0 = 1;
    while (2 * step0 <= bdim) step0 *= 2;
    int cnt[kProbeCands];
#pragma unroll
    for (int c = 0; c < kProbeCands; ++c) cnt[c] = 0;
    for (int i = tid; i < bdim; i += kProbeThreads) {
        const double a = cols_a[k * bdim + i];
        if (a == 0.0) {  // the product is 0, or NaN against an infinite norm
            const int lo = first_kept(s, bdim, step0, 1.0, 0.0), hi = first_kept(s, bdim, step0, 1.0, INFINITY);
#pragma unroll
            for (int c = 0; c < kProbeCands; ++c) cnt[c] += 0.0 >= taus[c] ? hi - lo : 0;
            continue;
        }
        int idx[kProbeCands];
#pragma unroll
        for (int c = 0; c < kProbeCands; ++c) idx[c] = 0;
        for (int step = step0; step > 0; step >>= 1)
#pragma unroll
            for (int c = 0; c < kProbeCands; ++c) {
                const int at = idx[c] + step;
                if (at <= bdim && !(a * s[at - 1] >= taus[c])) idx[c] = at;
            }
#pragma unroll
        for (int c = 0; c < kProbeCands; ++c) cnt[c] += bdim - idx[c];
    }
#pragma unroll
    for (int c = 0; c < kProbeCands; ++c) tally[c][tid] = cnt[c];
    __syncthreads();
    // sixteen threads add one threshold's counts
    const int c = tid >> 4, l = tid & 15;
    int v = 0;
    if (c < kProbeCands) {
#pragma unroll
        for (int u = 0; u < kProbeThreads / 16; ++u) v += tally[c][l + 16 * u];
    }
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if (l == 0) counts[k * kProbeStride + c] = v;
}

__global__ __launch_bounds__(kProbeThreads) void ratio_finish_kernel(int bdim, SearchState* __restrict__ states,
                                                                     const int32_t* __restrict__ before, int rounds) {
    __shared__ SearchState st;
    advance_state(states, before, rounds, bdim, &st);
    if (threadIdx.x == 0) states[rounds & 1] = st;
}

// Block k: over the products of this k, per threshold x the smallest one >= x
// and how many there are, and the largest product.  x > 0, so a zero norm of A
// has no product to give (0, or NaN against infinity).
__global__ __launch_bounds__(kProbeThreads) void norm_query_kernel(const double* __restrict__ rows_b,
                                                                   const double* __restrict__ cols_a, int bdim,
                                                                   StepQuery q, double* __restrict__ partials) {
    __shared__ double s[kSortMax];
    __shared__ double red[kProbeThreads / 64][kQueryPartial];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t k = blockIdx.x;
    for (int j = tid; j < bdim; j += kProbeThreads) s[j] = rows_b[k * bdim + j];
    __syncthreads();
    int step0 = 1;
    while (2 * step0 <= bdim) step0 *= 2;
    double least[kQueries], most = 0.0, kept[kQueries];  // counts below 2^20 are exact in FP64
#pragma unroll
    for (int c = 0; c < kQueries; ++c) {
        least[c] = INFINITY;
        kept[c] = 0.0;
    }
    for (int i = tid; i < bdim; i += kProbeThreads) {
        const double a = cols_a[k * bdim + i];
        const double top = a * s[bdim - 1];
        if (top > most) most = top;
#pragma unroll
        for (int c = 0; c < kQueries; ++c) {
            if (c >= q.count) break;
            const int at = first_kept(s, bdim, step0, a, q.x[c]);
            if (at < bdim) {
                least[c] = fmin(least[c], a * s[at]);
                kept[c] += double(bdim - at);
            }
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        most = fmax(most, __shfl_xor(most, o));
#pragma unroll
        for (int c = 0; c < kQueries; ++c) {
            least[c] = fmin(least[c], __shfl_xor(least[c], o));
            kept[c] += __shfl_xor(kept[c], o);
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < kQueries; ++c) {
            red[tid >> 6][c] = least[c];
            red[tid >> 6][kQueries + c] = kept[c];
        }
        red[tid >> 6][2 * kQueries] = most;
    }
    __syncthreads();
    if (tid < kQueryPartial) {
        double v = red[0][tid];
        for (int w = 1; w < kProbeThreads / 64; ++w)
            v = tid < kQueries ? fmin(v, red[w][tid]) : tid < 2 * kQueries ? v + red[w][tid] : fmax(v, red[w][tid]);
        partials[k * kQueryPartial + tid] = v;
    }
}

// One block: the partials of a query and of an error evaluation, each in a
// fixed order.
__global__ __launch_bounds__(1024) void step_answer_kernel(const double* __restrict__ partials, int bdim, int queries,
                                                           const double* __restrict__ sums,
                                                           const int32_t* __restrict__ counts, int64_t blocks,
                                                           StepAnswer* __restrict__ out) {
    __shared__ double red[16][kQueryPartial + 1];
    __shared__ long long redn[16][kQueries + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double least[kQueries], most = 0.0, sq = 0.0;
    long long kept[kQueries], dropped = 0;
#pragma unroll
    for (int c = 0; c < kQueries; ++c) {
        least[c] = INFINITY;
        kept[c] = 0;
    }
    if (queries > 0)
        for (int k = tid; k < bdim; k += 1024) {
            const double* p = partials + int64_t(k) * kQueryPartial;
#pragma unroll
            for (int c = 0; c < kQueries; ++c) {
                least[c] = fmin(least[c], p[c]);
                kept[c] += static_cast<long long>(p[kQueries + c]);
            }
            most = fmax(most, p[2 * kQueries]);
        }
    for (int64_t b = tid; b < blocks; b += 1024) {
        sq += sums[b];
        dropped += counts[b];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        most = fmax(most, __shfl_xor(most, o));
        sq += __shfl_xor(sq, o);
        dropped += __shfl_xor(dropped, o);
#pragma unroll
        for (int c = 0; c < kQueries; ++c) {
            least[c] = fmin(least[c], __shfl_xor(least[c], o));
            kept[c] += __shfl_xor(kept[c], o);
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < kQueries; ++c) {
            red[wave][c] = least[c];
            redn[wave][c] = kept[c];
        }
        red[wave][kQueries] = most;
        red[wave][kQueries + 1] = sq;
        redn[wave][kQueries] = dropped;
    }
    __syncthreads();
    if (tid != 0) return;
    for (int w = 1; w < 16; ++w) {
        for (int c = 0; c < kQueries; ++c) {
            red[0][c] = fmin(red[0][c], red[w][c]);
            redn[0][c] += redn[w][c];
        }
        red[0][kQueries] = fmax(red[0][kQueries], red[w][kQueries]);
        red[0][kQueries + 1] += red[w][kQueries + 1];
        redn[0][kQueries] += redn[w][kQueries];
    }
    for (int c = 0; c < kQueries; ++c) {
        out->least[c] = red[0][c];
        out->kept[c] = redn[0][c];
    }
    out->most = red[0][kQueries];
    out->sumsq = red[0][kQueries + 1];
    out->dropped = redn[0][kQueries];
}

hipError_t launch_norm_query(const double* rows_b, const double* cols_a, int64_t bdim, const StepQuery& q,
                             double* partials, hipStream_t s) {
    if (q.count < 1 || q.count > kQueries || bdim < 1 || bdim > kSortMax) return hipErrorInvalidValue;
    norm_query_kernel<<<unsigned(bdim), kProbeThreads, 0, s>>>(rows_b, cols_a, int(bdim), q, partials);
    return hipGetLastError();
}

hipError_t launch_step_answer(const double* partials, int64_t bdim, int queries, const double* sums,
                              const int32_t* counts, int64_t blocks, StepAnswer* out, hipStream_t s) {
    step_answer_kernel<<<1, 1024, 0, s>>>(partials, int(bdim), queries, sums, counts, blocks, out);
    return hipGetLastError();
}

hipError_t launch_norms_sort(const double* pyr_a, const double* pyr_b, int64_t bdim, int lv, double* rows_b,
                             double* cols_a, double* ksums, SearchState* state, const SearchState& init,
                             hipStream_t s) {
    if (bdim < 1 || bdim > kSortMax) return hipErrorInvalidValue;
    const int64_t side = int64_t(1) << lv;
    norms_sort_kernel<<<unsigned(bdim), kSortThreads, 0, s>>>(pyr_a + level_offset(lv), pyr_b + level_offset(lv), side,
                                                              bdim, rows_b, cols_a, ksums, state, init);
    return hipGetLastError();
}

hipError_t launch_ratio_probe(const double* rows_b, const double* cols_a, const double* ksums, int64_t bdim,
                              SearchState* states, int32_t* const* counts, int round, hipStream_t s) {
    ratio_probe_kernel<<<unsigned(bdim), kProbeThreads, 0, s>>>(rows_b, cols_a, ksums, int(bdim), states,
                                                                counts[(round + 1) & 1], counts[round & 1], round);
    return hipGetLastError();
}

hipError_t launch_ratio_finish(int64_t bdim, SearchState* states, int32_t* const* counts, int rounds, hipStream_t s) {
    if (rounds < 1) return hipErrorInvalidValue;
    ratio_finish_kernel<<<1, kProbeThreads, 0, s>>>(int(bdim), states, counts[(rounds + 1) & 1], rounds);
    return hipGetLastError();
}

}  // namespace spamm

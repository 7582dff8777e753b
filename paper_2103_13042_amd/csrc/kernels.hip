// gfx950 kernels of the SpAMM hot path.
//
//   leaf_sumsq_*      Frobenius norms of every leaf tile (Eq. 2), FP64 sums
//   pyramid_kernel    quadtree of node norms (Eq. 1), bottom-up, FP64
//   plan_*            norm-product tests (Algorithm 1 / Algorithm 2's bitmap),
//                     ballot bitmaps, scan, compaction into ascending k-lists
//   (in multiply)     cost-balanced static partition of output tiles
//   multiply_kernel   FP32 MFMA products of the kept leaf pairs into C
//
// Wave size is 64 throughout.
#include <hip/hip_runtime.h>

#include "device.h"
#include "dma.h"
#include "internal.h"
#include "norms.h"

namespace spamm {

// --------------------------------------------------------------------------
// Leaf norms (norms.h).

// words the first block of a norm pass sets to zero (a pair counter, the
// look-back state of the plan that follows)
__device__ __forceinline__ void clear_words(const NormJob& job) {
    if (job.clear && (blockIdx.x | blockIdx.y | blockIdx.z) == 0) {
        const int64_t cnt = job.clear_count > 0 ? job.clear_count : 1;
        for (int64_t e = threadIdx.x; e < cnt; e += blockDim.x) job.clear[e] = 0;
    }
}

// Grid (strip, column chunk, matrix), strips fastest: blocks dispatched
// together read 4 KiB row segments of different strips (2 MiB apart at
// N = 8192), which streams faster than neighbouring chunks of one strip
// (N = 8192, A and B: 83 against 92 us).
template <int LEAF, bool VEC, bool NT>
__global__ __launch_bounds__(kNormThreads) void leaf_sumsq_kernel(NormJob job, int64_t n, int64_t bdim) {
    const int m = blockIdx.z;
    clear_words(job);
    leaf_sumsq_strip<LEAF, VEC, NT>(job.x[m], n, bdim, blockIdx.x, blockIdx.y, job.sumsq[m], job.norms[m], job.ld);
}

// Small matrices (too few strips to fill the GPU with the kernel above): 1024
// threads per strip x 1024-column chunk, four row groups of LEAF/4 rows whose
// loads are all in flight at once; the four partial sums of a column group
// are added in row-group order through LDS, then across the tile's threads.
// Rows at 4-byte alignment (VEC false, n >= 4) as in leaf_sumsq_strip.
constexpr int kNormSmallThreads = 1024;

template <int LEAF, bool VEC>
__global__ __launch_bounds__(kNormSmallThreads) void leaf_sumsq_small_kernel(NormJob job, int64_t n, int64_t bdim) {
    constexpr int G = LEAF / 4;           // threads per tile (4 columns each)
    constexpr int RPG = LEAF / 4;         // rows per row group
    __shared__ double part[3][kNormCols / 4];
    const int m = blockIdx.z;
    clear_words(job);
    const float* __restrict__ x = job.x[m];
    const int t = threadIdx.x, cg = t & 255, rg = t >> 8;
    const int64_t strip = blockIdx.y, col = int64_t(blockIdx.x) * kNormCols + 4 * cg;
    const int64_t r0 = strip * LEAF + rg * RPG;
    double acc = 0.0;
    if (col < n) {
        f4 v[RPG];
        const int back = VEC || col + 4 <= n ? 0 : int(col + 4 - n);  // columns that the thread before holds
#pragma unroll
        for (int r = 0; r < RPG; ++r) {
            const int64_t row = r0 + r;
            v[r] = row < n ? load_row<VEC, false>(x + row * n + col - back) : f4{0.0f, 0.0f, 0.0f, 0.0f};
            if (!VEC) {
                v[r].x = back > 0 ? 0.0f : v[r].x;
                v[r].y = back > 1 ? 0.0f : v[r].y;
                v[r].z = back > 2 ? 0.0f : v[r].z;
            }
        }
        double a0 = 0.0, a1 = 0.0;
#pragma unroll
        for (int r = 0; r < RPG; ++r) {
            a0 += double(v[r].x) * double(v[r].x) + double(v[r].y) * double(v[r].y);
            a1 += double(v[r].z) * double(v[r].z) + double(v[r].w) * double(v[r].w);
        }
        acc = a0 + a1;
    }
    if (rg > 0) part[rg - 1][cg] = acc;
    __syncthreads();
    if (rg != 0) return;
    double s = ((acc + part[0][cg]) + part[1][cg]) + part[2][cg];
#pragma unroll
    for (int off = 1; off < G; off <<= 1) s += __shfl_xor(s, off);
    const int64_t tj = col / LEAF;
    if ((cg % G) == 0 && col < n && tj < bdim) {
        const int64_t i = strip * job.ld + tj;
        if (job.sumsq[m]) job.sumsq[m][i] = s;
        if (job.norms[m]) job.norms[m][i] = sqrt(s);
    }
}

// Any other leaf size: one block per tile, strided over its elements.
__global__ __launch_bounds__(kNormThreads) void leaf_sumsq_generic_kernel(NormJob job, int64_t n, int64_t bdim,
                                                                          int32_t leaf) {
    __shared__ double partial[kNormThreads / 64];
    const int m = blockIdx.z;
    clear_words(job);
    const float* __restrict__ x = job.x[m];
    const int64_t ti = blockIdx.y, tj = blockIdx.x;
    const int64_t rows = (ti * leaf + leaf < n ? leaf : n - ti * leaf);
    const int64_t cols = (tj * leaf + leaf < n ? leaf : n - tj * leaf);
    double acc = 0.0;
    for (int64_t e = threadIdx.x; e < rows * cols; e += kNormThreads) {
        const int64_t r = ti * leaf + e / cols, c = tj * leaf + e % cols;
        const double v = double(x[r * n + c]);
        acc += v * v;
    }
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) partial[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < kNormThreads / 64; ++w) s += partial[w];
        const int64_t t = ti * job.ld + tj;
        if (job.sumsq[m]) job.sumsq[m][t] = s;
        if (job.norms[m]) job.norms[m][t] = sqrt(s);
    }
}

constexpr double kInfinityCacheBytes = 256.0 * 1024 * 1024;  // MI355X's last-level cache
constexpr int64_t kSmallNormBlocks = 256;                      // one block per CU

template <int LEAF>
static hipError_t launch_leaf_fixed(const NormJob& job, int nmat, int64_t n, int64_t bdim, bool vec,
                                    hipStream_t s) {
    dim3 grid(unsigned((n + kNormCols - 1) / kNormCols), unsigned(bdim), unsigned(nmat));
    const bool nt = 4.0 * double(n) * double(n) * nmat > kInfinityCacheBytes;
    if constexpr (LEAF == 16 || LEAF == 32 || LEAF == 64) {
        // fewer blocks than CUs: the four-row-group form keeps more loads in flight
        if (n >= 4 && int64_t(grid.x) * grid.y * grid.z < kSmallNormBlocks) {
            if (vec)
                leaf_sumsq_small_kernel<LEAF, true><<<grid, kNormSmallThreads, 0, s>>>(job, n, bdim);
            else
                leaf_sumsq_small_kernel<LEAF, false><<<grid, kNormSmallThreads, 0, s>>>(job, n, bdim);
            return hipGetLastError();
        }
    }
    const dim3 sgrid(grid.y, grid.x, grid.z);  // strips fastest
    if (vec && nt)
        leaf_sumsq_kernel<LEAF, true, true><<<sgrid, kNormThreads, 0, s>>>(job, n, bdim);
    else if (vec)
        leaf_sumsq_kernel<LEAF, true, false><<<sgrid, kNormThreads, 0, s>>>(job, n, bdim);
    else if (nt)
        leaf_sumsq_kernel<LEAF, false, true><<<sgrid, kNormThreads, 0, s>>>(job, n, bdim);
    else
        leaf_sumsq_kernel<LEAF, false, false><<<sgrid, kNormThreads, 0, s>>>(job, n, bdim);
    return hipGetLastError();
}

hipError_t launch_leaf_norms(const NormJob& job, int nmat, int64_t n, int32_t leaf, bool vec, hipStream_t s) {
    const int64_t bdim = (n + leaf - 1) / leaf;
    switch (leaf) {
        case 16: return launch_leaf_fixed<16>(job, nmat, n, bdim, vec, s);
        case 32: return launch_leaf_fixed<32>(job, nmat, n, bdim, vec, s);
        case 64: return launch_leaf_fixed<64>(job, nmat, n, bdim, vec, s);
        case 128: return launch_leaf_fixed<128>(job, nmat, n, bdim, vec, s);
        case 256: return launch_leaf_fixed<256>(job, nmat, n, bdim, vec, s);
        default: break;
    }
    dim3 grid{unsigned(bdim), unsigned(bdim), unsigned(nmat)};
    leaf_sumsq_generic_kernel<<<grid, kNormThreads, 0, s>>>(job, n, bdim, leaf);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Pyramid.  One block per matrix walks the levels bottom-up.  A parent's
// sum of squares is (s00 + s01) + (s10 + s11) of its children: sums of
// non-negative FP64 values round monotonically, so a parent is never below any
// child, and neither is its square root.  That is what lets the plan drop a
// whole range of k on a parent's test without ever dropping a pair that the
// leaf test keeps.

constexpr int kPyrThreads = 1024;
constexpr int kPyrLdsTop = 6;                        // highest level kept in LDS
constexpr int kPyrLdsLevel = 1 << (2 * kPyrLdsTop);  // its node count

__device__ __forceinline__ void pyramid_build(double* __restrict__ sp, double* __restrict__ np, int64_t bdim,
                                              int lv) {
    const int64_t side = int64_t(1) << lv;
    if (bdim < side) {  // padding tiles of the leaf level: norm 0
        const int64_t base = level_offset(lv);
        for (int64_t idx = threadIdx.x; idx < side * side; idx += kPyrThreads) {
            const int64_t i = idx >> lv, j = idx & (side - 1);
            if (i >= bdim || j >= bdim) {
                sp[base + idx] = 0.0;
                np[base + idx] = 0.0;
            }
        }
    }
    // levels of at most kPyrLdsLevel nodes (l <= 6) are also kept in LDS, in
    // buffer l & 1, so the levels above the first such one read their children
    // there instead of waiting on the global writes of the level below
    __shared__ double lvl0[kPyrLdsLevel];      // levels 6, 4, 2, 0
    __shared__ double lvl1[kPyrLdsLevel / 4];  // levels 5, 3, 1
    for (int l = lv - 1; l >= 0; --l) {
        __syncthreads();
        const int64_t w = int64_t(1) << l, cw = 2 * w;
        const int64_t base = level_offset(l), cbase = level_offset(l + 1);
        // the leaf level (l + 1 == lv) is only in global memory
        const bool from_lds = l + 1 <= kPyrLdsTop && l + 1 < lv, to_lds = l <= kPyrLdsTop;
        const double* src = from_lds ? ((l + 1) & 1 ? lvl1 : lvl0) : sp + cbase;
        double* dst = (l & 1) ? lvl1 : lvl0;
#pragma unroll 4
        for (int64_t idx = threadIdx.x; idx < w * w; idx += kPyrThreads) {
            const int64_t i = idx >> l, j = idx & (w - 1);
            const double* c0 = src + (2 * i) * cw + 2 * j;
            const double* c1 = c0 + cw;
            const double v = (c0[0] + c0[1]) + (c1[0] + c1[1]);
            sp[base + idx] = v;
            np[base + idx] = sqrt(v);
            if (to_lds) dst[idx] = v;
        }
    }
}

__global__ __launch_bounds__(kPyrThreads) void pyramid_kernel(PyramidJob job, int64_t bdim, int lv, const int32_t* run) {
    if (closed(run)) return;
    pyramid_build(job.spyr[blockIdx.x], job.pyr[blockIdx.x], bdim, lv);
}

// The six levels above the leaves under one node of level lv - 6 (blockIdx.x,
// row-major), and the padding of its 64 x 64 leaves: the same sums as
// pyramid_build's.
constexpr int kSubtree = 6;

__global__ __launch_bounds__(kPyrThreads) void pyramid_subtree_kernel(PyramidJob job, int64_t bdim, int lv,
                                                                      const int32_t* run) {
    if (closed(run)) return;
    double* __restrict__ sp = job.spyr[blockIdx.y];
    double* __restrict__ np = job.pyr[blockIdx.y];
    const int64_t top = int64_t(1) << (lv - kSubtree), side = int64_t(1) << lv;
    const int64_t bi = blockIdx.x / top, bj = blockIdx.x % top;
    __shared__ double lvl[2][32 * 32];
    {   // 32 x 32 nodes of level lv - 1, one per thread, from its four leaves
        const int i = threadIdx.x >> 5, j = threadIdx.x & 31;
        const int64_t li = bi * 64 + 2 * i, lj = bj * 64 + 2 * j, leaves = level_offset(lv);
        double c[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const int64_t at = leaves + (li + u) * side + lj + v;
                if (li + u < bdim && lj + v < bdim) {
                    c[u][v] = sp[at];
                } else {
                    c[u][v] = 0.0;
                    sp[at] = 0.0;
                    np[at] = 0.0;
                }
            }
        const double s = (c[0][0] + c[0][1]) + (c[1][0] + c[1][1]);
        const int64_t at = level_offset(lv - 1) + (bi * 32 + i) * (side >> 1) + bj * 32 + j;
        sp[at] = s;
        np[at] = sqrt(s);
        lvl[0][threadIdx.x] = s;
    }
#pragma unroll
    for (int d = 2; d <= kSubtree; ++d) {
        __syncthreads();
        const int w = 64 >> d;  // nodes per side of level lv - d
        const double* src = lvl[d & 1];
        if (int(threadIdx.x) < w * w) {
            const int i = threadIdx.x / w, j = threadIdx.x % w;
            const double* c0 = src + 2 * i * 2 * w + 2 * j;
            const double* c1 = c0 + 2 * w;
            const double s = (c0[0] + c0[1]) + (c1[0] + c1[1]);
            const int64_t at = level_offset(lv - d) + (bi * w + i) * (side >> d) + bj * w + j;
            sp[at] = s;
            np[at] = sqrt(s);
            lvl[(d + 1) & 1][threadIdx.x] = s;
        }
    }
}

// From 128 leaves a side (rounded up) on the lower levels by subtrees, then the
// levels above by one block per matrix.  One block alone is bound by its own
// reads and writes: 9 us at 128 a side, 18 at 256, 95 at 512 with 256 of them
// padding, 197 at 1024; the two launches take 6, 9, 9 and 10.
constexpr int kSubtreeMinLevels = 7;

hipError_t launch_pyramid(const PyramidJob& job, int nmat, int64_t bdim, int lv, hipStream_t s, const int32_t* run) {
    if (lv < kSubtreeMinLevels) {
        pyramid_kernel<<<nmat, kPyrThreads, 0, s>>>(job, bdim, lv, run);
        return hipGetLastError();
    }
    const int above = lv - kSubtree;
    pyramid_subtree_kernel<<<dim3{1u << (2 * above), unsigned(nmat), 1u}, kPyrThreads, 0, s>>>(job, bdim, lv, run);
    pyramid_kernel<<<nmat, kPyrThreads, 0, s>>>(job, int64_t(1) << above, above, run);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Plan.  Block (jb, i) owns the 64 output tiles (i, 64*jb .. 64*jb+63) and
// walks k in chunks of 64.  A chunk is one pyramid node of 64 x 64 leaf tiles
// (level Lv-6) on each side; when that node product is below tau every leaf
// product in the chunk is too (a node norm bounds the norms below it), so the
// chunk is settled for all 64 tiles at once (uniform branch).  Otherwise the
// chunk's 64 x 64 block of B leaf norms is staged in LDS, each lane takes one
// k, and one ballot per tile gives the 64-bit bitmap of selected k.

constexpr int kPlanThreads = 256;

template <bool MASKS>
__device__ __forceinline__ void plan_mask_block(const double* __restrict__ pyr_a, const double* __restrict__ pyr_b,
                                                int64_t bdim, int lv, double tau, uint64_t* __restrict__ masks,
                                                int32_t* __restrict__ counts, int32_t* __restrict__ block_sums,
                                                int64_t jb, int64_t i) {
    __shared__ double sb[64][65];
    __shared__ int wsum[kPlanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t j0 = jb * 64;
    const int64_t side = int64_t(1) << lv;
    const int nw = int((bdim + 63) / 64);
    const double* la = pyr_a + level_offset(lv);
    const double* lb = pyr_b + level_offset(lv);
    int cnt[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) cnt[u] = 0;
    for (int c = 0; c < nw; ++c) {
        bool below;
        if (lv >= 6) {
            const int lc = lv - 6;
            const int64_t w = int64_t(1) << lc;
            below = !(pyr_a[level_offset(lc) + (i >> 6) * w + c] * pyr_b[level_offset(lc) + int64_t(c) * w + (j0 >> 6)] >=
                      tau);
        } else {
            below = !(pyr_a[0] * pyr_b[0] >= tau);
        }
        if (below) {
            if (MASKS && lane == 0) {
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const int64_t j = j0 + wave + 4 * u;
                    if (j < bdim) masks[(i * bdim + j) * nw + c] = 0;
                }
            }
            continue;
        }
        // stage the chunk's 64 x 64 B norms: all loads first, then the LDS writes
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int e = threadIdx.x + u * kPlanThreads;
            const int64_t k = int64_t(c) * 64 + (e >> 6), j = j0 + (e & 63);
            v[u] = (k < side && j < side) ? lb[k * side + j] : 0.0;
        }
        const int64_t k = int64_t(c) * 64 + lane;
        const double a = k < side ? la[i * side + k] : 0.0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int e = threadIdx.x + u * kPlanThreads;
            sb[e >> 6][e & 63] = v[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int jj = wave + 4 * u;
            const int64_t j = j0 + jj;
            const double p = a * sb[lane][jj];
            const bool bit = p >= tau && k < bdim && j < bdim;
            const uint64_t mk = __ballot(bit);
            if (MASKS && lane == 0 && j < bdim) masks[(i * bdim + j) * nw + c] = mk;
            cnt[u] += __popcll(mk);
        }
    }
    int tot = 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int64_t j = j0 + wave + 4 * u;
        if (j < bdim) {
            if (MASKS && lane == 0) counts[i * bdim + j] = cnt[u];
            tot += cnt[u];
        }
    }
    if (lane == 0) wsum[wave] = tot;
    __syncthreads();
    if (threadIdx.x == 0) block_sums[i * nw + jb] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

template <bool MASKS>
__global__ __launch_bounds__(kPlanThreads) void plan_mask_kernel(const double* __restrict__ pyr_a,
                                                                 const double* __restrict__ pyr_b, int64_t bdim,
                                                                 int lv, double tau, uint64_t* __restrict__ masks,
                                                                 int32_t* __restrict__ counts,
                                                                 int32_t* __restrict__ block_sums,
                                                                 const int32_t* run) {
    if (closed(run)) return;
    plan_mask_block<MASKS>(pyr_a, pyr_b, bdim, lv, tau, masks, counts, block_sums, blockIdx.x, blockIdx.y);
}

hipError_t launch_plan_mask(const double* pyr_a, const double* pyr_b, int64_t bdim, int lv, double tau,
                            uint64_t* masks, int32_t* counts, int32_t* block_sums, hipStream_t s,
                            const int32_t* run) {
    dim3 grid{unsigned((bdim + 63) / 64), unsigned(bdim), 1u};
    plan_mask_kernel<true><<<grid, kPlanThreads, 0, s>>>(pyr_a, pyr_b, bdim, lv, tau, masks, counts, block_sums, run);
    return hipGetLastError();
}

hipError_t launch_plan_count(const double* pyr_a, const double* pyr_b, int64_t bdim, int lv, double tau,
                             int32_t* block_sums, hipStream_t s) {
    dim3 grid{unsigned((bdim + 63) / 64), unsigned(bdim), 1u};
    plan_mask_kernel<false><<<grid, kPlanThreads, 0, s>>>(pyr_a, pyr_b, bdim, lv, tau, nullptr, nullptr, block_sums,
                                                          nullptr);
    return hipGetLastError();
}

// Exclusive scan of the block sums (one per 64 output tiles): one block, each
// thread a contiguous segment, wave scans with shuffles, then across waves.
constexpr int kScanThreads = 256;

__device__ __forceinline__ void plan_scan_block(const int32_t* __restrict__ block_sums, int64_t nb,
                                                int32_t* block_offsets, int32_t* offsets, int64_t nt,
                                                int64_t* __restrict__ pairs) {
    __shared__ int64_t wsum[kScanThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t seg = (nb + kScanThreads - 1) / kScanThreads;
    const int64_t b = tid * seg, e = (b + seg < nb ? b + seg : nb);
    int64_t local = 0;
    for (int64_t t = b; t < e; ++t) local += block_sums[t];
    int64_t incl = local;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int64_t run = incl - local;
    for (int w = 0; w < wave; ++w) run += wsum[w];
    if (block_offsets) {
        for (int64_t t = b; t < e; ++t) {
            block_offsets[t] = int32_t(run);
            run += block_sums[t];
        }
    }
    if (tid == kScanThreads - 1) {
        int64_t total = 0;
        for (int w = 0; w < kScanThreads / 64; ++w) total += wsum[w];
        if (offsets) offsets[nt] = int32_t(total);
        if (pairs) *pairs = total;
    }
}

__global__ __launch_bounds__(kScanThreads) void plan_scan_kernel(const int32_t* __restrict__ block_sums,
                                                                 int64_t nb, int32_t* block_offsets,
                                                                 int32_t* offsets, int64_t nt,
                                                                 int64_t* __restrict__ pairs, const int32_t* run) {
    if (closed(run)) return;
    plan_scan_block(block_sums, nb, block_offsets, offsets, nt, pairs);
}

hipError_t launch_plan_scan(const int32_t* block_sums, int64_t nblocks, int32_t* block_offsets, int32_t* offsets,
                            int64_t ntiles, int64_t* pairs, hipStream_t s, const int32_t* run) {
    plan_scan_kernel<<<1, kScanThreads, 0, s>>>(block_sums, nblocks, block_offsets, offsets, ntiles, pairs, run);
    return hipGetLastError();
}

// One wave per output tile t = (i, j): its offset is the offset of its block
// of 64 tiles plus the counts of the tiles before it in the block (a masked
// wave sum); then every lane whose bit is set writes its k at the offset plus
// the number of set bits below it (ascending k).
__device__ __forceinline__ void plan_fill_wave(const uint64_t* __restrict__ masks, const int32_t* __restrict__ counts,
                                               const int32_t* __restrict__ block_offsets, int64_t bdim,
                                               int32_t* __restrict__ offsets, int32_t* __restrict__ klist,
                                               int64_t t) {
    const int lane = threadIdx.x & 63;
    const int nw = int((bdim + 63) / 64);
    const int64_t i = t / bdim, j = t % bdim, jb = j >> 6;
    const int64_t jl = (jb * 64 + lane < bdim) ? jb * 64 + lane : -1;  // the block's tile for this lane
    int before = (jl >= 0 && (jl & 63) < (j & 63)) ? counts[i * bdim + jl] : 0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) before += __shfl_xor(before, off);
    int64_t base = int64_t(block_offsets[i * nw + jb]) + before;
    if (lane == 0) offsets[t] = int32_t(base);
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int w = 0; w < nw; ++w) {
        const uint64_t m = masks[t * nw + w];
        if ((m >> lane) & 1ull) klist[base + __popcll(m & below)] = w * 64 + lane;
        base += __popcll(m);
    }
}

__global__ __launch_bounds__(256) void plan_fill_kernel(const uint64_t* __restrict__ masks,
                                                        const int32_t* __restrict__ counts,
                                                        const int32_t* __restrict__ block_offsets, int64_t bdim,
                                                        int32_t* __restrict__ offsets, int32_t* __restrict__ klist,
                                                        const int32_t* run) {
    if (closed(run)) return;
    const int64_t t = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (t >= bdim * bdim) return;
    plan_fill_wave(masks, counts, block_offsets, bdim, offsets, klist, t);
}

hipError_t launch_plan_fill(const uint64_t* masks, const int32_t* counts, const int32_t* block_offsets,
                            int64_t bdim, int32_t* offsets, int32_t* klist, hipStream_t s, const int32_t* run) {
    const int64_t nt = bdim * bdim;
    plan_fill_kernel<<<unsigned((nt + 3) / 4), 256, 0, s>>>(masks, counts, block_offsets, bdim, offsets, klist, run);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// Multiply.
//
// A persistent grid of G workgroups (4 waves each).  Output tiles t = i*bdim+j
// are split into G contiguous row-major ranges of equal cost, where a tile
// costs kPairCost per kept pair plus one for writing it; the cost prefix is
// kPairCost*offsets[t] + t, so each group finds its range by binary search in
// the plan offsets.  Block ids are remapped so the groups on one XCD (ids
// congruent mod 8) own neighbouring ranges and share A/B tiles in that XCD's
// L2.
//
// A group first writes its pairs as packed (ti << 20 | tj << 10 | k) words into
// pair_scratch and streams them through a 128-entry LDS ring, refilled 64 at a
// time right after a stage commit (when no tile load is in flight), so the
// tile-load prefetch never waits on an index load.  The flat stream of (pair, k-chunk)
// items then runs through two register sets and two LDS stages: while the four
// waves multiply item it out of LDS, item it+1 sits in registers waiting to be
// stored to the other stage and the global loads of item it+2 are in flight.
// Tile loads are unconditional (out-of-range lanes read a valid address and
// select zero) so the wait before storing item it+1 leaves item it+2's loads
// outstanding.  Wave w computes
// the (w>>1, w&1) quadrant of the output tile with FP32 MFMA (32x32x2).
// In MFMA step s, lane
// group g takes k = g*(KC/G) + s, so a lane reads 4 consecutive A operands
// with one 16-byte LDS load; B rows are XOR-swizzled by lane group so the G
// groups read disjoint LDS banks.  Tiles are finished in ascending k and written
// from the accumulators; tiles without pairs are written as zeros.

constexpr int kMulThreads = 256;
constexpr int kPairCost = 4;
constexpr int kIdxBits = 10;  // packed pair = ti << 20 | tj << 10 | k  (all < 1024)
constexpr int32_t kIdxMask = (1 << kIdxBits) - 1;
constexpr int kRing = 512;  // packed pairs held in LDS (a power of two)

// Tile shapes per leaf: MFMA edge, k per pipeline stage, workgroups per CU.
template <int LEAF>
struct MulCfg;
template <>
struct MulCfg<128> {
    // one workgroup per CU: at two (256 registers per lane) the kernel spilled
    // to scratch, also with 16 k per stage
    static constexpr int MF = 32, KC = 32, OCC = 1;
};

template <int LEAF>
struct MulGeom {
    static constexpr int MF = MulCfg<LEAF>::MF;   // MFMA output edge
    static constexpr int KC = MulCfg<LEAF>::KC;   // k per pipeline stage
    static constexpr int QM = LEAF / 2;           // quadrant edge per wave
    static constexpr int NB = QM / MF;            // MFMA blocks per quadrant side
    static constexpr int G = 64 / MF;             // lane groups along k
    static constexpr int SPC = KC / G;            // MFMA steps per stage
    static constexpr int NCH = LEAF / KC;         // stages per leaf pair
    static constexpr int AST = KC + 4;            // A stage row stride (floats)
    static constexpr int BST = LEAF < 64 ? 64 : LEAF;  // B stage row stride (room for the swizzle)
    static constexpr int SWZ = 64 / G;            // B column swizzle unit
    static constexpr int ASZ = LEAF * AST;
    static constexpr int BSZ = KC * BST;
    static constexpr int STAGE = ASZ + BSZ;
    static constexpr int NV = LEAF * KC / 4 / kMulThreads;  // float4 per thread per operand
    static constexpr int ACC = (MF == 32 ? 16 : 4);         // accumulator floats per MFMA block
    static_assert(SPC % 4 == 0, "A reads are 4 steps wide");
    static_assert(NV >= 1 && NV * 4 * kMulThreads == LEAF * KC, "stage split");
};

template <int MF>
struct Mfma;
template <>
struct Mfma<32> {
    typedef f16v acc_t;
    static __device__ __forceinline__ acc_t step(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    // output element of accumulator register r for lane l: row, col in block
    static __device__ __forceinline__ int row(int r, int l) { return 8 * (r >> 2) + 4 * (l >> 5) + (r & 3); }
    static __device__ __forceinline__ int col(int, int l) { return l & 31; }
};
// First tile of logical group g: smallest t with (kPairCost*off[t] + t) * G >= g * total.
__device__ __forceinline__ int64_t partition_start(const int32_t* __restrict__ off, int64_t nt, int64_t g,
                                                   int64_t groups, int64_t total) {
    const int64_t target = g * total;
    int64_t lo = 0, hi = nt;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t(kPairCost) * off[mid] + mid) * groups >= target)
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// The multiply of the output tiles [t_begin, t_end) of one product, by one
// workgroup: lds holds the two staging buffers, ring the pair ring.
template <int LEAF, bool VEC>
__device__ __forceinline__ void mul_range(const float* __restrict__ A, const float* __restrict__ B,
                                          float* __restrict__ C, int64_t n, int64_t bdim,
                                          const int32_t* __restrict__ off, const int32_t* __restrict__ klist,
                                          int32_t* pairs, int64_t t_begin, int64_t t_end, float* lds,
                                          int32_t* ring) {
    using Gm = MulGeom<LEAF>;
    using M = Mfma<Gm::MF>;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wr = wave >> 1, wc = wave & 1;
    const int ir = lane % Gm::MF, g = lane / Gm::MF;
    const int64_t q_begin = off[t_begin], q_end = off[t_end];
    const int64_t nitems = (q_end - q_begin) * Gm::NCH;

    // packed (ti, tj, k) of every pair of the range
    for (int64_t q = q_begin + tid; q < q_end; q += kMulThreads) {
        int64_t lo = t_begin, hi = t_end - 1;  // tile of q: last t with off[t] <= q
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) >> 1;
            if (off[mid] <= q)
                lo = mid;
            else
                hi = mid - 1;
        }
        const int32_t ti = int32_t(lo / bdim), tj = int32_t(lo - int64_t(ti) * bdim);
        pairs[q] = (ti << (2 * kIdxBits)) | (tj << kIdxBits) | klist[q];
    }
    __syncthreads();
    const int64_t npairs = q_end - q_begin;
    for (int e = tid; e < kRing; e += kMulThreads) ring[e] = e < npairs ? pairs[q_begin + e] : 0;
    __syncthreads();
    int64_t rbase = 0;  // ring holds pairs [rbase, rbase + kRing)
    auto pk_of_item = [&](int64_t it) -> int32_t { return ring[(it / Gm::NCH) & (kRing - 1)]; };

    typename M::acc_t acc[Gm::NB][Gm::NB];
    auto zero_acc = [&]() {
#pragma unroll
        for (int a = 0; a < Gm::NB; ++a)
#pragma unroll
            for (int b = 0; b < Gm::NB; ++b)
#pragma unroll
                for (int r = 0; r < Gm::ACC; ++r) acc[a][b][r] = 0.0f;
    };
    auto store_tile = [&](int32_t ti, int32_t tj) {
#pragma unroll
        for (int a = 0; a < Gm::NB; ++a)
#pragma unroll
            for (int b = 0; b < Gm::NB; ++b)
#pragma unroll
                for (int r = 0; r < Gm::ACC; ++r) {
                    const int64_t row = int64_t(ti) * LEAF + wr * Gm::QM + a * Gm::MF + M::row(r, lane);
                    const int64_t col = int64_t(tj) * LEAF + wc * Gm::QM + b * Gm::MF + M::col(r, lane);
                    if (row < n && col < n) C[row * n + col] = acc[a][b][r];
                }
    };

    // global -> register staging of one (pair, chunk) item; every lane issues
    // every load (clamped to a valid address) and zeroes what lies outside C.
    // Rows that are not 16-byte aligned (VEC false) are read with 16-byte
    // loads at 4-byte alignment, which global loads accept; only chunks that
    // cross the matrix's edge are read element by element
    auto fetch = [&](int32_t pk, int ch, f4 (&ra)[Gm::NV], f4 (&rb)[Gm::NV]) {
        const int64_t ti = (uint32_t(pk) >> (2 * kIdxBits)) & kIdxMask, tj = (uint32_t(pk) >> kIdxBits) & kIdxMask,
                      kt = uint32_t(pk) & kIdxMask;
        const int64_t arow0 = ti * LEAF, acol0 = kt * LEAF + ch * Gm::KC;
        const int64_t brow0 = kt * LEAF + ch * Gm::KC, bcol0 = tj * LEAF;
        const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int v = 0; v < Gm::NV; ++v) {
            const int e = tid + v * kMulThreads;
            {
                const int r = e / (Gm::KC / 4), c4 = e % (Gm::KC / 4);
                const int64_t row = arow0 + r, col = acol0 + 4 * c4;
                if (VEC) {
                    const bool in = row < n && col < n;
                    const f4 x = *reinterpret_cast<const f4*>(A + (in ? row * n + col : 0));
                    ra[v] = in ? x : zero;
                } else if (row < n && col + 3 < n) {  // 4-byte aligned: one 16-byte load
                    ra[v] = *reinterpret_cast<const f4_dw*>(A + row * n + col);
                } else {
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const bool in = row < n && col + q4 < n;
                        const float x = A[in ? row * n + col + q4 : 0];
                        ra[v][q4] = in ? x : 0.0f;
                    }
                }
            }
            {
                const int r = e / (LEAF / 4), c4 = e % (LEAF / 4);
                const int64_t row = brow0 + r, col = bcol0 + 4 * c4;
                if (VEC) {
                    const bool in = row < n && col < n;
                    const f4 x = *reinterpret_cast<const f4*>(B + (in ? row * n + col : 0));
                    rb[v] = in ? x : zero;
                } else if (row < n && col + 3 < n) {
                    rb[v] = *reinterpret_cast<const f4_dw*>(B + row * n + col);
                } else {
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const bool in = row < n && col + q4 < n;
                        const float x = B[in ? row * n + col + q4 : 0];
                        rb[v][q4] = in ? x : 0.0f;
                    }
                }
            }
        }
    };
    auto commit = [&](int stage, const f4 (&ra)[Gm::NV], const f4 (&rb)[Gm::NV]) {
        float* sa = lds + stage * Gm::STAGE;
        float* sb = sa + Gm::ASZ;
#pragma unroll
        for (int v = 0; v < Gm::NV; ++v) {
            const int e = tid + v * kMulThreads;
            {
                const int r = e / (Gm::KC / 4), c4 = e % (Gm::KC / 4);
                *reinterpret_cast<f4*>(sa + r * Gm::AST + 4 * c4) = ra[v];
            }
            {
                const int r = e / (LEAF / 4), c4 = e % (LEAF / 4);
                const int swz = ((r / Gm::SPC) % Gm::G) * Gm::SWZ;
                *reinterpret_cast<f4*>(sb + r * Gm::BST + ((4 * c4) ^ swz)) = rb[v];
            }
        }
    };
    auto compute = [&](int stage) {
        const float* sa = lds + stage * Gm::STAGE;
        const float* sb = sa + Gm::ASZ + g * Gm::SPC * Gm::BST;
        const int swz = g * Gm::SWZ;
#pragma unroll
        for (int q = 0; q < Gm::SPC / 4; ++q) {
            f4 av[Gm::NB];
#pragma unroll
            for (int a = 0; a < Gm::NB; ++a)
                av[a] = *reinterpret_cast<const f4*>(sa + (wr * Gm::QM + a * Gm::MF + ir) * Gm::AST + g * Gm::SPC +
                                                     4 * q);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int s = 4 * q + u;
                float bv[Gm::NB];
#pragma unroll
                for (int b = 0; b < Gm::NB; ++b)
                    bv[b] = sb[s * Gm::BST + ((wc * Gm::QM + b * Gm::MF + ir) ^ swz)];
#pragma unroll
                for (int a = 0; a < Gm::NB; ++a)
#pragma unroll
                    for (int b = 0; b < Gm::NB; ++b) acc[a][b] = M::step(av[a][u], bv[b], acc[a][b]);
            }
        }
    };

    // output tile being accumulated: linear index t, coordinates (ti, tj);
    // tiles before it are written
    int64_t t = t_begin;
    int32_t ti = int32_t(t_begin / bdim), tj = int32_t(t_begin - int64_t(ti) * bdim);
    auto advance_tile = [&]() {
        store_tile(ti, tj);
        zero_acc();
        ++t;
        if (++tj == bdim) {
            tj = 0;
            ++ti;
        }
    };
    // one item of the stream: R_free receives item it+2, R_next (item it+1)
    // goes to LDS after the multiply of item it
    f4 ra0[Gm::NV], rb0[Gm::NV], ra1[Gm::NV], rb1[Gm::NV];
    auto step = [&](int64_t it, f4 (&fa)[Gm::NV], f4 (&fb)[Gm::NV], const f4 (&na)[Gm::NV],
                    const f4 (&nb)[Gm::NV]) {
        const int32_t pk = pk_of_item(it);
        const int64_t t_it =
            int64_t((uint32_t(pk) >> (2 * kIdxBits)) & kIdxMask) * bdim + ((uint32_t(pk) >> kIdxBits) & kIdxMask);
        while (t < t_it) advance_tile();  // tile t is complete (or has no pairs)
        const int64_t i2 = it + 2 < nitems ? it + 2 : nitems - 1;  // past the end: a harmless reload
        fetch(pk_of_item(i2), int(i2 % Gm::NCH), fa, fb);
        __syncthreads();
        compute(int(it & 1));
        if (it + 1 < nitems) commit(int((it + 1) & 1), na, nb);
        // every wave is past pair (it+1)/NCH - 1: recycle the older half of the ring
        if ((it + 1) / Gm::NCH >= rbase + kRing / 2) {
            for (int e = tid; e < kRing / 2; e += kMulThreads) {
                const int64_t p = rbase + kRing + e;
                ring[(rbase + e) & (kRing - 1)] = p < npairs ? pairs[q_begin + p] : 0;
            }
            rbase += kRing / 2;
        }
    };
    zero_acc();
    if (nitems > 0) {
        fetch(pk_of_item(0), 0, ra0, rb0);
        const int64_t i1 = nitems > 1 ? 1 : 0;
        fetch(pk_of_item(i1), int(i1 % Gm::NCH), ra1, rb1);
        commit(0, ra0, rb0);
    }
    for (int64_t it = 0; it < nitems; it += 2) {
        step(it, ra0, rb0, ra1, rb1);
        if (it + 1 >= nitems) break;
        step(it + 1, ra1, rb1, ra0, rb0);
    }
    while (t < t_end) advance_tile();
}


template <int LEAF, bool VEC>
__global__ __launch_bounds__(kMulThreads, MulCfg<LEAF>::OCC) void multiply_kernel(const float* __restrict__ A,
                                                                  const float* __restrict__ B, float* __restrict__ C,
                                                                  int64_t n, int64_t bdim,
                                                                  const int32_t* __restrict__ off,
                                                                  const int32_t* __restrict__ klist,
                                                                  int32_t* pairs) {
    __shared__ __attribute__((aligned(16))) float lds[2 * MulGeom<LEAF>::STAGE];
    __shared__ int32_t ring[kRing];
    // this group's range of output tiles
    const int64_t groups = gridDim.x;
    const int64_t bid = blockIdx.x;
    const int64_t lg = (bid & 7) * (groups >> 3) + (bid >> 3);
    const int64_t nt = bdim * bdim;
    const int64_t total = int64_t(kPairCost) * off[nt] + nt;
    const int64_t t_begin = partition_start(off, nt, lg, groups, total);
    const int64_t t_end = partition_start(off, nt, lg + 1, groups, total);
    if (t_begin >= t_end) return;
    mul_range<LEAF, VEC>(A, B, C, n, bdim, off, klist, pairs, t_begin, t_end, lds, ring);
}

template <int LEAF>
static hipError_t launch_mul(const float* a, const float* b, float* c, int64_t n, int64_t bdim,
                             const int32_t* offsets, const int32_t* klist, int32_t* pair_scratch, bool vec,
                             int num_cus, hipStream_t s) {
    const int64_t nt = bdim * bdim;
    int64_t groups = int64_t(num_cus) * MulCfg<LEAF>::OCC;
    const int64_t cap = ((nt + 7) / 8) * 8;
    if (groups > cap) groups = cap;
    groups = ((groups + 7) / 8) * 8;
    static int scratch_state[2] = {0, 0};
    const hipError_t ce = vec ? check_no_scratch(multiply_kernel<LEAF, true>, &scratch_state[1])
                              : check_no_scratch(multiply_kernel<LEAF, false>, &scratch_state[0]);
    if (ce != hipSuccess) return ce;
    if (vec)
        multiply_kernel<LEAF, true>
            <<<unsigned(groups), kMulThreads, 0, s>>>(a, b, c, n, bdim, offsets, klist, pair_scratch);
    else
        multiply_kernel<LEAF, false>
            <<<unsigned(groups), kMulThreads, 0, s>>>(a, b, c, n, bdim, offsets, klist, pair_scratch);
    return hipGetLastError();
}

hipError_t launch_multiply(const float* a, const float* b, float* c, int64_t n, int32_t leaf, int64_t bdim,
                           const int32_t* offsets, const int32_t* klist, int32_t* pair_scratch, bool vec,
                           int num_cus, hipStream_t s) {
    switch (leaf) {
        case 16: return launch_multiply_leaf16(a, b, c, n, bdim, offsets, klist, vec, s);
        case 128: return launch_mul<128>(a, b, c, n, bdim, offsets, klist, pair_scratch, vec, num_cus, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace spamm

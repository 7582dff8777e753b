// Batched products: two stages over all products of a batch, the leaf norms and
// the multiply of 64x64 blocks that test their own products (one launch per
// leaf class present), with the single-product device code.  A workgroup finds
// its product by a 64-ary search over the prefix of the stage's work, one read
// per lane; a binary search is a chain of reads as long as a small block's work.
// Products are taken largest first, so that the longest blocks start early.
//
// A batch of 48 products (n log-uniform in 256 .. 4096, exp decay, leaf 64): 577
// us with plan, cost and fill launches and the products in persistent
// single-tile ranges, 418 so.
#include <hip/hip_runtime.h>

#include "block_multiply.h"
#include "device.h"
#include "internal.h"
#include "norms.h"

namespace spamm {

namespace {
// the last p with base[p] <= x (base ascending, base[0] = 0); the whole wave
// calls it with the same x
__device__ __forceinline__ int batch_find(const int64_t* __restrict__ base, int count, int64_t x) {
    const int lane = threadIdx.x & 63;
    int lo = 0, len = count;
    while (len > 1) {
        const int step = (len + 63) / 64, at = lo + step * lane;
        const bool le = at < lo + len && base[at] <= x;
        const int cnt = __popcll(__ballot(le));  // monotone: lanes 0 .. cnt - 1
        const int end = lo + len;
        lo += step * (cnt - 1);
        len = end - lo < step ? end - lo : step;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

template <int LEAF, bool NT>
__device__ __forceinline__ void batch_strip(const float* x, double* norms, int64_t n, int64_t bdim, bool vec,
                                            int64_t b) {
    if (vec)
        leaf_sumsq_strip<LEAF, true, NT>(x, n, bdim, b % bdim, b / bdim, nullptr, norms, bdim);
    else
        leaf_sumsq_strip<LEAF, false, NT>(x, n, bdim, b % bdim, b / bdim, nullptr, norms, bdim);
}
}  // namespace

// One block per (tile row, 1024-column chunk) of A (blockIdx.y = 0) or B (1),
// tile rows fastest (as leaf_sumsq_kernel); a product's first block clears its
// pair counter.  NT: inputs of kBatchStreamBytes and more are read past the
// last-level cache, whose lines the multiply then finds free for its own reads
// and C (the 48 products of 1 GB in all: 460 -> 418 us a run; of 260 MB, which
// stay cached, 139 us against 148).
constexpr double kBatchStreamBytes = 512.0 * 1024 * 1024;

template <bool NT>
__global__ __launch_bounds__(kNormThreads) void batch_norms_kernel(const BatchProduct* __restrict__ P,
                                                                   const int64_t* __restrict__ strip_base, int count) {
    const int64_t bg = blockIdx.x;
    const int p = batch_find(strip_base, count, bg);
    const BatchProduct q = P[p];
    const int64_t b = bg - strip_base[p];
    const bool second = blockIdx.y != 0;
    if (b == 0 && !second && threadIdx.x == 0) *global_ptr(q.pairs) = 0;
    const float* x = global_ptr(second ? q.b : q.a);
    double* norms = global_ptr(second ? q.norms[1] : q.norms[0]);
    switch (q.leaf) {
        case 32: batch_strip<32, NT>(x, norms, q.n, q.bdim, q.vec != 0, b); break;
        case 64: batch_strip<64, NT>(x, norms, q.n, q.bdim, q.vec != 0, b); break;
        default: batch_strip<128, NT>(x, norms, q.n, q.bdim, q.vec != 0, b); break;
    }
}

// Products [0, count) of one leaf class, block_base their first blocks.  Two
// stages of operand tiles up to so many blocks (kTwoStageMaxN's reasons; 24
// products of 499 .. 1996, 6,700 blocks: 146 against 147 us, 48 of 256 .. 4096,
// 33,000 blocks: 475 against 462).
constexpr int64_t kTwoStageMaxBlocks = 8192;

template <int LEAF, int STAGES>
__global__ __launch_bounds__(kBlockThreads, block_occ(STAGES)) void multiply_batch_kernel(
    const BatchProduct* __restrict__ P, const int64_t* __restrict__ block_base, int count) {
    const int p = batch_find(block_base, count, blockIdx.x);
    const BatchProduct q = P[p];
    block_multiply<LEAF, kKept, STAGES>(global_ptr(q.a), global_ptr(q.b), global_ptr(q.c), q.n, int(q.bdim),
                                int((q.n + 63) / 64), global_ptr(q.norms[0]), global_ptr(q.norms[1]), q.bdim, q.tau,
                                reinterpret_cast<unsigned long long*>(global_ptr(q.pairs)), nullptr, nullptr,
                                BandJob{}, int(blockIdx.x - block_base[p]));
}

int64_t batch_strips(int64_t n, int64_t bdim) { return bdim * ((n + kNormCols - 1) / kNormCols); }

// A product of few block rows, all of them left over by block_at's strips, takes
// its blocks in launch order: it needs no more workgroups than blocks (4096
// products of n = 48, rounded up to one workgroup per XCD: 8 workgroups for 1
// block, 277 us against 66).  A class's products go from the largest to the
// smallest, so every product of whole strips still starts at a multiple of 8.
int64_t batch_blocks(int64_t n) {
    const int nb = int((n + 63) / 64);
    return dealt_rows(nb, kBlockOrder.H) == 0 ? int64_t(nb) * nb : block_grid(nb, kBlockOrder);
}

namespace {
template <int LEAF>
hipError_t launch_class(const BatchProduct* p, const int64_t* base, int32_t members, int64_t blocks, hipStream_t s) {
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    const bool two = blocks <= kTwoStageMaxBlocks;
    static int scratch_state[2] = {0, 0};
    const hipError_t e = two ? check_no_scratch(multiply_batch_kernel<LEAF, 2>, &scratch_state[1])
                             : check_no_scratch(multiply_batch_kernel<LEAF, 1>, &scratch_state[0]);
    if (e != hipSuccess) return e;
    if (two)
        multiply_batch_kernel<LEAF, 2><<<unsigned(blocks), kBlockThreads, 0, s>>>(p, base, members);
    else
        multiply_batch_kernel<LEAF, 1><<<unsigned(blocks), kBlockThreads, 0, s>>>(p, base, members);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_batch(const BatchProduct* prods, const int64_t* strip_base, const int64_t* block_base,
                        const int32_t* class_count, const int64_t* class_blocks, int64_t strips, double bytes,
                        int32_t count, hipStream_t s) {
    if (strips < 1 || strips > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid{unsigned(strips), 2u, 1u};
    if (bytes > kBatchStreamBytes)
        batch_norms_kernel<true><<<grid, kNormThreads, 0, s>>>(prods, strip_base, count);
    else
        batch_norms_kernel<false><<<grid, kNormThreads, 0, s>>>(prods, strip_base, count);
    hipError_t e = hipGetLastError();
    int32_t first = 0;
    for (int cls = 0; cls < kBatchClasses && e == hipSuccess; ++cls) {
        const int32_t members = class_count[cls];
        if (members == 0) continue;
        const BatchProduct* p = prods + first;
        const int64_t* base = block_base + first;
        e = cls == 0   ? launch_class<32>(p, base, members, class_blocks[cls], s)
            : cls == 1 ? launch_class<64>(p, base, members, class_blocks[cls], s)
                       : launch_class<128>(p, base, members, class_blocks[cls], s);
        first += members;
    }
    return e;
}

}  // namespace spamm

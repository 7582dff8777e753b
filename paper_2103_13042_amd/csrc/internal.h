// Internal interface between the host C-ABI (api.hip) and the gfx950 kernels
// (kernels.hip).  Not installed; the public interface is include/spamm.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace spamm {

// Level l of a norm pyramid starts at entry (4^l - 1) / 3 (levels 0..Lv).
__host__ __device__ inline int64_t level_offset(int l) { return ((int64_t(1) << (2 * l)) - 1) / 3; }

// Up to two matrices are processed by one launch of the norm and pyramid
// kernels (A and B of one product).
struct NormJob {
    const float* x[2];
    double* sumsq[2];     // leaf sums of squares, row stride ld, or null
    double* norms[2];     // leaf norms, row stride ld, or null
    int64_t ld;           // row stride of the outputs (bdim, or the padded pyramid side)
    int64_t* clear;       // device int64 words set to zero by the launch, or null
    int64_t clear_count;  // how many (1 when clear is set and this is 0)
};

// The leaf level of both pyramids is written by the norm pass (stride = side);
// the pyramid kernel zeroes its padding tiles and builds the levels above.
struct PyramidJob {
    double* spyr[2];  // [pyramid] sums of squares at every level (scratch)
    double* pyr[2];   // [pyramid] norms at every level (output)
};

// Norm pass: leaf sums of squares / norms of nmat matrices.
hipError_t launch_leaf_norms(const NormJob& job, int nmat, int64_t n, int32_t leaf, bool vec, hipStream_t s);

// Here and below, run: the launch does something only if *run (device memory) is
// not zero; null: always.

// Pyramid: bottom-up quadtree of sums of squares and norms for nmat matrices.
hipError_t launch_pyramid(const PyramidJob& job, int nmat, int64_t bdim, int lv, hipStream_t s,
                          const int32_t* run = nullptr);

// Plan: per output tile, the ballot bitmap of kept k (words of 64) and its
// count V; per block of 64 tiles (i, 64*jb ..) the sum of V (block b = i*nw + jb).
hipError_t launch_plan_mask(const double* pyr_a, const double* pyr_b, int64_t bdim, int lv, double tau,
                            uint64_t* masks, int32_t* counts, int32_t* block_sums, hipStream_t s,
                            const int32_t* run = nullptr);
// Plan counts only (no bitmaps): per block of 64 tiles the number of kept triples.
hipError_t launch_plan_count(const double* pyr_a, const double* pyr_b, int64_t bdim, int lv, double tau,
                             int32_t* block_sums, hipStream_t s);
// Plan: exclusive scan of the block sums into block_offsets; the total goes to
// offsets[T] and *pairs.  Each of the three outputs may be null; block_offsets
// and offsets may be the same array (they are written at disjoint indices).
hipError_t launch_plan_scan(const int32_t* block_sums, int64_t nblocks, int32_t* block_offsets, int32_t* offsets,
                            int64_t ntiles, int64_t* pairs, hipStream_t s, const int32_t* run = nullptr);
// Plan: per tile offset (block offset + prefix inside the block) and the
// compaction of its bitmap into an ascending k-list.
hipError_t launch_plan_fill(const uint64_t* masks, const int32_t* counts, const int32_t* block_offsets,
                            int64_t bdim, int32_t* offsets, int32_t* klist, hipStream_t s,
                            const int32_t* run = nullptr);

// Plan and macro-tile schedule in one launch (plan_macro.hip; leaf 32 and 64,
// bdim <= kPlanMacroMaxBdim): the outputs of launch_plan_mask +
// launch_plan_scan + launch_plan_fill (offsets, klist, pairs) and of
// launch_macro_schedule (uprefix, items); flags (mb words, mb = ceil(bdim /
// 2)) and the ticket after them must be zero before the launch
// (plan_macro_clear_words(bdim) words from flags).
constexpr int64_t kPlanMacroMaxBdim = 256;
struct PlanMacroOut {
    int32_t* offsets;
    int32_t* klist;
    int64_t* pairs;  // may be null
    int32_t* uprefix;
    uint32_t* items;
    unsigned long long* flags;
    unsigned int* ticket;
    const int32_t* run;
};
inline int64_t plan_macro_clear_words(int64_t bdim) { return (bdim + 1) / 2 + 1; }
// norms_a, norms_b: the leaf norms (row stride side); the pyramid above the
// leaf level is not used
hipError_t launch_plan_macro(const double* norms_a, const double* norms_b, int64_t side, int64_t bdim, double tau,
                             const PlanMacroOut& o, hipStream_t s);

// Small products, n <= kTileMaxN at leaf 32, 64 and 128 (multiply_tile.hip), n <=
// kSmallMaxN at leaf 16 (multiply_small.hip): the threshold test on the leaf
// norms na / nb (row stride ld) and the multiply of the kept pairs in one
// launch; adds the number of kept pairs to *pairs, which must be zero before
// (the norm pass clears it).  vec: n % 4 == 0 and a, b 16-byte aligned.
// kTileMaxN: a 32x32 tile of C per workgroup against a 64x64 block (one call,
// exp decay 0.05 and 0.01, tau 1e-6, leaf 32: n = 352 12.1 and 12.1 us against 16.0
// and 16.1; 1000 16.4 and 31.8 against 20.5 and 37.2; 1920 27.6 and 123 against 31
// and 138; 2047 30.7 and 167 against 31.5 and 142; leaf 64 and 128 alike).
constexpr int64_t kTileMaxN = 1920;
constexpr int64_t kSmallMaxN = 320;
hipError_t launch_tile_multiply(const float* a, const float* b, float* c, int64_t n, int32_t leaf, const double* na,
                                const double* nb, int64_t ld, double tau, int64_t* pairs, hipStream_t s);
hipError_t launch_small_multiply16(const float* a, const float* b, float* c, int64_t n, bool vec, int64_t bdim,
                                   const double* na, const double* nb, int64_t ld, double tau, int64_t* pairs,
                                   hipStream_t s);

// One 64x64 block of C per workgroup (multiply_block.hip).  test: the
// block tests the leaf norms itself, as launch_tile_multiply (*pairs zero
// before).  plan32: leaf 32, the items and prefix of a plan's macro-tile
// schedule.
//
// block_product: where the one-call path takes it or, at small n, the kernels
// above.  Leaf 16 and 32: any n (to the tile grid's 1024 per side).  Leaf 64 and
// 128 against the general path's plan, 128x128 macro tiles and fixup, which are two
// launches and their work list more, but read half the operands and share the
// work evenly, where blocks come in rounds of five a CU whose last is part empty.
// Measured on one call, leaf 64, exp decay 0.05, 0.01 and 0.005 (leaf 128 alike):
//  n <= 2048: blocks (2048: 32, 145, 152 us against 48, 144, 149);
//  to 3968, a multiple of 128: macro tiles (2560: 55, 213, 279 against 43, 237, 322;
//    3584: 69, 354, 647 against 65, 380, 718): the blocks gain on narrow bands, but
//    lose up to a third on wide ones (2688, decay 0.0065: 301 against 397);
//  to 5120: blocks (4096: 62, 467, 943 against 78, 428, 890; 5120: 96, 616, 1547
//    against 119, 584, 1448), but at leaf 128, whose macro tiles have no idle quarter,
//    they stay at multiples of 128 (4096: 94, 487, 920 against 81, 533, 1002, a tenth of the
//    tiles at random 173 against 200);
//  to 5120, ragged n: blocks, macro tiles at the edge cost more (2500: 43, 237, 321
//    against 57, 226, 294; 3001: 46, 325, 471 against 66, 296, 449).
constexpr int64_t kBlockCoarseFullN = 2048, kBlockCoarseRoundsN = 4096, kBlockCoarseMaxN = 5120;
inline bool block_product(int64_t n, int32_t leaf) {
    if (leaf == 16 || leaf == 32) return true;
    if (leaf != 64 && leaf != 128) return false;
    return n <= kBlockCoarseFullN ||
           (n <= kBlockCoarseMaxN && (n % 128 != 0 || (leaf == 64 && n >= kBlockCoarseRoundsN)));
}
hipError_t launch_block_test(const float* a, const float* b, float* c, int64_t n, int32_t leaf, int64_t bdim,
                             const double* na, const double* nb, int64_t ld, double tau, int64_t* pairs,
                             hipStream_t s);
hipError_t launch_block_plan32(const float* a, const float* b, float* c, int64_t n, int64_t bdim,
                               const uint32_t* items, const int32_t* uprefix, hipStream_t s);
// dropped: e plus the products dropped at tau (norm product not >= tau) but not
// at band.base; per block of C the FP64 sum of squares of the result and the
// number of products added.  Without a base e counts as zero and every
// product dropped at tau is added.
struct BandJob {
    double base = 0.0;
    int has_base = 0;
    int store = 0;              // whether e receives the result
    double* sums = nullptr;     // [ceil(n / 64)^2]
    int32_t* counts = nullptr;  // [ceil(n / 64)^2]
};
hipError_t launch_block_dropped(const float* a, const float* b, float* e, int64_t n, int32_t leaf, int64_t bdim,
                                const double* na, const double* nb, int64_t ld, double tau, const BandJob& band,
                                hipStream_t s);

// Multiply on single output tiles: persistent, cost-balanced multiply of the
// kept pairs into C (leaf 128 where the LDS-DMA kernel does not run: more than
// kLeaf128MaxBdim tiles per side, or no room for its item list; leaf 16 goes
// to launch_multiply_leaf16).
// pair_scratch holds bdim^3 int32 (each group's packed (tile, k) pairs).
hipError_t launch_multiply(const float* a, const float* b, float* c, int64_t n, int32_t leaf, int64_t bdim,
                           const int32_t* offsets, const int32_t* klist, int32_t* pair_scratch, bool vec,
                           int num_cus, hipStream_t s);

// Leaf 16: one wave per output tile, operands straight from global memory
// into MFMA registers (multiply_leaf16.hip); every tile of c is written.
hipError_t launch_multiply_leaf16(const float* a, const float* b, float* c, int64_t n, int64_t bdim,
                                  const int32_t* offsets, const int32_t* klist, bool vec, hipStream_t s);

// Multiply on 2x2 macro tiles, in two steps.  Schedule (leaf 32 and 64):
// per-macro-tile k bitmaps into words [mb*mb*4*nwords], union sizes into
// ucount [mb*mb], their exclusive prefix into uprefix [mb*mb + 1], and the
// union k lists as packed items into items [<= mb*mb*bdim].  Multiply (leaf
// 64, n >= 4; leaf 32 is launch_block_plan32): the persistent LDS-DMA kernel
// over that schedule, which also reads the plan's offsets for its cost model,
// writes four records per workgroup to bounds [4 * kSplitMaxGroups] and the partial sums of macro
// tiles shared between workgroups to fix_slots [kSplitMaxGroups * 2 * 128 *
// 128], which a second kernel adds into C; with fix_slots null no macro tile is
// shared.
struct MacroSchedule {
    uint64_t* words;
    int32_t *ucount, *uprefix;
    uint32_t* items;
    int64_t* bounds;
    float* fix_slots;
};
hipError_t launch_macro_schedule(const int32_t* offsets, const int32_t* klist, int64_t bdim, const MacroSchedule& ms,
                                 hipStream_t s, const int32_t* run = nullptr);
hipError_t launch_macro_multiply(const float* a, const float* b, float* c, int64_t n, int64_t bdim,
                                 const int32_t* offsets, const MacroSchedule& ms, int num_cus, hipStream_t s);
// Leaf 128 (4 <= n, bdim <= kLeaf128MaxBdim) on the LDS-DMA kernel: two items per kept pair (uprefix [bdim*bdim + 1], items
// [2 * pairs]), then the multiply and fixup kernels with one macro tile per
// output tile.
constexpr int64_t kLeaf128MaxBdim = 512;  // item fields: tile index < 512, k half < 1024
hipError_t launch_leaf128_schedule(const int32_t* offsets, const int32_t* klist, int64_t bdim, int32_t* uprefix,
                                   uint32_t* items, hipStream_t s);
hipError_t launch_leaf128_multiply(const float* a, const float* b, float* c, int64_t n, int64_t bdim,
                                   const int32_t* uprefix, const uint32_t* items, int64_t* bounds, float* fix_slots,
                                   int num_cus, hipStream_t s);

// --------------------------------------------------------------------------
// Learned threshold (learned.hip).

constexpr int kSumBlocks = 1024;  // partials of launch_sumsq
constexpr int kMlpIn = 129, kMlpHid = 128;

// Offsets into the flat parameter array and into the activation scratch of
// a batch (in floats).
struct MlpLayout {
    int64_t w1 = 0;
    int64_t b1 = w1 + int64_t(kMlpHid) * kMlpIn;
    int64_t w2 = b1 + kMlpHid;
    int64_t b2 = w2 + int64_t(kMlpHid) * kMlpHid;
    int64_t w3 = b2 + kMlpHid;
    int64_t b3 = w3 + kMlpHid;
    int64_t count = b3 + 1;
    // activations: H1 H2 D1 D2 [B][128] each, then y, dy [B]
    int64_t h1 = 0, h2 = 0, d1 = 0, d2 = 0, y = 0, dy = 0, acts_total = 0;
    static MlpLayout acts(int batch) {
        MlpLayout L{};
        const int64_t bh = int64_t(batch) * kMlpHid;
        L.h1 = 0;
        L.h2 = bh;
        L.d1 = 2 * bh;
        L.d2 = 3 * bh;
        L.y = 4 * bh;
        L.dy = L.y + batch;
        L.acts_total = L.dy + batch;
        return L;
    }
};

hipError_t launch_tau_features(const double* pyr_a, const double* pyr_b, int64_t bdim, int lv, float log_target,
                               float* out, hipStream_t s);
// *out = sum of x[q]^2 in FP64; partials holds kSumBlocks doubles.
hipError_t launch_sumsq(const float* x, int64_t count, double* partials, double* out, hipStream_t s);
hipError_t launch_mlp_forward(const float* params, const float* x, int batch, float* acts, float* y, hipStream_t s);
hipError_t launch_mlp_loss_grad(const float* params, const float* x, const float* t, int batch, float* acts,
                                float* grad, float* loss, hipStream_t s);
hipError_t launch_adam(float* params, const float* grad, float* m, float* v, int64_t count, float lr, float b1,
                       float b2, float eps, float c1, float c2, hipStream_t s);

// --------------------------------------------------------------------------
// Reduced-precision leaf products (split.hip, multiply_macro.hip).

constexpr int kPrecFp32 = 0, kPrecBf16 = 1, kPrecF16x3 = 2;

// Device pointers into a split buffer: scale exponents [2] (A, B), A planes
// (row-major, n x n halves), Bt planes (B transposed, n x n halves); the lo
// planes are used by f16x3 only.
struct SplitLayout {
    int32_t* exps;
    uint16_t *a_hi, *a_lo, *bt_hi, *bt_lo;
};

hipError_t launch_split(const float* a, const float* b, int64_t n, int64_t bdim, int lv, const double* pyr_a,
                        const double* pyr_b, int precision, const SplitLayout& L, hipStream_t s);
// The f16x3 scale exponents alone (int32 exps at header[0..1], the two
// largest leaf norms at header + 8 bytes).
hipError_t launch_split_scales(int64_t bdim, int lv, const double* pyr_a, const double* pyr_b, int32_t* header,
                               hipStream_t s);
// Reduced-precision products (kPrecBf16 or kPrecF16x3) straight from the FP32
// inputs (multiply_convert.hip), bitwise the same C as launch_split +
// launch_lowp_multiply: with the products tested on the leaf norms (row stride
// ld) and counted in *pairs, or from a plan's items.  exps: the split scale
// exponents (F16X3 only; may be null for BF16).  planes (may be null): nothing is
// done if *planes is not zero.
hipError_t launch_convert_test(const float* a, const float* b, int precision, const int32_t* exps, float* c, int64_t n,
                               int64_t bdim, const double* na, const double* nb, int64_t ld, double tau,
                               int64_t* pairs, const int32_t* planes, hipStream_t s);
hipError_t launch_convert_plan(const float* a, const float* b, int precision, const int32_t* exps, float* c, int64_t n,
                               int64_t bdim, const uint32_t* items, const int32_t* uprefix, hipStream_t s);
hipError_t launch_lowp_multiply(const SplitLayout& L, float* c, int64_t n, int64_t bdim, int precision,
                                const uint32_t* items, const int32_t* uprefix, int num_cus, hipStream_t s,
                                const int32_t* run = nullptr);

// BF16, one call, a caller with room for planes: which form multiplies is picked
// on the device from the leaf norms na, nb (row stride ld).  With V the kept pairs
// per output tile and U the k that any of a 2x2 block of tiles keeps, both
// estimated from 1024 such blocks and k, the planes are taken if 4 U - 3 V >=
// weight, unless every pair is kept and full_fp32 is set.  launch_split_choice
// writes *form (1: planes, 0: FP32 inputs), the planes if they are taken, and
// zeros to clear_count words at clear.  bf16_choice: whether there is a choice
// at this size, and its constants (multiply_convert.hip).
struct FormChoice {
    const double *na, *nb;
    int64_t ld;
    double tau;
    int32_t weight, full_fp32;
    int32_t* form;
    int64_t* clear;
    int64_t clear_count;
};
bool bf16_choice(int64_t n, int64_t bdim, FormChoice* choice);
hipError_t launch_split_choice(const float* a, const float* b, int64_t n, int64_t bdim, const FormChoice& choice,
                               const SplitLayout& L, hipStream_t s);

// --------------------------------------------------------------------------
// Batched products (batch.hip): one descriptor per product in device memory.

struct BatchProduct {
    const float* a;
    const float* b;
    float* c;
    double* norms[2];  // leaf norms of A, B [bdim][bdim]
    int64_t* pairs;    // this product's slot of the caller's pairs array
    int64_t n, bdim;
    int32_t leaf, vec;
    double tau;
};

// leaf classes of the batched multiply: 32, 64, 128
constexpr int kBatchClasses = 3;

// work of a product: norm-pass blocks per matrix, workgroups of the multiply
int64_t batch_strips(int64_t n, int64_t bdim);
int64_t batch_blocks(int64_t n);

// prods: class after class (class_count each).  strip_base, block_base [count]:
// the prefix of batch_strips over the batch, of batch_blocks within each class;
// strips and class_blocks: the totals; bytes: of all inputs.
hipError_t launch_batch(const BatchProduct* prods, const int64_t* strip_base, const int64_t* block_base,
                        const int32_t* class_count, const int64_t* class_blocks, int64_t strips, double bytes, int32_t count,
                        hipStream_t s);

}  // namespace spamm

// Multiply of the kept leaf pairs, one 64x64 block (I, J) of C per workgroup of
// four waves, wave q on the 32x32 quadrant (q >> 1, q & 1), at any leaf.
//
// k is walked in entries of 32.  An entry's four operand tiles (rows 2I + {0, 1}
// of A, columns 2J + {0, 1} of B, in tiles of 32) are copied straight into LDS,
// one tile per wave; a tile that no kept product reads is not copied.  With two
// stages this goes on while the entry before is multiplied and the waves meet
// once per entry, with one (the larger grids, kTwoStageMaxN) an entry is copied,
// then multiplied.  Four or six workgroups per CU keep every SIMD supplied with
// waves of as many different blocks, so one block's copies and barriers hide
// behind the others' MFMAs, and blocks of unequal length need no plan of the
// work split: the hardware hands out the next one.
//
// The entries come either from the leaf norms, the block testing its own
// products as Algorithm 2's blocks do (kKept, the one-call path: no plan
// launch; kDropped, the error searches below), or from the items of a plan and
// schedule, whose macro tiles at leaf 32 are these blocks (kPlanned).  Pairs and their
// order are the same, ascending k per output tile, at leaf 16 with the MFMA
// steps of the leaf-16 kernel: at leaf 16 and 32 C is bitwise the same either
// way.
//
// Bound by the matrix cores while the CUs are full: at N = 4096, the matrix
// 0.1 / (|i-j|^0.1 + 1) at leaf 32 with 15 % of the pairs kept, they are busy 70 %
// of the CUs' busy cycles (16 KiB of operands per 4 x 1024 cycles of MFMA work,
// a third of them past L2), and the launch ends with 5 % of the CUs' time idle.
// One call there 302 -> 220 us (register-staged 2x2 macro tiles in a static
// split of whole tiles, after a plan launch); exp decay 0.05, tau 1e-6, leaf 32:
// N = 2048 66 -> 33 us, 8192 287 -> 191; leaf 16: N = 2048 69 -> 33, 8192 601 ->
// 290; leaf 64: N = 2047 117 -> 36.
//
// Sizes that are no multiple of 32, rows at 4-byte alignment: rows and columns
// past the matrix are read from addresses inside it (they only reach parts of C
// that are not stored), a chunk across a row's end reads into the next row.
// Only the last entry, whose k reach past n, is loaded through registers with
// zeros; it comes last, after the copies.
// kDropped forms the error of a threshold search, E = the sum of the products
// dropped at tau, in one launch: C holds the E of a lower threshold `base`, the
// block adds the products dropped at tau but not at base, sums the squares of
// what that gives, and stores it only if asked to.  The products between two
// thresholds of a bisection are ever fewer, where E from nothing multiplies
// most of the matrix each time.
#include <hip/hip_runtime.h>

#include "block_multiply.h"

namespace spamm {

template <int LEAF, int FROM, int STAGES>
__global__ __launch_bounds__(kBlockThreads, block_occ(STAGES)) void multiply_block_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, int64_t n, int bdim, int nb,
    const double* __restrict__ na, const double* __restrict__ nbm, int64_t ld, double tau,
    unsigned long long* __restrict__ pairs, const uint32_t* __restrict__ items, const int32_t* __restrict__ uprefix,
    BandJob band) {
    block_multiply<LEAF, FROM, STAGES>(A, B, C, n, bdim, nb, na, nbm, ld, tau, pairs, items, uprefix, band, int(blockIdx.x));
}

namespace {
template <int LEAF, int FROM>
hipError_t launch_block_of(const float* a, const float* b, float* c, int64_t n, int64_t bdim, const double* na,
                           const double* nb, int64_t ld, double tau, int64_t* pairs, const uint32_t* items,
                           const int32_t* uprefix, const BandJob& band, hipStream_t s) {
    if (n < 1 || bdim != (n + LEAF - 1) / LEAF || bdim > 1024) return hipErrorInvalidValue;
    const bool two = n <= kTwoStageMaxN;
    static int scratch_state[2] = {0, 0};
    const hipError_t ce = two ? check_no_scratch(multiply_block_kernel<LEAF, FROM, 2>, &scratch_state[1])
                              : check_no_scratch(multiply_block_kernel<LEAF, FROM, 1>, &scratch_state[0]);
    if (ce != hipSuccess) return ce;
    const int blocks = int((n + 63) / 64);
    auto* count = reinterpret_cast<unsigned long long*>(pairs);
    if (two)
        multiply_block_kernel<LEAF, FROM, 2><<<block_grid(blocks, kBlockOrder), kBlockThreads, 0, s>>>(
            a, b, c, n, int(bdim), blocks, na, nb, ld, tau, count, items, uprefix, band);
    else
        multiply_block_kernel<LEAF, FROM, 1><<<block_grid(blocks, kBlockOrder), kBlockThreads, 0, s>>>(
            a, b, c, n, int(bdim), blocks, na, nb, ld, tau, count, items, uprefix, band);
    return hipGetLastError();
}

template <int FROM>
hipError_t launch_block_leaf(const float* a, const float* b, float* c, int64_t n, int32_t leaf, int64_t bdim,
                             const double* na, const double* nb, int64_t ld, double tau, int64_t* pairs,
                             const BandJob& band, hipStream_t s) {
    switch (leaf) {
        case 16:
            return launch_block_of<16, FROM>(a, b, c, n, bdim, na, nb, ld, tau, pairs, nullptr, nullptr, band, s);
        case 32:
            return launch_block_of<32, FROM>(a, b, c, n, bdim, na, nb, ld, tau, pairs, nullptr, nullptr, band, s);
        case 64:
            return launch_block_of<64, FROM>(a, b, c, n, bdim, na, nb, ld, tau, pairs, nullptr, nullptr, band, s);
        case 128:
            return launch_block_of<128, FROM>(a, b, c, n, bdim, na, nb, ld, tau, pairs, nullptr, nullptr, band, s);
        default: return hipErrorInvalidValue;
    }
}
}  // namespace

hipError_t launch_block_test(const float* a, const float* b, float* c, int64_t n, int32_t leaf, int64_t bdim,
                             const double* na, const double* nb, int64_t ld, double tau, int64_t* pairs,
                             hipStream_t s) {
    return launch_block_leaf<kKept>(a, b, c, n, leaf, bdim, na, nb, ld, tau, pairs, BandJob{}, s);
}

hipError_t launch_block_plan32(const float* a, const float* b, float* c, int64_t n, int64_t bdim,
                               const uint32_t* items, const int32_t* uprefix, hipStream_t s) {
    return launch_block_of<32, kPlanned>(a, b, c, n, bdim, nullptr, nullptr, 0, 0.0, nullptr, items, uprefix,
                                         BandJob{}, s);
}

hipError_t launch_block_dropped(const float* a, const float* b, float* e, int64_t n, int32_t leaf, int64_t bdim,
                                const double* na, const double* nb, int64_t ld, double tau, const BandJob& band,
                                hipStream_t s) {
    if (!band.sums || !band.counts) return hipErrorInvalidValue;
    return launch_block_leaf<kDropped>(a, b, e, n, leaf, bdim, na, nb, ld, tau, nullptr, band, s);
}

}  // namespace spamm

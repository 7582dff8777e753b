// The smallest products (n <= 320): the threshold test of Algorithm 1 and the
// multiply of the kept pairs in one launch after the leaf norm pass.  At these
// sizes a launch is a few microseconds of ramp and drain for well under a
// microsecond of work, and there are too few blocks of C to give every SIMD
// more than one wave.
//
// One workgroup of sixteen waves per 64x64 block (I, J) of C, whatever the
// leaf; k is walked in entries of 32 (block.h), at most ten of them, so that
// all operand tiles of the block fit in LDS: they are loaded at once, before
// the test is known, and nothing waits on memory a second time.
//  * every wave tests the leaf products of its lane's entry, nA * nB >= tau
//    (the comparison of the plan kernel, on the same leaf norms, so the kept
//    pairs are the same; the pyramid only skips subtrees whose leaf products
//    all fail).  Leaf 32: one product per quadrant of the block; leaf 64 and
//    128: one for the whole block; leaf 16: one for each of 16 output tiles
//    and both halves of the entry.  The entries that any product keeps form
//    the union list; block by block the kept pairs are added to the counter;
//  * leaf 32 and up: the waves are four k-groups of four (wave w: k-group
//    g = w >> 2, quadrant q = (w + g) & 3, so the four waves of a SIMD hold the
//    four quadrants and every SIMD gets a quarter of each quadrant's entries),
//    group g takes entries g, g + 4, ... of the list; each wave accumulates its
//    own in ascending k on v_mfma_f32_32x32x2f32 and the groups' partial tiles
//    are added in group order through LDS, so the result does not depend on
//    timing;
//  * leaf 16: one output tile per wave, v_mfma_f32_16x16x4f32 in the steps and
//    order of the leaf-16 kernel of the general path, so C is bitwise its C.
// Tiles with nothing kept are written as zeros (beta = 0).
//
// Bound by latency: launch, norms and operands from L2, reduction.  One call,
// n = 300: leaf 32 15.5 -> 13.7 us, leaf 64 45.6 -> 16.3, leaf 128 60 -> 17 (about
// what the host needs to enqueue two launches).
//
// Rows that are only 4-byte aligned (VEC false) are read by 16-byte loads at
// that alignment; a chunk that crosses the matrix's edge reads the last four
// columns and shifts them into place.
#include <hip/hip_runtime.h>

#include "block.h"
#include "device.h"
#include "dma.h"
#include "internal.h"

namespace spamm {

namespace {
constexpr int kSmallWaves = 16;
constexpr int kSmallThreads = kSmallWaves * 64;
constexpr int kSmallGroups = kSmallWaves / 4;
constexpr int kStripEntries = 10;       // 16 KiB of LDS each

// Which leaf products of entry `lane` of block (I, J) are kept.  Leaf 32 and
// up: bit q for quadrant q.  Leaf 16: bit 8 q + 4 a + 2 b + h for output tile
// (a, b) of quadrant q and half h of the entry.  *pairs: the kept leaf pairs
// that this block counts.
template <int LEAF>
__device__ __forceinline__ uint32_t small_test(const double* __restrict__ na, const double* __restrict__ nb,
                                               int64_t ld, int bdim, int n, int I, int J, double tau, int lane,
                                               int* pairs) {
    uint32_t mem = 0;
    *pairs = 0;
    if constexpr (LEAF >= 64) {
        constexpr int R = LEAF / 64, S = LEAF / 32;  // blocks and entries per leaf tile side
        const int ti = I / R, tj = J / R, k = lane / S;
        const int kc = k < bdim ? k : bdim - 1;
        const double x = na[ti * ld + kc], y = nb[kc * ld + tj];
        if (k < bdim && x * y >= tau) {
            *pairs = (I % R == 0 && J % R == 0 && lane % S == 0) ? 1 : 0;
            if (lane * 32 < n) {  // quadrants and entries with something inside the matrix
                const uint32_t rows = I * 64 + 32 < n ? 0xFu : 0x3u, cols = J * 64 + 32 < n ? 0xFu : 0x5u;
                mem = rows & cols;
            }
        }
    } else {
        constexpr int T = 64 / LEAF, H = 32 / LEAF;  // leaf tiles per block side and per entry
        double nav[T][H], nbv[H][T];
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const int ti = T * I + t < bdim ? T * I + t : bdim - 1, tj = T * J + t < bdim ? T * J + t : bdim - 1;
                const int k = H * lane + h, kc = k < bdim ? k : bdim - 1;
                nav[t][h] = na[ti * ld + kc];
                nbv[h][t] = nb[kc * ld + tj];
            }
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j)
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const bool in = H * lane + h < bdim && T * I + i < bdim && T * J + j < bdim;
                    const int bit = LEAF == 32 ? 2 * i + j : 8 * (2 * (i >> 1) + (j >> 1)) + 4 * (i & 1) + 2 * (j & 1) + h;
                    if (in && nav[i][h] * nbv[h][j] >= tau) mem |= 1u << bit;
                }
        *pairs = __popc(mem);
    }
    return mem;
}

// adds the block's kept pairs to the counter (one wave)
__device__ __forceinline__ void small_count(int cnt, int lane, unsigned long long* pairs) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (lane == 0 && cnt) atomicAdd(pairs, static_cast<unsigned long long>(cnt));
}

// what a wave accumulates: a 32x32 quadrant, or at leaf 16 one 16x16 tile
template <int LEAF>
struct SmallAcc {
    f16v acc;
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    }
    __device__ __forceinline__ void multiply(const float* t, uint32_t quads, int, int q, int lane) {
        if ((quads >> q) & 1) op_multiply(acc, t, q, lane);
    }
    // the quadrant's partial tiles of groups 1.. through LDS, added in group
    // order; group 0 (the caller's wave < 4) writes C
    __device__ __forceinline__ void finish(float* lds, float* __restrict__ C, int64_t n, int I, int J, int wave, int q,
                                           int lane) {
        float (*red)[4][16][64] = reinterpret_cast<float (*)[4][16][64]>(lds);
        const int grp = wave >> 2, ir = lane & 31, g = lane >> 5;
        if (grp > 0) {
#pragma unroll
            for (int r = 0; r < 16; ++r) red[grp - 1][q][r][lane] = acc[r];
        }
        __syncthreads();
        if (grp != 0) return;
#pragma unroll
        for (int h = 0; h < kSmallGroups - 1; ++h)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] += red[h][q][r][lane];
        const int64_t row0 = 64 * int64_t(I) + 32 * (q >> 1) + 4 * g, col = 64 * int64_t(J) + 32 * (q & 1) + ir;
        if (col >= n) return;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t row = row0 + 8 * (r >> 2) + (r & 3);
            if (row < n) C[row * n + col] = acc[r];
        }
    }
};

template <>
struct SmallAcc<16> {
    f4 acc;
    __device__ __forceinline__ void zero() { acc = f4{0.0f, 0.0f, 0.0f, 0.0f}; }
    // output tile (a, b) = (wave >> 2, wave & 3) of the block
    __device__ __forceinline__ void multiply(const float* t, uint32_t mem, int wave, int, int lane) {
        const int a = wave >> 2, b = wave & 3;
        op_multiply16(acc, t, a, b, (mem >> (8 * (2 * (a >> 1) + (b >> 1)) + 4 * (a & 1) + 2 * (b & 1))) & 3u, lane);
    }
    __device__ __forceinline__ void finish(float*, float* __restrict__ C, int64_t n, int I, int J, int wave, int,
                                           int lane) {
        const int64_t row0 = 64 * int64_t(I) + 16 * (wave >> 2) + 4 * (lane >> 4);
        const int64_t col = 64 * int64_t(J) + 16 * (wave & 3) + (lane & 15);
        if (col >= n) return;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (row0 + v < n) C[(row0 + v) * n + col] = acc[v];
    }
};
}  // namespace

// The union list's entries have ranks 0, 1, ... ; rank_entry finds the entry
// of a rank (-1: none), the same in every lane.
struct SmallUnion {
    uint64_t bal;
    int rank;
    __device__ __forceinline__ SmallUnion(uint32_t mem, int lane) {
        bal = __ballot(mem != 0);
        rank = __popcll(bal & (lane == 0 ? 0ull : (~0ull >> (64 - lane))));
    }
    __device__ __forceinline__ int size() const { return __popcll(bal); }
    __device__ __forceinline__ int entry(int r, int lane) const {
        const uint64_t sel = __ballot(((bal >> lane) & 1) && rank == r);
        return sel ? __builtin_ctzll(sel) : -1;
    }
};

template <int LEAF, bool VEC>
__global__ __launch_bounds__(kSmallThreads, 1) void multiply_strip_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, int64_t n, int bdim, int blocks,
    const double* __restrict__ na, const double* __restrict__ nb, int64_t ld, double tau,
    unsigned long long* __restrict__ pairs) {
    __shared__ __attribute__((aligned(16))) float strip[kStripEntries][4][kOpTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int I = blockIdx.x / blocks, J = blockIdx.x - I * blocks;
    const int grp = wave >> 2, q = (wave + grp) & 3;
    const int entries = (int(n) + 31) / 32;

    // four waves a tile: chunk v belongs to entry v, role wave / 4
    const int role = wave >> 2;
    const OpTile of(A, B, I, J, role);
    OpChunk<VEC> x[kStripEntries];
#pragma unroll
    for (int v = 0; v < kStripEntries; ++v) x[v].load(of, n, v, tid & 255, v < entries);
    int cnt;
    const uint32_t mem = small_test<LEAF>(na, nb, ld, bdim, int(n), I, J, tau, lane, &cnt);
    if (wave == 0) small_count(cnt, lane, pairs);
    const SmallUnion uni(mem, lane);
#pragma unroll
    for (int v = 0; v < kStripEntries; ++v)
        if (v < entries) op_commit<LEAF>(strip[v][role], role, tid & 255, x[v].value());
    __syncthreads();
    SmallAcc<LEAF> acc;
    acc.zero();
    for (int u = LEAF == 16 ? 0 : grp; u < uni.size(); u += LEAF == 16 ? 1 : kSmallGroups) {
        const int k = uni.entry(u, lane);
        acc.multiply(&strip[k][0][0], uint32_t(__shfl(int(mem), k)), wave, q, lane);
    }
    if (LEAF != 16) __syncthreads();  // the strip is reused by the reduction
    acc.finish(&strip[0][0][0], C, n, I, J, wave, q, lane);
}

template <int LEAF>
static hipError_t launch_strip(const float* a, const float* b, float* c, int64_t n, bool vec, int64_t bdim,
                               const double* na, const double* nb, int64_t ld, double tau, int64_t* pairs,
                               hipStream_t s) {
    static int scratch_state[2] = {0, 0};
    const hipError_t ce = vec ? check_no_scratch(multiply_strip_kernel<LEAF, true>, &scratch_state[1])
                              : check_no_scratch(multiply_strip_kernel<LEAF, false>, &scratch_state[0]);
    if (ce != hipSuccess) return ce;
    const int blocks = int((n + 63) / 64);
    auto* count = reinterpret_cast<unsigned long long*>(pairs);
    if (vec)
        multiply_strip_kernel<LEAF, true><<<unsigned(blocks * blocks), kSmallThreads, 0, s>>>(
            a, b, c, n, int(bdim), blocks, na, nb, ld, tau, count);
    else
        multiply_strip_kernel<LEAF, false><<<unsigned(blocks * blocks), kSmallThreads, 0, s>>>(
            a, b, c, n, int(bdim), blocks, na, nb, ld, tau, count);
    return hipGetLastError();
}

hipError_t launch_small_multiply(const float* a, const float* b, float* c, int64_t n, int32_t leaf, bool vec,
                                 int64_t bdim, const double* na, const double* nb, int64_t ld, double tau,
                                 int64_t* pairs, hipStream_t s) {
    static_assert(kSmallMaxN <= 32 * kStripEntries, "every operand tile of a block in LDS");
    if (n < 1 || n > kSmallMaxN || bdim != (n + leaf - 1) / leaf || (vec && n % 4 != 0)) return hipErrorInvalidValue;
    switch (leaf) {
        case 16: return launch_strip<16>(a, b, c, n, vec, bdim, na, nb, ld, tau, pairs, s);
        case 32: return launch_strip<32>(a, b, c, n, vec, bdim, na, nb, ld, tau, pairs, s);
        case 64: return launch_strip<64>(a, b, c, n, vec, bdim, na, nb, ld, tau, pairs, s);
        case 128: return launch_strip<128>(a, b, c, n, vec, bdim, na, nb, ld, tau, pairs, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace spamm

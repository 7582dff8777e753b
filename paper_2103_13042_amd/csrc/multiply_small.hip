// The smallest products at leaf 16 (n <= 320): the threshold test of Algorithm
// 1 and the multiply of the kept pairs in one launch after the leaf norm pass.
//
// One workgroup of sixteen waves per 64x64 block (I, J) of C, one 16x16 output
// tile per wave; k is walked in entries of 32 (block.h), at most ten of them, so
// that all operand tiles of the block fit in LDS: they are loaded at once,
// before the test is known, and nothing waits on memory a second time.
//  * every wave tests the leaf products of its lane's entry, nA * nB >= tau
//    (the comparison of the plan kernel, on the same leaf norms, so the kept
//    pairs are the same): one for each of 16 output tiles and both halves of
//    the entry.  The entries that any product keeps form the union list; block
//    by block the kept pairs are added to the counter;
//  * v_mfma_f32_16x16x4f32 in the steps and order of the leaf-16 kernel of the
//    general path, so C is bitwise its C.
// Tiles with nothing kept are written as zeros (beta = 0).
//
// Bound by latency: launch, norms and operands from L2.
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
constexpr int kStripEntries = 10;       // 16 KiB of LDS each

// Which leaf products of entry `lane` of block (I, J) are kept: bit 8 q + 4 a +
// 2 b + h for output tile (a, b) of quadrant q and half h of the entry.
__device__ __forceinline__ uint32_t small_test(const double* __restrict__ na, const double* __restrict__ nb,
                                               int64_t ld, int bdim, int I, int J, double tau, int lane) {
    uint32_t mem = 0;
    double nav[4][2], nbv[2][4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ti = 4 * I + t < bdim ? 4 * I + t : bdim - 1, tj = 4 * J + t < bdim ? 4 * J + t : bdim - 1;
            const int k = 2 * lane + h, kc = k < bdim ? k : bdim - 1;
            nav[t][h] = na[ti * ld + kc];
            nbv[h][t] = nb[kc * ld + tj];
        }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool in = 2 * lane + h < bdim && 4 * I + i < bdim && 4 * J + j < bdim;
                const int bit = 8 * (2 * (i >> 1) + (j >> 1)) + 4 * (i & 1) + 2 * (j & 1) + h;
                if (in && nav[i][h] * nbv[h][j] >= tau) mem |= 1u << bit;
            }
    return mem;
}

// adds the block's kept pairs to the counter (one wave)
__device__ __forceinline__ void small_count(int cnt, int lane, unsigned long long* pairs) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (lane == 0 && cnt) atomicAdd(pairs, static_cast<unsigned long long>(cnt));
}

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

template <bool VEC>
__global__ __launch_bounds__(kSmallThreads, 1) void multiply_strip_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, int64_t n, int bdim, int blocks,
    const double* __restrict__ na, const double* __restrict__ nb, int64_t ld, double tau,
    unsigned long long* __restrict__ pairs) {
    __shared__ __attribute__((aligned(16))) float strip[kStripEntries][4][kOpTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int I = blockIdx.x / blocks, J = blockIdx.x - I * blocks;
    const int entries = (int(n) + 31) / 32;

    // four waves a tile: chunk v belongs to entry v, role wave / 4
    const int role = wave >> 2;
    const OpTile of(A, B, I, J, role);
    OpChunk<VEC> x[kStripEntries];
#pragma unroll
    for (int v = 0; v < kStripEntries; ++v) x[v].load(of, n, v, tid & 255, v < entries);
    const uint32_t mem = small_test(na, nb, ld, bdim, I, J, tau, lane);
    if (wave == 0) small_count(__popc(mem), lane, pairs);
    const SmallUnion uni(mem, lane);
#pragma unroll
    for (int v = 0; v < kStripEntries; ++v)
        if (v < entries) op_commit<16>(strip[v][role], role, tid & 255, x[v].value());
    __syncthreads();
    const int a = wave >> 2, b = wave & 3;  // the wave's output tile
    const int first = 8 * (2 * (a >> 1) + (b >> 1)) + 4 * (a & 1) + 2 * (b & 1);
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int u = 0; u < uni.size(); ++u) {
        const int k = uni.entry(u, lane);
        op_multiply16(acc, &strip[k][0][0], a, b, (uint32_t(__shfl(int(mem), k)) >> first) & 3u, lane);
    }
    const int64_t row0 = 64 * int64_t(I) + 16 * a + 4 * (lane >> 4), col = 64 * int64_t(J) + 16 * b + (lane & 15);
    if (col >= n) return;
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (row0 + v < n) C[(row0 + v) * n + col] = acc[v];
}

hipError_t launch_small_multiply16(const float* a, const float* b, float* c, int64_t n, bool vec, int64_t bdim,
                                   const double* na, const double* nb, int64_t ld, double tau, int64_t* pairs,
                                   hipStream_t s) {
    static_assert(kSmallMaxN <= 32 * kStripEntries, "every operand tile of a block in LDS");
    if (n < 1 || n > kSmallMaxN || bdim != (n + 15) / 16 || (vec && n % 4 != 0)) return hipErrorInvalidValue;
    static int scratch_state[2] = {0, 0};
    const hipError_t ce = vec ? check_no_scratch(multiply_strip_kernel<true>, &scratch_state[1])
                              : check_no_scratch(multiply_strip_kernel<false>, &scratch_state[0]);
    if (ce != hipSuccess) return ce;
    const int blocks = int((n + 63) / 64);
    auto* count = reinterpret_cast<unsigned long long*>(pairs);
    if (vec)
        multiply_strip_kernel<true><<<unsigned(blocks * blocks), kSmallThreads, 0, s>>>(
            a, b, c, n, int(bdim), blocks, na, nb, ld, tau, count);
    else
        multiply_strip_kernel<false><<<unsigned(blocks * blocks), kSmallThreads, 0, s>>>(
            a, b, c, n, int(bdim), blocks, na, nb, ld, tau, count);
    return hipGetLastError();
}

}  // namespace spamm

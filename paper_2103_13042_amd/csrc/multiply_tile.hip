// Small products (n <= kTileMaxN, leaf 32 and up) in one launch after the leaf
// norms: a 32x32 tile (I, J) of C per workgroup of four waves, which share its k.
//
// k is walked in entries of 32.  Every wave tests all entries at once, one per
// lane (nA * nB >= tau, the comparison of the plan kernel on the same leaf norms),
// and takes every fourth kept one.  An entry's tiles of A and B are copied into
// 8 KiB of LDS of the wave's own, read into registers, and while the MFMAs run
// from there the next entry's copies land: no barrier until the four partial
// tiles are added, in wave order, so C does not depend on timing.
//
// At these sizes 64x64 blocks of C leave the chip idle: one workgroup a CU and one
// wave a SIMD at n = 1024, whose copies, LDS reads and barriers nothing hides, and
// the longest block decides.  Tiles give four times the workgroups, four waves a
// SIMD, for twice the operand traffic, which comes from L2.  One call, exp decay
// 0.05, tau 1e-6: n = 300 leaf 32 14.1 -> 11.5 us (sixteen waves a block, all
// operands in LDS first; now what the host needs for two launches), 1024 leaf 32
// 19.9 -> 15.8, leaf 64 22.0 -> 17.4, leaf 128 26.4 -> 21.
//
// Rows and columns past the matrix are read from addresses inside it (they only
// reach parts of C that are not stored), rows may be 4-byte aligned, a chunk
// across a row's end reads into the next row.  The entry whose k reach past n
// goes through registers with zeros.
#include <hip/hip_runtime.h>

#include "block.h"
#include "device.h"
#include "dma.h"
#include "internal.h"

namespace spamm {
namespace {

constexpr int kTileThreads = 256;
constexpr int kCountRun = 8;

template <int LEAF>
__global__ __launch_bounds__(kTileThreads, 4) void multiply_tile_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, int n, int tiles,
    const double* __restrict__ na, const double* __restrict__ nbm, int ld, double tau,
    unsigned long long* __restrict__ pairs) {
    constexpr int S = LEAF / 32;  // entries and tiles per leaf tile side
    __shared__ __attribute__((aligned(1024))) float lds[4 * 2 * kOpTile];  // per wave: an A and a B tile
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ir = lane & 31, g = lane >> 5;

    // XCD x takes an eighth of the tile rows (of A's rows, that is, for its L2), in
    // each the tiles nearest to the diagonal first: a CU, which gets every 32nd
    // workgroup, then has long and short ones
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int row0 = xcd * tiles / 8, rows = (xcd + 1) * tiles / 8 - row0;
    if (idx >= rows * tiles) return;
    const int I = row0 + idx % rows, step = idx / rows;
    const int near = I < tiles - 1 - I ? I : tiles - 1 - I;
    const int J = step <= 2 * near ? ((step & 1) ? I - (step + 1) / 2 : I + step / 2)
                  : I < tiles - 1 - I ? step
                                      : tiles - 1 - step;

    // entry e = lane: 32 k, kept if its leaf product is; tiles <= 64
    const int li = I / S, lj = J / S, lk = lane / S, bdim = (n + LEAF - 1) / LEAF;
    double nav = 0.0;
    bool keep = false;
    if (lane < tiles) {
        nav = na[li * ld + lk];
        keep = nav * nbm[lk * ld + lj] >= tau;
    }
    const uint64_t mask = __ballot(keep);
    // one workgroup counts the pairs of kCountRun leaf tiles of a row: 1024
    // additions to one address took 4 us at N = 1024, leaf 32
    if (wave == 3 && li * S == I && lj * S == J && lj % kCountRun == 0) {
        int count = 0;
#pragma unroll
        for (int c = 0; c < kCountRun; ++c) {
            const bool pair = lane < tiles && lk * S == lane && lj + c < bdim && nav * nbm[lk * ld + lj + c] >= tau;
            count += __popcll(__ballot(pair));
        }
        if (lane == 0 && count) atomicAdd(pairs, static_cast<unsigned long long>(count));
    }
    const int row = 32 * I + (tid >> 3), col = 32 * J + 4 * (tid & 7);  // this thread's part of C
    float* dst = C + row * n + col;
    f4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
    if (mask != 0) {
        // chunk 64 j + lane of a tile is row 8 j + lane / 8, position lane % 8
        // (a_at, b_at); rows of A and columns of B past the matrix moved inside
        float* ta = lds + wave * 2 * kOpTile;
        float* tb = ta + kOpTile;
        uint32_t a_off[4], b_off[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = 8 * j + (lane >> 3), p = lane & 7, k = r ^ ((r >> 4) & 1);
            const int row = 32 * I + r < n ? 32 * I + r : n - 1, col = 32 * J + 4 * p < n ? 32 * J + 4 * p : 32 * J;
            a_off[j] = uint32_t(row * n + 4 * (p ^ (r & 7))) * 4u;
            b_off[j] = uint32_t(k * n + col) * 4u;
        }
        auto copy = [&](int e) {
            const char* pa = reinterpret_cast<const char*>(A + 32 * e);
            const char* pb = reinterpret_cast<const char*>(B + 32 * e * n);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // opaque: else extended to 64 bits outside the loop, a vector add a copy
                asm volatile("" : "+v"(a_off[j]), "+v"(b_off[j]));
                copy_to_lds(reinterpret_cast<const float*>(pa + a_off[j]), reinterpret_cast<char*>(ta) + 1024 * j);
                copy_to_lds(reinterpret_cast<const float*>(pb + b_off[j]), reinterpret_cast<char*>(tb) + 1024 * j);
            }
        };
        // lane (ir, g) supplies A[ir][16 g + u] and B[16 g + u][ir] of MFMA step u
        f4 av[4];
        float bv[16];
        f16v acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
        auto multiply = [&]() {
#pragma unroll
            for (int u = 0; u < 16; ++u)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[u >> 2][u & 3], bv[u], acc, 0, 0, 0);
        };
        // the entries inside the matrix in turn to the waves
        const int whole = n / 32;
        uint64_t left = whole < 64 ? mask & ((1ull << whole) - 1) : mask;
        for (int w = 0; w < wave; ++w) left &= left - 1;
        if (left != 0) copy(__builtin_ctzll(left));
        while (left != 0) {
#pragma unroll
            for (int w = 0; w < 4; ++w) left &= left - 1;
            asm volatile("" ::: "memory");
            wait_vmcnt<0>();  // the entry's copies have landed
            asm volatile("" ::: "memory");
#pragma unroll
            for (int v = 0; v < 4; ++v) av[v] = *reinterpret_cast<const f4*>(ta + a_at(ir, 4 * g + v));
#pragma unroll
            for (int u = 0; u < 16; ++u) bv[u] = tb[b_at<32>(16 * g + u, ir)];
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): read before the next copies land
            asm volatile("" ::: "memory");
            if (left != 0) copy(__builtin_ctzll(left));
            multiply();
        }
        if (wave == 3 && whole < tiles && (mask >> whole & 1)) {  // k past the matrix: zeros
            const int ra = 32 * I + ir < n ? 32 * I + ir : n - 1, cb = 32 * J + ir < n ? 32 * J + ir : n - 1;
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int k = 32 * whole + 16 * g + u;
                av[u >> 2][u & 3] = k < n ? A[ra * n + k] : 0.0f;
                bv[u] = k < n ? B[k * n + cb] : 0.0f;
            }
            multiply();
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) ta[(8 * (r >> 2) + 4 * g + (r & 3)) * 32 + ir] = acc[r];
        __syncthreads();
#pragma unroll
        for (int w = 0; w < 4; ++w) sum += *reinterpret_cast<const f4*>(lds + w * 2 * kOpTile + 4 * tid);
    }
    if (row < n) {
        if (col + 4 <= n) {
            *reinterpret_cast<f4_dw*>(dst) = sum;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (col + c < n) dst[c] = sum[c];
        }
    }
}

template <int LEAF>
hipError_t launch_tile(const float* a, const float* b, float* c, int64_t n, const double* na, const double* nb,
                       int64_t ld, double tau, int64_t* pairs, hipStream_t s) {
    static int scratch_state = 0;
    const hipError_t ce = check_no_scratch(multiply_tile_kernel<LEAF>, &scratch_state);
    if (ce != hipSuccess) return ce;
    const int tiles = int((n + 31) / 32);
    multiply_tile_kernel<LEAF><<<unsigned((tiles + 7) / 8 * tiles * 8), kTileThreads, 0, s>>>(
        a, b, c, int(n), tiles, na, nb, int(ld), tau, reinterpret_cast<unsigned long long*>(pairs));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_tile_multiply(const float* a, const float* b, float* c, int64_t n, int32_t leaf, const double* na,
                                const double* nb, int64_t ld, double tau, int64_t* pairs, hipStream_t s) {
    if (n < 1 || n > kTileMaxN || ld > 2048) return hipErrorInvalidValue;
    switch (leaf) {
        case 32: return launch_tile<32>(a, b, c, n, na, nb, ld, tau, pairs, s);
        case 64: return launch_tile<64>(a, b, c, n, na, nb, ld, tau, pairs, s);
        case 128: return launch_tile<128>(a, b, c, n, na, nb, ld, tau, pairs, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace spamm

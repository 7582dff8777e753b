// Reduced-precision operands for the leaf products.
//
// bf16:  every element rounded to bfloat16 (round to nearest even).
// f16x3: per matrix one power-of-two scale s = 2^e, e = 15 - ceil(log2 M) with
//        M the largest leaf-tile Frobenius norm (so |s x| <= M s <= 2^15, inside
//        the FP16 range); hi = fp16(s x), lo = fp16(s x - hi), both round to
//        nearest even (s x and s x - hi are exact in FP32).
//
// A keeps its row-major layout; B is written transposed (Bt[j][k] = B[k][j])
// so that both MFMA operands read k-contiguous rows.  Both are HBM-bound
// streaming passes: 4 B read and 2 B (bf16) or 4 B (f16x3) written per element.
#include <hip/hip_runtime.h>

#include <cmath>

#include "device.h"
#include "internal.h"

namespace spamm {

// Of one matrix per block: the largest leaf norm, from the leaf level of its
// pyramid, and e from it.  One launch of two blocks, 12.8 us at bdim 256, bound
// by one CU's loads: clearing a maximum in memory, 128 blocks and a last launch to
// read it took 4.8 + 8.3 + 4.9 us and the gaps between them.
constexpr int kScaleThreads = 1024;

__global__ __launch_bounds__(kScaleThreads) void split_scale_kernel(const double* __restrict__ pyr_a,
                                                                    const double* __restrict__ pyr_b, int64_t bdim,
                                                                    int lv, int32_t* __restrict__ exps,
                                                                    double* __restrict__ mx) {
    const int64_t side = int64_t(1) << lv;
    const int m = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double* leaf = (m == 0 ? pyr_a : pyr_b) + level_offset(lv);
    double v = 0.0;
    constexpr int kRows = 16;  // of a wave, in flight at a time
    for (int64_t j = lane; j < bdim; j += 64)
        for (int64_t i0 = wave; i0 < bdim; i0 += kRows * (kScaleThreads / 64)) {
            double x[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const int64_t i = i0 + u * (kScaleThreads / 64);
                x[u] = i < bdim ? leaf[i * side + j] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kRows; ++u) v = fmax(v, x[u]);
        }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    __shared__ double part[kScaleThreads / 64];
    if (lane == 0) part[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kScaleThreads / 64; ++w) v = fmax(v, part[w]);
        mx[m] = v;
        int e = 0;
        if (v > 0.0) {
            int x = 0;
            const double f = frexp(v, &x);  // v = f 2^x, f in [0.5, 1)
            e = 15 - (f == 0.5 ? x - 1 : x);
        }
        exps[m] = e;
    }
}

template <int MODE>
struct Conv;

template <>
struct Conv<kPrecBf16> {
    static __device__ __forceinline__ void run(float x, float, uint16_t* hi, uint16_t*) {
        const __bf16 h = static_cast<__bf16>(x);
        *hi = __builtin_bit_cast(uint16_t, h);
    }
};

template <>
struct Conv<kPrecF16x3> {
    static __device__ __forceinline__ void run(float x, float s, uint16_t* hi, uint16_t* lo) {
        const float y = x * s;  // exact: s is a power of two
        const _Float16 h = static_cast<_Float16>(y);
        const _Float16 l = static_cast<_Float16>(y - static_cast<float>(h));
        *hi = __builtin_bit_cast(uint16_t, h);
        *lo = __builtin_bit_cast(uint16_t, l);
    }
};

// four elements of a row-major plane
template <int MODE>
__device__ __forceinline__ void split_row4(const f4* __restrict__ x4, int64_t q, float s, uint16_t* __restrict__ hi,
                                           uint16_t* __restrict__ lo) {
    const f4 v = x4[q];
    uint16_t h[4], l[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) Conv<MODE>::run(v[i], s, &h[i], &l[i]);
    const uint64_t hp = uint64_t(h[0]) | uint64_t(h[1]) << 16 | uint64_t(h[2]) << 32 | uint64_t(h[3]) << 48;
    reinterpret_cast<uint64_t*>(hi)[q] = hp;
    if (MODE == kPrecF16x3) {
        const uint64_t lp = uint64_t(l[0]) | uint64_t(l[1]) << 16 | uint64_t(l[2]) << 32 | uint64_t(l[3]) << 48;
        reinterpret_cast<uint64_t*>(lo)[q] = lp;
    }
}

// The 64 x 64 tile at (r0, c0) of B transposed, by 256 threads (tid) through LDS (n %
// 64 == 0): read rows of B coalesced, write rows of Bt (= columns of B) coalesced.
template <int MODE>
__device__ __forceinline__ void split_tile(const float* __restrict__ x, int64_t n, int64_t r0, int64_t c0, float s,
                                           uint16_t* __restrict__ hi, uint16_t* __restrict__ lo, float (*t)[65],
                                           int tid) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // 64 rows x 16 float4
        const int e = tid + 256 * u, r = e >> 4, c4 = e & 15;
        const f4 v = *reinterpret_cast<const f4*>(x + (r0 + r) * n + c0 + 4 * c4);
#pragma unroll
        for (int i = 0; i < 4; ++i) t[r][4 * c4 + i] = v[i];
    }
    __syncthreads();
    // Bt row j = c0 + jj holds B[r0 .. r0+63][c0 + jj]: 64 halves = 8 chunks of 8
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int e = tid + 256 * u, jj = e >> 3, ch = e & 7;
        uint16_t h[8], l[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            l[i] = 0;
            Conv<MODE>::run(t[8 * ch + i][jj], s, &h[i], &l[i]);
        }
        uint4 hp, lp;
        hp.x = h[0] | uint32_t(h[1]) << 16;
        hp.y = h[2] | uint32_t(h[3]) << 16;
        hp.z = h[4] | uint32_t(h[5]) << 16;
        hp.w = h[6] | uint32_t(h[7]) << 16;
        const int64_t off = (c0 + jj) * n + r0 + 8 * ch;
        *reinterpret_cast<uint4*>(hi + off) = hp;
        if (MODE == kPrecF16x3) {
            lp.x = l[0] | uint32_t(l[1]) << 16;
            lp.y = l[2] | uint32_t(l[3]) << 16;
            lp.z = l[4] | uint32_t(l[5]) << 16;
            lp.w = l[6] | uint32_t(l[7]) << 16;
            *reinterpret_cast<uint4*>(lo + off) = lp;
        }
    }
}

// A: row-major, 4 elements per thread per step (n % 4 == 0)
template <int MODE>
__global__ __launch_bounds__(256) void split_rows_kernel(const float* __restrict__ x, int64_t count,
                                                         const int32_t* __restrict__ exps, uint16_t* __restrict__ hi,
                                                         uint16_t* __restrict__ lo) {
    const float s = MODE == kPrecF16x3 ? ldexpf(1.0f, exps[0]) : 1.0f;
    const f4* x4 = reinterpret_cast<const f4*>(x);
    for (int64_t q = int64_t(blockIdx.x) * 256 + threadIdx.x; q < count / 4; q += int64_t(gridDim.x) * 256)
        split_row4<MODE>(x4, q, s, hi, lo);
}

// B transposed, one tile per block
template <int MODE>
__global__ __launch_bounds__(256) void split_transpose_kernel(const float* __restrict__ x, int64_t n,
                                                              const int32_t* __restrict__ exps,
                                                              uint16_t* __restrict__ hi, uint16_t* __restrict__ lo) {
    __shared__ float t[64][65];
    const float s = MODE == kPrecF16x3 ? ldexpf(1.0f, exps[1]) : 1.0f;
    split_tile<MODE>(x, n, int64_t(blockIdx.y) * 64, int64_t(blockIdx.x) * 64, s, hi, lo, t, threadIdx.x);
}

// The choice of launch_split_choice, then both BF16 planes if they are taken:
// blockIdx.y = 0 the rows of A, 1 the tiles of B.  Every block works the choice
// out by itself from the same 2x2 blocks of tiles and k, one per thread (spread
// evenly by multiples of the powers of a constant); block 0 writes it down.  A product
// that does not take the planes pays for this, so the grid is one large block a CU,
// each with few reads (2048 blocks of 256 threads took 18 us to end).
constexpr int kChoiceThreads = 1024;  // and blocks of tiles looked at
constexpr int kChoiceBlocks = 128;

__global__ __launch_bounds__(kChoiceThreads) void split_choice_kernel(const float* __restrict__ a,
                                                                      const float* __restrict__ b, int64_t n,
                                                                      int64_t bdim, FormChoice ch, SplitLayout L) {
    constexpr int kTiles = kChoiceThreads / 256;  // of B at a time
    __shared__ float t[kTiles][64][65];
    __shared__ int any[kChoiceThreads / 64], kept[kChoiceThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // multiples of 2^32 / 1.2207440846, its square and its cube
    auto at = [&](uint32_t step, int64_t len) {
        return int64_t((uint64_t(uint32_t(tid) * step + (step >> 1)) * uint64_t(len)) >> 32);
    };
    const int64_t i = 2 * at(3518319155u, bdim / 2), k = at(2882110345u, bdim), j = 2 * at(2360945575u, bdim / 2);
    const double* pa = ch.na + i * ch.ld + k;
    const double* pb = ch.nb + k * ch.ld + j;
    int mine = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) mine += pa[(q >> 1) * ch.ld] * pb[q & 1] >= ch.tau ? 1 : 0;
    const uint64_t hit = __ballot(mine > 0);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mine += __shfl_xor(mine, o);
    if (lane == 0) {
        any[wave] = __popcll(hit);
        kept[wave] = mine;
    }
    __syncthreads();
    int unions = 0, pairs = 0;  // of kChoiceThreads and of four times as many
#pragma unroll
    for (int w = 0; w < kChoiceThreads / 64; ++w) {
        unions += any[w];
        pairs += kept[w];
    }
    const bool planes = int64_t(16 * unions - 3 * pairs) * bdim >= int64_t(ch.weight) * 4 * kChoiceThreads &&
                        !(ch.full_fp32 && pairs == 4 * kChoiceThreads);
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        if (tid == 0) *ch.form = planes ? 1 : 0;
        for (int64_t w = tid; w < ch.clear_count; w += kChoiceThreads) ch.clear[w] = 0;
    }
    if (!planes) return;
    if (blockIdx.y == 0) {
        const f4* x4 = reinterpret_cast<const f4*>(a);
        const int64_t step = int64_t(gridDim.x) * kChoiceThreads, count = n * n / 4;
#pragma unroll 4
        for (int64_t q = int64_t(blockIdx.x) * kChoiceThreads + tid; q < count; q += step)
            split_row4<kPrecBf16>(x4, q, 1.0f, L.a_hi, nullptr);
        return;
    }
    const int64_t side = n / 64, sub = tid >> 8;  // side is even: four tiles at a time come out even
    for (int64_t e = int64_t(blockIdx.x) * kTiles; e < side * side; e += int64_t(gridDim.x) * kTiles) {
        split_tile<kPrecBf16>(b, n, (e + sub) / side * 64, (e + sub) % side * 64, 1.0f, L.bt_hi, nullptr, t[sub],
                              tid & 255);
        __syncthreads();  // t is used again
    }
}

hipError_t launch_split_choice(const float* a, const float* b, int64_t n, int64_t bdim, const FormChoice& choice,
                               const SplitLayout& L, hipStream_t s) {
    if (n % 128 != 0 || bdim * 64 != n || !choice.form) return hipErrorInvalidValue;
    split_choice_kernel<<<dim3{unsigned(kChoiceBlocks), 2u, 1u}, kChoiceThreads, 0, s>>>(a, b, n, bdim, choice, L);
    return hipGetLastError();
}

hipError_t launch_split_scales(int64_t bdim, int lv, const double* pyr_a, const double* pyr_b, int32_t* header,
                                      hipStream_t s) {
    // the header holds exps[2] (bytes 0..7) and the two maxima (bytes 8..23)
    split_scale_kernel<<<2, kScaleThreads, 0, s>>>(pyr_a, pyr_b, bdim, lv, header,
                                                   reinterpret_cast<double*>(header + 2));
    return hipGetLastError();
}

static hipError_t launch_split_planes(const float* a, const float* b, int64_t n, int precision, const SplitLayout& L,
                                      hipStream_t s) {
    const int64_t n4 = n * n / 4;
    const unsigned rows_grid = unsigned(n4 < 2048 * 256 ? (n4 + 255) / 256 : 2048);
    const dim3 tgrid{unsigned(n / 64), unsigned(n / 64), 1u};
    if (precision == kPrecBf16) {
        split_rows_kernel<kPrecBf16><<<rows_grid, 256, 0, s>>>(a, n * n, L.exps, L.a_hi, nullptr);
        split_transpose_kernel<kPrecBf16><<<tgrid, 256, 0, s>>>(b, n, L.exps, L.bt_hi, nullptr);
    } else {
        split_rows_kernel<kPrecF16x3><<<rows_grid, 256, 0, s>>>(a, n * n, L.exps, L.a_hi, L.a_lo);
        split_transpose_kernel<kPrecF16x3><<<tgrid, 256, 0, s>>>(b, n, L.exps, L.bt_hi, L.bt_lo);
    }
    return hipGetLastError();
}

hipError_t launch_split(const float* a, const float* b, int64_t n, int64_t bdim, int lv, const double* pyr_a,
                        const double* pyr_b, int precision, const SplitLayout& L, hipStream_t s) {
    hipError_t e = launch_split_scales(bdim, lv, pyr_a, pyr_b, L.exps, s);
    if (e != hipSuccess) return e;
    return launch_split_planes(a, b, n, precision, L, s);
}

}  // namespace spamm

// Reduced-precision leaf products (leaf 64, N a multiple of 128) straight from
// the FP32 inputs: bf16, or FP16 hi + lo with three products per k-step, the
// operand values and the order of sums of split.hip and multiply_lowp.hip, so
// that C is bitwise the same as through the split planes.
//
// One workgroup of four waves computes 64T x 64T of C, the kept k either tested on
// the leaf norms by the workgroup itself (kKept, the one-call path: no plan
// launch) or taken from a plan's items (kPlanned).  Operands come through
// registers in stages of KC = 64 / T k: A rows and B columns are loaded as FP32,
// converted once and written to LDS as planes of k-contiguous halves (B
// transposed on the way), in flight while the stage before is multiplied.
//  T = 2: 2x2 leaf tiles, one per wave.  Per 64 k the four waves convert 16,384
//         elements, write 64 KiB of LDS and read 128 for four leaf products.
//  T = 1: one leaf tile, a 32x32 quadrant per wave; four times the blocks.
// One LDS stage and three workgroups per CU: two stages and two workgroups
// measured the same or slower (N = 8192 with every pair kept 2,960 against
// 3,016 us, F16X3).  The kernel this replaced converted at the operand reads, in
// each of the four waves that read an operand.
//
// Bound by the loads: a macro tile reads 64 KiB per 64 k from L2 and past it, and
// at N = 16384, decay 0.01, half of that misses L2 (blocks that share panels are
// at different k); the matrix cores are busy 45 % of the time (F16X3; 15 % BF16).
// Loads are 16 bytes a lane: B by 8-byte loads, which suit the transposition,
// read L2 at 30 bytes a clock and CU against 52.
// One call, F16X3: N = 16384, decay 0.01, tau 1e-6 2,000 -> 1,261 us (314 of it the
// norms); 1024, 0.0126 122 -> 46; 4096, 0.0126 299 -> 170; 12800, 0.0126 1,090 ->
// 759.  BF16: 16384 1,546 -> 1,196; 1024 85 -> 36; 2816, 0.0126 127 -> 94.  With
// every pair kept, N = 8192: F16X3 3,650 -> 2,620, BF16 2,300 -> 1,890.
// Wide bands in BF16 go by planes where the caller has room for them (bf16_choice).
// hi and lo by mixed-precision FMAs, two instructions an element instead of three,
// measured 2 to 10 % slower.
#include <hip/hip_runtime.h>

#include "block_multiply.h"
#include "device.h"
#include "dma.h"
#include "internal.h"

namespace spamm {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b4 __attribute__((ext_vector_type(4)));

constexpr int kConvertThreads = 256;
constexpr int kConvertEntries = 1024;  // leaf tiles per side at most

template <int MODE, int T>
struct ConvertGeom {
    static constexpr bool F16 = MODE == kPrecF16x3;
    static constexpr int NP = F16 ? 2 : 1;  // planes per operand
    static constexpr int KC = 64 / T, R = 64 * T;
    static constexpr int PLANE = R * KC * 2;  // bytes
    static constexpr int STAGE = 2 * NP * PLANE;
    static constexpr int LIST = 2 * kConvertEntries;
};

// Byte of 16-byte chunk c (8 halves) of row r in a plane.  The 8 rows that a
// group of lanes reads at one c, and the rows 4 i + const (i = 0..7) that a group
// writes, fall in different banks.
template <int T>
__device__ __forceinline__ int plane_at(int r, int c) {
    if constexpr (T == 2)
        return (r >> 1) * 128 + ((((r & 1) << 2 | c) ^ (((r >> 1) ^ (r >> 4)) & 7)) * 16);
    else
        return r * 128 + ((c ^ ((r ^ (r >> 3)) & 7)) * 16);
}

// Strips run over so many columns that a round is the 96 blocks that an XCD's
// CUs hold at a time: these start together and stay near the same k, so the panels
// that they share stay in L2.  Strips of two rows, whose rounds span the whole
// band of a decaying matrix (F16X3, N = 16384, decay 0.01: 1,284 us, 1,343 at four
// rows and 24 columns, 1,392 at eight and eight); BF16, whose loads weigh more,
// four rows on the grids that give every XCD about two strips (N = 16384, decay
// 0.01 1,234 against 1,170 us; every pair kept, N = 8192 2,883 against 1,869, 10112
// 5,840 against 4,527).
template <int MODE>
BlockOrder convert_order(int nb) {
    return MODE == kPrecBf16 && nb >= 60 ? BlockOrder{4, 24} : BlockOrder{2, 48};
}

template <int MODE, int T, int FROM>
__global__ __launch_bounds__(kConvertThreads, 3) void multiply_convert_kernel(
    const float* __restrict__ A, const float* __restrict__ B, const int32_t* __restrict__ exps, float* __restrict__ C,
    int64_t n, int bdim, int nb, const double* __restrict__ na, const double* __restrict__ nbm, int64_t ld, double tau,
    unsigned long long* __restrict__ pairs, const uint32_t* __restrict__ items, const int32_t* __restrict__ uprefix,
    BlockOrder order, const int32_t* planes) {
    if (planes != nullptr && *planes != 0) return;
    using G = ConvertGeom<MODE, T>;
    constexpr bool F16 = G::F16;
    constexpr int KC = G::KC, R = G::R, PLANE = G::PLANE;
    __shared__ __attribute__((aligned(1024))) char lds[G::STAGE + G::LIST + 32];
    uint16_t* list = reinterpret_cast<uint16_t*>(lds + G::STAGE);
    int* wsum = reinterpret_cast<int*>(lds + G::STAGE + G::LIST);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const BlockAt at = block_at(blockIdx.x, nb, order);
    if (!at.valid) return;
    const int I = at.I, J = at.J;

    // ---- the leaf k with a kept product, ascending: list[e] = k << 4 | tiles
    int count = 0, kept = 0;
    {
        const uint32_t* plan = nullptr;
        int end = bdim;
        if constexpr (FROM == kPlanned) {
            const int64_t m = T == 2 ? int64_t(I) * nb + J : int64_t(I >> 1) * (nb >> 1) + (J >> 1);
            plan = items + uprefix[m];
            end = uprefix[m + 1] - uprefix[m];
        }
        for (int e0 = 0; e0 < end; e0 += kConvertThreads) {
            const int e = e0 + tid;
            uint32_t mem = 0, k = uint32_t(e);
            if (e < end) {
                if constexpr (FROM == kPlanned) {
                    k = (plan[e] >> 4) & 1023u;
                    mem = T == 2 ? plan[e] & 15u : (plan[e] >> (2 * (I & 1) + (J & 1))) & 1u;
                } else {
                    double nav[T], nbv[T];
#pragma unroll
                    for (int t = 0; t < T; ++t) {
                        nav[t] = na[(T * I + t) * ld + e];
                        nbv[t] = nbm[e * ld + T * J + t];
                    }
#pragma unroll
                    for (int t = 0; t < T * T; ++t)
                        if (nav[t / T] * nbv[t % T] >= tau) mem |= 1u << t;
                    kept += __popc(mem);
                }
            }
            const uint64_t bal = __ballot(mem != 0);
            if (lane == 0) wsum[wave] = __popcll(bal);
            __syncthreads();
            int pos = count + __popcll(bal & (lane == 0 ? 0ull : (~0ull >> (64 - lane))));
#pragma unroll
            for (int w = 0; w < kConvertThreads / 64; ++w) {
                if (w < wave) pos += wsum[w];
                count += wsum[w];
            }
            if (mem) list[pos] = uint16_t(k << 4 | mem);
            __syncthreads();
        }
    }
    count = __builtin_amdgcn_readfirstlane(count);
    if constexpr (FROM == kKept) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) kept += __shfl_xor(kept, o);
        if (lane == 0 && kept) atomicAdd(pairs, static_cast<unsigned long long>(kept));
    }
    if (count == 0) {
        constexpr int Q = R / 4;  // chunks of a row
#pragma unroll
        for (int u = 0; u < R * Q / kConvertThreads; ++u) {
            const int e = u * kConvertThreads + tid;
            float* at = C + (int64_t(I) * R + e / Q) * n + J * R + 4 * (e % Q);
            __builtin_nontemporal_store(f4{0, 0, 0, 0}, reinterpret_cast<f4_dw*>(at));  // c may be 4-byte aligned
        }
        return;
    }

    const float sa = F16 ? ldexpf(1.0f, exps[0]) : 1.0f, sb = F16 ? ldexpf(1.0f, exps[1]) : 1.0f;
    const float inv = F16 ? ldexpf(1.0f, -(exps[0] + exps[1])) : 1.0f;

    // ---- this thread's part of a stage: of A four k of four rows, of B four
    // columns of four k
    constexpr int AL = KC / 4, AR = kConvertThreads / AL;  // lanes per A row, rows per pass
    const int ar = tid / AL, aq = tid % AL;
    uint32_t a_off = uint32_t((int64_t(ar) * n + 4 * aq) * 4);
    // B: rows 4 bk .. + 3, columns 4 bc .. + 3 of the stage
    const int bk = (lane >> 3 & 1) + (T == 2 ? 2 * wave : 4 * wave + 2 * (lane >> 5));
    const int bc = (lane & 7) + (T == 2 ? lane >> 4 << 3 : (lane >> 4 & 1) << 3);
    uint32_t b_off = uint32_t((int64_t(4) * bk * n + 4 * bc) * 4);
    int a_at[4], b_at[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        a_at[p] = plane_at<T>(ar + p * AR, aq >> 1) + (aq & 1) * 8;
        b_at[p] = G::NP * PLANE + plane_at<T>(4 * bc + p, bk >> 1) + (bk & 1) * 8;
    }

    f4 xa[4], xb[4];
    auto load = [&](int k) {  // k: first of the stage
        const char* pa = reinterpret_cast<const char*>(A + int64_t(I) * R * n + k);
        const char* pb = reinterpret_cast<const char*>(B + int64_t(k) * n + J * R);
        // opaque: else extended to 64 bits outside the loop, a vector add a load
        asm volatile("" : "+v"(a_off), "+v"(b_off));
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            xa[p] = *reinterpret_cast<const f4*>(pa + int64_t(p) * AR * n * 4 + a_off);
            xb[p] = *reinterpret_cast<const f4*>(pb + int64_t(p) * n * 4 + b_off);
        }
    };
    // four k of one row (or column) to their place in the planes
    auto put = [&](char* at, const f4& x, float scale) {
        if constexpr (F16) {
            const f4 y = x * scale;
            const h4 hi = __builtin_convertvector(y, h4);
            const h4 lo = __builtin_convertvector(y - __builtin_convertvector(hi, f4), h4);
            *reinterpret_cast<h4*>(at) = hi;
            *reinterpret_cast<h4*>(at + PLANE) = lo;
        } else {
            *reinterpret_cast<b4*>(at) = __builtin_convertvector(x, b4);
        }
    };
    auto commit = [&](char* st) {
#pragma unroll
        for (int p = 0; p < 4; ++p) put(st + a_at[p], xa[p], sa);
#pragma unroll
        for (int p = 0; p < 4; ++p) put(st + b_at[p], f4{xb[0][p], xb[1][p], xb[2][p], xb[3][p]}, sb);
    };

    // ---- this wave's part of C: 32T x 32T at (wr, wc), T x T MFMA tiles
    const int wr = (wave >> 1) * 32 * T, wc = (wave & 1) * 32 * T;
    const int ir = lane & 31, g = lane >> 5;
    f16v acc[T][T];
#pragma unroll
    for (int u = 0; u < T; ++u)
#pragma unroll
        for (int v = 0; v < T; ++v)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[u][v][r] = 0.0f;
    auto compute = [&](const char* st) {
#pragma unroll
        for (int s = 0; s < KC / 16; ++s) {
            using V = typename std::conditional<F16, h8, b8>::type;
            V ah[T], al[T], bh[T], bl[T];
#pragma unroll
            for (int u = 0; u < T; ++u) {
                const char* pa = st + plane_at<T>(wr + 32 * u + ir, 2 * s + g);
                const char* pb = st + G::NP * PLANE + plane_at<T>(wc + 32 * u + ir, 2 * s + g);
                ah[u] = *reinterpret_cast<const V*>(pa);
                bh[u] = *reinterpret_cast<const V*>(pb);
                if constexpr (F16) {
                    al[u] = *reinterpret_cast<const V*>(pa + PLANE);
                    bl[u] = *reinterpret_cast<const V*>(pb + PLANE);
                }
            }
            if constexpr (F16) {
#pragma unroll
                for (int q = 0; q < T * T; ++q)
                    acc[q / T][q % T] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[q / T], bh[q % T], acc[q / T][q % T], 0, 0, 0);
#pragma unroll
                for (int q = 0; q < T * T; ++q)
                    acc[q / T][q % T] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[q / T], bl[q % T], acc[q / T][q % T], 0, 0, 0);
#pragma unroll
                for (int q = 0; q < T * T; ++q)
                    acc[q / T][q % T] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al[q / T], bh[q % T], acc[q / T][q % T], 0, 0, 0);
            } else {
#pragma unroll
                for (int q = 0; q < T * T; ++q)
                    acc[q / T][q % T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[q / T], bh[q % T], acc[q / T][q % T], 0, 0, 0);
            }
        }
    };

    // stage i: part i % T of entry i / T
    const int stages = count * T;
    auto entry = [&](int i) { return __builtin_amdgcn_readfirstlane(int(list[i / T])); };
    auto first_k = [&](int pk, int i) { return (pk >> 4) * 64 + (i % T) * KC; };
    int pk = entry(0);
    load(first_k(pk, 0));
    for (int i = 0; i < stages; ++i) {
        const int next = i + 1 < stages ? entry(i + 1) : 0;
        commit(lds);
        if (i + 1 < stages) load(first_k(next, i + 1));  // lands while this stage is multiplied
        __syncthreads();
        if (T == 1 || ((pk >> wave) & 1)) {
            __builtin_amdgcn_s_setprio(1);  // a wave with MFMAs to issue goes ahead of those that convert
            compute(lds);
            __builtin_amdgcn_s_setprio(0);
        }
        __syncthreads();
        pk = next;
    }
#pragma unroll
    for (int u = 0; u < T; ++u)
#pragma unroll
        for (int v = 0; v < T; ++v) {
            float* dst = C + (int64_t(I) * R + wr + 32 * u + 4 * g) * n + J * R + wc + 32 * v + ir;
#pragma unroll
            for (int r = 0; r < 16; ++r) __builtin_nontemporal_store(acc[u][v][r] * inv, &dst[(8 * (r >> 2) + (r & 3)) * n]);
        }
}
}  // namespace

// BF16 with room for planes.  From the FP32 inputs every workgroup loads four bytes
// an element; once the planes are there, two, for a pass over A and B (700 us at N =
// 16384) and a plan.  Both read a panel of A and of B for every k of a 2x2 block's
// union, U of them for V kept pairs per output tile.  Blocks of wide bands, at
// different k, share few panels in L2; where tiles are scattered (U well above V)
// nothing is shared, so U - V counts thrice on top of U.  One call, planes against
// FP32 inputs, V (bands: U = V + 1, scattered: U given):
//  N = 4608, band 57 476 and 395 us, scattered 18 (41) 293 and 342: weight 90,
//  scattered tiles only;
//  N = 6016, band 40 562 and 523, 56 686 and 729, scattered 15 (39) 477 and 590:
//  weight 58;
//  N = 7040, band 36 719 and 712, 53 887 and 1,022, scattered 7 (21) 457 and 531:
//  weight 45;
//  N = 8192, band 23 699 and 625, 49 1,131 and 1,272, 121 2,324 and 2,998, scattered 5
//  (17) 572 and 617, 21 (53) 1,008 and 1,678; 12288, band 24 1,592 and 1,524, 38
//  2,089 and 2,332, scattered 17 (50) 2,187 and 3,995; 16384, band 19 2,555 and 2,215,
//  30 3,251 and 3,432, 137 10,166 and 16,812: weight 30.
// With every pair kept all blocks start at k = 0 and share: where the strips of
// block_at come out even, N = 8192 2,278 and 1,864, 12288 7,291 and 6,830, but 11008
// 5,338 and 6,456, 11904 6,689 and 6,995, 20480 32,552 and 38,377.
// The choice costs a product that stays with its FP32 inputs 8 us, three launches
// that end at once: decay 0.1, N = 4352 45 -> 52, 8192 142 -> 150, 16384 550 -> 558.
// Below N = 4352 planes gain nothing (4096, scattered 17 (37): 228 and 224).
constexpr int64_t kChoiceMinN = 4352, kFullFp32MinN = 7680, kEvenMinN = 8192, kFullFp32MaxN = 16384;
bool bf16_choice(int64_t n, int64_t bdim, FormChoice* choice) {
    if (n < kChoiceMinN) return false;
    const int side = int(bdim / 2), dealt = dealt_rows(side, convert_order<kPrecBf16>(side).H);
    choice->weight = n < 5632 ? 90 : n < 6400 ? 58 : n < 8192 ? 45 : 30;
    choice->full_fp32 =
        n >= kFullFp32MinN && n <= kFullFp32MaxN && (dealt == side || (dealt > side && n < kEvenMinN));
    return true;
}

namespace {

// One leaf tile per workgroup up to this N, 2x2 above: four times the blocks
// against half the loads and LDS reads per product (decay 0.0126 and 0.1, one leaf
// tile against 2x2: F16X3 N = 1536 77 and 42 against 87 and 47 us, N = 2816 163
// and 51 against 128 and 54; BF16 1152 44 and 33 against 51 and 35, 2048 76
// and 37 against 67 and 38).
template <int MODE>
constexpr int64_t kConvertSmallN = MODE == kPrecF16x3 ? 2048 : 1536;

template <int MODE, int FROM>
hipError_t launch(const float* a, const float* b, const int32_t* exps, float* c, int64_t n, int64_t bdim,
                  const double* na, const double* nb, int64_t ld, double tau, int64_t* pairs, const uint32_t* items,
                  const int32_t* uprefix, const int32_t* planes, hipStream_t s) {
    if (n % 128 || n < 128 || bdim * 64 != n || bdim > kConvertEntries) return hipErrorInvalidValue;
    static int scratch_state[2] = {0, 0};
    const bool small = n <= kConvertSmallN<MODE>;
    const hipError_t ce = small ? check_no_scratch(multiply_convert_kernel<MODE, 1, FROM>, &scratch_state[0])
                                : check_no_scratch(multiply_convert_kernel<MODE, 2, FROM>, &scratch_state[1]);
    if (ce != hipSuccess) return ce;
    auto* count = reinterpret_cast<unsigned long long*>(pairs);
    const int side = int(small ? bdim : bdim / 2);
    const BlockOrder order = convert_order<MODE>(side);
    if (small)
        multiply_convert_kernel<MODE, 1, FROM><<<block_grid(side, order), kConvertThreads, 0, s>>>(
            a, b, exps, c, n, int(bdim), side, na, nb, ld, tau, count, items, uprefix, order, planes);
    else
        multiply_convert_kernel<MODE, 2, FROM><<<block_grid(side, order), kConvertThreads, 0, s>>>(
            a, b, exps, c, n, int(bdim), side, na, nb, ld, tau, count, items, uprefix, order, planes);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_convert_test(const float* a, const float* b, int precision, const int32_t* exps, float* c, int64_t n,
                               int64_t bdim, const double* na, const double* nb, int64_t ld, double tau,
                               int64_t* pairs, const int32_t* planes, hipStream_t s) {
    return precision == kPrecBf16
               ? launch<kPrecBf16, kKept>(a, b, exps, c, n, bdim, na, nb, ld, tau, pairs, nullptr, nullptr, planes, s)
               : launch<kPrecF16x3, kKept>(a, b, exps, c, n, bdim, na, nb, ld, tau, pairs, nullptr, nullptr, planes, s);
}

hipError_t launch_convert_plan(const float* a, const float* b, int precision, const int32_t* exps, float* c, int64_t n,
                               int64_t bdim, const uint32_t* items, const int32_t* uprefix, hipStream_t s) {
    return precision == kPrecBf16
               ? launch<kPrecBf16, kPlanned>(a, b, exps, c, n, bdim, nullptr, nullptr, 0, 0.0, nullptr, items, uprefix,
                                             nullptr, s)
               : launch<kPrecF16x3, kPlanned>(a, b, exps, c, n, bdim, nullptr, nullptr, 0, 0.0, nullptr, items, uprefix,
                                              nullptr, s);
}

}  // namespace spamm

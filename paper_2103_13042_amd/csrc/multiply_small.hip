// Small products: the threshold test of Algorithm 1 and the multiply of the
// kept pairs in one launch after the leaf norm pass, instead of the plan,
// schedule, multiply and fixup launches of the general path.  At these sizes
// every launch of the general path is a few microseconds of ramp and drain for
// well under a microsecond of work, and the multiply has too few macro tiles
// to give every SIMD more than one wave.
//
// One workgroup of sixteen waves per 64x64 block (I, J) of C, whatever the
// leaf.  k is walked in entries of 32 (at most 64 of them, one per lane): an
// entry stages the block's 64x32 part of A and 32x64 part of B as four 32x32
// operand tiles, rows 2I + {0, 1} of A and columns 2J + {0, 1} of B.
//  * every wave tests the leaf products of its lane's entry, nA * nB >= tau
//    (the comparison of the plan kernel, on the same leaf norms, so the kept
//    pairs are the same; the pyramid only skips subtrees whose leaf products
//    all fail).  Leaf 32: one product per quadrant of the block; leaf 64 and
//    128: one for the whole block; leaf 16: one for each of 16 output tiles
//    and both halves of the entry.  The entries that any product keeps form
//    the union list; block by block the kept pairs are added to the counter;
//  * leaf 32 and up: the waves are four k-groups of four (wave w: k-group
//    g = w >> 2, quadrant q = (w + g) & 3, so the four waves of a SIMD hold the
//    four quadrants and every SIMD gets a quarter of each quadrant's entries).
//    A step takes four entries of the list, one per group; each wave
//    accumulates its own in ascending k on v_mfma_f32_32x32x2f32 and the
//    groups' partial tiles are added in group order through LDS, so the result
//    does not depend on timing;
//  * leaf 16: one output tile per wave, v_mfma_f32_16x16x4f32 in the steps and
//    order of the leaf-16 kernel of the general path, so C is bitwise its C;
//    a step takes two entries.
// Tiles with nothing kept are written as zeros (beta = 0).
//
// multiply_strip_kernel (n <= 320: at most ten entries): all operand tiles of
// the block fit in LDS, so they are loaded at once, before the test is known,
// and nothing waits on memory a second time.  multiply_small_kernel (larger
// n): two steps of operand tiles in LDS, the next step's loads in flight
// during this step's MFMAs.
//
// Bound by latency up to n = 1024 (the test, the first operand loads, the
// reduction: about 7 us around 5 us of MFMA work in the fullest blocks), by
// the rounds of blocks above.  One call, exp decay 0.05, tau 1e-6: n = 1024
// leaf 32 21.1 -> 20.2 us, leaf 16 39.7 -> 23.3, leaf 64 51.9 -> 22.6; n = 1000
// leaf 128 99.7 -> 29.0; n = 203 leaf 32 37.3 -> 15.2 (that and smaller calls
// take what the host needs to enqueue them).
//
// Rows that are only 4-byte aligned (VEC false) are read by 16-byte loads at
// that alignment; a chunk that crosses the matrix's edge reads the last four
// columns and shifts them into place.
#include <hip/hip_runtime.h>

#include "device.h"
#include "dma.h"
#include "internal.h"

namespace spamm {

namespace {
constexpr int kSmallWaves = 16;
constexpr int kSmallThreads = kSmallWaves * 64;
constexpr int kSmallGroups = kSmallWaves / 4;
constexpr int kSmallTile = 32 * 32;     // floats of an operand tile
constexpr int kStripEntries = 10;       // 16 KiB of LDS each
constexpr int kStripMaxN = 32 * kStripEntries;

// entries per step of the staged kernel: two steps in LDS, and at leaf 16 (no
// k-groups) two workgroups per CU
template <int LEAF>
struct SmallStep {
    static constexpr int ENTRIES = LEAF == 16 ? 2 : kSmallGroups;
    static constexpr int OCC = LEAF == 16 ? 2 : 1;
};

// Where operand tile `role` of an entry lies: rows row0 + k * row_k of X from
// column col0 + k * col_k, the same arithmetic for A and B, so that no branch
// on the role stands between a load and the next one.
struct SmallTile {
    const float* X;
    int row0, row_k, col0, col_k;
    __device__ __forceinline__ SmallTile(const float* A, const float* B, int I, int J, int role) {
        const bool a = role < 2;
        X = a ? A : B;
        row0 = a ? 64 * I + 32 * role : 0;
        row_k = a ? 0 : 32;
        col0 = a ? 0 : 64 * J + 32 * (role - 2);
        col_k = a ? 32 : 0;
    }
};

// Chunk e (0 .. 255) of an operand tile of entry k: row e / 8, columns 4 (e % 8)
// .. + 3.  load() issues the load (of any address inside the matrix if the
// chunk lies outside or is not wanted; n >= 4); value() puts its floats in
// place, zeros outside the matrix, and is called when the chunk is needed.
template <bool VEC>
struct SmallChunk {
    f4 x;
    int back;  // columns past the matrix's edge, 4 or more: nothing of it is wanted
    __device__ __forceinline__ void load(const SmallTile& t, int64_t n, int k, int e, bool want) {
        const int row = t.row0 + k * t.row_k + (e >> 3), col = t.col0 + k * t.col_k + 4 * (e & 7);
        const int over = VEC ? 0 : (col + 4 > int(n) ? col + 4 - int(n) : 0);
        const bool in = want && row < int(n) && col < int(n);
        back = in ? over : 4;
        const float* p = t.X + (in ? int64_t(row) * n + col - over : 0);
        if constexpr (VEC)
            x = *reinterpret_cast<const f4*>(p);
        else
            x = *reinterpret_cast<const f4_dw*>(p);
    }
    __device__ __forceinline__ f4 value() const {
        f4 v;
        if constexpr (VEC) {
            v = back == 0 ? x : f4{0.0f, 0.0f, 0.0f, 0.0f};
        } else {
            v.x = back == 0 ? x.x : back == 1 ? x.y : back == 2 ? x.z : back == 3 ? x.w : 0.0f;
            v.y = back == 0 ? x.y : back == 1 ? x.z : back == 2 ? x.w : 0.0f;
            v.z = back == 0 ? x.z : back == 1 ? x.w : 0.0f;
            v.w = back == 0 ? x.w : 0.0f;
        }
        return v;
    }
};

// Operand tiles in LDS, rows of 32 floats, arranged so that the two (leaf 16:
// four) lane groups of an MFMA operand read fall in different banks.  A tiles:
// 16-byte chunks XOR-swizzled by the row.  B tiles: rows 16 .. 31 trade places
// in pairs (leaf 16: rows with bit 3 set do, and rows with bit 2 set have
// their column halves exchanged).
__device__ __forceinline__ int a_at(int row, int chunk) { return row * 32 + 4 * (chunk ^ (row & 7)); }

template <int LEAF>
__device__ __forceinline__ int b_at(int k, int col) {
    if (LEAF == 16) return (k ^ ((k >> 3) & 1)) * 32 + (col ^ (16 * ((k >> 2) & 1)));
    return (k ^ ((k >> 4) & 1)) * 32 + col;
}

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

// the quadrants of an entry with anything kept
template <int LEAF>
__device__ __forceinline__ uint32_t small_quadrants(uint32_t mem) {
    if constexpr (LEAF == 16)
        return (mem & 0xFFu ? 1u : 0u) | (mem & 0xFF00u ? 2u : 0u) | (mem & 0xFF0000u ? 4u : 0u) |
               (mem & 0xFF000000u ? 8u : 0u);
    else
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
    // quadrant (wa, wb) of the entry whose four operand tiles are at t.  Lane
    // (ir, g) supplies k = 16 g + u of MFMA step u: A[ir][16g + u], B[16g + u][ir]
    __device__ __forceinline__ void multiply(const float* t, uint32_t mem, int wave, int q, int lane) {
        if (!((mem >> q) & 1)) return;
        const int ir = lane & 31, g = lane >> 5;
        const float* ta = t + (q >> 1) * kSmallTile;
        // b_at(16 g + u, ir) for even and odd u, as offsets of u
        const float* tb = t + (2 + (q & 1)) * kSmallTile + 16 * g * 32 + ir;
        const float *tb0 = tb + 32 * g, *tb1 = tb - 32 * g;
        f4 av[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) av[v] = *reinterpret_cast<const f4*>(ta + a_at(ir, 4 * g + v));
#pragma unroll
        for (int u = 0; u < 16; ++u)
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[u >> 2][u & 3], (u & 1 ? tb1 : tb0)[u * 32], acc, 0, 0, 0);
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
    // output tile (a, b) = (wave >> 2, wave & 3) of the block: lane (r, g)
    // supplies k = 4 g + s of each half's MFMA step s
    __device__ __forceinline__ void multiply(const float* t, uint32_t mem, int wave, int, int lane) {
        const int a = wave >> 2, b = wave & 3, r = lane & 15, g = lane >> 4;
        const uint32_t keep = mem >> (8 * (2 * (a >> 1) + (b >> 1)) + 4 * (a & 1) + 2 * (b & 1));
        const float* ta = t + (a >> 1) * kSmallTile;
        const float* tb = t + (2 + (b >> 1)) * kSmallTile;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (!((keep >> h) & 1)) continue;
            const f4 av = *reinterpret_cast<const f4*>(ta + a_at(16 * (a & 1) + r, 4 * h + g));
            float bv[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) bv[s] = tb[b_at<16>(16 * h + 4 * g + s, 16 * (b & 1) + r)];
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s], bv[s], acc, 0, 0, 0);
        }
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

template <int LEAF>
__device__ __forceinline__ void small_commit(float* t, int role, int e, f4 v) {
    const int r = e >> 3, c4 = e & 7;
    *reinterpret_cast<f4*>(t + (role < 2 ? a_at(r, c4) : b_at<LEAF>(r, 4 * c4))) = v;
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

template <int LEAF, bool VEC>
__global__ __launch_bounds__(kSmallThreads, 1) void multiply_strip_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, int64_t n, int bdim, int blocks,
    const double* __restrict__ na, const double* __restrict__ nb, int64_t ld, double tau,
    unsigned long long* __restrict__ pairs) {
    __shared__ __attribute__((aligned(16))) float strip[kStripEntries][4][kSmallTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int I = blockIdx.x / blocks, J = blockIdx.x - I * blocks;
    const int grp = wave >> 2, q = (wave + grp) & 3;
    const int entries = (int(n) + 31) / 32;

    // four waves a tile: chunk v belongs to entry v, role wave / 4
    const int role = wave >> 2;
    const SmallTile of(A, B, I, J, role);
    SmallChunk<VEC> x[kStripEntries];
#pragma unroll
    for (int v = 0; v < kStripEntries; ++v) x[v].load(of, n, v, tid & 255, v < entries);
    int cnt;
    const uint32_t mem = small_test<LEAF>(na, nb, ld, bdim, int(n), I, J, tau, lane, &cnt);
    if (wave == 0) small_count(cnt, lane, pairs);
    const SmallUnion uni(mem, lane);
#pragma unroll
    for (int v = 0; v < kStripEntries; ++v)
        if (v < entries) small_commit<LEAF>(strip[v][role], role, tid & 255, x[v].value());
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

template <int LEAF, bool VEC>
__global__ __launch_bounds__(kSmallThreads, SmallStep<LEAF>::OCC) void multiply_small_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, int64_t n, int bdim, int blocks,
    const double* __restrict__ na, const double* __restrict__ nb, int64_t ld, double tau,
    unsigned long long* __restrict__ pairs) {
    constexpr int E = SmallStep<LEAF>::ENTRIES;
    __shared__ __attribute__((aligned(16))) float stage[2][E][4][kSmallTile];
    static_assert(LEAF == 16 || sizeof(stage) >= sizeof(float) * (kSmallGroups - 1) * 4 * 16 * 64, "reduction area");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int I = blockIdx.x / blocks, J = blockIdx.x - I * blocks;
    const int grp = wave >> 2, q = (wave + grp) & 3;

    int cnt;
    const uint32_t mem = small_test<LEAF>(na, nb, ld, bdim, int(n), I, J, tau, lane, &cnt);
    if (wave == 0) small_count(cnt, lane, pairs);
    const SmallUnion uni(mem, lane);
    const int steps = (uni.size() + E - 1) / E;

    // this wave's part of a step's 4 E operand tiles: chunks e0 + 64 v + lane of
    // tile wave / W; a tile that no kept product reads is not loaded
    constexpr int W = kSmallGroups / E;
    const int slot = wave / (4 * W), role = (wave / W) & 3, e0 = (wave % W) * 64 * E + lane;
    const SmallTile from(A, B, I, J, role);
    SmallChunk<VEC> x[E];
    auto fetch = [&](int s) {
        const int k = uni.entry(E * s + slot, lane);
        const uint32_t quads = k >= 0 ? small_quadrants<LEAF>(uint32_t(__shfl(int(mem), k))) : 0u;
        const uint32_t need = role == 0 ? 3u : role == 1 ? 12u : role == 2 ? 5u : 10u;
#pragma unroll
        for (int v = 0; v < E; ++v) x[v].load(from, n, k, e0 + 64 * v, (quads & need) != 0);
    };
    auto commit = [&](int s) {
#pragma unroll
        for (int v = 0; v < E; ++v) small_commit<LEAF>(stage[s & 1][slot][role], role, e0 + 64 * v, x[v].value());
    };
    SmallAcc<LEAF> acc;
    acc.zero();
    auto compute = [&](int s) {
#pragma unroll
        for (int e = 0; e < (LEAF == 16 ? E : 1); ++e) {
            const int of = LEAF == 16 ? e : grp;
            const int k = uni.entry(E * s + of, lane);
            if (k >= 0) acc.multiply(&stage[s & 1][of][0][0], uint32_t(__shfl(int(mem), k)), wave, q, lane);
        }
    };
    if (steps > 0) {
        fetch(0);
        commit(0);
    }
    __syncthreads();
    for (int s = 0; s < steps; ++s) {
        if (s + 1 < steps) fetch(s + 1);  // in flight during this step's MFMAs
        compute(s);
        if (s + 1 < steps) commit(s + 1);  // the stage step s-1 used; every wave is past it
        __syncthreads();
    }
    acc.finish(&stage[0][0][0][0], C, n, I, J, wave, q, lane);
}

template <int LEAF, bool VEC>
static hipError_t launch_small_of(const float* a, const float* b, float* c, int64_t n, int64_t bdim, const double* na,
                                  const double* nb, int64_t ld, double tau, int64_t* pairs, hipStream_t s) {
    const bool strip = n <= kStripMaxN;
    static int scratch_state[2] = {0, 0};
    const hipError_t ce = strip ? check_no_scratch(multiply_strip_kernel<LEAF, VEC>, &scratch_state[0])
                                : check_no_scratch(multiply_small_kernel<LEAF, VEC>, &scratch_state[1]);
    if (ce != hipSuccess) return ce;
    const int blocks = int((n + 63) / 64);
    auto* count = reinterpret_cast<unsigned long long*>(pairs);
    if (strip)
        multiply_strip_kernel<LEAF, VEC><<<unsigned(blocks * blocks), kSmallThreads, 0, s>>>(
            a, b, c, n, int(bdim), blocks, na, nb, ld, tau, count);
    else
        multiply_small_kernel<LEAF, VEC><<<unsigned(blocks * blocks), kSmallThreads, 0, s>>>(
            a, b, c, n, int(bdim), blocks, na, nb, ld, tau, count);
    return hipGetLastError();
}

bool small_product(int64_t n, int32_t leaf) {
    switch (leaf) {
        case 16:
        case 32: return n >= 4 && n <= kSmallFineMaxN;
        case 64:
        case 128: return n >= 4 && n <= kSmallCoarseMaxN;
        default: return false;
    }
}

hipError_t launch_small_multiply(const float* a, const float* b, float* c, int64_t n, int32_t leaf, bool vec,
                                 int64_t bdim, const double* na, const double* nb, int64_t ld, double tau,
                                 int64_t* pairs, hipStream_t s) {
    if (!small_product(n, leaf) || bdim != (n + leaf - 1) / leaf || (vec && n % 4 != 0)) return hipErrorInvalidValue;
    switch (leaf) {
        case 16:
            return vec ? launch_small_of<16, true>(a, b, c, n, bdim, na, nb, ld, tau, pairs, s)
                       : launch_small_of<16, false>(a, b, c, n, bdim, na, nb, ld, tau, pairs, s);
        case 32:
            return vec ? launch_small_of<32, true>(a, b, c, n, bdim, na, nb, ld, tau, pairs, s)
                       : launch_small_of<32, false>(a, b, c, n, bdim, na, nb, ld, tau, pairs, s);
        case 64:
            return vec ? launch_small_of<64, true>(a, b, c, n, bdim, na, nb, ld, tau, pairs, s)
                       : launch_small_of<64, false>(a, b, c, n, bdim, na, nb, ld, tau, pairs, s);
        default:
            return vec ? launch_small_of<128, true>(a, b, c, n, bdim, na, nb, ld, tau, pairs, s)
                       : launch_small_of<128, false>(a, b, c, n, bdim, na, nb, ld, tau, pairs, s);
    }
}

}  // namespace spamm

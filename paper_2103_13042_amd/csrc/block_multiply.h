// Device code of the multiply of one 64x64 block of C per workgroup (see
// multiply_block.hip), shared by the single-product and the batched kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "block.h"
#include "device.h"
#include "dma.h"
#include "internal.h"

namespace spamm {

constexpr int kBlockThreads = 256;
// Stages of operand tiles in LDS.  Two (36 KiB a workgroup, four per CU) copy an
// entry while the one before is multiplied; one (20 KiB, six per CU) waits for
// every copy but has half as many blocks again to hide it and the blocks'
// prologues.  With several rounds of blocks to run the latter is faster (one
// call, leaf 32: the 0.1 / (|i-j|^0.1 + 1) matrix at N = 8192 1451 -> 1406 us,
// exp decay 0.05 203 -> 192; leaf 16, N = 4096, decay 0.01 496 -> 460), with few
// blocks the former (leaf 32, N = 1000, decay 0.01: 38 against 45 us).
constexpr int block_occ(int stages) { return stages == 1 ? 5 : 4; }  // registers for so many at least
constexpr int64_t kTwoStageMaxN = 2048;                              // 1024 blocks: one round of four per CU
constexpr int kBlockEntries = 2048;  // k entries that the list holds (leaf 16, with its masks: a quarter)
constexpr int kKept = 0, kPlanned = 1, kDropped = 2;  // where a block's entries come from

// Blocks are dealt to the XCDs (workgroups congruent mod 8) by strips of H block
// rows, so that every XCD gets rows from all over the matrix; the rows left
// over, fewer than 8 H, are dealt block by block, so that every XCD gets as many
// blocks, unless they are nearly a round of strips.  A strip's blocks are taken
// outwards from the diagonal, the longest of decaying matrices first, in rounds
// of `run` columns over all strips of the XCD: the longest blocks of the whole
// matrix start first and the short ones fill the end (strip after strip the CUs
// idled 15 % of the launch at n = 4096), and the run keeps neighbours that share
// rows of A and columns of B in L2.
struct BlockOrder {
    int H, run;
};

struct BlockAt {
    int I, J;
    bool valid;
};

// rows in whole rounds of strips, a nearly whole last round included (its rows
// past the matrix have no blocks)
__host__ __device__ __forceinline__ int dealt_rows(int nb, int H) {
    return (nb + H) / (8 * H) * (8 * H);
}

__device__ __forceinline__ BlockAt block_at(int bid, int nb, BlockOrder order) {
    const int H = order.H;
    const int xcd = bid & 7, idx = bid >> 3;
    const int dealt = dealt_rows(nb, H), left = nb > dealt ? nb - dealt : 0;
    const int rows = dealt / 8;  // of an XCD's strips, whose blocks come first
    int I, mid, step;
    if (idx >= rows * nb) {
        const int r = (idx - rows * nb) * 8 + xcd;
        if (r >= left * nb) return {0, 0, false};
        I = mid = dealt + r % left;
        step = r / left;
    } else {
        const int col0 = idx / (rows * order.run) * order.run, in = idx - col0 * rows;  // rows > 0 here
        const int wide = nb - col0 < order.run ? nb - col0 : order.run;                 // columns of this run
        const int strip = in / (H * wide), of = in - strip * H * wide;
        const int row0 = H * (strip * 8 + xcd);
        I = row0 + of % H;
        if (I >= nb) return {0, 0, false};
        mid = row0 + H / 2 < nb ? row0 + H / 2 : nb - 1;
        step = col0 + of / H;
    }
    // columns mid, mid - 1, mid + 1, mid - 2, ... while both sides last, then the rest in order
    const int near = mid < nb - 1 - mid ? mid : nb - 1 - mid;
    int J;
    if (step <= 2 * near)
        J = (step & 1) ? mid - (step + 1) / 2 : mid + step / 2;
    else
        J = mid < nb - 1 - mid ? step : nb - 1 - step;
    return {I, J, true};
}
static inline unsigned block_grid(int nb, BlockOrder order) {
    const int H = order.H;
    const int dealt = dealt_rows(nb, H), left = nb > dealt ? nb - dealt : 0;
    return unsigned(((left * nb + 7) / 8 + dealt / 8 * nb) * 8);
}
// Of the FP32 blocks, whose kernel is bound by the matrix cores (strips of up to
// 8 rows measured the same, with fewer than two strips per XCD 6 % slower).
constexpr BlockOrder kBlockOrder{2, 8};

// The multiply of block `bid` (block_at) of one product by the calling
// workgroup; nothing if the grid has no such block.
template <int LEAF, int FROM, int STAGES>
__device__ __forceinline__ void block_multiply(const float* A, const float* B, float* C, int64_t n, int bdim, int nb,
                                               const double* na, const double* nbm, int64_t ld, double tau,
                                               unsigned long long* pairs, const uint32_t* items,
                                               const int32_t* uprefix, const BandJob& band, int bid) {
    constexpr bool TEST = FROM != kPlanned;
    constexpr int STAGE = 4 * kOpTile;
    // one LDS object (stages, then the list, in floats): see the copies' waits in dma.h
    constexpr int LIST = !TEST ? 0 : LEAF == 16 ? kBlockEntries / 4 : kBlockEntries / 2;
    constexpr int MASKS = TEST && LEAF == 16 ? kBlockEntries / 4 : 0;
    __shared__ __attribute__((aligned(1024))) float lds[STAGES * STAGE + LIST + MASKS + 8];
    uint16_t* list = reinterpret_cast<uint16_t*>(lds + STAGES * STAGE);
    uint32_t* masks = reinterpret_cast<uint32_t*>(lds + STAGES * STAGE + LIST);  // leaf 16: the 32 products of a list entry
    int* wsum = reinterpret_cast<int*>(lds + STAGES * STAGE + LIST + MASKS);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const BlockAt at = block_at(bid, nb, kBlockOrder);
    if (!at.valid) return;
    const int I = at.I, J = at.J;
    const int whole = int(n) / 32;  // entries inside the matrix

    auto chosen = [&](double p) {
        if constexpr (FROM == kDropped)
            return !(p >= tau) && (!band.has_base || p >= band.base);
        else
            return p >= tau;
    };
    constexpr int CAPACITY = LEAF == 16 ? kBlockEntries / 4 : kBlockEntries;
    const int entries = (int(n) + 31) / 32;
    int kept = 0;

    // ---- this wave's operand tile: chunk 64 j + lane of it is row 8 j + lane / 8,
    // position lane % 8; rows of A and columns of B past the matrix moved inside
    const OpTile of(A, B, I, J, wave);
    const bool is_a = wave < 2;
    const uint32_t need = wave == 0 ? 3u : wave == 1 ? 12u : wave == 2 ? 5u : 10u;
    uint32_t off[4];  // byte offsets from the entry's base
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = 8 * j + (lane >> 3), p = lane & 7;
        if (is_a) {
            const int row = of.row0 + r < int(n) ? r : int(n) - 1 - of.row0;
            off[j] = uint32_t((int64_t(row) * n + 4 * (p ^ (r & 7))) * 4);
        } else {
            const int k = LEAF == 16 ? r ^ ((r >> 3) & 1) : r ^ ((r >> 4) & 1);  // the row stored at r (b_at)
            const int c = LEAF == 16 ? p ^ (4 * ((k >> 2) & 1)) : p;
            const bool in = of.col0 + 4 * c < int(n);
            off[j] = uint32_t((int64_t(k) * n + (in ? 4 * c : 0)) * 4);
        }
    }
    const bool outside = is_a ? of.row0 >= int(n) : of.col0 >= int(n);  // nothing of the tile inside: never kept
    const char* base = reinterpret_cast<const char*>(of.X + (outside ? 0 : (is_a ? int64_t(of.row0) * n : of.col0)));
    const int64_t step = is_a ? 128 : 128 * n;  // bytes from an entry's tile to the next
    auto copy = [&](uint32_t pk, int st) {
        if (!(pk & need)) return;
        const char* src = base + int64_t(pk >> 4) * step;
        char* dst = reinterpret_cast<char*>(lds + st * STAGE + wave * kOpTile);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            asm volatile("" : "+v"(off[j]));  // else extended to 64 bits outside the loop, a vector add a copy
            copy_to_lds(reinterpret_cast<const float*>(src + off[j]), dst + 1024 * j);
        }
    };

    BlockAcc<LEAF> acc;
    acc.zero();
    const int run = n <= 2048 ? 2 : 4;
    bool none = true;  // no entry so far
    // one segment, but for leaf 128 beyond n = 65536
    for (int seg = 0; seg == 0 || (LEAF == 128 && seg < entries); seg += CAPACITY) {
        // ---- the entries of this segment: list[e] = k << 4 | quadrants (leaf 16: and masks[e])
        int count = 0;
        const uint32_t* plan = nullptr;
        if constexpr (TEST) {
            const int end = entries - seg < CAPACITY ? entries : seg + CAPACITY;
            for (int e0 = seg; e0 < end; e0 += kBlockThreads) {
                const int e = e0 + tid;
                uint32_t mem = 0, quads = 0;
                if constexpr (LEAF >= 64) {
                    constexpr int R = LEAF / 64, S = LEAF / 32;  // blocks and entries per leaf tile side
                    const int k = e / S < bdim ? e / S : bdim - 1;
                    if (e < end && chosen(na[(I / R) * ld + k] * nbm[k * ld + J / R])) {
                        kept += I % R == 0 && J % R == 0 && e % S == 0 ? 1 : 0;
                        mem = quads = (I * 64 + 32 < int(n) ? 0xFu : 0x3u) & (J * 64 + 32 < int(n) ? 0xFu : 0x5u);
                    }
                } else {
                    constexpr int T = 64 / LEAF, H = 32 / LEAF;  // leaf tiles per block side and per entry
                    double nav[T][H], nbv[H][T];
#pragma unroll
                    for (int t = 0; t < T; ++t)
#pragma unroll
                        for (int h = 0; h < H; ++h) {
                            const int ti = T * I + t < bdim ? T * I + t : bdim - 1;
                            const int tj = T * J + t < bdim ? T * J + t : bdim - 1;
                            const int k = H * e + h < bdim ? H * e + h : bdim - 1;
                            nav[t][h] = na[ti * ld + k];
                            nbv[h][t] = nbm[k * ld + tj];
                        }
#pragma unroll
                    for (int i = 0; i < T; ++i)
#pragma unroll
                        for (int j = 0; j < T; ++j)
#pragma unroll
                            for (int h = 0; h < H; ++h) {
                                const bool in = H * e + h < bdim && T * I + i < bdim && T * J + j < bdim;
                                const int q = LEAF == 32 ? 2 * i + j : 2 * (i >> 1) + (j >> 1);
                                const int bit = LEAF == 32 ? q : 8 * q + 4 * (i & 1) + 2 * (j & 1) + h;
                                if (in && chosen(nav[i][h] * nbv[h][j])) {
                                    mem |= 1u << bit;
                                    quads |= 1u << q;
                                }
                            }
                    kept += __popc(mem);
                }
                const uint64_t bal = __ballot(mem != 0);
                if (lane == 0) wsum[wave] = __popcll(bal);
                __syncthreads();
                int pos = count + __popcll(bal & (lane == 0 ? 0ull : (~0ull >> (64 - lane))));
#pragma unroll
                for (int w = 0; w < kBlockThreads / 64; ++w) {
                    if (w < wave) pos += wsum[w];
                    count += wsum[w];
                }
                if (mem) {
                    list[pos] = uint16_t(e << 4 | quads);
                    if constexpr (LEAF == 16) masks[pos] = mem;
                }
                __syncthreads();
            }
        } else {
            const int64_t m = int64_t(I) * nb + J;
            plan = items + uprefix[m];
            count = uprefix[m + 1] - uprefix[m];
        }
        count = __builtin_amdgcn_readfirstlane(count);
        none = none && count == 0;
        auto entry = [&](int e) -> uint32_t {  // k << 4 | quadrants
            if constexpr (TEST)
                return uint32_t(__builtin_amdgcn_readfirstlane(int(list[e])));
            else
                return plan[e] & 0x3FFFu;
        };
        const bool tail = count > 0 && int(entry(count - 1) >> 4) >= whole;
        const int full = tail ? count - 1 : count;

        uint32_t cur = full > 0 ? entry(0) : 0u;
        if (full > 0) copy(cur, 0);
        for (int e = 0; e < full; ++e) {
            const uint32_t next = e + 1 < full ? entry(e + 1) : 0u;
            uint32_t mask = cur;
            if constexpr (LEAF == 16) mask = uint32_t(__builtin_amdgcn_readfirstlane(int(masks[e])));
            asm volatile("" ::: "memory");
            wait_vmcnt<0>();  // this wave's copies of entry e have landed
            __builtin_amdgcn_s_waitcnt(0xC07F);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (STAGES == 2 && e + 1 < full) copy(next, (e + 1) & 1);  // the stage entry e - 1 used
            // a wave with MFMAs to issue goes ahead of those that copy or wait
            __builtin_amdgcn_s_setprio(1);
            acc.multiply(lds + (e & (STAGES - 1)) * STAGE, mask, e, run, wave, lane);
            __builtin_amdgcn_s_setprio(0);
            if (STAGES == 1 && e + 1 < count) {  // every wave is done with the stage
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0xC07F);
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                if (e + 1 < full) copy(next, 0);
            }
            cur = next;
        }
        if (tail) {
            const uint32_t pk = entry(count - 1);
            uint32_t mask = pk;
            if constexpr (LEAF == 16) mask = masks[count - 1];
            float* t = lds + (full & (STAGES - 1)) * STAGE + wave * kOpTile;  // a stage that no wave reads any more
            OpChunk<false> x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j].load(of, n, int(pk >> 4), 64 * j + lane, (pk & need) != 0);
#pragma unroll
            for (int j = 0; j < 4; ++j) op_commit<LEAF>(t, wave, 64 * j + lane, x[j].value());
            __syncthreads();
            acc.multiply(lds + (full & (STAGES - 1)) * STAGE, mask, full, run, wave, lane);
        }
        acc.finish(count, run);
        if (LEAF == 128) __syncthreads();  // the list and the stages are used again
    }
    if constexpr (TEST) {
        __syncthreads();  // the last entry of the list has been read
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) kept += __shfl_xor(kept, o);
        if (lane == 0) wsum[wave] = kept;
        __syncthreads();
        if (tid == 0) {
            const int total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
            if constexpr (FROM == kDropped)
                band.counts[I * nb + J] = total;
            else if (total)
                atomicAdd(pairs, static_cast<unsigned long long>(total));
        }
    }
    if (FROM != kDropped && none) {  // 16 bytes a store, the accumulators' layout has 4
        const int row = 64 * I + (tid >> 4), col = 64 * J + 4 * (tid & 15);
        if (col + 4 <= int(n)) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (row + 16 * u < int(n))
                    *reinterpret_cast<f4_dw*>(C + int64_t(row + 16 * u) * n + col) = f4{0, 0, 0, 0};
        } else {
            for (int u = 0; u < 4; ++u)
                for (int c = col; c < int(n); ++c)
                    if (row + 16 * u < int(n)) C[int64_t(row + 16 * u) * n + c] = 0.0f;
        }
        return;
    }
    if constexpr (FROM == kDropped) {
        double sq = 0.0;
        acc.each(n, I, J, wave, lane, [&](int64_t at, float v) {
            const float x = band.has_base ? C[at] + v : v;
            if (band.store) C[at] = x;
            sq += double(x) * double(x);
        });
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) sq += __shfl_xor(sq, o);
        __syncthreads();  // the list is no longer read
        double* red = reinterpret_cast<double*>(lds + STAGES * STAGE);
        if (lane == 0) red[wave] = sq;
        __syncthreads();
        if (tid == 0) band.sums[I * nb + J] = (red[0] + red[1]) + (red[2] + red[3]);
    } else {
        acc.each(n, I, J, wave, lane, [&](int64_t at, float v) { C[at] = v; });
    }
}


}  // namespace spamm

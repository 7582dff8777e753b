// Multiply of the kept leaf pairs on 2x2 blocks of output tiles ("macro
// tiles") at leaf 64 (and 128), and the schedule of such blocks at leaf 32 and
// 64.
//
// A macro tile (I, J) covers output tiles (2I+a, 2J+b), a, b in {0, 1}.  Its
// k-stream is the union of the four tiles' k-lists in ascending order; for each
// k the workgroup stages A[2I..2I+1, k] and B[k, 2J..2J+1] once and every wave
// whose own tile keeps that k multiplies its part.  One staged A/B pair thus
// feeds up to four leaf products, which halves the bytes per flop against one
// tile per workgroup for banded pair patterns, and every barrier is amortised
// over twice the MFMA work.
//
// The schedule step lists, for every macro tile in order, its union k values
// with the 4-bit membership of the four tiles (packed items); a workgroup
// streams its contiguous slice of that list with scalar loads, a few items
// ahead of the one it multiplies.
#include <hip/hip_runtime.h>

#include "device.h"
#include "dma.h"
#include "internal.h"
#include "macro.h"

namespace spamm {

// One wave per macro tile: k-bitmaps and union size (macro_words_wave).
__global__ __launch_bounds__(256) void macro_words_kernel(const int32_t* __restrict__ off,
                                                          const int32_t* __restrict__ klist, int64_t bdim, int64_t mb,
                                                          int nw, uint64_t* __restrict__ words,
                                                          int32_t* __restrict__ ucount, const int32_t* run) {
    __shared__ unsigned long long sw[4][4][16];  // [wave][tile][word]
    const int wave = threadIdx.x >> 6;
    const int64_t m = int64_t(blockIdx.x) * 4 + wave;
    if (closed(run) || m >= mb * mb) return;
    macro_words_wave(off, klist, bdim, mb, nw, words, ucount, m, sw[wave]);
}

// One wave per macro tile: its packed items (macro_items_wave).
__global__ __launch_bounds__(256) void macro_items_kernel(const uint64_t* __restrict__ words,
                                                          const int32_t* __restrict__ uprefix, int64_t mb, int nw,
                                                          uint32_t* __restrict__ items, const int32_t* run) {
    const int64_t m = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (closed(run) || m >= mb * mb) return;
    macro_items_wave(words, uprefix, mb, nw, items, m);
}

// ---------------------------------------------------------------------------
// Leaf 64: tiles move from global memory straight into LDS
// (global_load_lds_dwordx4) through two LDS stages of one item (64 k) each, so
// the copies of the next item are in flight while one is multiplied and no
// registers stage the data.
//
// Bound by the matrix cores: every pair of N = 8192 kept runs at 142 TFLOP/s,
// MFMAs alone at 155.  Vector instructions take the FP32 MFMAs' issue time and
// all waves' first LDS reads come at once after an item's barrier, so the loop
// has next to none of the former (scalar bases and counters, addresses as
// constants of the stage) and the latter are small; with 64-bit vector adds
// for the copies, stage-dependent read addresses and twice the first reads it
// ran at 127.  Banded patterns add items that few of the four tiles keep.
// Multiply alone, +-1/(1+|i-j|)^2, tau 1e-6, N = 8192: 466 -> 440 us, leaf 128
// 842 -> 790; exp decay 0.01, tau 1e-6: 1058 -> 964, leaf 128 1237 -> 1127.
//
// EDGE (N not a multiple of 128): macro tiles and k-chunks may reach past the
// matrix, and rows may be only 4-byte aligned, which the copies accept.  One
// call, leaf 128, N = 6000, exp decay 0.01: 1379 (register-staged, the kernel
// that took these sizes) -> 925 -> 882 us.
//
// Sixteen waves: wave w computes the 32x32 quadrant (w >> 3 & 1, w >> 2 & 1)
// of output tile (w + (w >> 2)) & 3 of the macro tile.  Waves are dealt to the
// four SIMDs round-robin (w, w+4, w+8, w+12 on one SIMD), so each output tile
// has one wave on every SIMD and the MFMA load of an item is the same on all
// SIMDs whichever of the four tiles keep its k.
//
// LDS rows are stored without padding; 16-byte chunks are XOR-swizzled so the
// MFMA operand reads are free of bank conflicts.
//
// Completion of the copies is tracked by hand with s_waitcnt vmcnt: with two
// stages, a wave's vector-memory operations issued after its copies of item
// it are exactly the kDmaStores stores of each macro tile it finished since
// (shared tiles included: their partial sums are stored the same way), so
// the wait counts those stores whatever number of copies the item needed.
// Empty asm statements with a memory clobber keep the compiler from moving
// LDS or global accesses across the hand-placed waits and the barrier.
//
// Work split: workgroup g takes the items between boundaries g and g+1 of the
// item-level cost partition (split_bound), so a macro tile may be shared by
// consecutive workgroups.  Each sharer writes its partial sums to its own
// slot instead of C; macro_fixup_kernel, launched next on the stream, adds the
// partials of every shared tile in workgroup order and writes C.
template <bool EDGE>
__global__ __launch_bounds__(kDmaThreads, 1) void multiply_macro_dma_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C, int64_t n, int64_t bdim,
    int64_t mb, const uint32_t* __restrict__ items, const int32_t* __restrict__ uprefix,
    const int32_t* __restrict__ offsets, int64_t* __restrict__ bounds, float* __restrict__ fix_slots) {
    constexpr int LEAF = 64, KC = kDmaKC, SPC = KC / 2;
    static_assert(KC == LEAF && kDmaStages == 2, "an item is one stage, its parity the stage");
    constexpr int ABYTES = 2 * LEAF * KC * 4, BBYTES = KC * 2 * LEAF * 4;
    constexpr int STAGE_BYTES = ABYTES + BBYTES;
    // one LDS object (the stages, the partition boundaries, the last chunks of
    // the matrices' last rows): a second __shared__ array makes the compiler
    // wait for every outstanding copy before each LDS read
    __shared__ __attribute__((aligned(1024))) char lds[kDmaStages * STAGE_BYTES + 6 * sizeof(int64_t) +
                                                       8 * sizeof(float)];
    int64_t(*sbound)[2] = reinterpret_cast<int64_t(*)[2]>(lds + kDmaStages * STAGE_BYTES);
    // the A stages, then the B stages: an operand's stages are less than 64 KiB apart
    auto a_stage = [&](int st) { return lds + st * ABYTES; };
    auto b_stage = [&](int st) { return lds + kDmaStages * ABYTES + st * BBYTES; };

    // the wave index as a scalar, so that what derives from it (the tile, the
    // copy half and its membership tests) stays in scalar registers
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // waves w, w+4, w+8, w+12 share a SIMD: give them different output tiles
    // (and each tile one wave per quadrant), so every SIMD holds one wave of
    // each tile and the MFMA work of an item is spread evenly whichever tiles
    // keep its k
    const int tile = (wave + (wave >> 2)) & 3, wa = tile >> 1, wb = tile & 1, qr = (wave >> 3) & 1,
              qc = (wave >> 2) & 1;
    const int ir = lane & 31, g = lane >> 5;

    const int64_t groups = gridDim.x;
    const int64_t bid = blockIdx.x;
    const int64_t lg = (bid & 7) * (groups >> 3) + (bid >> 3);
    const int64_t nm = mb * mb;
    // boundaries lg, lg+1 and lg-1, one wave each
    if (wave < 3) {
        const SplitBound sbd = split_bound(wave < 2 ? lg + wave : lg - 1, groups, mb, bdim, fix_slots == nullptr,
                                           uprefix, offsets, items);
        if (lane == 0) {
            sbound[wave][0] = sbd.m;
            sbound[wave][1] = sbd.p;
        }
    }
    // EDGE: the chunk of A's (0 .. 3) and B's (4 .. 7) last row that crosses its
    // end, with zeros past it
    float* last_chunk = reinterpret_cast<float*>(lds + kDmaStages * STAGE_BYTES + 6 * sizeof(int64_t));
    if (EDGE && tid >= 256 && tid < 264) {
        const int64_t col = n / 4 * 4 + (tid & 3);
        last_chunk[tid & 7] = col < n ? (tid & 4 ? B : A)[(n - 1) * n + col] : 0.0f;
    }
    __syncthreads();
    const int64_t m_first = sbound[0][0], p_begin = sbound[0][1];
    const int64_t m_next = sbound[1][0], p_end = sbound[1][1];
    const bool has_items = p_begin < p_end;
    const bool head_split = has_items && p_begin > uprefix[m_first];
    const bool tail_split = has_items && m_next < nm && p_end > uprefix[m_next];
    // record for macro_fixup_kernel: boundary lg; the macro tile it opens
    // for sharing (boundary lg lies inside it and boundary lg-1 does not), or
    // -1; and lg if this workgroup then holds the rest of that tile (it is
    // the last of the two contributors), else -1
    if (tid < 4) {
        const bool inside = m_first < nm && p_begin > uprefix[m_first];
        const bool opens = inside && !(sbound[2][0] == m_first && sbound[2][1] > uprefix[m_first]);
        const int64_t v = tid < 2    ? sbound[0][tid]
                          : tid == 2 ? (opens ? m_first : int64_t(-1))
                                     : (opens && has_items && p_end >= uprefix[m_first + 1] ? lg : int64_t(-1));
        bounds[4 * lg + tid] = v;
    }
    const int64_t m_begin = m_first, m_end = m_next + (tail_split ? 1 : 0);
    if (m_begin >= m_end) return;

    // this group's slice of the item list (wave-uniform); past the end the
    // last item repeats (a harmless reload)
    const uint32_t* ip = items + p_begin;
    const int32_t npairs = int32_t(p_end - p_begin);
    int32_t pp = 0;
    uint32_t last = 0;
    auto produce = [&]() -> uint32_t {
        if (pp < npairs) last = ip[pp];
        ++pp;
        return last;
    };

    f16v acc;
    auto zero_acc = [&]() {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    };
    // EDGE: macro tiles of the last row and column may reach past the matrix
    auto at_edge = [&](int64_t I, int64_t J) { return I == mb - 1 || J == mb - 1; };
    // exactly kDmaStores stores per wave: the accumulators of finished macro
    // tile m to C, or for a tile shared with other workgroups to this
    // workgroup's slot (a 128 x 128 row-major tile; side 1 if this workgroup
    // holds the tile's first item, the tile being its last, side 0 otherwise,
    // the tile being its first).  Returns how many times kDmaStores the copy
    // waits may count: 0 where stores outside the matrix were left out (a
    // count that is too low only waits for more)
    auto store_macro = [&](int64_t m, bool shared) -> int {
        const int64_t I = m / mb, J = m - (m / mb) * mb;
        float* base;
        int64_t ld;
        if (shared) {
            const int side = p_begin <= int64_t(uprefix[m]) ? 1 : 0;
            base = fix_slots + (lg * 2 + side) * int64_t(kSplitSlotFloats);
            ld = 2 * LEAF;
        } else {
            base = C + 2 * I * LEAF * n + 2 * J * LEAF;
            ld = n;
        }
        const int row0 = wa * LEAF + qr * 32 + 4 * g, col0 = wb * LEAF + qc * 32 + ir;
        float* dst = base + row0 * ld + col0;
        if (EDGE && !shared && at_edge(I, J)) {  // inside the matrix only
            const int rows = int(n - 2 * I * LEAF), cols = int(n - 2 * J * LEAF);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (row0 + 8 * (r >> 2) + (r & 3) < rows && col0 < cols) dst[(8 * (r >> 2) + (r & 3)) * ld] = acc[r];
            return 0;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[(8 * (r >> 2) + (r & 3)) * ld] = acc[r];
        return 1;
    };

    // copies of item (pair item pi, chunk ch) into stage st: KC/32 A and KC/32
    // B instructions of 1 KiB per wave.  A is staged as 128 rows of KC; B as
    // two column halves (one per output tile column), each KC rows of 64.
    // Waves 0-7 copy the first half of each operand (A rows of output tile row
    // 0, B columns of tile column 0), waves 8-15 the second; a half that no
    // tile keeping the item's k reads is not copied (the membership bits tell),
    // so an item kept by one tile moves half the bytes.  The copy waits count
    // only the stores issued after a wave's copies, which holds for any number
    // of copies per wave with two stages.
    constexpr int ACH = KC / 4;  // 16-byte chunks per A row
    constexpr int BHALF = KC * LEAF * 4;  // bytes of one B column half
    auto aswz = [](int r) { return KC == 32 ? ((r >> 1) & 7) : (r & 15); };
    const int half = wave >> 3;
    const uint32_t need_a = half ? 12u : 3u, need_b = half ? 10u : 5u;
    // each copy's address: the item's part (uniform: a scalar base) plus the
    // lane's part, the same for every item (a 32-bit byte offset computed
    // once: row r of the copy's block times n, plus its swizzled chunk), so
    // the copies of an item cost no per-lane address arithmetic (the offset is
    // opaque where it is used: an extension to 64 bits outside the loop would
    // cost each copy a 64-bit vector add, and vector instructions take the FP32
    // MFMAs' issue time, 3 to 4 cycles each: 155 TFLOP/s of them alone, 130 with
    // 4 additions per MFMA)
    uint32_t a_off[KC / 32], b_off[KC / 32];
#pragma unroll
    for (int j = 0; j < KC / 32; ++j) {
        {  // A: 1024 / (4 KC) rows per instruction
            const int blk = wave * (KC / 32) + j;
            const int r = blk * (256 / KC) + lane / ACH, p = lane % ACH;
            a_off[j] = uint32_t((int64_t(r) * n + 4 * (p ^ aswz(r))) * 4);
        }
        {  // B: 4 rows of 16 chunks of one half per instruction
            const int blk = (wave & 7) * (KC / 32) + j;
            const int r = blk * 4 + (lane >> 4), p = lane & 15;
            b_off[j] = uint32_t((int64_t(r) * n + half * LEAF + 4 * (p ^ (8 * ((r / SPC) & 1)))) * 4);
        }
    }
    // EDGE: rows and columns outside the matrix are read from addresses inside
    // it: their products only reach parts of C that are not stored.  In the
    // last macro row the lane's rows, in the last macro column its columns,
    // are moved inside by other offsets, as cheap as the ones above (the
    // workgroups of the last macro row see no other items: with the addresses
    // worked out per item they ended last, 10 % behind the others).
    const int last_m = int(mb) - 1;
    uint32_t a_edge[KC / 32], b_edge[KC / 32];
    if (EDGE) {
#pragma unroll
        for (int j = 0; j < KC / 32; ++j) {
            const int blka = wave * (KC / 32) + j, blkb = (wave & 7) * (KC / 32) + j;
            const int ra = blka * (256 / KC) + lane / ACH, rb = blkb * 4 + (lane >> 4);
            const int in_rows = int(n - 1 - 2 * int64_t(last_m) * LEAF);  // last row inside, from the macro row's first
            a_edge[j] = uint32_t((int64_t(ra < in_rows ? ra : in_rows) * n + 4 * ((lane % ACH) ^ aswz(ra))) * 4);
            const int cb = half * LEAF + 4 * ((lane & 15) ^ (8 * ((rb / SPC) & 1)));
            const bool in = 2 * int64_t(last_m) * LEAF + cb < n;
            b_edge[j] = uint32_t((int64_t(rb) * n + (in ? cb : 0)) * 4);
        }
    }
    // EDGE, an item whose k reach past n (rare): any address inside for what
    // lies outside; a chunk that crosses a row's end reads into the next row,
    // and in the matrix's last row the last four floats.  patch_tail then
    // clears k >= n and mends the last row.
    const uint32_t whole_kt = uint32_t(n / LEAF);  // k-chunks inside the matrix
    auto in_tail = [&](uint32_t pi) { return ((pi >> 4) & 1023u) >= whole_kt; };
    // the lane as a value of its own in these rare blocks, so that what they
    // compute from it does not stay in registers over the whole loop
    auto edge_lane = [&]() { return opaque(lane); };
    auto edge_source = [&](const float* X, int64_t row, int64_t col) -> const float* {
        const int64_t r = row < n ? row : n - 1;
        const int64_t e = r * n + (col < n ? col : 0), last = n * n - 4;
        return X + (e < last ? e : last);
    };
    auto copy_item = [&](uint32_t pi, int st) {
        const int64_t I = pi >> 23, J = (pi >> 14) & 511, kt = (pi >> 4) & 1023;
        if (EDGE && in_tail(pi)) {
            const int lane = edge_lane();
            if (pi & need_a) {
#pragma unroll 1
                for (int j = 0; j < KC / 32; ++j) {
                    const int blk = wave * (KC / 32) + j;
                    const int r = blk * (256 / KC) + lane / ACH, p = lane % ACH;
                    copy_to_lds(edge_source(A, 2 * I * LEAF + r, kt * LEAF + 4 * (p ^ aswz(r))),
                                a_stage(st) + blk * 1024);
                }
            }
            if (pi & need_b) {
#pragma unroll 1
                for (int j = 0; j < KC / 32; ++j) {
                    const int blk = (wave & 7) * (KC / 32) + j;
                    const int r = blk * 4 + (lane >> 4), p = lane & 15;
                    copy_to_lds(edge_source(B, kt * LEAF + r,
                                            2 * J * LEAF + half * LEAF + 4 * (p ^ (8 * ((r / SPC) & 1)))),
                                b_stage(st) + half * BHALF + blk * 1024);
                }
            }
            return;
        }
        if (pi & need_a) {
            const char* base = reinterpret_cast<const char*>(A + 2 * I * LEAF * n + kt * LEAF);
#pragma unroll
            for (int j = 0; j < KC / 32; ++j) {
                const int blk = wave * (KC / 32) + j;
                asm volatile("" : "+v"(a_off[j]));  // see a_off
                const uint32_t off = EDGE && int(I) == last_m ? a_edge[j] : a_off[j];
                copy_to_lds(reinterpret_cast<const float*>(base + off), a_stage(st) + blk * 1024);
            }
        }
        if (pi & need_b) {
            const char* base = reinterpret_cast<const char*>(B + (kt * LEAF) * n + 2 * J * LEAF);
#pragma unroll
            for (int j = 0; j < KC / 32; ++j) {
                const int blk = (wave & 7) * (KC / 32) + j;
                asm volatile("" : "+v"(b_off[j]));
                const uint32_t off = EDGE && int(J) == last_m ? b_edge[j] : b_off[j];
                copy_to_lds(reinterpret_cast<const float*>(base + off), b_stage(st) + half * BHALF + blk * 1024);
            }
        }
    };
    // EDGE, an item whose k reach past n, after this wave's copies of it have
    // landed: zeros for every k >= n of the chunks this wave copied, and the
    // elements of the matrix's last row whose chunk crosses its end
    auto patch_tail = [&](uint32_t pi, int st) {
        const int I = int(pi >> 23), J = int((pi >> 14) & 511), kt = int((pi >> 4) & 1023);
        const int lane = edge_lane();
        // dst: the chunk of (row, col); k: the index of the two that is one
        auto mend = [&](char* dst, int row, int col, int k, int last) {
            f4* d = reinterpret_cast<f4*>(dst);
            if (k >= int(n)) {
                *d = f4{0.0f, 0.0f, 0.0f, 0.0f};
            } else if (col < int(n) && col + 4 > int(n)) {
                f4 v = row == int(n) - 1 ? *reinterpret_cast<const f4*>(last_chunk + last) : *d;
                v.y = col + 1 < int(n) ? v.y : 0.0f;
                v.z = col + 2 < int(n) ? v.z : 0.0f;
                v.w = 0.0f;
                *d = v;
            }
        };
        if (pi & need_a) {
#pragma unroll 1
            for (int j = 0; j < KC / 32; ++j) {
                const int blk = wave * (KC / 32) + j;
                const int r = blk * (256 / KC) + lane / ACH, p = lane % ACH;
                const int col = kt * LEAF + 4 * (p ^ aswz(r));
                mend(a_stage(st) + blk * 1024 + lane * 16, 2 * I * LEAF + r, col, col, 0);
            }
        }
        if (pi & need_b) {
#pragma unroll 1
            for (int j = 0; j < KC / 32; ++j) {
                const int blk = (wave & 7) * (KC / 32) + j;
                const int r = blk * 4 + (lane >> 4), p = lane & 15;
                const int row = kt * LEAF + r;
                mend(b_stage(st) + half * BHALF + blk * 1024 + lane * 16, row,
                     2 * J * LEAF + half * LEAF + 4 * (p ^ (8 * ((r / SPC) & 1))), row, 4);
            }
        }
    };
    // operands are read in groups of GRP MFMA steps, one group ahead of the
    // MFMAs that use them, so the LDS latency hides behind MFMA work; small
    // groups, as all 16 waves read their first ones at once after the barrier.
    // The stage is a constant, so that every address is one of a_chunk, b_col
    // plus an offset in the instruction.
    constexpr int GRP = 4, NGRP = SPC / GRP;
    static_assert(SPC % GRP == 0, "operand groups");
    const int a_row = wa * 64 + qr * 32 + ir, cc = qc * 32 + ir;  // cc: column within tile column wb's half of B
    int a_chunk[SPC / 4];  // opaque: else a base and eight offsets, added for every read
#pragma unroll
    for (int q = 0; q < SPC / 4; ++q)
        a_chunk[q] = opaque(a_row * (KC * 4) + ((g * (SPC / 4) + q) ^ aswz(a_row)) * 16);
    const char* b_col = b_stage(0) + wb * BHALF + g * SPC * (LEAF * 4) + ((cc >> 2) ^ (8 * g)) * 16 + (cc & 3) * 4;
    auto compute = [&](auto stage) {
        constexpr int st = decltype(stage)::value;
        f4 av[2][GRP / 4];
        float bv[2][GRP];
        auto load = [&](int grp, int buf) {
#pragma unroll
            for (int q = 0; q < GRP / 4; ++q) {
                av[buf][q] = *reinterpret_cast<const f4*>(a_stage(st) + a_chunk[grp * (GRP / 4) + q]);
            }
#pragma unroll
            for (int u = 0; u < GRP; ++u) {
                bv[buf][u] = *reinterpret_cast<const float*>(b_col + st * BBYTES + (grp * GRP + u) * (LEAF * 4));
            }
        };
        // a wave in its MFMA block goes first in its SIMD's issue arbitration,
        // ahead of the waves that issue their copies or wait at the barrier,
        // so the matrix unit is not left idle while copies are issued
        __builtin_amdgcn_s_setprio(1);
        load(0, 0);
#pragma unroll
        for (int grp = 0; grp < NGRP; ++grp) {
            if (grp + 1 < NGRP) load(grp + 1, (grp + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);  // keep the next group's reads ahead of these MFMAs
#pragma unroll
            for (int u = 0; u < GRP; ++u)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[grp & 1][u >> 2][u & 3], bv[grp & 1][u], acc, 0, 0, 0);
        }
        __builtin_amdgcn_s_setprio(0);
    };

    uint32_t cur = produce(), next = produce();
    copy_item(cur, 0);
    int32_t out_m = int32_t(m_begin);
    // finish macro tile out_m: its C tile, or this workgroup's partial sums of
    // a shared tile
    auto finish = [&]() -> int {
        const int stored = store_macro(out_m, (out_m == m_first && head_split) || (out_m == m_next && tail_split));
        zero_acc();
        ++out_m;
        return stored;
    };
    zero_acc();
    // item `cur` from stage st, its parity
    auto step = [&](auto st) {
        const uint32_t pi = cur;
        const int32_t m_it = int32_t(pi >> 23) * int32_t(mb) + int32_t((pi >> 14) & 511);
        int stores = 0;
        while (out_m < m_it) stores += finish();
        // this wave's copies of the item are complete once at most the stores
        // issued since are outstanding
        asm volatile("" ::: "memory");
        wait_copies<0>(stores);
        if (EDGE && in_tail(pi)) {
            asm volatile("" ::: "memory");
            patch_tail(pi, st);
            asm volatile("" ::: "memory");
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's LDS reads of the item before are done
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        copy_item(next, 1 - st);  // the next item -> the stage that the one before used
        if ((pi >> tile) & 1) compute(st);
        cur = next;
        next = produce();
    };
    for (int32_t it = 0; it < npairs; it += 2) {
        step(std::integral_constant<int, 0>{});
        if (it + 1 == npairs) break;
        step(std::integral_constant<int, 1>{});
    }
    while (out_m < m_end) finish();
    __builtin_amdgcn_s_waitcnt(0);  // no copy into LDS may outlive the workgroup
}

// One workgroup per interior boundary g = 1 .. G-1 of the split multiply,
// from the records the multiply kernel left in bounds[4g ..]: (macro tile,
// item position) of boundary g, the shared macro tile M boundary g opens (or
// -1) and M's last contributor (or -1: found here from the later
// boundaries).  M's contributors are workgroups g-1 (slot side 1), g, g+1, ...
// (side 0; those with empty ranges skipped); their partial sums are added in
// that order and written to C.
__global__ __launch_bounds__(kDmaThreads) void macro_fixup_kernel(float* __restrict__ C, int64_t n, int64_t mb,
                                                                  const int32_t* __restrict__ uprefix,
                                                                  const int64_t* __restrict__ bounds,
                                                                  const float* __restrict__ fix_slots,
                                                                  int64_t groups) {
    constexpr int LEAF = 64;
    // element e = tid + 1024 j of the 128 x 128 tile: row e / 128, column e % 128
    constexpr int EL = (2 * LEAF * 2 * LEAF) / kDmaThreads;
    const int tid = threadIdx.x;
    const int64_t nm = mb * mb, gb = int64_t(blockIdx.x) + 1;
    const int64_t m = bounds[4 * gb + 2], last = bounds[4 * gb + 3];
    if (m < 0) return;
    auto slot = [&](int64_t c, int side) { return fix_slots + (c * 2 + side) * int64_t(kSplitSlotFloats); };
    float sum[EL];
    if (last >= 0) {  // two contributors, gb-1 and gb
        const float* s0 = slot(gb - 1, 1);
        const float* s1 = slot(gb, 0);
#pragma unroll
        for (int j = 0; j < EL; ++j) sum[j] = s0[tid + j * kDmaThreads] + s1[tid + j * kDmaThreads];
    } else {  // gb-1, then the non-empty ones of gb .. the one holding the tile's last item
        const float* s0 = slot(gb - 1, 1);
#pragma unroll
        for (int j = 0; j < EL; ++j) sum[j] = s0[tid + j * kDmaThreads];
        auto pos = [&](int64_t c) { return c >= groups ? int64_t(uprefix[nm]) : bounds[4 * c + 1]; };
        const int64_t u1 = uprefix[m + 1];
        for (int64_t c = gb, pc = pos(gb); pc < u1; ++c) {
            const int64_t pn = pos(c + 1);
            if (pc < pn) {
                const float* sc = slot(c, 0);
#pragma unroll
                for (int j = 0; j < EL; ++j) sum[j] += sc[tid + j * kDmaThreads];
            }
            pc = pn;
        }
    }
    const int64_t I = m / mb, J = m - (m / mb) * mb;
    const int64_t rows = n - 2 * I * LEAF, cols = n - 2 * J * LEAF;  // inside the matrix (any number past the tile's)
    float* dst = C + 2 * I * LEAF * n + 2 * J * LEAF;
#pragma unroll
    for (int j = 0; j < EL; ++j) {
        const int e = tid + j * kDmaThreads;
        if (e / (2 * LEAF) < rows && e % (2 * LEAF) < cols) dst[(e / (2 * LEAF)) * n + e % (2 * LEAF)] = sum[j];
    }
}

// Leaf 128 on the same kernel: a 128x128 output tile
// is a macro tile of four 64x64 quarters that all keep every k, so each kept
// pair (i, k, j) becomes two items (one per 64-wide half of k) with all four
// membership bits set.  One wave per output tile t: its items at
// 2 offsets[t] .., and uprefix[t] = 2 offsets[t].
__global__ __launch_bounds__(256) void leaf128_items_kernel(const int32_t* __restrict__ off,
                                                            const int32_t* __restrict__ klist, int64_t bdim,
                                                            int32_t* __restrict__ uprefix,
                                                            uint32_t* __restrict__ items) {
    const int lane = threadIdx.x & 63;
    const int64_t t = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (t > bdim * bdim) return;
    if (lane == 0) uprefix[t] = 2 * off[t];
    if (t == bdim * bdim) return;
    const uint32_t i = uint32_t(t / bdim), j = uint32_t(t - (t / bdim) * bdim);
    for (int32_t q = off[t] + lane; q < off[t + 1]; q += 64) {
        const uint32_t k = uint32_t(klist[q]);
        items[2 * int64_t(q)] = mi_pack(i, j, 2 * k, 15u);
        items[2 * int64_t(q) + 1] = mi_pack(i, j, 2 * k + 1, 15u);
    }
}

hipError_t launch_leaf128_schedule(const int32_t* offsets, const int32_t* klist, int64_t bdim, int32_t* uprefix,
                                   uint32_t* items, hipStream_t s) {
    leaf128_items_kernel<<<unsigned((bdim * bdim + 1 + 3) / 4), 256, 0, s>>>(offsets, klist, bdim, uprefix, items);
    return hipGetLastError();
}

// The LDS-DMA multiply over mb x mb macro tiles and its fixup; fix_slots ==
// nullptr: no macro tile is shared between workgroups.
static hipError_t launch_dma(const float* a, const float* b, float* c, int64_t n, int64_t bdim, int64_t mb,
                             const uint32_t* items, const int32_t* uprefix, const int32_t* offsets, int64_t* bounds,
                             float* fix_slots, int num_cus, hipStream_t s) {
    if (n < 4 || !bounds) return hipErrorInvalidValue;
    const bool edge = n % 128 != 0;
    static int scratch_state[2] = {0, 0};
    const hipError_t ce = edge ? check_no_scratch(multiply_macro_dma_kernel<true>, &scratch_state[1])
                               : check_no_scratch(multiply_macro_dma_kernel<false>, &scratch_state[0]);
    if (ce != hipSuccess) return ce;
    const int64_t cap = ((mb * mb + 7) / 8) * 8;
    int64_t groups = int64_t(num_cus);
    if (groups > cap) groups = cap;
    groups = ((groups + 7) / 8) * 8;
    if (groups > kSplitMaxGroups) groups = kSplitMaxGroups;
    if (edge)
        multiply_macro_dma_kernel<true><<<unsigned(groups), kDmaThreads, 0, s>>>(a, b, c, n, bdim, mb, items, uprefix,
                                                                                offsets, bounds, fix_slots);
    else
        multiply_macro_dma_kernel<false><<<unsigned(groups), kDmaThreads, 0, s>>>(a, b, c, n, bdim, mb, items,
                                                                                 uprefix, offsets, bounds, fix_slots);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || groups < 2 || !fix_slots) return e;
    macro_fixup_kernel<<<unsigned(groups - 1), kDmaThreads, 0, s>>>(c, n, mb, uprefix, bounds, fix_slots, groups);
    return hipGetLastError();
}

hipError_t launch_leaf128_multiply(const float* a, const float* b, float* c, int64_t n, int64_t bdim,
                                   const int32_t* uprefix, const uint32_t* items, int64_t* bounds, float* fix_slots,
                                   int num_cus, hipStream_t s) {
    // one macro tile per 128x128 output tile
    return launch_dma(a, b, c, n, 2 * bdim, bdim, items, uprefix, nullptr, bounds, fix_slots, num_cus, s);
}

hipError_t launch_macro_schedule(const int32_t* offsets, const int32_t* klist, int64_t bdim, const MacroSchedule& ms,
                                 hipStream_t s, const int32_t* run) {
    const int64_t mb = (bdim + 1) / 2, nm = mb * mb;
    const int nw = int((bdim + 63) / 64);
    macro_words_kernel<<<unsigned((nm + 3) / 4), 256, 0, s>>>(offsets, klist, bdim, mb, nw, ms.words, ms.ucount, run);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = launch_plan_scan(ms.ucount, nm, ms.uprefix, ms.uprefix, nm, nullptr, s, run);
    if (e != hipSuccess) return e;
    macro_items_kernel<<<unsigned((nm + 3) / 4), 256, 0, s>>>(ms.words, ms.uprefix, mb, nw, ms.items, run);
    return hipGetLastError();
}

hipError_t launch_macro_multiply(const float* a, const float* b, float* c, int64_t n, int64_t bdim,
                                 const int32_t* offsets, const MacroSchedule& ms, int num_cus, hipStream_t s) {
    return launch_dma(a, b, c, n, bdim, (bdim + 1) / 2, ms.items, ms.uprefix, offsets, ms.bounds, ms.fix_slots, num_cus,
                      s);
}

}  // namespace spamm

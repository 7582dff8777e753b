// Device code shared by the kernels that multiply one 64x64 block of C per
// workgroup (multiply_small.hip, multiply_block.hip): k is walked in entries of
// 32, an entry's operands are four 32x32 tiles (rows 2I + {0, 1} of A, columns
// 2J + {0, 1} of B, in tiles of 32) in LDS.
#pragma once

#include <hip/hip_runtime.h>

#include "device.h"

namespace spamm {

constexpr int kOpTile = 32 * 32;  // floats of an operand tile

// Where operand tile `role` of an entry lies: rows row0 + k * row_k of X from
// column col0 + k * col_k, the same arithmetic for A and B, so that no branch
// on the role stands between a load and the next one.
struct OpTile {
    const float* X;
    int row0, row_k, col0, col_k;
    __device__ __forceinline__ OpTile(const float* A, const float* B, int I, int J, int role) {
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
// chunk lies outside or is not wanted); value() puts its floats in place, zeros
// outside the matrix, and is called when the chunk is needed.
template <bool VEC>
struct OpChunk {
    f4 x;
    int back;  // columns past the matrix's edge, 4 or more: nothing of it is wanted
    __device__ __forceinline__ void load(const OpTile& t, int64_t n, int k, int e, bool want) {
        const int row = t.row0 + k * t.row_k + (e >> 3), col = t.col0 + k * t.col_k + 4 * (e & 7);
        const int over = VEC ? 0 : (col + 4 > int(n) ? col + 4 - int(n) : 0);
        const bool in = want && row < int(n) && col < int(n);
        back = in ? over : 4;
        const float* p = t.X + (in ? int64_t(row) * n + col - over : 0);
        if constexpr (VEC) {
            x = *reinterpret_cast<const f4*>(p);
        } else if (n >= 4) {
            x = *reinterpret_cast<const f4_dw*>(p);
        } else {  // no four floats in a row of the matrix
            const float* q = t.X + (in ? int64_t(row) * n : 0);
            x = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (e < int(n)) x[e] = q[e];
            back = in ? 0 : 4;
        }
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

// chunk e of an operand tile (roles 0, 1: A; 2, 3: B) into the tile at t
template <int LEAF>
__device__ __forceinline__ void op_commit(float* t, int role, int e, f4 v) {
    const int r = e >> 3, c4 = e & 7;
    *reinterpret_cast<f4*>(t + (role < 2 ? a_at(r, c4) : b_at<LEAF>(r, 4 * c4))) = v;
}

// acc += quadrant (q >> 1, q & 1) of the entry whose four operand tiles are at t
// (leaf 32 and up): lane (ir, g) supplies k = 16 g + u of MFMA step u, A[ir][16g
// + u] and B[16g + u][ir].  FIRST: acc = instead of acc +=.
template <bool FIRST = false>
__device__ __forceinline__ void op_multiply(f16v& acc, const float* t, int q, int lane) {
    const int ir = lane & 31, g = lane >> 5;
    const float* ta = t + (q >> 1) * kOpTile;
    // b_at(16 g + u, ir) for even and odd u, as offsets of u
    const float* tb = t + (2 + (q & 1)) * kOpTile + 16 * g * 32 + ir;
    const float *tb0 = tb + 32 * g, *tb1 = tb - 32 * g;
    f4 av[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) av[v] = *reinterpret_cast<const f4*>(ta + a_at(ir, 4 * g + v));
#pragma unroll
    for (int u = 0; u < 16; ++u)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[u >> 2][u & 3], (u & 1 ? tb1 : tb0)[u * 32],
                                                   FIRST && u == 0 ? f16v{} : acc, 0, 0, 0);
}

// acc += output tile (a, b) of the block (leaf 16) for the halves of the entry
// in keep (bits 0 and 1): lane (r, g) supplies k = 4 g + s of each half's step s
__device__ __forceinline__ void op_multiply16(f4& acc, const float* t, int a, int b, uint32_t keep, int lane) {
    const int r = lane & 15, g = lane >> 4;
    const float* ta = t + (a >> 1) * kOpTile;
    const float* tb = t + (2 + (b >> 1)) * kOpTile;
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

// What a wave of four accumulates: its quadrant, at leaf 16 as 2x2 tiles.
// Leaf 32 and up: every `run` entries of the block's list (a power of two) the
// accumulators are added to a total and start again, so that a long list does
// not grow the rounding error of one long chain, for 16 additions a run.
// N = 1024, exp decay 0.05, leaf 32, relative to FP64: one chain 4.1e-7, runs of
// 4 1.5e-7, of 2 1.2e-7 (2 % of the call's time at large N, none below 2048).
template <int LEAF>
struct BlockAcc {
    f16v acc, total;
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int r = 0; r < 16; ++r) total[r] = 0.0f;
    }
    // e: the entry's index in the list.  A run starts without clearing the
    // accumulators: vector instructions take the MFMAs' issue time, 3 to 4
    // cycles each of the 64 of an MFMA (this and the copies' addresses: N = 4096
    // paper matrix 231 -> 220 us, exp decay 0.01 at leaf 64 496 -> 476).
    __device__ __forceinline__ void multiply(const float* t, uint32_t quads, int e, int run, int q, int lane) {
        const bool kept = (quads >> q) & 1;
        if ((e & (run - 1)) == 0) {
            if (kept)
                op_multiply<true>(acc, t, q, lane);
            else
                acc = f16v{};
        } else if (kept) {
            op_multiply(acc, t, q, lane);
        }
        if (((e + 1) & (run - 1)) == 0) add();
    }
    // after the last of `count` entries
    __device__ __forceinline__ void finish(int count, int run) {
        if (count & (run - 1)) add();
    }
    __device__ __forceinline__ void add() {
#pragma unroll
        for (int r = 0; r < 16; ++r) total[r] += acc[r];
    }
    // f(element of the matrix, its sum) for every element of the quadrant inside it
    template <typename F>
    __device__ __forceinline__ void each(int64_t n, int I, int J, int q, int lane, F f) const {
        const int64_t row0 = 64 * int64_t(I) + 32 * (q >> 1) + 4 * (lane >> 5);
        const int64_t col = 64 * int64_t(J) + 32 * (q & 1) + (lane & 31);
        if (col >= n) return;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t row = row0 + 8 * (r >> 2) + (r & 3);
            if (row < n) f(row * n + col, total[r]);
        }
    }
};

template <>
struct BlockAcc<16> {
    f4 acc[4];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[x] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    // mem: bit 8 q + 4 a + 2 b + h for output tile (a, b) of quadrant q, half h
    __device__ __forceinline__ void multiply(const float* t, uint32_t mem, int, int, int q, int lane) {
        const uint32_t keep = (mem >> (8 * q)) & 0xFFu;
#pragma unroll
        for (int x = 0; x < 4; ++x)
            op_multiply16(acc[x], t, 2 * (q >> 1) + (x >> 1), 2 * (q & 1) + (x & 1), (keep >> (2 * x)) & 3u, lane);
    }
    __device__ __forceinline__ void finish(int, int) {}
    template <typename F>
    __device__ __forceinline__ void each(int64_t n, int I, int J, int q, int lane, F f) const {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const int64_t row0 = 64 * int64_t(I) + 32 * (q >> 1) + 16 * (x >> 1) + 4 * (lane >> 4);
            const int64_t col = 64 * int64_t(J) + 32 * (q & 1) + 16 * (x & 1) + (lane & 15);
            if (col >= n) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (row0 + v < n) f((row0 + v) * n + col, acc[x][v]);
        }
    }
};

}  // namespace spamm

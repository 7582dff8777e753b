// Device code of the macro-tile schedule (leaf 32 and 64): the bitmaps, union
// sizes and packed items of a product's 2x2 blocks of output tiles, one wave
// per macro tile.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"

namespace spamm {

// One wave per macro tile m: k-bitmaps of its four tiles (zero for tiles
// outside the grid) and the size of their union.  sw: the wave's 4 x 16 words
// of LDS scratch.
__device__ __forceinline__ void macro_words_wave(const int32_t* __restrict__ off, const int32_t* __restrict__ klist,
                                                 int64_t bdim, int64_t mb, int nw, uint64_t* __restrict__ words,
                                                 int32_t* __restrict__ ucount, int64_t m,
                                                 unsigned long long (*sw)[16]) {
    const int lane = threadIdx.x & 63;
    const int64_t I = m / mb, J = m - (m / mb) * mb;
    sw[lane >> 4][lane & 15] = 0ull;
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): zeroing done before the ORs
    for (int ab = 0; ab < 4; ++ab) {
        const int64_t ti = 2 * I + (ab >> 1), tj = 2 * J + (ab & 1);
        if (ti >= bdim || tj >= bdim) continue;
        const int64_t t = ti * bdim + tj;
        const int32_t q0 = off[t], q1 = off[t + 1];
        for (int32_t q = q0 + lane; q < q1; q += 64) {
            const int32_t k = klist[q];
            atomicOr(&sw[ab][k >> 6], 1ull << (k & 63));
        }
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);
    int cnt = 0;
    if (lane < nw) {
        const uint64_t u = sw[0][lane] | sw[1][lane] | sw[2][lane] | sw[3][lane];
        cnt = __popcll(u);
    }
    if (lane < 4 * nw) words[(m * 4 + lane / nw) * nw + lane % nw] = sw[lane / nw][lane % nw];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (lane == 0) ucount[m] = cnt;
}

// packed pair item: I << 23 | J << 14 | k << 4 | membership (bit a*2+b)
__device__ __forceinline__ uint32_t mi_pack(uint32_t I, uint32_t J, uint32_t k, uint32_t mem) {
    return (I << 23) | (J << 14) | (k << 4) | mem;
}

// One wave per macro tile m: its union k values in ascending order, as packed
// items at items[uprefix[m] ..].
__device__ __forceinline__ void macro_items_wave(const uint64_t* __restrict__ words,
                                                 const int32_t* __restrict__ uprefix, int64_t mb, int nw,
                                                 uint32_t* __restrict__ items, int64_t m) {
    const int lane = threadIdx.x & 63;
    const uint32_t I = uint32_t(m / mb), J = uint32_t(m - (m / mb) * mb);
    const uint64_t* wp = words + m * 4 * nw;
    int64_t base = uprefix[m];
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int w = 0; w < nw; ++w) {
        const uint64_t w0 = wp[w], w1 = wp[nw + w], w2 = wp[2 * nw + w], w3 = wp[3 * nw + w];
        const uint64_t u = w0 | w1 | w2 | w3;
        if ((u >> lane) & 1ull) {
            const uint32_t mem = uint32_t((w0 >> lane) & 1) | uint32_t(((w1 >> lane) & 1) << 1) |
                                 uint32_t(((w2 >> lane) & 1) << 2) | uint32_t(((w3 >> lane) & 1) << 3);
            items[base + __popcll(u & below)] = mi_pack(I, J, uint32_t(w) * 64 + lane, mem);
        }
        base += __popcll(u);
    }
}

}  // namespace spamm

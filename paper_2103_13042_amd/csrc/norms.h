// Device code of the leaf norm pass, shared by the single-product and the
// batched kernels.
//
// A block of 256 threads reads a strip of `leaf` rows by 1024 columns; each
// thread owns 4 adjacent columns and sums their squares down the strip in FP64
// (an FP32 square is exact in FP64), then the leaf/4 threads of one tile
// combine their sums with an xor butterfly.  Rows are read as whole 4 KiB
// segments per block, so the pass streams HBM at full coalescing.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.h"

namespace spamm {

constexpr int kNormThreads = 256;
constexpr int kNormCols = kNormThreads * 4;

// NT: nontemporal loads, for a pass whose input is larger than the
// infinity cache: A and B are read once here, and keeping them out of the
// caches leaves room for the multiply's tiles (measured on the N = 8192 step:
// norm pass 112 -> 90 us, multiply unchanged).  Below that size the multiply
// profits from what the pass leaves in the cache (batch of small products:
// 2 % slower with NT).  ALIGNED: the address is a multiple of 16, else of 4.
template <bool ALIGNED, bool NT>
__device__ __forceinline__ f4 load_row(const float* p) {
    if constexpr (ALIGNED) {
        const f4* q = reinterpret_cast<const f4*>(p);
        if constexpr (NT)
            return __builtin_nontemporal_load(q);
        else
            return *q;
    } else {
        const f4_dw* q = reinterpret_cast<const f4_dw*>(p);
        if constexpr (NT)
            return __builtin_nontemporal_load(q);
        else
            return *q;
    }
}

// strip `strip` (tile row) x column chunk `chunk` of x; tile (strip, tj) goes to
// sumsq / norms[strip * ld + tj] (either may be null)
//
// Rows that are not 16-byte aligned (VEC false: n % 4 != 0, or x itself only
// 4-byte aligned) are read by the same 16-byte loads at 4-byte alignment,
// which global loads accept.  The thread whose four columns cross the
// matrix's edge reads the row's last four instead and drops the ones that its
// neighbour holds, so no lane runs a loop of its own (one 64-row column of
// 4-byte loads by that thread took as long as the strip: n = 5003, leaf 64,
// one matrix 42 -> 20 us, as fast as n = 5000).
template <int LEAF, bool VEC, bool NT = false>
__device__ __forceinline__ void leaf_sumsq_strip(const float* __restrict__ x, int64_t n, int64_t bdim, int64_t strip,
                                                 int64_t chunk, double* sumsq, double* norms, int64_t ld) {
    constexpr int G = LEAF / 4;  // threads per tile
    const int64_t r0 = strip * LEAF;
    const int64_t r1 = r0 + LEAF < n ? r0 + LEAF : n;
    const int t = threadIdx.x;
    const int64_t col = chunk * kNormCols + 4 * t;  // columns 4t .. 4t+3 of the chunk
    double acc0 = 0.0, acc1 = 0.0;
    if (!VEC && n < 4) {  // no four columns to read
        for (int64_t r = r0; r < r1; ++r)
            for (int64_t c = col; c < n; ++c) acc0 += double(x[r * n + c]) * double(x[r * n + c]);
    } else if (col < n) {
        const int back = VEC || col + 4 <= n ? 0 : int(col + 4 - n);  // columns that the thread before holds
        const float* p = x + r0 * n + col - back;
        auto add = [&](f4 v) {
            if (!VEC) {
                v.x = back > 0 ? 0.0f : v.x;
                v.y = back > 1 ? 0.0f : v.y;
                v.z = back > 2 ? 0.0f : v.z;
            }
            acc0 += double(v.x) * double(v.x) + double(v.y) * double(v.y);
            acc1 += double(v.z) * double(v.z) + double(v.w) * double(v.w);
        };
        int64_t r = r0;
#pragma unroll 4
        for (; r + 1 < r1; r += 2) {
            const f4 v = load_row<VEC, NT>(p);
            const f4 w = load_row<VEC, NT>(p + n);
            p += 2 * n;
            add(v);
            add(w);
        }
        if (r < r1) add(load_row<VEC, NT>(p));
    }
    double s = acc0 + acc1;
#pragma unroll
    for (int off = 1; off < G; off <<= 1) s += __shfl_xor(s, off);
    const int64_t tj = col / LEAF;
    if ((t % G) == 0 && tj < bdim) {
        const int64_t i = strip * ld + tj;
        if (sumsq) sumsq[i] = s;
        if (norms) norms[i] = sqrt(s);
    }
}

}  // namespace spamm

// Device-side types shared by the kernel sources of libspamm.so.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace spamm {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
// four floats read with one 16-byte load from a 4-byte aligned address
// (global loads accept it)
typedef float f4_dw __attribute__((ext_vector_type(4), aligned(4)));

// p as a pointer into global memory.  A pointer read from memory (a
// descriptor array) carries no address space, so the compiler emits flat
// accesses through it, which also count against the LDS wait counter (an LDS
// wait then waits for every load in flight too); the integer round trip gives
// it the global address space, which the compiler keeps through inlining.
template <typename T>
__device__ __forceinline__ T* global_ptr(T* p) {
    return (T*)(__attribute__((address_space(1))) T*)reinterpret_cast<uintptr_t>(p);
}

// A launch that runs only if *run is not zero (null: always), so that one stream
// can hold both forms of a step and the device pick.
__device__ __forceinline__ bool closed(const int32_t* run) { return run != nullptr && *run == 0; }

// v, as a value the compiler knows nothing about (what is computed from it is
// neither shared with other code nor moved out of a loop)
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

}  // namespace spamm

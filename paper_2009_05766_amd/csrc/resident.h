// For kernels whose workgroups are resident together and exchange data while they run (whole iterations in one launch).
//
// A device-wide barrier is split: a workgroup arrives when its new parameters are in memory and looks for the others' arrival
// only where it needs their rows, half an iteration later.  What the workgroups exchange (and only that) is
// stored and loaded at device scope, past the caches of one XCD, so no cache is written back or dropped: a wave's stores have
// arrived when its vmcnt is zero.
#pragma once
#include "vec.h"

namespace netmax {

__device__ __forceinline__ void store4_device(float *p, f32x4 v)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    unsigned long long *q = reinterpret_cast<unsigned long long *>(p);
    __hip_atomic_store(q, __builtin_bit_cast(unsigned long long, f32x2{v[0], v[1]}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, __builtin_bit_cast(unsigned long long, f32x2{v[2], v[3]}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x4 load4_device(const float *p)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const unsigned long long *q = reinterpret_cast<const unsigned long long *>(p);
    const f32x2 a = __builtin_bit_cast(f32x2, __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const f32x2 b = __builtin_bit_cast(f32x2, __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return f32x4{a[0], a[1], b[0], b[1]};
}
__device__ __forceinline__ void stores_arrived() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ __forceinline__ unsigned arrivals(unsigned *counter) { return __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// A wave that has polled `patience` times in vain raises *fault; it and all that see the flag (they look at every 64th poll) do not
// go on waiting, so the kernel always ends.
__device__ __forceinline__ bool gives_up(long long polls, int *fault, long long patience)
{
    if (polls > patience) {
        __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    return polls % 64 == 0 && __hip_atomic_load(fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}
// Waits until the counter has reached `target`; `seen`: what it was a moment ago.
__device__ __forceinline__ void await_arrivals(unsigned *counter, unsigned seen, unsigned target, int *fault, long long patience)
{
    long long polls = 0;
    while ((patience == 0 || (int)(seen - target) < 0) && !gives_up(++polls, fault, patience)) {
        __builtin_amdgcn_s_sleep(1);
        seen = arrivals(counter);
    }
    asm volatile("" ::: "memory");           // what is read behind the wait is not asked for before it
}

// A new parameter, for this launch's workgroups or (the last iteration's) for what follows the launch.
__device__ __forceinline__ void store_row(float *at, float x, bool more)
{
    if (more) __hip_atomic_store(at, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *at = x;
}
// Element at a 32-bit byte offset: the base stays in scalar registers.  (By way of an integer the pointer would lose its address space, and
// every load be one that may also be of LDS and is waited for as such.)
template <class T> __device__ __forceinline__ T *at_bytes(T *base, uint32_t bytes) { return (T *)((const char *)base + bytes); }

// j / d for 0 <= j < 2^32 / d: the high half of j times ceil(2^32 / d), which of d = 1 has no 32 bits; j itself there.
struct DivBy {
    uint32_t magic, one;
    __device__ __host__ __forceinline__ explicit DivBy(int d) : magic((uint32_t)((0x100000000ull + (uint32_t)d - 1) / (uint32_t)d)), one(d == 1 ? 0xFFFFFFFFu : 0u) {}
    __device__ __forceinline__ int operator()(int j) const { return (int)(__umulhi((uint32_t)j, magic) | ((uint32_t)j & one)); }
};

// The value that lane (l ^ MASK) holds, MASK in {1, 2, 4, 8}, by data-parallel-primitive moves inside the vector unit
// (no trip through the LDS crossbar as a general lane shuffle takes): quad permutations [1,0,3,2] and [2,3,0,1] for
// 1 and 2; for 4 the mirror of each group of eight lanes (l -> l ^ 7) followed by the reversal of each quad (^ 3); for 8 the rotation of
// each group of sixteen by eight.
template <int MASK>
__device__ __forceinline__ float xor_lane(float v)
{
    static_assert(MASK == 1 || MASK == 2 || MASK == 4 || MASK == 8, "lane distances inside a group of sixteen");
    int x = __float_as_int(v);
    if (MASK == 1) x = __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false);
    if (MASK == 2) x = __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false);
    if (MASK == 4) {
        x = __builtin_amdgcn_update_dpp(x, x, 0x141, 0xF, 0xF, false);
        x = __builtin_amdgcn_update_dpp(x, x, 0x1B, 0xF, 0xF, false);
    }
    if (MASK == 8) x = __builtin_amdgcn_update_dpp(x, x, 0x128, 0xF, 0xF, false);
    return __int_as_float(x);
}

// The value, hidden from the optimiser: what is computed from it inside a loop is computed there, not once before
// the loop (address arithmetic of all phases kept in registers across the whole iteration starves the inner loops).
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

}  // namespace netmax

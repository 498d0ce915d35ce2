// Cross-workgroup hand-over of scan aggregates through global memory (gfx950), shared by the scan
// kernels and by the projection GEMM that scans its own output tile.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ssm {

__device__ __forceinline__ float2 cmul(float2 a, float2 b)
{
    // (one rounding order wherever it is inlined)
    return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.x, b.y, a.y * b.x));
}
// a * b + c
__device__ __forceinline__ float2 cfma(float2 a, float2 b, float2 c)
{
    return make_float2(fmaf(a.x, b.x, fmaf(-a.y, b.y, c.x)), fmaf(a.x, b.y, fmaf(a.y, b.x, c.y)));
}

// Cross-workgroup hand-over without fences: every descriptor word is one 64-bit value that
// carries a float in its upper half and a tag in its lower half, written and read with relaxed
// device-scope atomics (write-through / cache-bypassing accesses).  A word whose tag is non-zero
// is complete by construction, so no ordering between different words is ever needed and no
// cache write-back or invalidate is paid.
//   tag 1: aggregate (state for zero incoming state), no reset among the workgroup's steps
//   tag 2: aggregate, a reset among the steps (the product of the transition is zero)
//   tag 3: inclusive state
__device__ __forceinline__ void publish_word(unsigned long long *w, float v, unsigned tag)
{
    __hip_atomic_store(w, ((unsigned long long)__float_as_uint(v) << 32) | tag, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long poll_word(const unsigned long long *w)
{
    return __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float word_value(unsigned long long w) { return __uint_as_float((unsigned)(w >> 32)); }
__device__ __forceinline__ unsigned word_tag(unsigned long long w) { return (unsigned)(w & 0xffffffffu); }

// Waits (bounded) until both words of a pair carry a tag >= min_tag.  Returns false on give-up.
__device__ __forceinline__ bool wait_pair(const unsigned long long *w, unsigned min_tag, unsigned spin_limit,
                                          float2 &value, unsigned &tag)
{
    unsigned spins = 0;
    while (true) {
        const unsigned long long w0 = poll_word(w), w1 = poll_word(w + 1);
        if (word_tag(w0) >= min_tag && word_tag(w1) >= min_tag) {
            value = make_float2(word_value(w0), word_value(w1));
            tag = word_tag(w0);
            return true;
        }
        if (spins >= spin_limit) return false;
        ++spins;
        __builtin_amdgcn_s_sleep(2);
    }
}

// Stores that go through the XCD's L2 to memory at once instead of staying there until the launch ends, when the next one waits for the whole L2 to
// be written back (boundaries between launches: 2.0 us behind a kernel that writes little, 3.2 to 4 behind one that writes 16 MB).
// What the products and their scans write is not read again in the launch.  Forward and gradient pass of 16 x 256 tokens, H = P = 512: 131.4 ->
// 128.4 us; 16 x 64, 256, 256: 46.6 -> 45.3; 4 x 4096, 256, 256: 158.9 -> 156.8; the 64 launches of a roll-out of 1024 x 16: 625 -> 617; launches of
// several rounds within 0.5 % either way.  Outputs and states take it by the rule of store_rule.h; the slabs of the reductions always, at any width (a few MB, written
// once and read by the next launch; limited to widths of whole lines: 1 to 2.5 % slower on twelve of eighteen layers).
__device__ __forceinline__ void store_through(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_through(float2 *p, float2 v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p), __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace ssm

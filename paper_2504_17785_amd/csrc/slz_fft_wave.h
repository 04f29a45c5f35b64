// Device pieces of the transform kernels: LDS and global access by offset, butterflies, and the counters through which waves of
// one workgroup follow each other.
#pragma once
#include <hip/hip_runtime.h>

typedef double d2 __attribute__((ext_vector_type(2)));
#define FFT_FENCE() __builtin_amdgcn_sched_barrier(0)

// LDS by byte offset (32-bit addresses in the LDS address space)
#define LDS_AS __attribute__((address_space(3)))
__device__ __forceinline__ d2 lds_get(uint32_t byte) { return *(const LDS_AS d2 *)(uintptr_t)byte; }
__device__ __forceinline__ void lds_put(uint32_t byte, d2 v) { *(LDS_AS d2 *)(uintptr_t)byte = v; }

// global memory as "uniform base + 32-bit lane offset": one address register for all loads
__device__ __forceinline__ d2 lane_get(const d2 *uniform_base, uint32_t lane) {
    return *reinterpret_cast<const d2 *>(reinterpret_cast<const char *>(uniform_base) + lane * 16u);
}

__device__ __forceinline__ void lane_put(d2 *uniform_base, uint32_t lane, d2 v) {
    *reinterpret_cast<d2 *>(reinterpret_cast<char *>(uniform_base) + lane * 16u) = v;
}

template <int V> struct fft_int { static constexpr int value = V; };

// x w for a plain complex factor
__device__ __forceinline__ d2 cmul(d2 x, d2 w) {
    d2 r;
    r.x = __builtin_fma(-x.y, w.y, x.x * w.x);
    r.y = __builtin_fma(x.y, w.x, x.x * w.y);
    return r;
}
// inverse radix-2, a +- w b with w = c (1 + i t) given as (c, t); TURN: w is further multiplied by -i
template <bool TURN>
__device__ __forceinline__ void inv2(d2 &a, d2 &b, d2 ct) {
    const double ur = __builtin_fma(-ct.y, b.y, b.x), ui = __builtin_fma(ct.y, b.x, b.y);
    const double vr = TURN ? ui : ur, vi = TURN ? -ur : ui;
    b.x = __builtin_fma(-ct.x, vr, a.x);
    b.y = __builtin_fma(-ct.x, vi, a.y);
    a.x = __builtin_fma(ct.x, vr, a.x);
    a.y = __builtin_fma(ct.x, vi, a.y);
}
// forward radix-2 whose twiddle is i w: the second block of every pair of blocks
__device__ __forceinline__ void fwd2i(d2 &a, d2 &b, d2 ct) {
    const double vr = __builtin_fma(-ct.y, b.x, -b.y), vi = __builtin_fma(-ct.y, b.y, b.x);
    b.x = __builtin_fma(-ct.x, vr, a.x);
    b.y = __builtin_fma(-ct.x, vi, a.y);
    a.x = __builtin_fma(ct.x, vr, a.x);
    a.y = __builtin_fma(ct.x, vi, a.y);
}
// inverse radix-4: half-sizes t and 2 t over (a0, a1, a2, a3) with v the twiddle of half-size 2 t and its powers
__device__ __forceinline__ void inv4(d2 &a0, d2 &a1, d2 &a2, d2 &a3, d2 v, d2 v2, d2 v3) {
    const d2 b1 = cmul(a1, v2), b2 = cmul(a2, v), b3 = cmul(a3, v3);
    const d2 s = a0 + b1, d = a0 - b1, e = b2 + b3, f = b2 - b3;
    a0 = s + e;
    a2 = s - e;
    a1.x = d.x + f.y; a1.y = d.y - f.x;
    a3.x = d.x - f.y; a3.y = d.y + f.x;
}

// a +- b and a -+ i b
__device__ __forceinline__ void add2(d2 &a, d2 &b) { const d2 t = b; b = a - t; a = a + t; }
__device__ __forceinline__ void add2i(d2 &a, d2 &b) {                 // b <- a + i b, a <- a - i b  (twiddle -i)
    const d2 t = b;
    b.x = a.x - t.y; b.y = a.y + t.x;
    a.x = a.x + t.y; a.y = a.y - t.x;
}

// forward radix-4: strides 2 n and n over (a0, a1, a2, a3) with v, v^2, v^3
__device__ __forceinline__ void fwd4(d2 &a0, d2 &a1, d2 &a2, d2 &a3, d2 v, d2 v2, d2 v3) {
    const d2 b1 = cmul(a1, v), b2 = cmul(a2, v2), b3 = cmul(a3, v3);
    const d2 s = a0 + b2, d = a0 - b2, e = b1 + b3, f = b1 - b3;
    a0 = s + e;
    a1 = s - e;
    a2.x = d.x - f.y; a2.y = d.y + f.x;
    a3.x = d.x + f.y; a3.y = d.y - f.x;
}

// inverse half-sizes 1, 2, 4: constant twiddles
#define FFT_SQRT_HALF 0.70710678118654752440
__device__ __forceinline__ void inv8(d2 *s) {
    const double r2 = FFT_SQRT_HALF;
#pragma unroll
    for (int k = 0; k < 8; k += 2) add2(s[k], s[k + 1]);
#pragma unroll
    for (int k = 0; k < 8; k += 4) { add2(s[k], s[k + 2]); add2i(s[k + 1], s[k + 3]); }
    add2(s[0], s[4]);
    add2i(s[2], s[6]);
    {   // twiddle sqrt(1/2) (1 - i)
        const double p = s[5].x + s[5].y, q = s[5].y - s[5].x;
        s[5].x = __builtin_fma(-r2, p, s[1].x); s[5].y = __builtin_fma(-r2, q, s[1].y);
        s[1].x = __builtin_fma(r2, p, s[1].x); s[1].y = __builtin_fma(r2, q, s[1].y);
    }
    {   // twiddle sqrt(1/2) (-1 - i)
        const double p = s[7].y - s[7].x, q = s[7].x + s[7].y;
        s[7].x = __builtin_fma(-r2, p, s[3].x); s[7].y = __builtin_fma(r2, q, s[3].y);
        s[3].x = __builtin_fma(r2, p, s[3].x); s[3].y = __builtin_fma(-r2, q, s[3].y);
    }
}

// forward radix-8 with u .. u^7: the values of sum_k x_k (u z)^k at z = 1, -1, i, -i, w, -w, iw, -iw, w = (1 + i) / sqrt(2)
__device__ __forceinline__ void fwd8(d2 *x, const d2 *u) {
    const double r2 = FFT_SQRT_HALF;
#pragma unroll
    for (int k = 1; k < 8; k++) x[k] = cmul(x[k], u[k - 1]);
    const d2 s04 = x[0] + x[4], d04 = x[0] - x[4], s26 = x[2] + x[6], d26 = x[2] - x[6];
    const d2 s15 = x[1] + x[5], d15 = x[1] - x[5], s37 = x[3] + x[7], d37 = x[3] - x[7];
    const d2 e0 = s04 + s26, e1 = s04 - s26, o0 = s15 + s37, o1 = s15 - s37;
    d2 e2, e3, o2, o3;
    e2.x = d04.x - d26.y; e2.y = d04.y + d26.x;
    e3.x = d04.x + d26.y; e3.y = d04.y - d26.x;
    o2.x = d15.x - d37.y; o2.y = d15.y + d37.x;
    o3.x = d15.x + d37.y; o3.y = d15.y - d37.x;
    x[0] = e0 + o0;
    x[1] = e0 - o0;
    x[2].x = e1.x - o1.y; x[2].y = e1.y + o1.x;
    x[3].x = e1.x + o1.y; x[3].y = e1.y - o1.x;
    const double p2 = o2.x - o2.y, q2 = o2.x + o2.y, p3 = o3.x - o3.y, q3 = o3.x + o3.y;
    x[4].x = __builtin_fma(r2, p2, e2.x); x[4].y = __builtin_fma(r2, q2, e2.y);
    x[5].x = __builtin_fma(-r2, p2, e2.x); x[5].y = __builtin_fma(-r2, q2, e2.y);
    x[6].x = __builtin_fma(-r2, q3, e3.x); x[6].y = __builtin_fma(r2, p3, e3.y);
    x[7].x = __builtin_fma(r2, q3, e3.x); x[7].y = __builtin_fma(-r2, p3, e3.y);
}

// acc += y 2^s for the bits y of (integer + 1.5 * 2^52): the bits of that constant lie above bit 50, so they leave the word with any
// shift of 13 or more; a shift past 32 only concerns the upper half
template <int s>
__device__ __forceinline__ void add_shifted(uint64_t &acc, uint64_t y) {
    if constexpr (s >= 32) {
        // one 32-bit operation (spelled out: the compiler widens the plain expression to a 64-bit addition with its moves)
        uint32_t hi = (uint32_t)(acc >> 32);
        asm("v_lshl_add_u32 %0, %1, %2, %0" : "+v"(hi) : "v"((uint32_t)y), "n"(s - 32));
        acc = ((uint64_t)hi << 32) | (uint32_t)acc;
    } else {
        acc += y << s;
    }
}

// The two waves of a ciphertext follow each other through two counters per wave in LDS: `done` (its part of an exchange has
// been written) and `free` (it has read what the other wave may overwrite next).  Both waves are resident in the same
// workgroup and take the same sequence of steps, so every wait ends.  LDS operations of one wave execute in order, so a
// counter written after data (or after reads) is seen after them.
__device__ __forceinline__ void fft_signal(uint32_t flag, uint32_t value) {
    asm volatile("" ::: "memory");
    __hip_atomic_store((LDS_AS uint32_t *)(uintptr_t)flag, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ uint32_t fft_peek(uint32_t flag) {
    return __hip_atomic_load((const LDS_AS uint32_t *)(uintptr_t)flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// `seen`: what an earlier fft_peek returned, so that a counter that has long arrived costs no LDS round trip here
__device__ __forceinline__ void fft_wait(uint32_t flag, uint32_t seen, uint32_t value) {
    asm volatile("" ::: "memory");
    while ((int32_t)((uint32_t)__builtin_amdgcn_readfirstlane(seen) - value) < 0) {
        __builtin_amdgcn_s_sleep(1);
        seen = fft_peek(flag);
    }
    asm volatile("" ::: "memory");
}

// Counters of the four waves of a component from `flags` on, one read for all of them.  As in fft_wait, every wave of the workgroup is
// resident and takes the same sequence of exchanges, so every wait ends.
__device__ __forceinline__ uint32_t peek_four(uint32_t flags, uint32_t lane) { return fft_peek(flags + 4u * (lane & 3u)); }
__device__ __forceinline__ void wait_four(uint32_t flags, uint32_t lane, uint32_t seen, uint32_t value) {
    asm volatile("" ::: "memory");
    while (__builtin_amdgcn_ballot_w64((int32_t)(seen - value) < 0)) {
        __builtin_amdgcn_s_sleep(1);
        seen = peek_four(flags, lane);
    }
    asm volatile("" ::: "memory");
}

// Values are complete here: pure arithmetic would otherwise be sunk past the waits below into the block that uses it.
__device__ __forceinline__ void pin(d2 &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void pin(uint64_t &v) { asm volatile("" : "+v"(v)); }

// A copy of the lane number that the compiler cannot trace back: the LDS addresses made from it are computed where they are
// used (a few 32-bit operations) instead of being kept in registers across the whole step.
__device__ __forceinline__ uint32_t fresh(uint32_t lane) {
    asm volatile("" : "+v"(lane));
    return lane;
}

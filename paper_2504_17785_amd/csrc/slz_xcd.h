// Workgroups of one XCD that work together through its L2, and pairs of them.
//
// Memory order.  The vector L1 caches are not coherent; an XCD's L2 is shared by all its compute units.  What one workgroup writes for another goes
// to the L2 by plain stores (the L1 writes through, s_waitcnt vmcnt(0) waits for the L2's acknowledgement), and is read by agent-scope loads, which
// pass the L1.  This holds inside one XCD only, so workgroups find each other by the XCC_ID they run on; words that workgroups of
// different XCDs share are written and read by agent-scope atomics alone.
#pragma once
#include "slz_internal.h"
#include "slz_fft_wave.h"

__device__ __forceinline__ uint32_t slz_xcc_id() {
    uint32_t v;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
    return v & 15u;
}
__device__ __forceinline__ uint32_t ld_agent(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// This wave's stores have reached the L2; then the word is written there.
__device__ __forceinline__ void slz_xcd_report(uint32_t *word, uint32_t value) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if ((threadIdx.x & 63u) == 0) __hip_atomic_store(word, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Waits for a workgroup that runs and takes the same sequence of steps, so it ends.
__device__ __forceinline__ void slz_xcd_await(const uint32_t *word, uint32_t value) {
    asm volatile("" ::: "memory");
    while ((int32_t)(__builtin_amdgcn_readfirstlane(ld_agent(word)) - value) < 0) {}
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ d2 lane_get_l2(const d2 *uniform_base, uint32_t lane) {
    const double *p = reinterpret_cast<const double *>(reinterpret_cast<const char *>(uniform_base) + lane * 16u);
    d2 r;
    r.x = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    r.y = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return r;
}

// Pairs.  A workgroup takes a number on its XCD; two with successive numbers are a pair, the second of which asks for ciphertexts for both until
// there are none left.  First all workgroups of the launch have to have come, within `patience` of the one that waits longest; otherwise all leave, those
// that come later too, and a launch behind this one that pairs nothing takes the ciphertexts.  So a launch ends whatever places it is given (one
// compute unit of an XCD, under a mask of compute units, holds one of these workgroups and never a pair), and takes twice the compute units of the kernel that
// pairs nothing only where they stand idle: beside other calls two of them do less than one on each of two ciphertexts.  200 steps of N = 2048 by
// several contexts on streams of their own, us with one workgroup / pairs at once / this: 2 x 64 ciphertexts
// 1877 / 1383 / 1389, 2 x 100: 1880 / 2429 / 2115, 3 x 80: 1890 / 2942 / 2109, 4 x 60: 1890 / 2694 / 2228; 2 x 128, where each finds all compute units free in
// turn, 1903 / 2673 / 2692; N = 4096, 3 x 80: 3398 / 6804 / 3925.  It costs a call of its own 1 to 3 us.
// Once all have come, the two of a pair wait for each other alone, and both run; a first one without a second leaves.
#define SLZ_PAIR_MAX 128u                           // pairs of a launch: 256 workgroups
#define SLZ_PAIR_NONE 0xffffffffu
#define SLZ_PAIR_PATIENCE 2000u                     // 20 us of the 100 MHz clock; where there is room the last one comes within 1 (16 workgroups) to 6 us (256) of the first
struct slz_pairs {
    uint32_t *ctl;            // words, zero at the start: [0] ciphertexts taken, [16] whether there are pairs, [32] workgroups that have come and, times 2^16, pairs,
                              // [64 + 32 x] numbers of XCD x, then [16][128] pair + 1 by XCD and number / 2, then a line of 32 words per pair: [8] progress of
                              // its waves, [8] the ciphertext at hand
    uint32_t patience;
};
#define SLZ_PAIR_MET 576u
#define SLZ_PAIR_LINES (SLZ_PAIR_MET + 16u * 128u)
#define SLZ_PAIR_WORDS (SLZ_PAIR_LINES + 32u * SLZ_PAIR_MAX)
__device__ __forceinline__ uint32_t *slz_pair_line(slz_pairs P, uint32_t pair) { return P.ctl + SLZ_PAIR_LINES + 32u * pair; }

// One thread: 2 pair + (0 first, 1 second), or SLZ_PAIR_NONE
__device__ __forceinline__ uint32_t slz_pair_join(slz_pairs P) {
    enum : uint32_t { GO = 1, LEAVE = 2 };
    const uint32_t x = slz_xcc_id();
    uint32_t *decision = P.ctl + 16, *numbers = P.ctl + 64 + 32 * x;
    auto settle = [&](uint32_t value) -> uint32_t {                 // the word has one value after zero: whoever comes first writes it
        uint32_t seen = 0;
        return __hip_atomic_compare_exchange_strong(decision, &seen, value, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? value : seen;
    };
    const uint32_t number = __hip_atomic_fetch_add(numbers, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t second = number & 1u;
    uint32_t *met = P.ctl + SLZ_PAIR_MET + 128 * x + number / 2;
    const uint32_t before = __hip_atomic_fetch_add(P.ctl + 32, 1u + (second << 16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t pair = (before >> 16) + 1;
    if (second) __hip_atomic_store(met, pair, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const uint64_t since = wall_clock64();
    uint32_t found = (before & 0xffffu) + 1 == gridDim.x ? settle(GO) : 0;
    while (!found) {
        found = ld_agent(decision);
        if (!found && wall_clock64() - since >= P.patience) found = settle(LEAVE);
    }
    if (found == LEAVE) return SLZ_PAIR_NONE;
    if (second) return 2 * (pair - 1) + 1;
    // All have taken their numbers.  Read by an atomic addition like those that made it, as it is looked at once: a first workgroup that overlooked its
    // second would leave that one waiting.  (Of a zero that the compiler sees it makes a load.)
    uint32_t zero = 0;
    asm volatile("" : "+v"(zero));
    if (__hip_atomic_fetch_add(numbers, zero, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == number + 1) return SLZ_PAIR_NONE;
    while (!(pair = ld_agent(met))) {}                              // the second is past its number, and writes this next
    return 2 * (pair - 1);
}
// One thread of either workgroup: the pair's ciphertext of this round, or one past the last
__device__ __forceinline__ uint32_t slz_pair_next(slz_pairs P, uint32_t pair, uint32_t second, uint32_t round) {
    uint32_t *word = slz_pair_line(P, pair) + 8;
    if (second) {
        const uint32_t c = __hip_atomic_fetch_add(P.ctl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(word, ((round + 1) << 16) | c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        return c;
    }
    for (;;) {
        const uint32_t w = ld_agent(word);
        if (w >> 16 == round + 1) return w & 0xffffu;
    }
}

// Two workgroups per ciphertext of every XCD's share, and the most that a context has memory for
static inline uint32_t slz_pairs_grid(uint32_t batch) { return 16u * ((batch + 7) / 8); }
static inline uint32_t slz_pairs_most(const slz_ctx *ctx) { return slz_pairs_grid(ctx->max_batch < SLZ_PAIR_MAX ? ctx->max_batch : SLZ_PAIR_MAX); }
// host (slz_fft.hip)
void slz_pairs_clear(slz_ctx *ctx, hipStream_t s);

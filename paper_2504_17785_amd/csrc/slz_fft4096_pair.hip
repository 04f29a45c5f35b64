// Blind rotation for N = 4096, k = 1, l = 1, up to 128 ciphertexts: two workgroups of one XCD on each ciphertext, a component each, as in
// slz_fft2048_pair.hip.  Passes, layouts and maps are those of slz_fft4096.hip, where the eight waves of one workgroup do both components; key,
// tables and the error bound too.  The spectrum is 32 KiB; the group without the accumulator finds its copy in its own buffers and leaves its sums there.
// What bounds it: 34 k cycles per step, 17 k of them the late group's three pieces in turn, one chain of passes per wave, beside the
// key's way: 320 KiB per step and workgroup are 10 bytes per clock of the 13 to 20 that a compute unit gets from beyond the L2.  Measured, us per
// step, before (one workgroup) / now: 1 ciphertext 16.4 / 14.5, 100: 16.5 / 14.75, 128: 16.6 / 15.1; with group 0 at the priority of group 1 15.7;
// key words requested earlier, eight or sixteen loads at a time, 15.3.
#include "slz_fft.h"
#include "slz_fft_wave.h"
#include "slz_modarith.h"
#include "slz_fused_common.h"
#include "slz_xcd.h"

#define F12P_THREADS 512
#define F12P_BUF (544u * 16u)                        // bytes of a wave's buffer: 512 points, padded
#define F12P_FLAGS_OFF (8u * F12P_BUF + F12_LDS_TAB * 16u)
#define F12P_LDS_BYTES (F12P_FLAGS_OFF + 128u)        // done and free per wave and group; spectrum written, sums written per wave; two words

struct fft4096p_args {
    const uint64_t *lwe_in;
    const uint64_t *luts;
    const uint32_t *lut_idx;
    const d2 *key;            // [n][F12_KEY_STEP]
    const d2 *tab;            // F12_TAB_LEN entries
    uint64_t *acc_out;
    uint64_t *lwe_out;
    slz_pairs pairs;
    d2 *mail;                 // [pair][parity of the step][component][quarter][512]
    uint32_t n, n_steps, batch, beta;
    double f1[6][2];          // lane-uniform twiddles of the second forward layer: (v, v^2, v^3) of its two blocks
};

__global__ void __launch_bounds__(F12P_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_fft4096_pair(fft4096p_args A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const uint32_t lds = (uint32_t)(uintptr_t)(LDS_AS unsigned char *)lds_raw;
    const uint32_t beta = A.beta;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t late = wave >> 2, g = wave & 3u;                                         // group 0: front and pieces 3 and 4, group 1: pieces 0 to 2
    const uint32_t C0 = lds + late * 4u * F12P_BUF, R0 = lds + wave * F12P_BUF;             // the group's buffers; this wave's
    const uint32_t tab0 = lds + 8u * F12P_BUF;
    const uint32_t flags = lds + F12P_FLAGS_OFF;
    const uint32_t done = flags + 32u * late, freed = done + 16u, my_done = done + 4u * g, my_free = freed + 4u * g;
    const uint32_t spec_done = flags + 64u + 4u * g, sums_done = flags + 80u, told = flags + 96u;
    for (uint32_t i = threadIdx.x; i < F12_LDS_TAB; i += F12P_THREADS) lds_put(tab0 + 16u * i, A.tab[i]);
    if (threadIdx.x < 32) *(LDS_AS uint32_t *)(uintptr_t)(flags + 4u * threadIdx.x) = 0;
    auto broadcast = [&](uint32_t v) -> uint32_t {                                          // thread 0's value to all
        __syncthreads();
        if (threadIdx.x == 0) *(LDS_AS uint32_t *)(uintptr_t)told = v;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(*(const LDS_AS uint32_t *)(uintptr_t)told);
    };
    const uint32_t place = broadcast(threadIdx.x == 0 ? slz_pair_join(A.pairs) : 0u);
    if (place == SLZ_PAIR_NONE) return;
    const uint32_t h = place & 1u, box = place >> 1;                                        // component; pair
    uint32_t *line = slz_pair_line(A.pairs, box);
    d2 *mail = A.mail + (size_t)box * 8192u;

    const double magic = 6755399441055744.0, r2 = FFT_SQRT_HALF;      // 1.5 * 2^52: adding it rounds to an integer
    uint32_t ex = 0;                                                  // exchanges between the waves of the group so far
    uint32_t tick = 0;                                                // steps so far
    for (uint32_t round = 0;; round++) {
        const uint32_t c = broadcast(threadIdx.x == 0 ? slz_pair_next(A.pairs, box, h, round) : 0u);
        if (c >= A.batch) return;
        auto work = [&](auto group) __attribute__((always_inline)) {          // one per group: their registers have nothing to do with each other
        constexpr bool late = decltype(group)::value;
        const uint64_t *lwe = A.lwe_in + (size_t)c * (A.n + 1);
        uint64_t accr[8], acci[8];                                    // negated coefficients 256 e + 64 g + lane and 2048 more of component h
        const uint32_t li = 64u * g + fresh(lane);
        if (h == 1 && !late) {
            const uint32_t bt = slz_modswitch(lwe[A.n], 13);
            const uint32_t r = (8192u - bt) & 8191u;
            const uint64_t *lut = A.luts + (size_t)(A.lut_idx ? A.lut_idx[c] : 0) * 4096u;
#pragma unroll
            for (int e = 0; e < 8; e++) {
                accr[e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 256u * e + li, r, 4096u);
                acci[e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 2048u + 256u * e + li, r, 4096u);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; e++) accr[e] = acci[e] = 0;
        }

        // The accumulator is written to its component's buffers whenever it is complete: here and at the end of every step.
        auto stage = [&](int e) {
            LDS_AS uint64_t *S = (LDS_AS uint64_t *)(uintptr_t)C0 + 64u * g;
            S[256 * e + lane] = accr[e];
            S[2048 + 256 * e + lane] = acci[e];
        };
        if (!late) {
#pragma unroll
            for (int e = 0; e < 8; e++) stage(e);
            fft_signal(my_done, ++ex);
        }
        uint64_t mask = lwe[0];
        d2 kb[8][2];                                                  // key words of the next piece
        constexpr size_t PIECE = F12_KEY_STEP / SLZ_FFT_PIECES;       // pieces and steps follow each other at the same distance
        const d2 *kp = A.key + (g * 8u * 4u + h) * 64u + (late ? 0 : 3 * PIECE);          // [piece][quarter][k][row, component][lane]
        // four loads at a time, spread over the passes: more of them together would fill the memory pipeline's queue and hold the wave; the row of
        // this workgroup's component comes first, as its spectrum does
        auto request = [&](int part) __attribute__((always_inline)) {
            const uint32_t kl = fresh(lane);
#pragma unroll
            for (int k = 2 * part; k < 2 * part + 2; k++)
#pragma unroll
                for (int r = 0; r < 2; r++) kb[k][r] = lane_get(kp + (4 * k + 2 * (r ^ h)) * 64, kl);
            if (part == 3) kp += PIECE;
            FFT_FENCE();
        };
#pragma unroll
        for (int part = 0; part < 4; part++) request(part);
        // F4 and both components' spectra at this wave's quarter of the points
        auto spectra = [&](d2 (&D)[2][8]) __attribute__((always_inline)) {
            int z;
            asm volatile("s_mov_b32 %0, 0" : "=s"(z));
            const uint32_t ln = fresh(lane);
            d2 f4[6];
            const d2 *t4 = A.tab + F12_F4_OFF + g * 384u + z;
#pragma unroll
            for (int q = 0; q < 6; q++) f4[q] = lane_get(t4 + 64 * q, ln);
            // lane = b8..b3; register = b2 b1 b0
            const uint32_t r0 = R0 + z + 16u * (17u * (16u * (ln >> 5) + 8u * ((ln >> 4) & 1u) + 2u * ((ln >> 1) & 1u) + (ln & 1u)) +
                                                8u * ((ln >> 3) & 1u) + 4u * ((ln >> 2) & 1u));
#pragma unroll
            for (int k = 0; k < 8; k++) D[0][k] = lds_get(r0 + 16 * (17 * 4 * (k >> 2) + (k & 3)));
            slz_xcd_await(line + 4u * (h ^ 1u) + g, tick + 1);
            const d2 *from_there = mail + ((((tick & 1u) * 2u + (h ^ 1u)) * 4u + g) * 512u);
#pragma unroll
            for (int k = 0; k < 8; k++) D[1][k] = lane_get_l2(from_there + k, 8u * ln);
            FFT_FENCE();
#pragma unroll
            for (int cc = 0; cc < 2; cc++)
#pragma unroll
                for (int b = 0; b < 2; b++) fwd4(D[cc][4 * b], D[cc][4 * b + 1], D[cc][4 * b + 2], D[cc][4 * b + 3], f4[3 * b], f4[3 * b + 1], f4[3 * b + 2]);
        };
        auto run_piece = [&](auto which, auto place_in_group, const d2 (&D)[2][8], uint32_t step) __attribute__((always_inline)) {
            constexpr int piece = decltype(which)::value;
            constexpr bool FIRST = decltype(place_in_group)::value == 0, LAST = piece == 2 || piece == 4;
            int z;
            asm volatile("s_mov_b32 %0, 0" : "=s"(z));
            const uint32_t T = C0 + z, R = R0 + z;
            d2 x[8];
            const uint32_t tb = tab0 + z;
            d2 S[8];
            FFT_FENCE();
            const uint32_t free_seen = peek_four(freed, lane);
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const d2 k0 = kb[k][0], k1 = kb[k][1], a = D[0][k], b = D[1][k];
                S[k].x = __builtin_fma(-b.y, k1.y, __builtin_fma(b.x, k1.x, __builtin_fma(-a.y, k0.y, a.x * k0.x)));
                S[k].y = __builtin_fma(b.y, k1.x, __builtin_fma(b.x, k1.y, __builtin_fma(a.y, k0.x, a.x * k0.y)));
                pin(S[k]);
            }
            FFT_FENCE();
            // the group's next key words (the next step's after the last piece, if there is one) arrive during this inverse transform
            const bool more = !LAST || step + 1 < A.n_steps;
            if (LAST) kp += (piece == 2 ? 2 : 3) * PIECE;
            if (more) request(0);
            inv8(S);                                              // I1: half-sizes 1, 2, 4
            if (!FIRST) wait_four(freed, lane, free_seen, ex);    // the waves that read this one's buffer have done so
            {
                const uint32_t ln = fresh(lane);                  // b8..b3; register = b2 b1 b0
                const uint32_t w = R + 16u * (17u * (16u * (ln >> 5) + 8u * ((ln >> 4) & 1u) + (ln & 7u)) + 8u * ((ln >> 3) & 1u));
#pragma unroll
                for (int k = 0; k < 8; k++) lds_put(w + 16 * k, S[k]);
            }
            if (more) request(1);
            {   // I2: half-sizes 8, 16, 32; lane = b8 b7 b6 b2 b1 b0; register = b5 b4 b3
                const uint32_t ln = fresh(lane);
                const uint32_t r0 = R + 16u * (17u * (16u * (ln >> 5) + 8u * ((ln >> 4) & 1u)) + 8u * ((ln >> 3) & 1u) + (ln & 7u));
                const uint32_t t2 = tb + F12_I2_OFF * 16u + 16u * (ln & 7u);
                const d2 i2v = lds_get(t2), i2v2 = lds_get(t2 + 128), i2v3 = lds_get(t2 + 256), i2w0 = lds_get(t2 + 384), i2w1 = lds_get(t2 + 512);
#pragma unroll
                for (int m = 0; m < 8; m++) x[m] = lds_get(r0 + 16 * 17 * m);
                FFT_FENCE();
                inv4(x[0], x[1], x[2], x[3], i2v, i2v2, i2v3);
                inv4(x[4], x[5], x[6], x[7], i2v, i2v2, i2v3);
                inv2<false>(x[0], x[4], i2w0); inv2<false>(x[1], x[5], i2w1);
                inv2<true>(x[2], x[6], i2w0); inv2<true>(x[3], x[7], i2w1);
                const uint32_t w = R + 16u * (17u * (16u * (ln >> 5) + 4u * ((ln >> 4) & 1u) + 8u * ((ln >> 3) & 1u)) + (ln & 7u));
#pragma unroll
                for (int m = 0; m < 8; m++) lds_put(w + 16 * (17 * (m >> 1) + 8 * (m & 1)), x[m]);
            }
            if (more) request(2);
            {   // I3: half-sizes 64, 128, 256; lane = b5..b0; register = b8 b7 b6
                const uint32_t ln = fresh(lane);
                const uint32_t t3 = tb + F12_I3_OFF * 16u + 16u * ln;
                const d2 v = lds_get(t3), v2 = lds_get(t3 + 1024), v3 = lds_get(t3 + 2048), w0 = lds_get(t3 + 3072), w1 = lds_get(t3 + 4096);
                const uint32_t r0 = R + 16u * (17u * (ln >> 4) + (ln & 15u));
#pragma unroll
                for (int m = 0; m < 8; m++) x[m] = lds_get(r0 + 16 * 17 * (16 * (m >> 2) + 4 * ((m >> 1) & 1) + 8 * (m & 1)));
                FFT_FENCE();
                inv4(x[0], x[1], x[2], x[3], v, v2, v3);
                inv4(x[4], x[5], x[6], x[7], v, v2, v3);
                inv2<false>(x[0], x[4], w0); inv2<false>(x[1], x[5], w1);
                inv2<true>(x[2], x[6], w0); inv2<true>(x[3], x[7], w1);
#pragma unroll
                for (int m = 0; m < 8; m++) lds_put(r0 + 16 * 17 * 4 * m, x[m]);
            }
            fft_signal(my_done, ++ex);
            if (more) request(3);
            {   // I4: half-sizes 512 and 1024 with the twist; lane = b5..b0, wave = b7 b6; register = b10 b9 b8
                const uint32_t ln = fresh(lane);
                const uint32_t t4 = tb + F12_I4_OFF * 16u + 16u * (64u * g + ln);
                const d2 w0 = lds_get(t4);
                d2 c1[2], c2[2];
                c1[0] = lds_get(t4 + 4096); c2[0] = lds_get(t4 + 8192);
                FFT_FENCE();
                wait_four(done, lane, peek_four(done, lane), ex);
                const uint32_t r0 = T + 16u * (17u * (4u * g + (ln >> 4)) + (ln & 15u));
#pragma unroll
                for (int e = 0; e < 8; e++) x[e] = lds_get(r0 + (e >> 1) * F12P_BUF + 16 * 17 * 16 * (e & 1));
                fft_signal(my_free, ex);
                FFT_FENCE();
                inv2<false>(x[0], x[2], w0); inv2<true>(x[1], x[3], w0);
                inv2<false>(x[4], x[6], w0); inv2<true>(x[5], x[7], w0);
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    FFT_FENCE();
                    if (e + 1 < 4) { c1[(e + 1) & 1] = lds_get(t4 + 4096 * (3 + 2 * e)); c2[(e + 1) & 1] = lds_get(t4 + 4096 * (4 + 2 * e)); }
                    FFT_FENCE();
                    d2 a = cmul(x[e], c1[e & 1]), b = x[e + 4];
                    inv2<false>(a, b, c2[e & 1]);
                    // coefficients 256 e + .. (a) and 1024 + 256 e + .. (b turned by -45 degrees), rounded
                    const uint64_t y0 = (uint64_t)__double_as_longlong(a.x + magic), y1 = (uint64_t)__double_as_longlong(a.y + magic);
                    const uint64_t y2 = (uint64_t)__double_as_longlong(__builtin_fma(b.x + b.y, r2, magic));
                    const uint64_t y3 = (uint64_t)__double_as_longlong(__builtin_fma(b.y - b.x, r2, magic));
                    add_shifted<SLZ_FFT_PIECE_BITS * piece>(accr[e], y0);
                    add_shifted<SLZ_FFT_PIECE_BITS * piece>(acci[e], y1);
                    add_shifted<SLZ_FFT_PIECE_BITS * piece>(accr[e + 4], y2);
                    add_shifted<SLZ_FFT_PIECE_BITS * piece>(acci[e + 4], y3);
                    if (piece == 0) {                             // the bits of `magic` that shift 0 has left
                        accr[e] -= 0x4338000000000000ull; acci[e] -= 0x4338000000000000ull;
                        accr[e + 4] -= 0x4338000000000000ull; acci[e + 4] -= 0x4338000000000000ull;
                    }
                    pin(accr[e]); pin(acci[e]); pin(accr[e + 4]); pin(acci[e + 4]);
                }
            }
        };
        if constexpr (late) {
            __builtin_amdgcn_s_setprio(1);                            // it has the longer half: 15.7 -> 14.75 us per step at 100 ciphertexts
            for (uint32_t step = 0; step < A.n_steps; step++) {
                d2 D[2][8];
                fft_wait(spec_done, fft_peek(spec_done), tick + 1);
                spectra(D);
#pragma unroll
                for (int e = 0; e < 8; e++) accr[e] = acci[e] = 0;
                run_piece(fft_int<0>(), fft_int<0>(), D, step);
                run_piece(fft_int<1>(), fft_int<1>(), D, step);
                run_piece(fft_int<2>(), fft_int<2>(), D, step);
                wait_four(freed, lane, peek_four(freed, lane), ex);   // the sums go into this wave's buffer
                LDS_AS uint64_t *M = (LDS_AS uint64_t *)(uintptr_t)R0 + fresh(lane);
#pragma unroll
                for (int e = 0; e < 8; e++) { M[64 * e] = accr[e]; M[512 + 64 * e] = acci[e]; }
                fft_signal(sums_done + 4u * g, ++tick);
            }
            return;
        }
        for (uint32_t step = 0; step < A.n_steps; step++) {
            // an opaque zero in every table and buffer address keeps the loads inside the step
            int z;
            asm volatile("s_mov_b32 %0, 0" : "=s"(z));
            const uint32_t T = C0 + z, R = R0 + z;
            const uint32_t tab = tab0 + z;
            d2 D[2][8];
            {
                d2 x[8];
                const uint32_t at = slz_modswitch(mask, 13);
                mask = lwe[step + 1];                                 // the next step's word (the body after the last step)
                wait_four(done, lane, peek_four(done, lane), ex);
                // ---- 1. digits ----
                {
                    // word (idx - at) mod 8192 of X^at ACC: twelve bits of address, the thirteenth is the sign; its opposite (bit 15 of t)
                    // tells where the stored, negated word has to be negated again
                    const uint32_t rnd = 1u << (31 - beta), t0 = 8u * (64u * g + fresh(lane)) + 0x8000u - 8u * at;
                    auto word = [&](uint32_t t) { return *(const LDS_AS uint64_t *)(uintptr_t)(T + (t & 0x7ff8u)); };
                    auto digit = [&](uint32_t t, uint64_t a, uint64_t own) {
                        const uint32_t m = (uint32_t)((int32_t)(t << 16) >> 31);
                        uint32_t lo = (uint32_t)a ^ m, hi = (uint32_t)(a >> 32) ^ m;
                        asm("v_cmp_ne_u32_e32 vcc, 0, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %3, vcc\n\tv_addc_co_u32_e32 %1, vcc, %1, %4, vcc"
                            : "+v"(lo), "+v"(hi) : "v"(m), "v"((uint32_t)own), "v"((uint32_t)(own >> 32)) : "vcc");
                        return (double)((int32_t)(hi + rnd) >> (32 - beta));
                    };
                    uint64_t a[2][8];
#pragma unroll
                    for (int i = 0; i < 8; i++) a[0][i] = word(t0 + 2048u * i);
#pragma unroll
                    for (int i = 0; i < 8; i++) a[1][i] = word(t0 + 16384u + 2048u * i);
                    fft_signal(my_free, ex);
#pragma unroll
                    for (int i = 0; i < 8; i++) x[i].x = digit(t0 + 2048u * i, a[0][i], accr[i]);
#pragma unroll
                    for (int i = 0; i < 8; i++) x[i].y = digit(t0 + 16384u + 2048u * i, a[1][i], acci[i]);
                }
                // ---- 2. forward transform ----
                // F1: stride 1024 with the twiddle (1 + i) / sqrt(2), whose sums of digits are exact; strides 512 and 256
                const uint32_t free_seen = peek_four(freed, lane);
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const double p = x[e + 4].x - x[e + 4].y, q = x[e + 4].x + x[e + 4].y;
                    x[e + 4].x = __builtin_fma(-r2, p, x[e].x); x[e + 4].y = __builtin_fma(-r2, q, x[e].y);
                    x[e].x = __builtin_fma(r2, p, x[e].x); x[e].y = __builtin_fma(r2, q, x[e].y);
                }
                auto f1 = [&](int q) { d2 w; w.x = A.f1[q + z][0]; w.y = A.f1[q + z][1]; return w; };
                fwd4(x[0], x[1], x[2], x[3], f1(0), f1(1), f1(2));
                fwd4(x[4], x[5], x[6], x[7], f1(3), f1(4), f1(5));
                wait_four(freed, lane, free_seen, ex);                // every wave has read its rotated words
                {
                    const uint32_t ln = fresh(lane);
                    // b7 b6 are this wave's, b5 b4 / b3..b0 the lane's; e = b10 b9 b8
                    const uint32_t w = T + 16u * (17u * ((g & 1u) * 8u + (g >> 1) + (ln >> 5) * 4u + ((ln >> 4) & 1u) * 2u) + (ln & 15u));
#pragma unroll
                    for (int e = 0; e < 8; e++) lds_put(w + (e >> 1) * F12P_BUF + 16 * 17 * 16 * (e & 1), x[e]);
                }
                fft_signal(my_done, ++ex);
                d2 u[7];
                {
                    const uint32_t ln = fresh(lane);
                    const uint32_t tf = tab + F12_F2_OFF * 16u + 16u * (2u * g + (ln >> 5));
#pragma unroll
                    for (int t = 0; t < 7; t++) u[t] = lds_get(tf + 128 * t);
                    FFT_FENCE();
                    wait_four(done, lane, peek_four(done, lane), ex);
                    // lane = b8 b4 b3..b0; register = b7 b6 b5
                    const uint32_t r0 = R + 16u * (17u * (16u * (ln >> 5) + 2u * ((ln >> 4) & 1u)) + (ln & 15u));
                    auto slot = [](int m) { return 16 * 17 * ((m >> 2) + 8 * ((m >> 1) & 1) + 4 * (m & 1)); };
#pragma unroll
                    for (int m = 0; m < 8; m++) x[m] = lds_get(r0 + slot(m));
                    FFT_FENCE();
                    fwd8(x, u);
#pragma unroll
                    for (int m = 0; m < 8; m++) lds_put(r0 + slot(m), x[m]);
                }
                {
                    const uint32_t ln = fresh(lane);
                    // lane = b8 b7 b6 b5 b1 b0; register = b4 b3 b2
                    const uint32_t tf = tab + F12_F3_OFF * 16u + 16u * (16u * g + (ln >> 2));
#pragma unroll
                    for (int t = 0; t < 7; t++) u[t] = lds_get(tf + 1024 * t);
                    const uint32_t r0 = R + 16u * (17u * (16u * (ln >> 5) + ((ln >> 4) & 1u) + 8u * ((ln >> 3) & 1u) + 4u * ((ln >> 2) & 1u)) + (ln & 3u));
#pragma unroll
                    for (int m = 0; m < 8; m++) x[m] = lds_get(r0 + 16 * (17 * 2 * (m >> 2) + 4 * (m & 3)));
                    FFT_FENCE();
                    fwd8(x, u);
                    const uint32_t w = R + 16u * (17u * (16u * (ln >> 5) + 8u * ((ln >> 4) & 1u)) + 8u * ((ln >> 3) & 1u) + 4u * ((ln >> 2) & 1u) + (ln & 3u));
                    // for the other component's workgroup (positions b8 .. b0 of the quarter in order), for this wave, and for the late group's
                    d2 *post = mail + ((((tick & 1u) * 2u + h) * 4u + g) * 512u);
                    const uint32_t pl = (ln >> 2) * 32u + (ln & 3u);
#pragma unroll
                    for (int m = 0; m < 8; m++) lane_put(post + 4 * m, pl, x[m]);
#pragma unroll
                    for (int m = 0; m < 8; m++) {
                        const int slot = 16 * 17 * (2 * (m >> 2) + ((m >> 1) & 1) + 4 * (m & 1));
                        lds_put(w + 4 * F12P_BUF + slot, x[m]);
                        lds_put(w + slot, x[m]);
                    }
                }
                fft_signal(spec_done, tick + 1);
                slz_xcd_report(line + 4u * h + g, tick + 1);
            }
            spectra(D);
            run_piece(fft_int<3>(), fft_int<0>(), D, step);
            run_piece(fft_int<4>(), fft_int<1>(), D, step);
            wait_four(freed, lane, peek_four(freed, lane), ex);       // the words below go into all four buffers
            tick++;
            wait_four(sums_done, lane, peek_four(sums_done, lane), tick);     // of all four: the next spectrum goes into the late group's buffers
            const LDS_AS uint64_t *M = (const LDS_AS uint64_t *)(uintptr_t)(R0 + 4u * F12P_BUF) + fresh(lane);
#pragma unroll
            for (int e = 0; e < 8; e++) { accr[e] += M[64 * e]; acci[e] += M[512 + 64 * e]; }
#pragma unroll
            for (int e = 0; e < 8; e++) stage(e);
            fft_signal(my_done, ++ex);
        }

        const uint32_t lo = 64u * g + fresh(lane);
        if (A.acc_out) {
            uint64_t *dst = A.acc_out + ((size_t)c * 2 + h) * 4096u;
#pragma unroll
            for (int e = 0; e < 8; e++) { dst[256u * e + lo] = (uint64_t)0 - accr[e]; dst[2048u + 256u * e + lo] = (uint64_t)0 - acci[e]; }
        }
        if (A.lwe_out) {
            uint64_t *dst = A.lwe_out + (size_t)c * 4097u;
            if (h == 0) {
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const uint32_t idx = 256u * e + lo;
                    if (idx == 0) dst[0] = (uint64_t)0 - accr[0];
                    else dst[4096u - idx] = accr[e];
                    dst[2048u - idx] = acci[e];
                }
            } else if (lo == 0) {
                dst[4096] = (uint64_t)0 - accr[0];
            }
        }
        };
        if (late) work(fft_int<1>());
        else work(fft_int<0>());
    }
}

// ---- host side ------------------------------------------------------------------------------------------------------

int slz_fft4096_pair_setup() {
    SLZ_HIP(hipFuncSetAttribute((const void *)k_fft4096_pair, hipFuncAttributeMaxDynamicSharedMemorySize, F12P_LDS_BYTES));
    return SLZ_OK;
}

int slz_fft4096_pair_launch(slz_ctx *ctx, const uint64_t *lwe_in, const uint64_t *luts, const uint32_t *lut_idx, const void *key,
                            uint32_t n_steps, uint64_t *acc_out, uint64_t *lwe_out, uint32_t batch, uint32_t workgroups, uint32_t patience, hipStream_t s) {
    if (!ctx->pair_ctl || batch > SLZ_PAIR_MAX || workgroups > slz_pairs_most(ctx)) return SLZ_E_INVALID_ARG;
    fft4096p_args A;
    A.lwe_in = lwe_in; A.luts = luts; A.lut_idx = lut_idx; A.key = (const d2 *)key; A.tab = (const d2 *)ctx->fft_tab;
    A.acc_out = acc_out; A.lwe_out = lwe_out;
    A.pairs = slz_pairs{ctx->pair_ctl, patience};
    A.mail = (d2 *)ctx->pair_mail;
    A.n = ctx->prm.n; A.n_steps = n_steps; A.batch = batch; A.beta = ctx->prm.pbs_base_log;
    for (int q = 0; q < 6; q++)
        for (int t = 0; t < 2; t++) A.f1[q][t] = ctx->fft_f1[q][t];
    slz_pairs_clear(ctx, s);
    hipLaunchKernelGGL(k_fft4096_pair, dim3(workgroups), dim3(F12P_THREADS), F12P_LDS_BYTES, s, A);
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

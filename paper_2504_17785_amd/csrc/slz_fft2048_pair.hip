// Blind rotation for N = 2048, k = 1, l = 1, up to 128 ciphertexts: two workgroups of one XCD (slz_xcd.h) on each ciphertext, a component
// each.  Passes, layouts and maps are those of slz_fft2048_team.hip, where the eight waves of one workgroup do both components; key, tables and
// the error bound too (the two rows' products are added in the order own, other).
//
// Four waves (group 0) keep the component's accumulator, transform its digits and post the spectrum for the other workgroup, 16 KiB through
// the XCD's L2 and a word per wave; then both groups read both spectra at their quarter of the points and take the key pieces side by side:
// group 0 pieces 3 and 4, group 1, which has waited meanwhile, pieces 0 to 2.  Group 1's sums go to group 0 through LDS.  The mail has two sides, by the parity of the
// step: what is posted two steps later overwrites it, after the other workgroup's spectrum of the step between, which it posts when all its
// waves are done with the first.
// What bounds it: 15.3 k cycles per step, a chain of 4.9 k from the accumulator to the spectrum (one wave per SIMD), 2 k for the way to
// the other workgroup, and 8.3 k for three pieces, where the exchanges of five pieces keep the LDS busy for two thirds of the time.  Measured, us per step,
// before (one workgroup) / now: 1 ciphertext 9.2 / 6.4, 64: 9.3 / 6.5, 128: 9.3 / 6.6; without the priority of group 1 6.6.  129 and more
// would need a second round.
#include "slz_fft.h"
#include "slz_fft_wave.h"
#include "slz_modarith.h"
#include "slz_fused_common.h"
#include "slz_xcd.h"

#define FP_THREADS 512
#define FP_BUF (272u * 16u)                         // bytes of a wave's buffer for one piece: 256 points, padded
#define FP_SLOT (4u * FP_BUF)                       // bytes of a group's buffers for one piece
#define FP_LATE_OFF (2u * FP_SLOT)                  // buffers of the group with three pieces
#define FP_SPEC_OFF (5u * FP_SLOT)                  // spectrum of this workgroup's component
#define FP_SUM_OFF (6u * FP_SLOT)                   // the late group's sums: [wave][real, imaginary][4][64 lanes]
#define FP_TAB_OFF (FP_SUM_OFF + 16384u)
#define FP_FLAGS_OFF (FP_TAB_OFF + (FFT_F2_LEN + FFT_T_LEN) * 16u)
#define FP_LDS_BYTES (FP_FLAGS_OFF + 128u)          // done and free per wave and group; spectrum written, sums written per wave; two words

struct fft2048p_args {
    const uint64_t *lwe_in;
    const uint64_t *luts;
    const uint32_t *lut_idx;
    const d2 *key;            // [n][FFT_KEY_STEP]
    const d2 *tab;            // FFT_TAB_LEN entries
    uint64_t *acc_out;
    uint64_t *lwe_out;
    slz_pairs pairs;
    d2 *mail;                 // [pair][parity of the step][component][quarter][256]
    uint32_t n, n_steps, batch, beta;
    double f1[15][2];         // lane-uniform twiddles of the first two forward layers: (v, v^2, v^3) of block 0 and of the next four blocks
};

__global__ void __launch_bounds__(FP_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_fft2048_pair(fft2048p_args A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const uint32_t lds = (uint32_t)(uintptr_t)(LDS_AS unsigned char *)lds_raw;
    const uint32_t beta = A.beta;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t late = wave >> 2, g = wave & 3u;                                         // group 0: front and pieces 3 and 4, group 1: pieces 0 to 2
    const uint32_t C0 = lds + late * FP_LATE_OFF, R0 = C0 + g * FP_BUF;                     // the group's buffers; this wave's
    const uint32_t S0 = lds + FP_SPEC_OFF + g * FP_BUF, M0 = lds + FP_SUM_OFF + g * 4096u;
    const uint32_t tab0 = lds + FP_TAB_OFF;                                                 // F2 table, then the T tables
    const uint32_t flags = lds + FP_FLAGS_OFF;
    const uint32_t done = flags + 32u * late, freed = done + 16u, my_done = done + 4u * g, my_free = freed + 4u * g;
    const uint32_t spec_done = flags + 64u + 4u * g, sums_done = flags + 80u + 4u * g, told = flags + 96u;
    for (uint32_t i = threadIdx.x; i < FFT_F2_LEN + FFT_T_LEN; i += FP_THREADS)
        lds_put(tab0 + 16u * i, A.tab[i < FFT_F2_LEN ? FFT_F2_OFF + i : FFT_T_OFF + i - FFT_F2_LEN]);
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
    d2 *mail = A.mail + (size_t)box * 4096u;

    // twiddles of I2, I3 and I4, the same for every piece and step
    d2 v, v2, v3, w30, w31, w40, w41;
    {
        const uint32_t tt = tab0 + FFT_F2_LEN * 16u, t2 = tt + FFT_T2_OFF * 16u + 16u * (lane & 3u), t3 = tt + FFT_T3_OFF * 16u + 16u * (lane & 15u);
        const uint32_t t4 = tt + FFT_T4_OFF * 16u + 16u * lane;
        v = lds_get(t2); v2 = lds_get(t2 + 64); v3 = lds_get(t2 + 128);
        w30 = lds_get(t3); w31 = lds_get(t3 + 256);
        w40 = lds_get(t4); w41 = lds_get(t4 + 1024);
        pin(v); pin(v2); pin(v3); pin(w30); pin(w31); pin(w40); pin(w41);
    }

    const double magic = 6755399441055744.0, r2 = FFT_SQRT_HALF;      // 1.5 * 2^52: adding it rounds to an integer
    uint32_t ex = 0;                                                  // exchanges between the waves of the group so far
    uint32_t tick = 0;                                                // steps so far
    for (uint32_t round = 0;; round++) {
        const uint32_t c = broadcast(threadIdx.x == 0 ? slz_pair_next(A.pairs, box, h, round) : 0u);
        if (c >= A.batch) return;
        const uint64_t *lwe = A.lwe_in + (size_t)c * (A.n + 1);
        uint64_t accr[4], acci[4];                                    // negated coefficients 256 e + 64 g + lane and 1024 more of component h
        const uint32_t li = 64u * g + fresh(lane);
        if (h == 1 && !late) {
            const uint32_t bt = slz_modswitch(lwe[A.n], 12);
            const uint32_t r = (4096u - bt) & 4095u;
            const uint64_t *lut = A.luts + (size_t)(A.lut_idx ? A.lut_idx[c] : 0) * 2048u;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                accr[e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 256u * e + li, r, 2048u);
                acci[e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 1024u + 256u * e + li, r, 2048u);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++) accr[e] = acci[e] = 0;
        }

        // The accumulator is written to its component's buffers whenever it is complete: here and at the end of every step.
        auto stage = [&](int e) {
            LDS_AS uint64_t *S = (LDS_AS uint64_t *)(uintptr_t)C0 + 64u * g;
            S[256 * e + lane] = accr[e];
            S[1024 + 256 * e + lane] = acci[e];
        };
        if (!late) {
#pragma unroll
            for (int e = 0; e < 4; e++) stage(e);
            fft_signal(my_done, ++ex);
        }
        uint64_t mask = lwe[0];
        // key words: [piece][half b9][k' = b2 b1 b0][row, component][lane' = b8..b3]; here the lane is b7..b2, the register b1 b0
        d2 kb[3][4][2];
        const d2 *kp = A.key + ((g >> 1) * 8u * 4u + h) * 64u + (size_t)(late ? 0u : 3u) * (FFT_KEY_STEP / SLZ_FFT_PIECES);     // from the group's first piece on
        // four loads at a time, spread over the passes: more of them together would fill the memory pipeline's queue and hold the wave; the row of
        // this workgroup's component comes first, as its spectrum does
        auto request = [&](int q, int piece, int half) __attribute__((always_inline)) {
            const uint32_t ln = fresh(lane), kl = (ln & 1u) * 4u * 4u * 64u + (g & 1u) * 32u + (ln >> 1);
#pragma unroll
            for (int k = 2 * half; k < 2 * half + 2; k++)
#pragma unroll
                for (int r = 0; r < 2; r++) kb[q][k][r] = lane_get(kp + (size_t)piece * (FFT_KEY_STEP / SLZ_FFT_PIECES) + (4 * k + 2 * (r ^ h)) * 64, kl);
            FFT_FENCE();
        };
#pragma unroll
        for (int q = 0; q < 2; q++) { request(q, q, 0); request(q, q, 1); }
        // F5 and both components' spectra at this wave's quarter of the points
        auto spectra = [&](d2 (&D)[2][4]) __attribute__((always_inline)) {
            int z;
            asm volatile("s_mov_b32 %0, 0" : "=s"(z));
            const uint32_t ln0 = fresh(lane);
            // F5 (registers b1 b0) takes the two components' spectra at this wave's quarter of the points
            const uint32_t from_here = S0 + z + 16u * (17u * ((ln0 >> 4) * 4u + (ln0 & 3u)) + ((ln0 >> 2) & 3u) * 4u);
            const d2 *from_there = mail + ((((tick & 1u) * 2u + (h ^ 1u)) * 4u + g) * 256u);
            d2 f5[3];
            {
                const d2 *t5 = A.tab + FFT_F3_OFF + (g >> 1) * 384u + z;
                const uint32_t l5 = (ln0 & 1u) * 192u + (g & 1u) * 32u + (ln0 >> 1);
#pragma unroll
                for (int t = 0; t < 3; t++) f5[t] = lane_get(t5 + 64 * t, l5);
            }
#pragma unroll
            for (int k = 0; k < 4; k++) D[0][k] = lds_get(from_here + 16 * k);
            slz_xcd_await(line + 4u * (h ^ 1u) + g, tick + 1);
#pragma unroll
            for (int k = 0; k < 4; k++) D[1][k] = lane_get_l2(from_there + k, 4u * ln0);
            FFT_FENCE();
#pragma unroll
            for (int cc = 0; cc < 2; cc++) fwd4(D[cc][0], D[cc][1], D[cc][2], D[cc][3], f5[0], f5[1], f5[2]);
        };
        // the group's key pieces, COUNT of them from FIRST on, side by side
        auto run_pieces = [&](auto first, auto how_many, const d2 (&D)[2][4], uint32_t step) __attribute__((always_inline)) {
            constexpr int FIRST = decltype(first)::value, COUNT = decltype(how_many)::value;
            int z;
            asm volatile("s_mov_b32 %0, 0" : "=s"(z));
            const uint32_t T = C0 + z, R = R0 + z;
            const uint32_t tt = tab0 + z + FFT_F2_LEN * 16u;
            d2 x[COUNT][4];
            FFT_FENCE();
            const uint32_t free_seen = peek_four(freed, lane);
#pragma unroll
            for (int q = 0; q < COUNT; q++)
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const d2 k0 = kb[q][k][0], k1 = kb[q][k][1], a = D[0][k], b = D[1][k];
                    x[q][k].x = __builtin_fma(-b.y, k1.y, __builtin_fma(b.x, k1.x, __builtin_fma(-a.y, k0.y, a.x * k0.x)));
                    x[q][k].y = __builtin_fma(b.y, k1.x, __builtin_fma(b.x, k1.y, __builtin_fma(a.y, k0.x, a.x * k0.y)));
                    pin(x[q][k]);
                }
            FFT_FENCE();
            // the next step's key words (if there is one) arrive during this inverse transform and the front
            const bool more = step + 1 < A.n_steps;
            kp += FFT_KEY_STEP;
            const uint32_t ln = fresh(lane);
            const uint32_t t5 = tt + FFT_T5_OFF * 16u + 16u * (64u * g + ln);
            // base addresses of the layouts: I1 (map Y), I2 in map Y and in map X, I3, I4
            const uint32_t w1 = R + 16u * (17u * ((ln >> 4) * 4u + (ln & 3u)) + ((ln >> 2) & 3u) * 4u);
            const uint32_t r2b = R + 16u * (17u * ((ln >> 4) * 4u) + (ln & 15u));                            // also I4 in map X
            const uint32_t w2 = R + 16u * (17u * (((ln >> 2) & 3u) * 4u + (ln >> 4)) + (ln & 3u));
            const uint32_t r3 = R + 16u * (17u * (ln >> 4) + (ln & 15u));
            // A piece's points are read for the next pass as soon as they are written, and arrive while the other pieces go through this one.
#pragma unroll
            for (int q = 0; q < COUNT; q++) {                     // I1: half-sizes 1, 2; lane = b7..b2; register = b1 b0
                add2(x[q][0], x[q][1]); add2(x[q][2], x[q][3]);
                add2(x[q][0], x[q][2]); add2i(x[q][1], x[q][3]);
                if (FIRST == 0 && q == 0) wait_four(freed, lane, free_seen, ex);  // the waves that read this one's buffers have done so (group 0: before it staged)
#pragma unroll
                for (int k = 0; k < 4; k++) lds_put(w1 + q * FP_SLOT + 16 * k, x[q][k]);
#pragma unroll
                for (int m = 0; m < 4; m++) x[q][m] = lds_get(r2b + q * FP_SLOT + 16 * 17 * m);
                FFT_FENCE();
            }
            if (more) request(0, 0, 0);
#pragma unroll
            for (int q = 0; q < COUNT; q++) {                     // I2: half-sizes 4, 8; lane = b7 b6 b5 b4 b1 b0; register = b3 b2
                inv4(x[q][0], x[q][1], x[q][2], x[q][3], v, v2, v3);
#pragma unroll
                for (int m = 0; m < 4; m++) lds_put(w2 + q * FP_SLOT + 16 * 4 * m, x[q][m]);
#pragma unroll
                for (int m = 0; m < 4; m++) x[q][m] = lds_get(r3 + q * FP_SLOT + 16 * 17 * 4 * m);
                FFT_FENCE();
            }
            if (more) request(0, 0, 1);
#pragma unroll
            for (int q = 0; q < COUNT; q++) {                     // I3: half-sizes 16, 32; lane = b7 b6 b3..b0; register = b5 b4
                inv2<false>(x[q][0], x[q][1], w30); inv2<false>(x[q][2], x[q][3], w30);
                inv2<false>(x[q][0], x[q][2], w31); inv2<true>(x[q][1], x[q][3], w31);
#pragma unroll
                for (int m = 0; m < 4; m++) lds_put(r3 + q * FP_SLOT + 16 * 17 * 4 * m, x[q][m]);
#pragma unroll
                for (int m = 0; m < 4; m++) x[q][m] = lds_get(r2b + q * FP_SLOT + 16 * 17 * m);
                FFT_FENCE();
            }
            if (more) request(1, 1, 0);
#pragma unroll
            for (int q = 0; q < COUNT; q++) {                     // I4: half-sizes 64, 128; lane = b5..b0; register = b7 b6
                inv2<false>(x[q][0], x[q][1], w40); inv2<false>(x[q][2], x[q][3], w40);
                inv2<false>(x[q][0], x[q][2], w41); inv2<true>(x[q][1], x[q][3], w41);
#pragma unroll
                for (int m = 0; m < 4; m++) lds_put(r2b + q * FP_SLOT + 16 * 17 * m, x[q][m]);
            }
            fft_signal(my_done, ++ex);
            if (more) request(1, 1, 1);
            {   // I5: half-sizes 256 and 512 with the twist; lane = b5..b0, wave = b7 b6; register = b9 b8
                const d2 w0 = lds_get(t5);
                d2 c1[2], c2[2];
#pragma unroll
                for (int e = 0; e < 2; e++) { c1[e] = lds_get(t5 + 4096 * (1 + 2 * e)); c2[e] = lds_get(t5 + 4096 * (2 + 2 * e)); }
                FFT_FENCE();
                wait_four(done, lane, peek_four(done, lane), ex);
                const uint32_t r0 = T + 16u * (17u * ((ln >> 4) * 4u + g) + (ln & 15u));
#pragma unroll
                for (int q = 0; q < COUNT; q++)
#pragma unroll
                    for (int e = 0; e < 4; e++) x[q][e] = lds_get(r0 + q * FP_SLOT + e * FP_BUF);
                fft_signal(my_free, ex);
                FFT_FENCE();
                auto finish = [&](auto which, d2 (&y)[4]) __attribute__((always_inline)) {
                    constexpr int piece = decltype(which)::value;
                    inv2<false>(y[0], y[1], w0); inv2<false>(y[2], y[3], w0);
#pragma unroll
                    for (int e = 0; e < 2; e++) {
                        d2 a = cmul(y[e], c1[e]), b = y[e + 2];
                        inv2<false>(a, b, c2[e]);
                        // coefficients 256 e + .. (a) and 512 + 256 e + .. (b turned by -45 degrees), rounded
                        const uint64_t y0 = (uint64_t)__double_as_longlong(a.x + magic), y1 = (uint64_t)__double_as_longlong(a.y + magic);
                        const uint64_t y2 = (uint64_t)__double_as_longlong(__builtin_fma(b.x + b.y, r2, magic));
                        const uint64_t y3 = (uint64_t)__double_as_longlong(__builtin_fma(b.y - b.x, r2, magic));
                        add_shifted<SLZ_FFT_PIECE_BITS * piece>(accr[e], y0);
                        add_shifted<SLZ_FFT_PIECE_BITS * piece>(acci[e], y1);
                        add_shifted<SLZ_FFT_PIECE_BITS * piece>(accr[e + 2], y2);
                        add_shifted<SLZ_FFT_PIECE_BITS * piece>(acci[e + 2], y3);
                        if (piece == 0) {                         // the bits of `magic` that shift 0 has left
                            accr[e] -= 0x4338000000000000ull; acci[e] -= 0x4338000000000000ull;
                            accr[e + 2] -= 0x4338000000000000ull; acci[e + 2] -= 0x4338000000000000ull;
                        }
                    }
                };
                finish(fft_int<FIRST>(), x[0]);
                finish(fft_int<FIRST + 1>(), x[1]);
                if constexpr (COUNT == 3) finish(fft_int<FIRST + 2>(), x[2]);
#pragma unroll
                for (int e = 0; e < 4; e++) { pin(accr[e]); pin(acci[e]); }
            }
        };
        if (late) {
            __builtin_amdgcn_s_setprio(1);                            // it has the longer half: 6.63 -> 6.46 us per step
            for (uint32_t step = 0; step < A.n_steps; step++) {
                d2 D[2][4];
                request(2, 2, 0);                                     // of this step: the others were asked for a step ahead
                request(2, 2, 1);
                fft_wait(spec_done, fft_peek(spec_done), tick + 1);
                spectra(D);
#pragma unroll
                for (int e = 0; e < 4; e++) accr[e] = acci[e] = 0;
                run_pieces(fft_int<0>(), fft_int<3>(), D, step);
                LDS_AS uint64_t *M = (LDS_AS uint64_t *)(uintptr_t)M0 + fresh(lane);
#pragma unroll
                for (int e = 0; e < 4; e++) { M[64 * e] = accr[e]; M[256 + 64 * e] = acci[e]; }
                fft_signal(sums_done, tick + 1);
                tick++;
            }
            continue;
        }
        for (uint32_t step = 0; step < A.n_steps; step++) {
            // an opaque zero in every table and buffer address keeps the loads inside the step
            int z;
            asm volatile("s_mov_b32 %0, 0" : "=s"(z));
            const uint32_t T = C0 + z, R = R0 + z;
            const uint32_t tab = tab0 + z;
            // slots of a wave's buffer by the bits of a point: map X (A = b5 b4 b7 b6, B = b3..b0) and map Y (A = b7 b6 b3 b2, B = b5 b4 b1 b0)
            d2 D[2][4];
            {
                d2 x[4];
                const uint32_t at = slz_modswitch(mask, 12);
                mask = lwe[step + 1];                                 // the next step's word (the body after the last step)
                wait_four(done, lane, peek_four(done, lane), ex);
                // ---- 1. digits ----
                {
                    const uint32_t rnd = 1u << (31 - beta), t0 = 8u * (64u * g + fresh(lane)) + 0x4000u - 8u * at;
                    auto word = [&](uint32_t t) { return *(const LDS_AS uint64_t *)(uintptr_t)(T + (t & 0x3ff8u)); };
                    auto digit = [&](uint32_t t, uint64_t a, uint64_t own) {
                        const uint32_t m = (uint32_t)((int32_t)(t << 17) >> 31);
                        uint32_t lo = (uint32_t)a ^ m, hi = (uint32_t)(a >> 32) ^ m;
                        asm("v_cmp_ne_u32_e32 vcc, 0, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %3, vcc\n\tv_addc_co_u32_e32 %1, vcc, %1, %4, vcc"
                            : "+v"(lo), "+v"(hi) : "v"(m), "v"((uint32_t)own), "v"((uint32_t)(own >> 32)) : "vcc");
                        return (double)((int32_t)(hi + rnd) >> (32 - beta));
                    };
                    uint64_t a[2][4];
#pragma unroll
                    for (int i = 0; i < 4; i++) { a[0][i] = word(t0 + 2048u * i); a[1][i] = word(t0 + 8192u + 2048u * i); }
                    fft_signal(my_free, ex);
#pragma unroll
                    for (int i = 0; i < 4; i++) { x[i].x = digit(t0 + 2048u * i, a[0][i], accr[i]); x[i].y = digit(t0 + 8192u + 2048u * i, a[1][i], acci[i]); }
                }
                // ---- 2. forward transform ----
                const uint32_t free_seen = peek_four(freed, lane);
                auto f1 = [&](int q) { d2 w; w.x = A.f1[q + z][0]; w.y = A.f1[q + z][1]; return w; };
                fwd4(x[0], x[1], x[2], x[3], f1(0), f1(1), f1(2));
                wait_four(freed, lane, free_seen, ex);                // every wave has read its rotated words
                const uint32_t ln = fresh(lane);
                {
                    // b7 b6 are this wave's, b5 b4 / b3..b0 the lane's; register = b9 b8 = buffer
                    const uint32_t w = T + 16u * (17u * ((ln >> 4) * 4u + g) + (ln & 15u));
#pragma unroll
                    for (int e = 0; e < 4; e++) lds_put(w + e * FP_BUF, x[e]);
                }
                fft_signal(my_done, ++ex);
                const uint32_t tf3 = tab + FFT_F2_OFF * 16u + 16u * (4u * g + (ln >> 4));
                const d2 u0 = lds_get(tf3), u1 = lds_get(tf3 + 256), u2 = lds_get(tf3 + 512);
                // F4: block 4 x + q with x = b9 b8 b7 b6 and q = b5 b4
                const uint32_t tf4 = tab + FFT_F2_OFF * 16u + 16u * (16u * (3u + 3u * ((ln >> 2) & 3u)) + 4u * g + (ln >> 4));
                const d2 v0 = lds_get(tf4), v1 = lds_get(tf4 + 256), v2 = lds_get(tf4 + 512);
                FFT_FENCE();
                wait_four(done, lane, peek_four(done, lane), ex);
                {   // F2: lane = b5..b0; register = b7 b6
                    const uint32_t r0 = R + 16u * (17u * ((ln >> 4) * 4u) + (ln & 15u));
#pragma unroll
                    for (int m = 0; m < 4; m++) x[m] = lds_get(r0 + 16 * 17 * m);
                    const int b = 3 + 3 * (int)g;
                    fwd4(x[0], x[1], x[2], x[3], f1(b), f1(b + 1), f1(b + 2));
#pragma unroll
                    for (int m = 0; m < 4; m++) lds_put(r0 + 16 * 17 * m, x[m]);
                }
                {   // F3: lane = b7 b6 b3..b0; register = b5 b4
                    const uint32_t r0 = R + 16u * (17u * (ln >> 4) + (ln & 15u));
#pragma unroll
                    for (int m = 0; m < 4; m++) x[m] = lds_get(r0 + 16 * 17 * 4 * m);
                    fwd4(x[0], x[1], x[2], x[3], u0, u1, u2);
#pragma unroll
                    for (int m = 0; m < 4; m++) lds_put(r0 + 16 * 17 * 4 * m, x[m]);
                }
                {   // F4: lane = b7 b6 b5 b4 b1 b0; register = b3 b2
                    const uint32_t r0 = R + 16u * (17u * (((ln >> 2) & 3u) * 4u + (ln >> 4)) + (ln & 3u));
#pragma unroll
                    for (int m = 0; m < 4; m++) x[m] = lds_get(r0 + 16 * 4 * m);
                    fwd4(x[0], x[1], x[2], x[3], v0, v1, v2);
                    // for the late group, and for the other component's workgroup (positions b7 .. b0 of the quarter in order)
                    const uint32_t w = S0 + z + 16u * (17u * ((ln >> 4) * 4u) + (ln & 15u));
                    d2 *post = mail + ((((tick & 1u) * 2u + h) * 4u + g) * 256u);
                    const uint32_t pl = (ln >> 2) * 16u + (ln & 3u);
#pragma unroll
                    for (int m = 0; m < 4; m++) lane_put(post + 4 * m, pl, x[m]);
#pragma unroll
                    for (int m = 0; m < 4; m++) lds_put(w + 16 * 17 * m, x[m]);
                }
                fft_signal(spec_done, tick + 1);
                slz_xcd_report(line + 4u * h + g, tick + 1);
            }
            spectra(D);
            run_pieces(fft_int<3>(), fft_int<2>(), D, step);
            wait_four(freed, lane, peek_four(freed, lane), ex);   // the words below go into all four buffers
            fft_wait(sums_done, fft_peek(sums_done), tick + 1);
            const LDS_AS uint64_t *M = (const LDS_AS uint64_t *)(uintptr_t)M0 + fresh(lane);
#pragma unroll
            for (int e = 0; e < 4; e++) { accr[e] += M[64 * e]; acci[e] += M[256 + 64 * e]; }
#pragma unroll
            for (int e = 0; e < 4; e++) stage(e);
            fft_signal(my_done, ++ex);
            tick++;
        }

        const uint32_t lo = 64u * g + fresh(lane);
        if (A.acc_out) {
            uint64_t *dst = A.acc_out + ((size_t)c * 2 + h) * 2048u;
#pragma unroll
            for (int e = 0; e < 4; e++) { dst[256u * e + lo] = (uint64_t)0 - accr[e]; dst[1024u + 256u * e + lo] = (uint64_t)0 - acci[e]; }
        }
        if (A.lwe_out) {
            uint64_t *dst = A.lwe_out + (size_t)c * 2049u;
            if (h == 0) {
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const uint32_t idx = 256u * e + lo;
                    if (idx == 0) dst[0] = (uint64_t)0 - accr[0];
                    else dst[2048u - idx] = accr[e];
                    dst[1024u - idx] = acci[e];
                }
            } else if (lo == 0) {
                dst[2048] = (uint64_t)0 - accr[0];
            }
        }
    }
}

// ---- host side ------------------------------------------------------------------------------------------------------

int slz_fft2048_pair_setup() {
    SLZ_HIP(hipFuncSetAttribute((const void *)k_fft2048_pair, hipFuncAttributeMaxDynamicSharedMemorySize, FP_LDS_BYTES));
    return SLZ_OK;
}

int slz_fft2048_pair(slz_ctx *ctx, const uint64_t *lwe_in, const uint64_t *luts, const uint32_t *lut_idx, const void *key,
                     uint32_t n_steps, uint64_t *acc_out, uint64_t *lwe_out, uint32_t batch, uint32_t workgroups, uint32_t patience, hipStream_t s) {
    if (!ctx->pair_ctl || batch > SLZ_PAIR_MAX || workgroups > slz_pairs_most(ctx)) return SLZ_E_INVALID_ARG;
    fft2048p_args A;
    A.lwe_in = lwe_in; A.luts = luts; A.lut_idx = lut_idx; A.key = (const d2 *)key; A.tab = (const d2 *)ctx->fft_tab;
    A.acc_out = acc_out; A.lwe_out = lwe_out;
    A.pairs = slz_pairs{ctx->pair_ctl, patience};
    A.mail = (d2 *)ctx->pair_mail;
    A.n = ctx->prm.n; A.n_steps = n_steps; A.batch = batch; A.beta = ctx->prm.pbs_base_log;
    for (int q = 0; q < 15; q++)
        for (int t = 0; t < 2; t++) A.f1[q][t] = ctx->fft_f1[q][t];
    slz_pairs_clear(ctx, s);
    hipLaunchKernelGGL(k_fft2048_pair, dim3(workgroups), dim3(FP_THREADS), FP_LDS_BYTES, s, A);
    SLZ_HIP(hipGetLastError());
    return slz_fft2048_team(ctx, lwe_in, luts, lut_idx, key, n_steps, acc_out, lwe_out, batch, s, ctx->pair_ctl);
}

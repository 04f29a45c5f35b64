// Blind rotation for N = 4096, k = 1, l = 1 (5-bit messages) through exact double-precision transforms (slz_fft.h).
//
// One workgroup of eight waves owns a ciphertext for the whole rotation (up to 128 ciphertexts: two, slz_fft4096_pair.hip).  Four waves share each component: wave (h, g) keeps a quarter
// of component h of the accumulator in registers (eight points, i.e. sixteen words, per lane) and transforms it together with the
// other three; between the transforms it holds the spectra of both components at quarter g of the 2048 points and makes the products
// for output component h, so that products need no exchange.  Per CMux step:
//   1. the accumulator goes through LDS to be rotated; subtract, round, one signed digit per coefficient; digits c and c + 2048 are the
//      real and imaginary part of one of 2048 points
//   2. forward transform: a radix-2 layer with the constant 45-degree twiddle (on integers), radix 4, two radix-8 layers, radix 4
//   3. for each of the five key pieces: products and their sum over the two rows, inverse transform (decimation in time; half-sizes 1, 2,
//      4 with constant twiddles, 8 and 16 as radix 4, 32, 64 and 128 as radix 4, 256, 512, 1024 with the twist), rounding to integers,
//      shifted add into the accumulator.
// Radix 4 and 8 instead of pairs of radix-2 butterflies cost a few instructions (28 against 24, 80 against 72) and round less: with
// them five pieces of 13 bits are proven (slz_fft_error_bound), with radix 2 alone it would take six of 11.
// Positions: p = 0 .. 2047 with bits b10 .. b0; before the forward and after the inverse transform p is the coefficient, in between the
// bit-reversed evaluation point.  Layouts (registers / lane bits from the top / wave):
//   F1, I4: b10 b9 b8 / b5..b0 / b7 b6     F2: b7 b6 b5 / b8 b4 b3 b2 b1 b0 / b10 b9     F3: b4 b3 b2 / b8 b7 b6 b5 b1 b0 / b10 b9
//   F4, I1: b2 b1 b0 / b8..b3 / b10 b9     I2: b5 b4 b3 / b8 b7 b6 b2 b1 b0 / b10 b9     I3: b8 b7 b6 / b5..b0 / b10 b9
// so that only F1 -> F2, F3 -> F4 (across the components) and I3 -> I4 cross waves.  A wave's buffer holds the 512 points with the same
// b10 b9; an exchange places a point at 17 * A + B (16-byte slots) with five bits in A and four in B, by which 16 neighbouring
// lanes touch 16 different columns when writing and when reading (the counter still shows conflicts, see below), and every register is one lane
// base plus an immediate:
//   F1 -> F2, F2 -> F3: A = b8 b6 b5 b4 b7, B = b3 b2 b1 b0     F3 -> F4: A = b8 b7 b2 b4 b3, B = b6 b5 b1 b0
//   I1 -> I2: A = b8 b7 b5 b4 b3, B = b6 b2 b1 b0               I2 -> I3: A = b8 b6 b7 b5 b4, B = b3 b2 b1 b0
//   I3 -> I4: A = b8 b7 b6 b5 b4, B = b3 b2 b1 b0
// What bounds it: 3 096 vector instructions per wave and step, 27.5 k cycles of a SIMD's two waves, and 18 exchanges per step, which keep the
// LDS busy for 23 k cycles, 4.9 k of them counted as bank conflicts (of which accesses is not known); of 39.6 k cycles per step (100 and 256
// ciphertexts alike) 70 % issue vector instructions, the rest is what the two waves of a SIMD do not hide of each other's exchanges.  With a full
// chip the clock falls from 2.35 to 2.0 GHz.  One ciphertext per compute unit: the exchange
// buffers and tables of two would not fit LDS, and eight waves on one ciphertext also give the lower latency.  Of the two waves on a SIMD
// the one behind gets the priority (20.2 us per step at 100 ciphertexts without, 18.8 with); key words are requested one piece ahead, four
// loads at a time (18.8, 17.7); the twiddles of I2 stay in registers (1024 ciphertexts: 68.6, 67.6).  Measured, us per step (in brackets: two
// residues): 1 ciphertext 16.8 (26.7), 100: 17.6 (27.4), 256: 19.9 (29.7), 1024: 68 to 70 (115); a lookup of 100 with 800 steps 13.3 ms (21.2).
#include "slz_fft.h"
#include "slz_fft_wave.h"
#include "slz_modarith.h"
#include "slz_fused_common.h"
#include "slz_xcd.h"

#define F12_THREADS 512
#define F12_BUF (544u * 16u)                        // bytes of a wave's buffer: 512 points, padded
#define F12_FLAGS_OFF (8u * F12_BUF + F12_LDS_TAB * 16u)
#define F12_LDS_BYTES (F12_FLAGS_OFF + 64u)         // done and free per wave

struct fft4096_args {
    const uint64_t *lwe_in;
    const uint64_t *luts;
    const uint32_t *lut_idx;
    const d2 *key;            // [n][F12_KEY_STEP]
    const d2 *tab;            // F12_TAB_LEN entries
    uint64_t *acc_out;
    uint64_t *lwe_out;
    const uint32_t *taken;    // where it is given: ciphertexts that a launch before this one has done (slz_xcd.h)
    uint32_t n, n_steps, batch, beta;
    double f1[6][2];          // lane-uniform twiddles of the second forward layer: (v, v^2, v^3) of its two blocks
};

__global__ void __launch_bounds__(F12_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_fft4096_blind_rotate(fft4096_args A) {
    if (A.taken && blockIdx.x < *A.taken) return;                     // one workgroup per ciphertext
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const uint32_t lds = (uint32_t)(uintptr_t)(LDS_AS unsigned char *)lds_raw;
    const uint32_t beta = A.beta;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t h = wave >> 2, g = wave & 3u;
    const uint32_t C0 = lds + h * 4u * F12_BUF, R0 = lds + wave * F12_BUF;                  // buffers of component h; this wave's
    const uint32_t tab0 = lds + 8u * F12_BUF;
    const uint32_t flags = lds + F12_FLAGS_OFF;
    const uint32_t done = flags + 16u * h, freed = done + 32u, my_done = flags + 4u * wave, my_free = my_done + 32u;
    const uint32_t his_done = flags + 4u * (wave ^ 4u), his_free = his_done + 32u;          // the wave at the same quarter of the other component
    for (uint32_t i = threadIdx.x; i < F12_LDS_TAB; i += F12_THREADS) lds_put(tab0 + 16u * i, A.tab[i]);
    if (threadIdx.x < 16) *(LDS_AS uint32_t *)(uintptr_t)(flags + 4u * threadIdx.x) = 0;
    __syncthreads();

    // twiddles of I2, the same for every piece and step
    d2 i2v, i2v2, i2v3, i2w0, i2w1;
    {
        const uint32_t t2 = tab0 + F12_I2_OFF * 16u + 16u * (lane & 7u);
        i2v = lds_get(t2); i2v2 = lds_get(t2 + 128); i2v3 = lds_get(t2 + 256); i2w0 = lds_get(t2 + 384); i2w1 = lds_get(t2 + 512);
        pin(i2v); pin(i2v2); pin(i2v3); pin(i2w0); pin(i2w1);
    }

    const double magic = 6755399441055744.0, r2 = FFT_SQRT_HALF;      // 1.5 * 2^52: adding it rounds to an integer
    uint32_t ex = 0;                                                  // exchanges between waves so far
    for (uint32_t c = blockIdx.x; c < A.batch; c += gridDim.x) {
        const uint64_t *lwe = A.lwe_in + (size_t)c * (A.n + 1);
        uint64_t accr[8], acci[8];                                    // negated coefficients 256 e + 64 g + lane and 2048 more of component h
        const uint32_t li = 64u * g + fresh(lane);
        if (h == 1) {
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
#pragma unroll
        for (int e = 0; e < 8; e++) stage(e);
        fft_signal(my_done, ++ex);
        uint64_t mask = lwe[0];
        d2 kb[8][2];                                                  // key words of the next piece
        const d2 *kp = A.key + (g * 8u * 4u + h) * 64u;               // [piece][quarter][k][row, component][lane]
        // four loads at a time, spread over the passes: more of them together would fill the memory pipeline's queue and hold the wave
        auto request = [&](int part) __attribute__((always_inline)) {
            const uint32_t kl = fresh(lane);
#pragma unroll
            for (int k = 2 * part; k < 2 * part + 2; k++)
#pragma unroll
                for (int r = 0; r < 2; r++) kb[k][r] = lane_get(kp + (4 * k + 2 * r) * 64, kl);
            if (part == 3) kp += F12_KEY_STEP / SLZ_FFT_PIECES;        // pieces and steps follow each other at the same distance
            FFT_FENCE();
        };
        if (A.n_steps)
#pragma unroll
            for (int part = 0; part < 4; part++) request(part);
        for (uint32_t step = 0; step < A.n_steps; step++) {
            // The SIMD serves its older wave first, here that of component 0, which would run ahead through the pieces and then wait for the
            // other's spectra while that one runs alone: of the two waves on a SIMD the one that is behind gets the priority.
            auto pace = [&]() {
                if ((int32_t)(ex - (uint32_t)__builtin_amdgcn_readfirstlane(fft_peek(his_done))) > 0) __builtin_amdgcn_s_setprio(0);
                else __builtin_amdgcn_s_setprio(2);
            };
            // an opaque zero in every table and buffer address keeps the loads inside the step
            int z;
            asm volatile("s_mov_b32 %0, 0" : "=s"(z));
            uint32_t T = C0 + z, R = R0 + z;
            const uint32_t tab = tab0 + z;
            d2 x[8];
            d2 D[2][8];
            {
                const uint32_t at = slz_modswitch(mask, 13);
                mask = lwe[step + 1];                                 // the next step's word (the body after the last step)
                pace();
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
                    for (int e = 0; e < 8; e++) lds_put(w + (e >> 1) * F12_BUF + 16 * 17 * 16 * (e & 1), x[e]);
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
#pragma unroll
                    for (int m = 0; m < 8; m++) lds_put(w + 16 * 17 * (2 * (m >> 2) + ((m >> 1) & 1) + 4 * (m & 1)), x[m]);
                }
                fft_signal(my_done, ++ex);
                {
                    const uint32_t ln = fresh(lane);
                    d2 f4[6];
                    const d2 *t4 = A.tab + F12_F4_OFF + g * 384u + z;
#pragma unroll
                    for (int q = 0; q < 6; q++) f4[q] = lane_get(t4 + 64 * q, ln);
                    FFT_FENCE();
                    fft_wait(his_done, fft_peek(his_done), ex);
                    // lane = b8..b3; register = b2 b1 b0
                    const uint32_t r0 = lds + z + g * F12_BUF + 16u * (17u * (16u * (ln >> 5) + 8u * ((ln >> 4) & 1u) + 2u * ((ln >> 1) & 1u) + (ln & 1u)) +
                                                                      8u * ((ln >> 3) & 1u) + 4u * ((ln >> 2) & 1u));
#pragma unroll
                    for (int cc = 0; cc < 2; cc++)
#pragma unroll
                        for (int k = 0; k < 8; k++) D[cc][k] = lds_get(r0 + cc * 4 * F12_BUF + 16 * (17 * 4 * (k >> 2) + (k & 3)));
                    fft_signal(my_free, ex);
#pragma unroll
                    for (int cc = 0; cc < 2; cc++)
#pragma unroll
                        for (int b = 0; b < 2; b++) fwd4(D[cc][4 * b], D[cc][4 * b + 1], D[cc][4 * b + 2], D[cc][4 * b + 3], f4[3 * b], f4[3 * b + 1], f4[3 * b + 2]);
                }
            }
            // ---- 3. key pieces ----
            auto run_piece = [&](auto which) __attribute__((always_inline)) {
                constexpr int piece = decltype(which)::value;
                asm volatile("s_mov_b32 %0, 0" : "=s"(z));
                T = C0 + z;
                R = R0 + z;
                const uint32_t tb = tab0 + z;
                d2 S[8];
                pace();
                FFT_FENCE();
                const uint32_t free_seen = piece ? peek_four(freed, lane) : fft_peek(his_free);
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const d2 k0 = kb[k][0], k1 = kb[k][1], a = D[0][k], b = D[1][k];
                    S[k].x = __builtin_fma(-b.y, k1.y, __builtin_fma(b.x, k1.x, __builtin_fma(-a.y, k0.y, a.x * k0.x)));
                    S[k].y = __builtin_fma(b.y, k1.x, __builtin_fma(b.x, k1.y, __builtin_fma(a.y, k0.x, a.x * k0.y)));
                    pin(S[k]);
                }
                FFT_FENCE();
                // the next piece's key words (the next step's after the last piece, if there is one) arrive during this inverse transform
                const bool more = piece < SLZ_FFT_PIECES - 1 || step + 1 < A.n_steps;
                if (more) request(0);
                inv8(S);                                              // I1: half-sizes 1, 2, 4
                if (piece) wait_four(freed, lane, free_seen, ex);     // the waves that read this one's buffer have done so
                else fft_wait(his_free, free_seen, ex);
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
                    for (int e = 0; e < 8; e++) x[e] = lds_get(r0 + (e >> 1) * F12_BUF + 16 * 17 * 16 * (e & 1));
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
            run_piece(fft_int<0>());
            run_piece(fft_int<1>());
            run_piece(fft_int<2>());
            run_piece(fft_int<3>());
            run_piece(fft_int<4>());
            wait_four(freed, lane, peek_four(freed, lane), ex);       // the words below go into all four buffers
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
    }
}

// ---- host side ------------------------------------------------------------------------------------------------------

int slz_fft4096_supported(const slz_params *p) {
    return p->N == 4096 && p->k == 1 && p->pbs_level == 1 && p->pbs_base_log <= 30 && slz_fft_error_bound(4096, 2, p->pbs_base_log) < 0.499;
}

int slz_fft4096_setup() {
    SLZ_HIP(hipFuncSetAttribute((const void *)k_fft4096_blind_rotate, hipFuncAttributeMaxDynamicSharedMemorySize, F12_LDS_BYTES));
    return slz_fft4096_pair_setup();
}

static int all_of_them(slz_ctx *ctx, const uint64_t *lwe_in, const uint64_t *luts, const uint32_t *lut_idx, const void *key,
                       uint32_t n_steps, uint64_t *acc_out, uint64_t *lwe_out, uint32_t batch, hipStream_t s, const uint32_t *taken) {
    fft4096_args A;
    A.lwe_in = lwe_in; A.luts = luts; A.lut_idx = lut_idx; A.key = (const d2 *)key; A.tab = (const d2 *)ctx->fft_tab;
    A.acc_out = acc_out; A.lwe_out = lwe_out; A.taken = taken;
    A.n = ctx->prm.n; A.n_steps = n_steps; A.batch = batch; A.beta = ctx->prm.pbs_base_log;
    for (int q = 0; q < 6; q++)
        for (int t = 0; t < 2; t++) A.f1[q][t] = ctx->fft_f1[q][t];
    hipLaunchKernelGGL(k_fft4096_blind_rotate, dim3(slz_fused_grid(batch, 1)), dim3(F12_THREADS), F12_LDS_BYTES, s, A);
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

// Steps from which on two workgroups take each of `batch` ciphertexts.  What pairs cost beside the steps they have to win back: us with one workgroup / two, the
// launches around them included: 4 steps 73 / 70 at 1 ciphertext, 76 / 81 at 64; 8 steps 144 / 138 at 64, 144 / 152 at 100; 32 steps 538 / 508 at 80,
// 538 / 533 at 100, 537 / 553 at 128; 48 steps 802 / 810 at 120, 64 steps 1065 / 1048.
uint32_t slz_fft4096_pair_steps(uint32_t batch) { return batch <= 64 ? 8 : batch <= 100 ? 32 : 64; }

int slz_fft4096_blind_rotate(slz_ctx *ctx, const uint64_t *lwe_in, const uint64_t *luts, const uint32_t *lut_idx, const void *key,
                             uint32_t n_steps, uint64_t *acc_out, uint64_t *lwe_out, uint32_t batch, hipStream_t s) {
    // up to 128 ciphertexts two workgroups on each: 14.5 to 15.1 us per step against 16.4 to 16.6 (slz_fft2048.hip: when not)
    if (slz_pairs_acquire(ctx, n_steps >= slz_fft4096_pair_steps(batch) && slz_pairs_fit(batch, s), s))
        return slz_pairs_release(ctx, slz_fft4096_pair(ctx, lwe_in, luts, lut_idx, key, n_steps, acc_out, lwe_out, batch, slz_pairs_grid(batch), SLZ_PAIR_PATIENCE, s), s);
    return all_of_them(ctx, lwe_in, luts, lut_idx, key, n_steps, acc_out, lwe_out, batch, s, nullptr);
}

int slz_fft4096_pair(slz_ctx *ctx, const uint64_t *lwe_in, const uint64_t *luts, const uint32_t *lut_idx, const void *key,
                     uint32_t n_steps, uint64_t *acc_out, uint64_t *lwe_out, uint32_t batch, uint32_t workgroups, uint32_t patience, hipStream_t s) {
    const int rc = slz_fft4096_pair_launch(ctx, lwe_in, luts, lut_idx, key, n_steps, acc_out, lwe_out, batch, workgroups, patience, s);
    return rc == SLZ_OK ? all_of_them(ctx, lwe_in, luts, lut_idx, key, n_steps, acc_out, lwe_out, batch, s, ctx->pair_ctl) : rc;
}

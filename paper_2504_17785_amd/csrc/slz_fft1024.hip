// Blind rotation for N = 1024, k = 1, l = 1 through exact double-precision transforms (slz_fft.h).
//
// A wavefront transforms both components of a ciphertext, 8 of the 512 points of each per lane, so every exchange stays inside the
// wave and the products with the key need none.  Per CMux step:
//   front    the accumulator (negated, in registers) goes through LDS to be rotated; subtract, round, one signed digit per coefficient;
//            forward transform (merged twiddles, nine radix-2 layers)
//   pieces   for each of the five key pieces: products and their sum over the two rows, inverse transform (decimation in time, nine
//            radix-2 stages), rounding to integers, shifted add into the accumulator.
// Positions p = b8 .. b0.  Layouts (registers / lane bits from the top):
//   F1, I3: b8 b7 b6 / b5..b0     F2, I2: b5 b4 b3 / b8 b7 b6 b2 b1 b0     F3, I1: b2 b1 b0 / b8..b3
// Exchanges between the first two layouts place a point at 72 (b8 b7 b6) + (b5..b0), between the last two at 72 (b8 b7 b6) +
// 9 (b5 b4 b3) + (b2 b1 b0): 16 neighbouring lanes always touch 16 different columns of 16 bytes, writing and reading.
// Bound and shape: FP64 issue.  A step is about 4.2 k VALU instructions per ciphertext; registers (accumulator 64, spectra 64, transform 64,
// key words 64 of 256) allow two waves per SIMD.  The two components of a wave hide each other's LDS round trips.  Smaller batches
// leave compute units with fewer than eight ciphertexts, so waves share one (SHARE below).  Measured with 630 steps and the
// keyswitch (in brackets: two 50-bit residues on the same card): one ciphertext 3.7 ms (4.6), 512: 5.6 (7.0), 777: 7.8 (13.1),
// 2048: 15.4 (24.4), 8192: 60.3 (102).
#include "slz_fft.h"
#include "slz_fft_wave.h"
#include "slz_modarith.h"
#include "slz_fused_common.h"

#define F10_WAVES 8
#define F10_THREADS (64 * F10_WAVES)
#define F10_BUF (576u * 16u)                        // bytes of one component's exchange buffer: 512 points, padded
#define F10_WBUF (2u * F10_BUF)
#define F10_FLAGS_OFF (F10_WAVES * F10_WBUF + F10_LDS_TAB * 16u)
#define F10_FLAGS 32u
#define F10_LDS_BYTES (F10_FLAGS_OFF + 4u * F10_FLAGS)
#define F10_RING 4                                  // positions of the key (four words each) in registers at a time during the products
#define F10_EARLY 4                                 // positions requested by the end of the previous piece

struct fft1024_args {
    const uint64_t *lwe_in;
    const uint64_t *luts;
    const uint32_t *lut_idx;
    const d2 *key;            // [n][F10_KEY_STEP]
    const d2 *tab;            // F10_TAB_LEN entries
    uint64_t *acc_out;
    uint64_t *lwe_out;
    uint32_t n, n_steps, batch, beta;
    double f1[4][2];          // lane-uniform twiddles of the first three forward layers
};

// SHARE: waves per ciphertext.
//   1  a wave does everything
//   2  the first wave runs the front and two pieces, the second one three pieces
//   4  the first wave runs the front and a piece, the others one, one and two pieces
//   8  (one ciphertext per workgroup) the first two waves run the front of one component each, the next five one piece each
// Waves that share a ciphertext read the spectra, three layers before their end, from the front's exchange buffers; sums return
// through the buffers of the wave that made them.
template <int BETA, int SHARE>
__global__ void __launch_bounds__(F10_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_fft1024_blind_rotate(fft1024_args A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const uint32_t lds = (uint32_t)(uintptr_t)(LDS_AS unsigned char *)lds_raw;
    const uint32_t beta = BETA > 0 ? (uint32_t)BETA : A.beta;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr uint32_t GROUPS = F10_WAVES / SHARE;
    // wave w sits on SIMD w mod 4: with SHARE = 2 a front and its helper have a SIMD to themselves (measured up to 5 % faster than the
    // next ciphertext's helper there), with SHARE = 4 a ciphertext has two
    const uint32_t group = SHARE == 1 ? wave : SHARE == 2 ? (wave & 3u) : SHARE == 4 ? wave & 1u : 0u;
    const uint32_t T0 = lds + wave * F10_WBUF;                        // this wave's two buffers
    const uint32_t O0 = SHARE == 1 ? T0 : lds + group * F10_WBUF;   // the front's
    const uint32_t component_stride = SHARE == 8 ? F10_WBUF : F10_BUF;                   // between the components of the spectra there
    const uint32_t tab0 = lds + F10_WAVES * F10_WBUF;
    const uint32_t flags = lds + F10_FLAGS_OFF;
    // counters, in steps: spectra written (per front wave), spectra read and sums written (per wave), progress (per wave)
    const uint32_t spectra_done = flags + 4u * (SHARE == 8 ? 0u : group), spectra_read = flags + 32u, sums_done = flags + 64u,
                   progress = flags + 96u;
    for (uint32_t i = threadIdx.x; i < F10_LDS_TAB; i += F10_THREADS) lds_put(tab0 + 16u * i, A.tab[i]);
    if (threadIdx.x < F10_FLAGS) *(LDS_AS uint32_t *)(uintptr_t)(flags + 4u * threadIdx.x) = 0;
    __syncthreads();
    constexpr uint32_t HELPERS = SHARE == 8 ? 5 : SHARE - 1;
    auto helper = [&](uint32_t q) { return SHARE == 8 ? 2u + q : SHARE == 4 ? group + 2u * (q + 1u) : group + 4u; };

    const double magic = 6755399441055744.0;                          // 1.5 * 2^52: adding it rounds to an integer
    uint32_t tick = 0;                                                // steps so far
    // One loop per kind of wave.  FIRST .. LAST: pieces of this wave; COMPS: components of the accumulator that it owns (2, 1 or 0)
    auto rotate = [&](auto first_piece, auto last_piece, auto comps) __attribute__((always_inline)) {
        constexpr int FIRST = decltype(first_piece)::value, LAST = decltype(last_piece)::value, COMPS = decltype(comps)::value;
        constexpr bool front = COMPS > 0, alone = SHARE == 1;
        constexpr int NA = COMPS == 1 ? 1 : 2;                        // components held (a helper's are its sums)
        for (uint32_t c = blockIdx.x + group * gridDim.x; c < A.batch; c += GROUPS * gridDim.x) {
            const uint64_t *lwe = A.lwe_in + (size_t)c * (A.n + 1);
            uint64_t accr[NA][8], acci[NA][8];                        // negated coefficients 64 e + lane and 512 + 64 e + lane
            const uint32_t li = fresh(lane);
#pragma unroll
            for (int cc = 0; cc < NA; cc++) {
                if (front && (COMPS == 2 ? cc == 1 : wave == 1)) {
                    const uint32_t bt = slz_modswitch(lwe[A.n], 11);
                    const uint32_t r = (2048u - bt) & 2047u;
                    const uint64_t *lut = A.luts + (size_t)(A.lut_idx ? A.lut_idx[c] : 0) * 1024u;
#pragma unroll
                    for (int e = 0; e < 8; e++) {
                        accr[cc][e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 64u * e + li, r, 1024u);
                        acci[cc][e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 512u + 64u * e + li, r, 1024u);
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 8; e++) accr[cc][e] = acci[cc][e] = 0;
                }
            }
            // The accumulator is written to its buffer whenever it is complete: here and at the end of every step.  A helper's sums too.
            auto stage = [&](int cc, int e) {
                LDS_AS uint64_t *S = (LDS_AS uint64_t *)(uintptr_t)(T0 + cc * F10_BUF);
                S[64 * e + lane] = accr[cc][e];
                S[512 + 64 * e + lane] = acci[cc][e];
            };
            auto stage_all = [&]() {
#pragma unroll
                for (int cc = 0; cc < NA; cc++)
#pragma unroll
                    for (int e = 0; e < 8; e++) stage(cc, e);
            };
            if constexpr (front) stage_all();
            uint64_t mask = front ? lwe[0] : 0;
            for (uint32_t step = 0; step < A.n_steps; step++) {
                // an opaque zero in every table and buffer address keeps the loads inside the step
                int z;
                asm volatile("s_mov_b32 %0, 0" : "=s"(z));
                tick++;
                if (alone) {
                    // of the two waves on a SIMD the one that is behind gets the priority (the SIMD by itself serves the older one)
                    if ((int32_t)(tick - (uint32_t)__builtin_amdgcn_readfirstlane(fft_peek(progress + 4u * (wave ^ 4u)))) > 0) __builtin_amdgcn_s_setprio(0);
                    else __builtin_amdgcn_s_setprio(2);
                    fft_signal(progress + 4u * wave, tick);
                }
                // the helper, younger on its SIMD than the front, has three pieces to the front's two: 630 steps of 513 ciphertexts 7.4 ms with,
                // 8.5 without, 777: 7.7 and 8.5, 1024: 8.3 and 8.6 (SHARE = 4, where the front's chain is the longer one: 400 ciphertexts 10.1 with, 9.6 without)
                if (SHARE == 2 && !front) __builtin_amdgcn_s_setprio(2);
                const d2 *kp = A.key + (size_t)step * F10_KEY_STEP + FIRST * 2048u + z;
                d2 kb[8][4];
                const uint32_t kl = fresh(lane);
                auto request = [&](int k) {
#pragma unroll
                    for (int q = 0; q < 4; q++) kb[k][q] = lane_get(kp + (4 * k + q) * 64, kl);
                };
                if constexpr (front) {
                    uint32_t T = T0 + z;
                    d2 x[NA][8];
                    const uint32_t at = slz_modswitch(mask, 11);
                    mask = lwe[step + 1];                             // the next step's word (the body after the last step)
                    // ---- digits ----
                    {
                        // word (idx - at) mod 2048 of X^at ACC: ten bits of address, the eleventh is the sign; its opposite (bit 13 of t)
                        // tells where the stored, negated word has to be negated again
                        const uint32_t rnd = 1u << (31 - beta), t0 = 8u * fresh(lane) + 0x2000u - 8u * at;
                        auto word = [&](int cc, uint32_t t) { return *(const LDS_AS uint64_t *)(uintptr_t)(T + cc * F10_BUF + (t & 0x1ff8u)); };
                        auto digit = [&](uint32_t t, uint64_t a, uint64_t own) {
                            const uint32_t m = (uint32_t)((int32_t)(t << 18) >> 31);
                            uint32_t lo = (uint32_t)a ^ m, hi = (uint32_t)(a >> 32) ^ m;
                            asm("v_cmp_ne_u32_e32 vcc, 0, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %3, vcc\n\tv_addc_co_u32_e32 %1, vcc, %1, %4, vcc"
                                : "+v"(lo), "+v"(hi) : "v"(m), "v"((uint32_t)own), "v"((uint32_t)(own >> 32)) : "vcc");
                            return (double)((int32_t)(hi + rnd) >> (32 - beta));
                        };
                        // eight words are in flight while the previous eight become digits
                        uint64_t a[2][8];
#pragma unroll
                        for (int i = 0; i < 8; i++) a[0][i] = word(0, t0 + 512u * i);
#pragma unroll
                        for (int g = 0; g < 2 * NA; g++) {            // real, imaginary parts of the first component, of the second
                            FFT_FENCE();
                            if (g + 1 < 2 * NA) {
#pragma unroll
                                for (int i = 0; i < 8; i++) a[(g + 1) & 1][i] = word((g + 1) >> 1, t0 + 4096u * ((g + 1) & 1) + 512u * i);
                            }
                            FFT_FENCE();
#pragma unroll
                            for (int i = 0; i < 8; i++) {
                                const uint32_t t = t0 + 4096u * (g & 1) + 512u * i;
                                if ((g & 1) == 0) x[g >> 1][i].x = digit(t, a[g & 1][i], accr[g >> 1][i]);
                                else x[g >> 1][i].y = digit(t, a[g & 1][i], acci[g >> 1][i]);
                            }
                        }
                    }
                    // ---- forward transform: layers 1..6 ----
                    auto f1 = [&](int q) { d2 w; w.x = A.f1[q + z][0]; w.y = A.f1[q + z][1]; return w; };
                    const uint32_t ln = fresh(lane);
                    const uint32_t aL = T + 16u * ln, aT = T + 1152u * (ln >> 3) + 16u * (ln & 7u);
                    d2 v[4];
#pragma unroll
                    for (int t = 0; t < 4; t++) v[t] = lds_get(tab0 + z + F10_F2_OFF * 16u + 16u * (ln >> 3) + 128u * t);
#pragma unroll
                    for (int cc = 0; cc < NA; cc++) {
                        d2 *y = x[cc];
#pragma unroll
                        for (int e = 0; e < 4; e++) inv2<false>(y[e], y[e + 4], f1(0));
#pragma unroll
                        for (int e = 0; e < 2; e++) { inv2<false>(y[e], y[e + 2], f1(1)); fwd2i(y[e + 4], y[e + 6], f1(1)); }
                        inv2<false>(y[0], y[1], f1(2)); fwd2i(y[2], y[3], f1(2)); inv2<false>(y[4], y[5], f1(3)); fwd2i(y[6], y[7], f1(3));
                        FFT_FENCE();
#pragma unroll
                        for (int e = 0; e < 8; e++) lds_put(aL + cc * F10_BUF + 16 * 72 * e, y[e]);
#pragma unroll
                        for (int m = 0; m < 8; m++) y[m] = lds_get(aT + cc * F10_BUF + 16 * 8 * m);
                    }
#pragma unroll
                    for (int cc = 0; cc < NA; cc++) {
                        FFT_FENCE();
                        d2 *y = x[cc];
#pragma unroll
                        for (int e = 0; e < 4; e++) inv2<false>(y[e], y[e + 4], v[0]);
#pragma unroll
                        for (int e = 0; e < 2; e++) { inv2<false>(y[e], y[e + 2], v[1]); fwd2i(y[e + 4], y[e + 6], v[1]); }
                        inv2<false>(y[0], y[1], v[2]); fwd2i(y[2], y[3], v[2]); inv2<false>(y[4], y[5], v[3]); fwd2i(y[6], y[7], v[3]);
                        FFT_FENCE();
#pragma unroll
                        for (int m = 0; m < 8; m++) lds_put(aT + cc * F10_BUF + 16 * 9 * m, y[m]);
                    }
                    if constexpr (!alone) fft_signal(spectra_done + (SHARE == 8 ? 4u * wave : 0u), tick);
                }
                // ---- layers 7..9 ----
                if constexpr (FIRST <= LAST) {
                    d2 D[2][8];
                    {
                        d2 f3[4];
#pragma unroll
                        for (int q = 0; q < 4; q++) f3[q] = lane_get(A.tab + F10_F3_OFF + 64 * q + z, kl);
                        // key words of the first positions are requested one phase ahead of their use, here and at the end of every piece
                        if constexpr (front) {
#pragma unroll
                            for (int k = 0; k < F10_EARLY; k++) request(k);
                        } else {
#pragma unroll
                            for (int k = 0; k < 8; k++) request(k);
                        }
                        FFT_FENCE();
                        if constexpr (!front) {
                            fft_wait(spectra_done, fft_peek(spectra_done), tick);
                            if (SHARE == 8) fft_wait(spectra_done + 4u, fft_peek(spectra_done + 4u), tick);
                        }
                        const uint32_t lr = fresh(lane), rd = O0 + z + 1152u * (lr >> 3) + 144u * (lr & 7u);
#pragma unroll
                        for (int cc = 0; cc < 2; cc++)
#pragma unroll
                            for (int i = 0; i < 4; i++) {
                                D[cc][i] = lds_get(rd + cc * component_stride + 16 * i);
                                D[cc][i + 4] = lds_get(rd + cc * component_stride + 16 * (i + 4));
                            }
                        if (SHARE < 8 && !front) fft_signal(spectra_read + 4u * wave, tick);
#pragma unroll
                        for (int cc = 0; cc < 2; cc++) {
                            d2 *y = D[cc];
#pragma unroll
                            for (int e = 0; e < 4; e++) inv2<false>(y[e], y[e + 4], f3[0]);
#pragma unroll
                            for (int e = 0; e < 2; e++) { inv2<false>(y[e], y[e + 2], f3[1]); fwd2i(y[e + 4], y[e + 6], f3[1]); }
                            inv2<false>(y[0], y[1], f3[2]); fwd2i(y[2], y[3], f3[2]); inv2<false>(y[4], y[5], f3[3]); fwd2i(y[6], y[7], f3[3]);
                        }
                    }
                    if constexpr (!front) {
#pragma unroll
                        for (int cc = 0; cc < NA; cc++)
#pragma unroll
                            for (int e = 0; e < 8; e++) accr[cc][e] = acci[cc][e] = 0;
                    }
                    // ---- key pieces ----
                    auto run_piece = [&](auto which, auto early) __attribute__((always_inline)) {
                        constexpr int piece = decltype(which)::value, ahead = decltype(early)::value;
                        constexpr bool more = piece < LAST;
                        asm volatile("s_mov_b32 %0, 0" : "=s"(z));
                        const uint32_t T = T0 + z;
                        d2 S[2][8];
#pragma unroll
                        for (int k = 0; k < 8; k++) {
                            FFT_FENCE();
#pragma unroll
                            for (int n = (k ? k + F10_RING - 1 : ahead); n < 8 && n < k + F10_RING; n++)
                                if (n >= ahead) request(n);
                            FFT_FENCE();
#pragma unroll
                            for (int cc = 0; cc < 2; cc++) {
                                const d2 k0 = kb[k][cc], k1 = kb[k][2 + cc], a = D[0][k], b = D[1][k];
                                S[cc][k].x = __builtin_fma(-b.y, k1.y, __builtin_fma(b.x, k1.x, __builtin_fma(-a.y, k0.y, a.x * k0.x)));
                                S[cc][k].y = __builtin_fma(b.y, k1.x, __builtin_fma(b.x, k1.y, __builtin_fma(a.y, k0.x, a.x * k0.y)));
                                pin(S[cc][k]);
                            }
                        }
                        FFT_FENCE();
                        if (!alone && front && piece == FIRST) {     // its buffers are where the others read the spectra
#pragma unroll
                            for (uint32_t q = 0; q < HELPERS; q++) fft_wait(spectra_read + 4u * helper(q), fft_peek(spectra_read + 4u * helper(q)), tick);
                        }
                        const uint32_t ln = fresh(lane);
                        const uint32_t aK = T + 1152u * (ln >> 3) + 144u * (ln & 7u), aT = T + 1152u * (ln >> 3) + 16u * (ln & 7u), aL = T + 16u * ln;
                        const uint32_t t2 = tab0 + z + F10_I2_OFF * 16u + 16u * (ln & 7u), t3 = tab0 + z + F10_I3_OFF * 16u + 16u * ln;
                        // I1: half-sizes 1, 2, 4
                        d2 w2[4];
#pragma unroll
                        for (int cc = 0; cc < 2; cc++) {
                            inv8(S[cc]);
#pragma unroll
                            for (int k = 0; k < 8; k++) lds_put(aK + cc * F10_BUF + 16 * k, S[cc][k]);
#pragma unroll
                            for (int m = 0; m < 8; m++) S[cc][m] = lds_get(aT + cc * F10_BUF + 16 * 9 * m);
                            if (cc == 0) {
#pragma unroll
                                for (int t = 0; t < 4; t++) w2[t] = lds_get(t2 + 128 * t);
                            }
                            FFT_FENCE();
                        }
                        // I2: half-sizes 8, 16, 32
                        d2 w3[2];
#pragma unroll
                        for (int cc = 0; cc < 2; cc++) {
                            d2 *x = S[cc];
#pragma unroll
                            for (int m = 0; m < 8; m += 2) inv2<false>(x[m], x[m + 1], w2[0]);
#pragma unroll
                            for (int m = 0; m < 8; m += 4) { inv2<false>(x[m], x[m + 2], w2[1]); inv2<true>(x[m + 1], x[m + 3], w2[1]); }
                            inv2<false>(x[0], x[4], w2[2]); inv2<true>(x[2], x[6], w2[2]);
                            inv2<false>(x[1], x[5], w2[3]); inv2<true>(x[3], x[7], w2[3]);
#pragma unroll
                            for (int m = 0; m < 8; m++) lds_put(aT + cc * F10_BUF + 16 * 8 * m, x[m]);
#pragma unroll
                            for (int f = 0; f < 8; f++) x[f] = lds_get(aL + cc * F10_BUF + 16 * 72 * f);
                            if (cc == 0) {
#pragma unroll
                                for (int t = 0; t < 2; t++) w3[t] = lds_get(t3 + 1024 * t);
                            }
                            FFT_FENCE();
                        }
                        // I3: half-sizes 64, 128, 256 with the twist
                        kp += 2048u;
                        d2 c1[2], c2[2];
                        c1[0] = lds_get(t3 + 2048); c2[0] = lds_get(t3 + 3072);
                        FFT_FENCE();
#pragma unroll
                        for (int cc = 0; cc < 2; cc++) {
                            d2 *x = S[cc];
#pragma unroll
                            for (int f = 0; f < 8; f += 2) inv2<false>(x[f], x[f + 1], w3[0]);
#pragma unroll
                            for (int f = 0; f < 8; f += 4) { inv2<false>(x[f], x[f + 2], w3[1]); inv2<true>(x[f + 1], x[f + 3], w3[1]); }
#pragma unroll
                            for (int f = 0; f < 4; f++) {
                                const int e = 4 * cc + f;
                                FFT_FENCE();
                                if (e + 1 < 8) {
                                    c1[(e + 1) & 1] = lds_get(t3 + 2048 + 2048 * ((e + 1) & 3));
                                    c2[(e + 1) & 1] = lds_get(t3 + 3072 + 2048 * ((e + 1) & 3));
                                }
                                FFT_FENCE();
                                d2 a = cmul(x[f], c1[e & 1]), b = x[f + 4];
                                inv2<false>(a, b, c2[e & 1]);
                                // coefficients 64 f + lane (a) and 256 + 64 f + lane (b turned by -45 degrees), rounded
                                const uint64_t y0 = (uint64_t)__double_as_longlong(a.x + magic), y1 = (uint64_t)__double_as_longlong(a.y + magic);
                                const uint64_t y2 = (uint64_t)__double_as_longlong(__builtin_fma(b.x + b.y, FFT_SQRT_HALF, magic));
                                const uint64_t y3 = (uint64_t)__double_as_longlong(__builtin_fma(b.y - b.x, FFT_SQRT_HALF, magic));
                                uint64_t &r0 = accr[NA == 2 ? cc : 0][f], &r1 = acci[NA == 2 ? cc : 0][f];
                                uint64_t &r2 = accr[NA == 2 ? cc : 0][f + 4], &r3 = acci[NA == 2 ? cc : 0][f + 4];
                                add_shifted<SLZ_FFT_PIECE_BITS * piece>(r0, y0);
                                add_shifted<SLZ_FFT_PIECE_BITS * piece>(r1, y1);
                                add_shifted<SLZ_FFT_PIECE_BITS * piece>(r2, y2);
                                add_shifted<SLZ_FFT_PIECE_BITS * piece>(r3, y3);
                                if (piece == 0) {                    // the bits of `magic` that shift 0 has left
                                    r0 -= 0x4338000000000000ull; r1 -= 0x4338000000000000ull;
                                    r2 -= 0x4338000000000000ull; r3 -= 0x4338000000000000ull;
                                }
                                pin(r0); pin(r1); pin(r2); pin(r3);
                                if (!more && (alone || !front)) { stage(cc, f); stage(cc, f + 4); }
                                if (more) {
                                    FFT_FENCE();
#pragma unroll
                                    for (int q = 0; q < 2; q++)
                                        kb[e / 2][2 * (e & 1) + q] = lane_get(kp + (4 * (e / 2) + 2 * (e & 1) + q) * 64, kl);
                                }
                            }
                        }
                    };
                    fft_int<F10_EARLY> four;
                    fft_int<front ? F10_EARLY : 8> begin;
                    run_piece(fft_int<FIRST>(), begin);
                    if constexpr (FIRST + 1 <= LAST) run_piece(fft_int<FIRST + 1>(), four);
                    if constexpr (FIRST + 2 <= LAST) run_piece(fft_int<FIRST + 2>(), four);
                    if constexpr (FIRST + 3 <= LAST) run_piece(fft_int<FIRST + 3>(), four);
                    if constexpr (FIRST + 4 <= LAST) run_piece(fft_int<FIRST + 4>(), four);
                    if constexpr (!front) fft_signal(sums_done + 4u * wave, tick);
                }
                if constexpr (front && !alone) {
                    // the other waves' sums
#pragma unroll 1
                    for (uint32_t q = 0; q < HELPERS; q++) {
                        const uint32_t w = helper(q), flag = sums_done + 4u * w;
                        fft_wait(flag, fft_peek(flag), tick);
#pragma unroll
                        for (int cc = 0; cc < NA; cc++) {
                            const LDS_AS uint64_t *S = (const LDS_AS uint64_t *)(uintptr_t)(lds + z + w * F10_WBUF + (COMPS == 1 ? wave : cc) * F10_BUF);
#pragma unroll
                            for (int e = 0; e < 8; e++) { accr[cc][e] += S[64 * e + lane]; acci[cc][e] += S[512 + 64 * e + lane]; }
                        }
                    }
                    stage_all();
                }
            }

            if constexpr (!front) continue;
            const uint32_t lo = fresh(lane);
#pragma unroll
            for (int cc = 0; cc < NA; cc++) {
                const uint32_t h = COMPS == 1 ? wave : cc;
                if (A.acc_out) {
                    uint64_t *dst = A.acc_out + ((size_t)c * 2 + h) * 1024u;
#pragma unroll
                    for (int e = 0; e < 8; e++) { dst[64u * e + lo] = (uint64_t)0 - accr[cc][e]; dst[512u + 64u * e + lo] = (uint64_t)0 - acci[cc][e]; }
                }
                if (A.lwe_out) {
                    uint64_t *dst = A.lwe_out + (size_t)c * 1025u;
                    if (h == 0) {
#pragma unroll
                        for (int e = 0; e < 8; e++) {
                            const uint32_t idx = 64u * e + lo;
                            if (idx == 0) dst[0] = (uint64_t)0 - accr[cc][0];
                            else dst[1024u - idx] = accr[cc][e];
                            dst[512u - idx] = acci[cc][e];
                        }
                    } else if (lo == 0) {
                        dst[1024] = (uint64_t)0 - accr[cc][0];
                    }
                }
            }
        }
    };
    fft_int<0> none;
    fft_int<1> one;
    fft_int<2> both;
    fft_int<4> last;
    if constexpr (SHARE == 1) rotate(none, last, both);
    else if constexpr (SHARE == 2) {
        if (wave < 4) rotate(none, one, both);
        else rotate(both, last, none);
    } else if constexpr (SHARE == 4) {
        if (wave < 2) rotate(none, none, both);
        else if (wave < 4) rotate(both, both, none);
        else if (wave < 6) rotate(one, one, none);
        else rotate(fft_int<3>(), last, none);
    } else {
        if (wave < 2) rotate(one, none, one);
        else if (wave == 2) rotate(fft_int<0>(), fft_int<0>(), none);
        else if (wave == 3) rotate(fft_int<1>(), fft_int<1>(), none);
        else if (wave == 4) rotate(fft_int<2>(), fft_int<2>(), none);
        else if (wave == 5) rotate(fft_int<3>(), fft_int<3>(), none);
        else if (wave == 6) rotate(fft_int<4>(), fft_int<4>(), none);
    }
}

// ---- host side ------------------------------------------------------------------------------------------------------

int slz_fft1024_setup() {
    const void *const kernels[6] = {(const void *)k_fft1024_blind_rotate<0, 8>, (const void *)k_fft1024_blind_rotate<0, 4>,
                                    (const void *)k_fft1024_blind_rotate<23, 2>, (const void *)k_fft1024_blind_rotate<0, 2>,
                                    (const void *)k_fft1024_blind_rotate<23, 1>, (const void *)k_fft1024_blind_rotate<0, 1>};
    for (const void *k : kernels) SLZ_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, F10_LDS_BYTES));
    return SLZ_OK;
}

// Largest batches of SHARE = 8, 4 and 2: one, two and four ciphertexts per compute unit.  Past each line the form would need a second
// round (1100 in two rounds of SHARE = 2: 17.0 ms, with SHARE = 1: 12.4), before it the next form leaves waves idle (512 with
// SHARE = 2: 7.1 ms, with 4: 5.6; 777 with SHARE = 1: 9.9 ms, with 2: 7.8).
#define F10_MAX_8 256
#define F10_MAX_4 512
#define F10_MAX_2 1024

int slz_fft1024_blind_rotate(slz_ctx *ctx, const uint64_t *lwe_in, const uint64_t *luts, const uint32_t *lut_idx, const void *key,
                             uint32_t n_steps, uint64_t *acc_out, uint64_t *lwe_out, uint32_t batch, hipStream_t s) {
    fft1024_args A;
    A.lwe_in = lwe_in; A.luts = luts; A.lut_idx = lut_idx; A.key = (const d2 *)key; A.tab = (const d2 *)ctx->fft_tab;
    A.acc_out = acc_out; A.lwe_out = lwe_out;
    A.n = ctx->prm.n; A.n_steps = n_steps; A.batch = batch; A.beta = ctx->prm.pbs_base_log;
    for (int q = 0; q < 4; q++)
        for (int t = 0; t < 2; t++) A.f1[q][t] = ctx->fft_f1[q][t];
    const uint32_t grid = slz_fused_grid(batch, 1);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(F10_THREADS), F10_LDS_BYTES, s, A); };
    // The base 2^23 of the parameter sets as a constant: 1024 ciphertexts with SHARE = 2 8.96 ms instead of 9.20, 1025 with SHARE = 1 12.04
    // instead of 12.30.  With SHARE = 8 and 4 the base as an argument is as fast (200: 3.64, 512: 5.63 against 5.67).
    const bool b23 = A.beta == 23;
    if (batch <= F10_MAX_8) launch(k_fft1024_blind_rotate<0, 8>);
    else if (batch <= F10_MAX_4) launch(k_fft1024_blind_rotate<0, 4>);
    else if (batch <= F10_MAX_2) b23 ? launch(k_fft1024_blind_rotate<23, 2>) : launch(k_fft1024_blind_rotate<0, 2>);
    else b23 ? launch(k_fft1024_blind_rotate<23, 1>) : launch(k_fft1024_blind_rotate<0, 1>);
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

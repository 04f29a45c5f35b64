// Blind rotation for N = 512, k = 1, l = 2 through exact double-precision transforms (slz_fft.h), bases up to 2^14.
//
// A half-wave transforms one polynomial, 8 of its 256 points per lane, so a wave holds both components of the ciphertext, and every
// exchange stays inside the wave.  Per CMux step:
//   front    the accumulator (negated, in registers) goes through LDS to be rotated; subtract, round, two signed digits per coefficient;
//            forward transforms of both levels (merged twiddles, radix-2 layers)
//   pieces   for each of the three key pieces (22 bits): products and their sum over the four rows, inverse transform (decimation in
//            time), rounding to integers, shifted add into the accumulator.
// Positions p = b7 .. b0.  Layouts (registers / lane bits from the top; c: component):
//   F1, I3: b7 b6 b5 / c b4..b0     F2, I2: b4 b3 b2 / c b7 b6 b5 b1 b0     spectra, I1: row or c, b1 b0 / b7..b2
// Exchanges between the first two layouts place a point at 68 (b7 b6 b5) + 32 c + (b4..b0), between the last two at
// 280 c + 140 b7 + 8 b6 + 4 b5 + 72 b4 + 34 b3 + 17 b2 + (b1 b0): 16 neighbouring lanes always touch 16 different columns of 16 bytes,
// writing and reading.
// Bound and shape: FP64 issue for large batches; a small one waits for the chain of a step, which is why its waves share the work (SHARE
// below).  A step is about 1.9 k VALU instructions per ciphertext, of 256 registers 190 to 250 are in use, two waves per SIMD.
// Measured with 128 steps and the keyswitch (in brackets: two 50-bit residues on the same card): 8 ciphertexts 0.51 ms (0.87),
// 512: 0.61 (1.21), 1024: 0.88 (2.40), 16384: 11.7 (38.3).
#include "slz_fft.h"
#include "slz_fft_wave.h"
#include "slz_modarith.h"
#include "slz_fused_common.h"

#define F9_WAVES 8
#define F9_THREADS (64 * F9_WAVES)
#define F9_BUF (576u * 16u)                         // bytes of the exchange buffer of two polynomials of 256 points, padded
#define F9_WBUF (2u * F9_BUF)
#define F9_FLAGS_OFF (F9_WAVES * F9_WBUF + F9_LDS_TAB * 16u)
#define F9_FLAGS 24u
#define F9_LDS_BYTES (F9_FLAGS_OFF + 4u * F9_FLAGS)
#define F9_RING 3                                   // positions of the key (eight words each) in registers at a time during the products
#define F9_EARLY 2                                  // positions requested before the last stages of the previous piece

struct fft512_args {
    const uint64_t *lwe_in;
    const uint64_t *luts;
    const uint32_t *lut_idx;
    const d2 *key;            // [n][F9_KEY_STEP]
    const d2 *tab;            // F9_TAB_LEN entries
    uint64_t *acc_out;
    uint64_t *lwe_out;
    uint32_t n, n_steps, batch, beta;
    double f1[4][2];          // lane-uniform twiddles of the first three forward layers
};

// three radix-2 layers over eight registers: one twiddle, one and its sibling's i w, two and their siblings'
__device__ __forceinline__ void fwd8(d2 *y, d2 w0, d2 w1, d2 w2, d2 w3) {
#pragma unroll
    for (int e = 0; e < 4; e++) inv2<false>(y[e], y[e + 4], w0);
#pragma unroll
    for (int e = 0; e < 2; e++) { inv2<false>(y[e], y[e + 2], w1); fwd2i(y[e + 4], y[e + 6], w1); }
    inv2<false>(y[0], y[1], w2); fwd2i(y[2], y[3], w2); inv2<false>(y[4], y[5], w3); fwd2i(y[6], y[7], w3);
}

// SHARE: waves per ciphertext.
//   1  a wave does everything
//   4  the first wave runs the front, the others a piece each
//   8  (one ciphertext per workgroup) the first two waves run the front for a level each, the next three a piece each
// Waves that share a ciphertext read the spectra, two layers before their end, from the front's exchange buffers; sums return
// through the buffer of the wave that made them.
template <int SHARE>
__global__ void __launch_bounds__(F9_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_fft512_blind_rotate(fft512_args A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const uint32_t lds = (uint32_t)(uintptr_t)(LDS_AS unsigned char *)lds_raw;
    const uint32_t beta = A.beta;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr uint32_t GROUPS = F9_WAVES / SHARE, HELPERS = SHARE == 1 ? 0 : 3;
    // wave w sits on SIMD w mod 4: with SHARE = 4 a ciphertext has two SIMDs to itself
    const uint32_t group = SHARE == 1 ? wave : SHARE == 4 ? wave & 1u : 0u;
    const uint32_t T0 = lds + wave * F9_WBUF;                         // this wave's two buffers
    const uint32_t O0 = SHARE == 1 ? T0 : lds + group * F9_WBUF;      // the front's
    constexpr uint32_t level_stride = SHARE == 8 ? F9_WBUF : F9_BUF;  // between the levels of the spectra there
    const uint32_t tab0 = lds + F9_WAVES * F9_WBUF;
    const uint32_t flags = lds + F9_FLAGS_OFF;
    // counters, in steps: spectra written (per front wave), sums written and progress (per wave)
    const uint32_t spectra_done = flags + 4u * (SHARE == 8 ? 0u : group), sums_done = flags + 32u, progress = flags + 64u;
    auto helper = [&](uint32_t q) { return SHARE == 8 ? 2u + q : group + 2u * (q + 1u); };
    for (uint32_t i = threadIdx.x; i < F9_LDS_TAB; i += F9_THREADS) lds_put(tab0 + 16u * i, A.tab[i]);
    if (threadIdx.x < F9_FLAGS) *(LDS_AS uint32_t *)(uintptr_t)(flags + 4u * threadIdx.x) = 0;
    __syncthreads();

    const double magic = 6755399441055744.0;                          // 1.5 * 2^52: adding it rounds to an integer
    uint32_t tick = 0;                                                // steps so far
    // One loop per kind of wave.  FIRST .. LAST: pieces of this wave; LEVELS: digit levels whose front it runs (2, 1 or 0)
    auto rotate = [&](auto first_piece, auto last_piece, auto levels) __attribute__((always_inline)) {
        constexpr int FIRST = decltype(first_piece)::value, LAST = decltype(last_piece)::value, LEVELS = decltype(levels)::value;
        constexpr bool front = LEVELS > 0, alone = SHARE == 1;
        for (uint32_t c = blockIdx.x + group * gridDim.x; c < A.batch; c += GROUPS * gridDim.x) {
            const uint64_t *lwe = A.lwe_in + (size_t)c * (A.n + 1);
            uint64_t accr[8], acci[8];                                // negated coefficients 32 e + (lane & 31) and 256 more, component lane >> 5
            const uint32_t li = fresh(lane);
#pragma unroll
            for (int e = 0; e < 8; e++) accr[e] = acci[e] = 0;
            if (front && (li >> 5)) {
                const uint32_t bt = slz_modswitch(lwe[A.n], 10);
                const uint32_t r = (1024u - bt) & 1023u;
                const uint64_t *lut = A.luts + (size_t)(A.lut_idx ? A.lut_idx[c] : 0) * 512u;
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    accr[e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 32u * e + (li & 31u), r, 512u);
                    acci[e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 256u + 32u * e + (li & 31u), r, 512u);
                }
            }
            // The accumulator is written to the first buffer whenever it is complete: here and at the end of every step.  A helper's sums
            // too.  Word `coefficient + 512 component`.
            auto stage = [&](int e) {
                LDS_AS uint64_t *S = (LDS_AS uint64_t *)(uintptr_t)(T0 + 4096u * (lane >> 5) + 8u * (lane & 31u));
                S[32 * e] = accr[e];
                S[256 + 32 * e] = acci[e];
            };
            auto stage_all = [&]() {
#pragma unroll
                for (int e = 0; e < 8; e++) stage(e);
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
                const d2 *kp = A.key + (size_t)step * F9_KEY_STEP + FIRST * 2048u + z;
                d2 kb[4][8];
                const uint32_t kl = fresh(lane);
                auto request = [&](int k) {
#pragma unroll
                    for (int q = 0; q < 8; q++) kb[k][q] = lane_get(kp + (8 * k + q) * 64, kl);
                };
                if constexpr (front) {
                    const uint32_t T = T0 + z;
                    d2 x[LEVELS][8];
                    const uint32_t at = slz_modswitch(mask, 10);
                    mask = lwe[step + 1];                             // the next step's word (the body after the last step)
                    // ---- digits ----
                    {
                        // word (idx - at) mod 1024 of X^at ACC: nine bits of address, the tenth is the sign; its opposite (bit 12 of t)
                        // tells where the stored, negated word has to be negated again
                        const uint32_t ld = fresh(lane);
                        const uint32_t rnd = 1u << (31 - 2 * beta), up = 1u << (31 - beta), t0 = 8u * (ld & 31u) + 0x1000u - 8u * at, Tc = T + 4096u * (ld >> 5);
                        auto word = [&](uint32_t t) { return *(const LDS_AS uint64_t *)(uintptr_t)(Tc + (t & 0xff8u)); };
                        uint64_t a[16];
#pragma unroll
                        for (int i = 0; i < 16; i++) a[i] = word(t0 + 2048u * (i >> 3) + 256u * (i & 7));
                        FFT_FENCE();
#pragma unroll
                        for (int i = 0; i < 16; i++) {
                            const uint32_t t = t0 + 2048u * (i >> 3) + 256u * (i & 7), m = (uint32_t)((int32_t)(t << 19) >> 31);
                            const uint64_t own = i < 8 ? accr[i & 7] : acci[i & 7];
                            uint32_t lo = (uint32_t)a[i] ^ m, hi = (uint32_t)(a[i] >> 32) ^ m;
                            asm("v_cmp_ne_u32_e32 vcc, 0, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %3, vcc\n\tv_addc_co_u32_e32 %1, vcc, %1, %4, vcc"
                                : "+v"(lo), "+v"(hi) : "v"(m), "v"((uint32_t)own), "v"((uint32_t)(own >> 32)) : "vcc");
                            // the lower digit (level 1) keeps its sign, which carries into the upper one
                            const uint32_t v = hi + rnd;
                            const double d0 = (double)((int32_t)(v + up) >> (32 - beta)), d1 = (double)((int32_t)(v << beta) >> (32 - beta));
                            if constexpr (LEVELS == 2) {
                                if (i < 8) { x[0][i].x = d0; x[1][i].x = d1; }
                                else { x[0][i & 7].y = d0; x[1][i & 7].y = d1; }
                            } else {
                                const double d = wave == 0 ? d0 : d1;
                                if (i < 8) x[0][i].x = d;
                                else x[0][i & 7].y = d;
                            }
                        }
                    }
                    // ---- forward transform: layers 1..6 ----
                    auto f1 = [&](int q) { d2 w; w.x = A.f1[q + z][0]; w.y = A.f1[q + z][1]; return w; };
                    const uint32_t ln = fresh(lane);
                    const uint32_t aL = T + 16u * ln, aT = T + 1088u * ((ln >> 2) & 7u) + 512u * (ln >> 5) + 16u * (ln & 3u),
                                   aW = T + 16u * (ln & 15u) + 2240u * (ln >> 4);
                    d2 v[4];
#pragma unroll
                    for (int t = 0; t < 4; t++) v[t] = lds_get(tab0 + z + F9_F2_OFF * 16u + 16u * ((ln >> 2) & 7u) + 128u * t);
#pragma unroll
                    for (int lv = 0; lv < LEVELS; lv++) {
                        fwd8(x[lv], f1(0), f1(1), f1(2), f1(3));
                        FFT_FENCE();
#pragma unroll
                        for (int e = 0; e < 8; e++) lds_put(aL + lv * F9_BUF + 16 * 68 * e, x[lv][e]);
#pragma unroll
                        for (int m = 0; m < 8; m++) x[lv][m] = lds_get(aT + lv * F9_BUF + 16 * 4 * m);
                    }
#pragma unroll
                    for (int lv = 0; lv < LEVELS; lv++) {
                        FFT_FENCE();
                        fwd8(x[lv], v[0], v[1], v[2], v[3]);
                        FFT_FENCE();
#pragma unroll
                        for (int m = 0; m < 8; m++) lds_put(aW + lv * F9_BUF + 16 * (72 * (m >> 2) + 34 * ((m >> 1) & 1) + 17 * (m & 1)), x[lv][m]);
                    }
                    if constexpr (!alone) fft_signal(spectra_done + (SHARE == 8 ? 4u * wave : 0u), tick);
                }
                if constexpr (FIRST <= LAST) {
                    // ---- layers 7 and 8; D[2 component + level] ----
                    d2 D[4][4];
                    {
                        d2 f3[2];
#pragma unroll
                        for (int q = 0; q < 2; q++) f3[q] = lane_get(A.tab + F9_F3_OFF + 64 * q + z, kl);
                        // key words of the first positions are requested ahead of their use, here and in every piece
#pragma unroll
                        for (int k = 0; k < (front ? F9_EARLY : F9_RING); k++) request(k);
                        FFT_FENCE();
                        if constexpr (!front) {
                            fft_wait(spectra_done, fft_peek(spectra_done), tick);
                            if (SHARE == 8) fft_wait(spectra_done + 4u, fft_peek(spectra_done + 4u), tick);
                        }
                        const uint32_t lr = fresh(lane);
                        const uint32_t rd = O0 + z + 272u * (lr & 3u) + 1152u * ((lr >> 2) & 1u) + 64u * ((lr >> 3) & 3u) + 2240u * (lr >> 5);
#pragma unroll
                        for (int r = 0; r < 4; r++)
#pragma unroll
                            for (int k = 0; k < 4; k++) D[r][k] = lds_get(rd + (r & 1) * level_stride + 16 * (k + 280 * (r >> 1)));
#pragma unroll
                        for (int r = 0; r < 4; r++) {
                            d2 *y = D[r];
                            inv2<false>(y[0], y[2], f3[0]); inv2<false>(y[1], y[3], f3[0]);
                            inv2<false>(y[0], y[1], f3[1]); fwd2i(y[2], y[3], f3[1]);
                        }
                    }
                    if constexpr (!front) {
#pragma unroll
                        for (int e = 0; e < 8; e++) accr[e] = acci[e] = 0;
                    }
                    // ---- key pieces ----
                    auto run_piece = [&](auto which, auto early) __attribute__((always_inline)) {
                        constexpr int piece = decltype(which)::value, ahead = decltype(early)::value;
                        constexpr bool more = piece < LAST;
                        asm volatile("s_mov_b32 %0, 0" : "=s"(z));
                        const uint32_t T = T0 + z;
                        d2 S[2][4];
#pragma unroll
                        for (int k = 0; k < 4; k++) {
                            FFT_FENCE();
#pragma unroll
                            for (int n = (k ? k + F9_RING - 1 : ahead); n < 4 && n < k + F9_RING; n++)
                                if (n >= ahead) request(n);
                            FFT_FENCE();
#pragma unroll
                            for (int cc = 0; cc < 2; cc++) {
                                double sx = 0, sy = 0;
#pragma unroll
                                for (int r = 0; r < 4; r++) {
                                    const d2 w = kb[k][2 * r + cc], a = D[r][k];
                                    sx = __builtin_fma(-a.y, w.y, r ? __builtin_fma(a.x, w.x, sx) : a.x * w.x);
                                    sy = __builtin_fma(a.y, w.x, r ? __builtin_fma(a.x, w.y, sy) : a.x * w.y);
                                }
                                S[cc][k].x = sx; S[cc][k].y = sy;
                                pin(S[cc][k]);
                            }
                        }
                        FFT_FENCE();
                        const uint32_t ln = fresh(lane);
                        const uint32_t aR = T + 272u * (ln & 3u) + 1152u * ((ln >> 2) & 1u) + 64u * ((ln >> 3) & 3u) + 2240u * (ln >> 5);
                        const uint32_t aL = T + 16u * ln, aT = T + 1088u * ((ln >> 2) & 7u) + 512u * (ln >> 5) + 16u * (ln & 3u),
                                       aW = T + 16u * (ln & 15u) + 2240u * (ln >> 4);
                        const uint32_t t2 = tab0 + z + F9_I2_OFF * 16u + 16u * (ln & 3u), t3 = tab0 + z + F9_I3_OFF * 16u + 16u * (ln & 31u);
                        // I1: half-sizes 1 and 2
#pragma unroll
                        for (int cc = 0; cc < 2; cc++) {
                            d2 *s = S[cc];
                            add2(s[0], s[1]); add2(s[2], s[3]);
                            add2(s[0], s[2]); add2i(s[1], s[3]);
#pragma unroll
                            for (int k = 0; k < 4; k++) lds_put(aR + 16 * (k + 280 * cc), s[k]);
                        }
                        d2 x[8], w2[4], w3[2];
#pragma unroll
                        for (int t = 0; t < 4; t++) w2[t] = lds_get(t2 + 64 * t);
#pragma unroll
                        for (int m = 0; m < 8; m++) x[m] = lds_get(aW + 16 * (72 * (m >> 2) + 34 * ((m >> 1) & 1) + 17 * (m & 1)));
                        kp += 2048u;
                        if (more) {
                            FFT_FENCE();
#pragma unroll
                            for (int k = 0; k < F9_EARLY; k++) request(k);
                            FFT_FENCE();
                        }
                        // I2: half-sizes 4, 8, 16
#pragma unroll
                        for (int m = 0; m < 8; m += 2) inv2<false>(x[m], x[m + 1], w2[0]);
#pragma unroll
                        for (int m = 0; m < 8; m += 4) { inv2<false>(x[m], x[m + 2], w2[1]); inv2<true>(x[m + 1], x[m + 3], w2[1]); }
                        inv2<false>(x[0], x[4], w2[2]); inv2<true>(x[2], x[6], w2[2]);
                        inv2<false>(x[1], x[5], w2[3]); inv2<true>(x[3], x[7], w2[3]);
                        FFT_FENCE();
#pragma unroll
                        for (int m = 0; m < 8; m++) lds_put(aT + 16 * 4 * m, x[m]);
                        // I3: half-sizes 32, 64, 128 with the twist
                        d2 c1[4], c2[4];
#pragma unroll
                        for (int t = 0; t < 2; t++) w3[t] = lds_get(t3 + 512 * t);
#pragma unroll
                        for (int f = 0; f < 8; f++) x[f] = lds_get(aL + 16 * 68 * f);
#pragma unroll
                        for (int f = 0; f < 4; f++) { c1[f] = lds_get(t3 + 1024 + 1024 * f); c2[f] = lds_get(t3 + 1536 + 1024 * f); }
                        FFT_FENCE();
#pragma unroll
                        for (int f = 0; f < 8; f += 2) inv2<false>(x[f], x[f + 1], w3[0]);
#pragma unroll
                        for (int f = 0; f < 8; f += 4) { inv2<false>(x[f], x[f + 2], w3[1]); inv2<true>(x[f + 1], x[f + 3], w3[1]); }
#pragma unroll
                        for (int f = 0; f < 4; f++) {
                            FFT_FENCE();
                            d2 a = cmul(x[f], c1[f]), b = x[f + 4];
                            inv2<false>(a, b, c2[f]);
                            // coefficients 32 f + (lane & 31) (a) and 128 more (b turned by -45 degrees), rounded
                            const uint64_t y0 = (uint64_t)__double_as_longlong(a.x + magic), y1 = (uint64_t)__double_as_longlong(a.y + magic);
                            const uint64_t y2 = (uint64_t)__double_as_longlong(__builtin_fma(b.x + b.y, FFT_SQRT_HALF, magic));
                            const uint64_t y3 = (uint64_t)__double_as_longlong(__builtin_fma(b.y - b.x, FFT_SQRT_HALF, magic));
                            add_shifted<F9_PIECE_BITS * piece>(accr[f], y0);
                            add_shifted<F9_PIECE_BITS * piece>(acci[f], y1);
                            add_shifted<F9_PIECE_BITS * piece>(accr[f + 4], y2);
                            add_shifted<F9_PIECE_BITS * piece>(acci[f + 4], y3);
                            if (piece == 0) {                        // the bits of `magic` that shift 0 has left
                                accr[f] -= 0x4338000000000000ull; acci[f] -= 0x4338000000000000ull;
                                accr[f + 4] -= 0x4338000000000000ull; acci[f + 4] -= 0x4338000000000000ull;
                            }
                            pin(accr[f]); pin(acci[f]); pin(accr[f + 4]); pin(acci[f + 4]);
                            if (!more && (alone || !front)) { stage(f); stage(f + 4); }
                        }
                    };
                    fft_int<F9_EARLY> some;
                    fft_int<front ? F9_EARLY : F9_RING> begin;
                    run_piece(fft_int<FIRST>(), begin);
                    if constexpr (FIRST + 1 <= LAST) run_piece(fft_int<FIRST + 1>(), some);
                    if constexpr (FIRST + 2 <= LAST) run_piece(fft_int<FIRST + 2>(), some);
                    if constexpr (!front) fft_signal(sums_done + 4u * wave, tick);
                }
                if constexpr (front && !alone) {
                    // the other waves' sums
#pragma unroll 1
                    for (uint32_t q = 0; q < HELPERS; q++) {
                        const uint32_t w = helper(q), flag = sums_done + 4u * w;
                        fft_wait(flag, fft_peek(flag), tick);
                        const LDS_AS uint64_t *S = (const LDS_AS uint64_t *)(uintptr_t)(lds + z + w * F9_WBUF + 4096u * (lane >> 5) + 8u * (lane & 31u));
#pragma unroll
                        for (int e = 0; e < 8; e++) { accr[e] += S[32 * e]; acci[e] += S[256 + 32 * e]; }
                    }
                    stage_all();
                }
            }

            if (!front || (SHARE == 8 && wave != 0)) continue;
            const uint32_t l5 = fresh(lane) & 31u, h = lane >> 5;
            if (A.acc_out) {
                uint64_t *dst = A.acc_out + ((size_t)c * 2 + h) * 512u;
#pragma unroll
                for (int e = 0; e < 8; e++) { dst[32u * e + l5] = (uint64_t)0 - accr[e]; dst[256u + 32u * e + l5] = (uint64_t)0 - acci[e]; }
            }
            if (A.lwe_out) {
                uint64_t *dst = A.lwe_out + (size_t)c * 513u;
                if (h == 0) {
#pragma unroll
                    for (int e = 0; e < 8; e++) {
                        const uint32_t idx = 32u * e + l5;
                        if (idx == 0) dst[0] = (uint64_t)0 - accr[0];
                        else dst[512u - idx] = accr[e];
                        dst[256u - idx] = acci[e];
                    }
                } else if (l5 == 0) {
                    dst[512] = (uint64_t)0 - accr[0];
                }
            }
        }
    };
    fft_int<0> zero;
    fft_int<1> one;
    fft_int<2> two;
    if constexpr (SHARE == 1) rotate(zero, two, two);
    else if constexpr (SHARE == 4) {
        if (wave < 2) rotate(one, zero, two);
        else if (wave < 4) rotate(zero, zero, zero);
        else if (wave < 6) rotate(one, one, zero);
        else rotate(two, two, zero);
    } else {
        if (wave < 2) rotate(one, zero, one);
        else if (wave == 2) rotate(zero, zero, zero);
        else if (wave == 3) rotate(one, one, zero);
        else if (wave == 4) rotate(two, two, zero);
    }
}

// ---- host side ------------------------------------------------------------------------------------------------------

int slz_fft512_setup() {
    const void *const kernels[3] = {(const void *)k_fft512_blind_rotate<1>, (const void *)k_fft512_blind_rotate<4>, (const void *)k_fft512_blind_rotate<8>};
    for (const void *k : kernels) SLZ_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, F9_LDS_BYTES));
    return SLZ_OK;
}

// Largest batches of SHARE = 8 and 4: one and two ciphertexts per compute unit.  256 ciphertexts take 0.50 ms with 8 waves each and 0.61 ms
// with 4; 300 take 0.61 ms with 4 and 0.99 ms in two rounds of 8; 1024 take 0.88 ms with one wave each, and two would gain 1 %, 8 % for 600.
#define F9_MAX_8 256
#define F9_MAX_4 512

int slz_fft512_blind_rotate(slz_ctx *ctx, const uint64_t *lwe_in, const uint64_t *luts, const uint32_t *lut_idx, const void *key,
                            uint32_t n_steps, uint64_t *acc_out, uint64_t *lwe_out, uint32_t batch, hipStream_t s) {
    fft512_args A;
    A.lwe_in = lwe_in; A.luts = luts; A.lut_idx = lut_idx; A.key = (const d2 *)key; A.tab = (const d2 *)ctx->fft_tab;
    A.acc_out = acc_out; A.lwe_out = lwe_out;
    A.n = ctx->prm.n; A.n_steps = n_steps; A.batch = batch; A.beta = ctx->prm.pbs_base_log;
    for (int q = 0; q < 4; q++)
        for (int t = 0; t < 2; t++) A.f1[q][t] = ctx->fft_f1[q][t];
    const uint32_t grid = slz_fused_grid(batch, 1);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(F9_THREADS), F9_LDS_BYTES, s, A); };
    if (batch <= F9_MAX_8) launch(k_fft512_blind_rotate<8>);
    else if (batch <= F9_MAX_4) launch(k_fft512_blind_rotate<4>);
    else launch(k_fft512_blind_rotate<1>);
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

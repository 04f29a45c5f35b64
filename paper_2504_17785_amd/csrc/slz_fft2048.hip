// Blind rotation for N = 2048, k = 1, l = 1 through exact double-precision transforms (slz_fft.h).
//
// Two wavefronts own one ciphertext for the whole rotation.  Wave h keeps component h of the accumulator in registers
// (32 words per lane) and transforms it; between the transforms, wave g holds the spectra of both components at the half g of
// the 1024 points, so the products with the key need no exchange of their own.  Per CMux step and wave:
//   1. the accumulator goes through LDS to be rotated; subtract, round, one signed digit per coefficient; digits c and
//      c + 1024 are the real and imaginary part of one of 1024 points, 16 per lane
//   2. forward transform (merged twiddles, five radix-4 layers) with two LDS exchanges, the second one across the two waves
//   3. for each of the five key pieces: products and their sum over the two rows, inverse transform (decimation in time, ten
//      radix-2 stages) with two LDS exchanges, the first one across the two waves; rounding to integers, shifted add into
//      the accumulator.
// Positions: p = 0 .. 1023 with bits b9 .. b0; before the forward and after the inverse transform p is the coefficient, in
// between the bit-reversed evaluation point.  Layouts (registers / lane bits from the top / wave):
//   F1, I3: b9..b6 / b5..b0      F2: b5..b2 / b9..b6 b1 b0      F3, I1: component b2..b0 / b8..b3 / wave b9
//   I2: b6..b3 / b9 b8 b7 b2 b1 b0
// Exchanges place a point at 272 * (two bits) + 17 * (four bits) + (four bits) of a wave's buffer: the odd stride spreads the bits in
// the middle over the 16 columns (of 16 bytes) that LDS serves at a time, so that with the orders below 16 neighbouring lanes always
// touch 16 different columns when writing and when reading, and every register's slot is one lane base plus an immediate:
//   F1 -> F2: b9 b8 / b7 b6 b5 b4 / b3 b2 b1 b0     F2 -> F3: b9 b8 / b5 b2 b4 b3 / b7 b6 b1 b0
//   I1 -> I2 and I2 -> I3: b9 b8 / b3 b6 b5 b4 / b7 b2 b1 b0
// The accumulator is kept negated (and so are the key's spectra): X^a ACC - ACC is then one exclusive-or and one addition with
// carry per word.
// Bound and shape: a step is about 4.8 k VALU instructions per wave (3.8 k of them FP64); two 50-bit residues took 17.3 k
// wave-instructions per ciphertext.  Registers decide the rest: accumulator 64, spectra 64, transform 64 of 256, two waves per
// SIMD; key words stream from L2 (320 KiB per step, every ciphertext reads all of it) through what is left.  Eight waves (four
// ciphertexts) share one workgroup, i.e. one copy of the tables in LDS, and only the two waves of a ciphertext wait for each other.
// Two waves hide little of each other's LDS round trips, so loads are requested in groups ahead of the arithmetic, and results are
// written while the next ones are computed.  Measured with 742 steps (in brackets: two residues on the same card): 1024 ciphertexts
// 20.2 ms (31.5), 4096: 80.6 (126.6), 301: 11.5 (15.4).
// Batches up to 128 go to slz_fft2048_pair.hip, up to 256 to slz_fft2048_team.hip.  From 257 to 512 a compute unit has two ciphertexts; two pairs work on each (SHARE = 2).
#include "slz_fft.h"
#include "slz_fft_wave.h"
#include "slz_modarith.h"
#include "slz_fused_common.h"
#include "slz_xcd.h"

#define FFT_WAVES 8                                 // waves per workgroup: four ciphertexts share one copy of the tables
#define FFT_PAIRS (FFT_WAVES / 2)
#define FFT_TEAM_MAX 256                            // batches up to this: slz_fft2048_team.hip; up to twice this: two pairs per ciphertext
#define FFT_THREADS (64 * FFT_WAVES)
#define FFT_BUF (4u * 272u * 16u)                   // bytes of a wave's exchange buffer: 1024 points, padded
#define FFT_EARLY 4                                 // positions (of four key words each) requested during the last inverse stage: each of its
                                                    // eight butterflies frees the registers of half a position
#define FFT_RING 4                                  // positions in registers at a time during the products
#define FFT_FLAGS_OFF (FFT_WAVES * FFT_BUF + FFT_LDS_TAB * 16u)
#define FFT_FLAGS 40u                               // per wave: done and free; for shared ciphertexts also spectra written, read, sums written
#define FFT_LDS_BYTES (FFT_FLAGS_OFF + 4u * FFT_FLAGS)

struct fft_args {
    const uint64_t *lwe_in;
    const uint64_t *luts;
    const uint32_t *lut_idx;
    const d2 *key;            // [n][FFT_KEY_STEP]
    const d2 *tab;            // FFT_TAB_LEN entries
    uint64_t *acc_out;
    uint64_t *lwe_out;
    uint32_t n, n_steps, batch, beta;
    double f1[15][2];         // lane-uniform twiddles of the first two forward layers: (v, v^2, v^3) of block 0 and of the next four blocks
};

// SHARE = 1: a workgroup's four pairs of waves take a ciphertext each.  SHARE = 2, for batches of at most two ciphertexts per
// compute unit: two pairs work on each.  One owns the accumulator, runs step 1, the forward transform and two key pieces; the other
// reads the spectra from the owner's exchange buffers and takes three pieces (its first piece's key words wait in registers by then); its sums
// come back through its exchange buffers.  The owners of a workgroup's two ciphertexts sit on different SIMDs.
// The base is an argument: an instance with 23 as a constant measured the same (256 ciphertexts 8.28 ms, 301: 12.95, 1024: 20.2).
template <int SHARE>
__global__ void __launch_bounds__(FFT_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_fft_blind_rotate(fft_args A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const uint32_t lds = (uint32_t)(uintptr_t)(LDS_AS unsigned char *)lds_raw;
    const uint32_t beta = A.beta;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr bool SHARED = SHARE == 2;
    constexpr uint32_t GROUPS = FFT_PAIRS / SHARE;                    // ciphertexts of a workgroup at a time
    const uint32_t h = wave & 1u, pair = wave >> 1, group = pair / SHARE;
    const uint32_t T0 = lds + wave * FFT_BUF, Tp0 = lds + (wave & ~1u) * FFT_BUF;   // buffer of component h; of both components
    const uint32_t tab0 = lds + FFT_WAVES * FFT_BUF;
    const uint32_t flags = lds + FFT_FLAGS_OFF;
    const uint32_t my_done = flags + 4u * wave, my_free = my_done + 32u, his_done = flags + 4u * (wave ^ 1u), his_free = his_done + 32u;
    for (uint32_t i = threadIdx.x; i < FFT_LDS_TAB; i += FFT_THREADS) lds_put(tab0 + 16u * i, A.tab[i]);
    if (threadIdx.x < FFT_FLAGS) *(LDS_AS uint32_t *)(uintptr_t)(flags + 4u * threadIdx.x) = 0;
    // SHARE = 2, counted in steps: spectra written (per owner wave), spectra read, sums written (per wave of the group)
    const uint32_t own = 6u * group;                                  // first wave of this group's owner pair
    const uint32_t spectra_done = flags + 64u + 4u * own, spectra_read = flags + 96u + 8u * SHARE * group, sums_done = flags + 128u;
    __syncthreads();

    const double magic = 6755399441055744.0;                          // 1.5 * 2^52: adding it rounds to an integer
    uint32_t seq = 0;                                                 // exchanges of this pair so far
    uint32_t tick = 0;                                                // SHARE = 2: steps so far
    // One loop per kind of wave, so that each keeps only its own values in registers.  ROLE 0: owner, 1: helper, 2: the pair has the
    // ciphertext to itself.
    auto rotate = [&](auto role) __attribute__((always_inline)) {
        constexpr int ROLE = decltype(role)::value;
        constexpr bool owner = ROLE != 1;
        for (uint32_t c = blockIdx.x + group * gridDim.x; c < A.batch; c += GROUPS * gridDim.x) {
            const uint64_t *lwe = A.lwe_in + (size_t)c * (A.n + 1);
            uint64_t accr[16], acci[16];                                  // negated coefficients 64 e + lane and 1024 + 64 e + lane of component h
            const uint32_t li = fresh(lane);
            if (owner && h == 1) {
                const uint32_t bt = slz_modswitch(lwe[A.n], 12);
                const uint32_t r = (4096u - bt) & 4095u;
                const uint64_t *lut = A.luts + (size_t)(A.lut_idx ? A.lut_idx[c] : 0) * 2048u;
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    accr[e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 64u * e + li, r, 2048u);
                    acci[e] = (uint64_t)0 - slz_rot_coeff([&](uint32_t j) { return lut[j]; }, 1024u + 64u * e + li, r, 2048u);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; e++) accr[e] = acci[e] = 0;
            }

            // The owner's accumulator is written to its buffer whenever it is complete: here and at the end of every step.
            auto stage = [&](int e) {
                LDS_AS uint64_t *S = (LDS_AS uint64_t *)(uintptr_t)T0;
                S[64 * e + lane] = accr[e];
                S[1024 + 64 * e + lane] = acci[e];
            };
            if constexpr (owner) {
#pragma unroll
                for (int e = 0; e < 16; e++) stage(e);
            }
            uint64_t mask = owner ? lwe[0] : 0;
            for (uint32_t step = 0; step < A.n_steps; step++) {
                // an opaque zero in every table and buffer address keeps the loads inside the step
                int z;
                asm volatile("s_mov_b32 %0, 0" : "=s"(z));
                uint32_t T = T0 + z;
                tick++;
                if (!SHARED) {
                    // The SIMD serves its older wave first, which would let half of the ciphertexts of a compute unit run ahead and leave
                    // the SIMDs half empty at the end: of the two waves on a SIMD the one that is behind gets the priority.
                    if ((int32_t)(seq - (uint32_t)__builtin_amdgcn_readfirstlane(fft_peek(flags + 4u * (wave ^ 4u)))) > 0) __builtin_amdgcn_s_setprio(0);
                    else __builtin_amdgcn_s_setprio(2);
                }
                // the owner's front and two pieces are the longer chain: 742 steps of 257 ciphertexts 11.5 ms with, 12.4 without, 301: 11.4 and
                // 12.3, 512: 11.6 and 12.6
                if (SHARED && owner) __builtin_amdgcn_s_setprio(2);
                const d2 *kp = A.key + (size_t)step * FFT_KEY_STEP + h * 2048u + z;
                d2 kb[8][4];
                uint32_t kl = fresh(lane);
                auto request = [&](int k) {
#pragma unroll
                    for (int q = 0; q < 4; q++) kb[k][q] = lane_get(kp + (4 * k + q) * 64, kl);
                };
                d2 x[16];
                if constexpr (owner) {
                    const uint32_t at = slz_modswitch(mask, 12);
                    mask = lwe[step + 1];                                     // the next step's word (the body after the last step)
                    // ---- 1. digits ----
                    {
                        // word (idx - at) mod 4096 of X^at ACC: eleven bits of address, the twelfth is the sign; its opposite (bit 14 of t)
                        // tells where the stored, negated word has to be negated again
                        const uint32_t rnd = 1u << (31 - beta), t0 = 8u * fresh(lane) + 0x4000u - 8u * at;
                        auto word = [&](uint32_t t) { return *(const LDS_AS uint64_t *)(uintptr_t)(T + (t & 0x3ff8u)); };
                        auto digit = [&](uint32_t t, uint64_t a, uint64_t own) {
                            const uint32_t m = (uint32_t)((int32_t)(t << 17) >> 31);
                            uint32_t lo = (uint32_t)a ^ m, hi = (uint32_t)(a >> 32) ^ m;
                            asm("v_cmp_ne_u32_e32 vcc, 0, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %3, vcc\n\tv_addc_co_u32_e32 %1, vcc, %1, %4, vcc"
                                : "+v"(lo), "+v"(hi) : "v"(m), "v"((uint32_t)own), "v"((uint32_t)(own >> 32)) : "vcc");
                            return (double)((int32_t)(hi + rnd) >> (32 - beta));
                        };
                        // eight words are in flight while the previous eight become digits
                        uint64_t a[2][8];
#pragma unroll
                        for (int i = 0; i < 8; i++) a[0][i] = word(t0 + 512u * i);
#pragma unroll
                        for (int g = 0; g < 4; g++) {                        // real parts 0..7, 8..15, imaginary parts 0..7, 8..15
                            FFT_FENCE();
                            if (g < 3) {
#pragma unroll
                                for (int i = 0; i < 8; i++) a[(g + 1) & 1][i] = word(t0 + 4096u * (g + 1) + 512u * i);
                            }
                            FFT_FENCE();
#pragma unroll
                            for (int i = 0; i < 8; i++) {
                                const uint32_t t = t0 + 4096u * g + 512u * i;
                                if (g < 2) x[8 * g + i].x = digit(t, a[g & 1][i], accr[8 * g + i]);
                                else x[8 * (g - 2) + i].y = digit(t, a[g & 1][i], acci[8 * (g - 2) + i]);
                            }
                        }
                    }
                    // ---- 2. forward transform ----
                    auto f1 = [&](int q) { d2 w; w.x = A.f1[q + z][0]; w.y = A.f1[q + z][1]; return w; };
#pragma unroll
                    for (int e = 0; e < 4; e++) fwd4(x[e], x[e + 4], x[e + 8], x[e + 12], f1(0), f1(1), f1(2));
                    {
                        // results go out as they are made; the next layer's twiddles are requested ahead of the values they meet
                        const uint32_t ln = fresh(lane);
                        const uint32_t w = T + (ln >> 4) * 272u + (ln & 15u) * 16u;                              // b5 b4 / b3 b2 b1 b0
                        const uint32_t r = T + (ln >> 4) * 4352u + ((ln >> 2) & 3u) * 1088u + (ln & 3u) * 16u;   // b9 b8 / b7 b6 / b1 b0
                        const uint32_t tf = tab0 + z + FFT_F2_OFF * 16u + 16u * (ln >> 2);
                        d2 v[3], u[2][3];
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            fwd4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3], f1(3 + 3 * q), f1(4 + 3 * q), f1(5 + 3 * q));
                            FFT_FENCE();
#pragma unroll
                            for (int e = 4 * q; e < 4 * q + 4; e++) lds_put(w + 16 * (272 * (e >> 2) + 68 * (e & 3)), x[e]);
                        }
#pragma unroll
                        for (int t = 0; t < 3; t++) v[t] = lds_get(tf + 256 * t);
#pragma unroll
                        for (int i = 0; i < 4; i++)
#pragma unroll
                            for (int m = i; m < 16; m += 4) x[m] = lds_get(r + 16 * (17 * (m >> 2) + 4 * (m & 3)));
#pragma unroll
                        for (int t = 0; t < 3; t++) u[0][t] = lds_get(tf + 256 * (3 + t));
                        FFT_FENCE();
#pragma unroll
                        for (int i = 0; i < 4; i++) fwd4(x[i], x[i + 4], x[i + 8], x[i + 12], v[0], v[1], v[2]);
                        const uint32_t le = fresh(lane);
                        const uint32_t o = T + (le >> 4) * 4352u + (le & 15u) * 16u;                             // b9 b8 / b7 b6 b1 b0
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            FFT_FENCE();
                            if (q < 3) {
#pragma unroll
                                for (int t = 0; t < 3; t++) u[(q + 1) & 1][t] = lds_get(tf + 256 * (6 + 3 * q + t));
                            }
                            FFT_FENCE();
                            fwd4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3], u[q & 1][0], u[q & 1][1], u[q & 1][2]);
                            FFT_FENCE();
#pragma unroll
                            for (int i = 4 * q; i < 4 * q + 4; i++)
                                lds_put(o + 16 * 17 * (((i >> 3) & 1) * 8 + (i & 1) * 4 + ((i >> 2) & 1) * 2 + ((i >> 1) & 1)), x[i]);
                        }
                        if (SHARED) {
                            fft_signal(spectra_done + 4u * h, tick);
                        } else {
                            seq++;
                            fft_signal(my_done, seq);
                        }
                    }
                }
                d2 D[2][8];
                {
                    d2 f3[6];
                    const d2 *tabF3 = A.tab + FFT_F3_OFF + h * 384u + z;
#pragma unroll
                    for (int q = 0; q < 6; q++) f3[q] = lane_get(tabF3 + 64 * q, kl);
                    // key words of the first positions are requested one phase ahead of their use, here and at the end of every piece
                    if constexpr (!owner) {
                        kp += 2u * 4096u;                                 // the helper begins with piece 2
#pragma unroll
                        for (int k = 0; k < 8; k++) request(k);
                    } else {
#pragma unroll
                        for (int k = 0; k < FFT_EARLY; k++) request(k);
                    }
                    FFT_FENCE();
                    if (SHARED) {
                        fft_wait(spectra_done, fft_peek(spectra_done), tick);
                        fft_wait(spectra_done + 4u, fft_peek(spectra_done + 4u), tick);
                    } else {
                        fft_wait(his_done, fft_peek(his_done), seq);
                    }
                    const uint32_t lr = fresh(lane);                                                        // b8 b7 b6 b5 b4 b3
                    const uint32_t rd = (SHARED ? lds + own * FFT_BUF : Tp0) + z + h * 8704u + (lr >> 5) * 4352u + ((lr >> 2) & 1u) * 2176u + (lr & 3u) * 272u + ((lr >> 3) & 3u) * 64u;
#pragma unroll
                    for (int cc = 0; cc < 2; cc++)
#pragma unroll
                        for (int k = 0; k < 8; k++) D[cc][k] = lds_get(rd + cc * FFT_BUF + 16 * (68 * (k >> 2) + (k & 3)));
                    if (SHARED) fft_signal(spectra_read + 4u * (wave % (2u * SHARE)), tick);
                    else fft_signal(my_free, seq);
#pragma unroll
                    for (int cc = 0; cc < 2; cc++)
#pragma unroll
                        for (int b = 0; b < 2; b++) fwd4(D[cc][4 * b], D[cc][4 * b + 1], D[cc][4 * b + 2], D[cc][4 * b + 3], f3[3 * b], f3[3 * b + 1], f3[3 * b + 2]);
                }
                // ---- 3. key pieces ----
                // `early`: positions requested before the piece begins; `next`: the piece that this wave takes afterwards, or -1
                auto run_piece = [&](auto which, auto early, auto then) __attribute__((always_inline)) {
                    constexpr int piece = decltype(which)::value, ahead = decltype(early)::value, next = decltype(then)::value;
                    asm volatile("s_mov_b32 %0, 0" : "=s"(z));
                    T = T0 + z;
                    d2 S[2][8];
                    FFT_FENCE();
                    const uint32_t free_seen = fft_peek(his_free);
#pragma unroll
                    for (int k = 0; k < 8; k++) {
                        FFT_FENCE();
#pragma unroll
                        for (int n = (k ? k + FFT_RING - 1 : ahead); n < 8 && n < k + FFT_RING; n++)
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
                    // I1: half-sizes 1, 2, 4
                    const double r2 = FFT_SQRT_HALF;
                    inv8(S[0]);
#pragma unroll
                    for (int k = 0; k < 8; k++) pin(S[0][k]);
                    fft_wait(his_free, free_seen, seq);                  // the other wave has read the previous exchange
                    if (SHARED && piece == 0) {                            // the owner writes where all waves of the group read the spectra
#pragma unroll
                        for (uint32_t q = 0; q < 2 * SHARE; q++) fft_wait(spectra_read + 4u * q, fft_peek(spectra_read + 4u * q), tick);
                    }
                    {
                        const uint32_t ln = fresh(lane);                                                    // b8 b7 b6 b5 b4 b3
                        const uint32_t w = Tp0 + z + h * 8704u + (ln >> 5) * 4352u + (ln & 1u) * 2176u + ((ln >> 1) & 7u) * 272u + ((ln >> 4) & 1u) * 128u;
#pragma unroll
                        for (int k = 0; k < 8; k++) lds_put(w + 16 * k, S[0][k]);
                        inv8(S[1]);
#pragma unroll
                        for (int k = 0; k < 8; k++) lds_put(w + FFT_BUF + 16 * k, S[1][k]);
                    }
                    seq++;
                    fft_signal(my_done, seq);
                    // I2: half-sizes 8, 16, 32, 64; twiddles are requested ahead of the values they meet
                    const uint32_t t2 = tab0 + z + FFT_I2_OFF * 16u + 16u * (fresh(lane) & 7u);
                    const uint32_t t3 = tab0 + z + FFT_I3_OFF * 16u + 16u * fresh(lane);
                    {
                        const d2 w0 = lds_get(t2), w1 = lds_get(t2 + 128);
                        FFT_FENCE();
                        fft_wait(his_done, fft_peek(his_done), seq);
                        const uint32_t ln = fresh(lane);
                        const uint32_t r0 = T + (ln >> 4) * 4352u + (ln & 15u) * 16u;                       // b9 b8 / b7 b2 b1 b0
                        auto slot = [](int m) { return 16 * 17 * ((m & 1) * 8 + (m >> 1)); };                // register m = b6 b5 b4 b3
#pragma unroll
                        for (int m = 0; m < 16; m++) x[m] = lds_get(r0 + slot(m));
                        const d2 w2 = lds_get(t2 + 256), w3 = lds_get(t2 + 384);
                        FFT_FENCE();
#pragma unroll
                        for (int m = 0; m < 16; m += 2) inv2<false>(x[m], x[m + 1], w0);
                        FFT_FENCE();
#pragma unroll
                        for (int m = 0; m < 16; m += 4) { inv2<false>(x[m], x[m + 2], w1); inv2<true>(x[m + 1], x[m + 3], w1); }
                        FFT_FENCE();
                        const d2 w4 = lds_get(t2 + 512), w5 = lds_get(t2 + 640), w6 = lds_get(t2 + 768), w7 = lds_get(t2 + 896);
                        FFT_FENCE();
#pragma unroll
                        for (int m = 0; m < 16; m += 8) {
                            inv2<false>(x[m], x[m + 4], w2); inv2<true>(x[m + 2], x[m + 6], w2);
                            inv2<false>(x[m + 1], x[m + 5], w3); inv2<true>(x[m + 3], x[m + 7], w3);
                        }
                        // the last stage's results go out two butterflies at a time
                        auto put = [&](int m) { lds_put(r0 + slot(m), x[m]); };
                        FFT_FENCE();
                        inv2<false>(x[0], x[8], w4); inv2<true>(x[4], x[12], w4);
                        inv2<false>(x[1], x[9], w5); inv2<true>(x[5], x[13], w5);
                        FFT_FENCE();
                        put(0); put(8); put(4); put(12); put(1); put(9); put(5); put(13);
                        inv2<false>(x[2], x[10], w6); inv2<true>(x[6], x[14], w6);
                        inv2<false>(x[3], x[11], w7); inv2<true>(x[7], x[15], w7);
                        put(2); put(10); put(6); put(14); put(3); put(11); put(7); put(15);
                    }
                    // I3: half-sizes 128, 256, 512 with the twist
                    {
                        FFT_FENCE();
                        const d2 w0 = lds_get(t3);
                        const uint32_t ln = fresh(lane);                                                    // b5 b4 b3 b2 b1 b0
                        const uint32_t r0 = T + ((ln >> 3) & 1u) * 2176u + (ln >> 4) * 272u + (ln & 7u) * 16u;
#pragma unroll
                        for (int e = 0; e < 16; e += 4)
#pragma unroll
                            for (int q = 0; q < 4; q++) {
                                const int f = e + (q >> 1) + 2 * (q & 1);          // b9 b8 b7 b6, in the order of the butterflies below
                                x[f] = lds_get(r0 + 16 * (272 * (f >> 2) + 68 * (f & 1) + 8 * ((f >> 1) & 1)));
                            }
                        fft_signal(my_free, seq);
                        const d2 w1 = lds_get(t3 + 1024), w2 = lds_get(t3 + 2048);
                        FFT_FENCE();
#pragma unroll
                        for (int e = 0; e < 16; e += 4) { inv2<false>(x[e], x[e + 2], w0); inv2<true>(x[e + 1], x[e + 3], w0); }
                        FFT_FENCE();
                        kp += 4096u;
                        d2 c1[2], c2[2];
                        c1[0] = lds_get(t3 + 3072); c2[0] = lds_get(t3 + 4096);
                        FFT_FENCE();
#pragma unroll
                        for (int e = 0; e < 16; e += 8) {
                            inv2<false>(x[e], x[e + 4], w1); inv2<true>(x[e + 2], x[e + 6], w1);
                            inv2<false>(x[e + 1], x[e + 5], w2); inv2<true>(x[e + 3], x[e + 7], w2);
                        }
#pragma unroll
                        for (int e = 0; e < 8; e++) {
                            FFT_FENCE();
                            if (e + 1 < 8) { c1[(e + 1) & 1] = lds_get(t3 + 1024 * (5 + 2 * e)); c2[(e + 1) & 1] = lds_get(t3 + 1024 * (6 + 2 * e)); }
                            FFT_FENCE();
                            d2 a = cmul(x[e], c1[e & 1]), b = x[e + 8];
                            inv2<false>(a, b, c2[e & 1]);
                            // coefficients 64 e + lane (a) and 512 + 64 e + lane (b turned by -45 degrees), rounded
                            const uint64_t y0 = (uint64_t)__double_as_longlong(a.x + magic), y1 = (uint64_t)__double_as_longlong(a.y + magic);
                            const uint64_t y2 = (uint64_t)__double_as_longlong(__builtin_fma(b.x + b.y, r2, magic));
                            const uint64_t y3 = (uint64_t)__double_as_longlong(__builtin_fma(b.y - b.x, r2, magic));
                            add_shifted<SLZ_FFT_PIECE_BITS * piece>(accr[e], y0);
                            add_shifted<SLZ_FFT_PIECE_BITS * piece>(acci[e], y1);
                            add_shifted<SLZ_FFT_PIECE_BITS * piece>(accr[e + 8], y2);
                            add_shifted<SLZ_FFT_PIECE_BITS * piece>(acci[e + 8], y3);
                            if (piece == 0) {                            // the bits of `magic` that shift 0 has left
                                accr[e] -= 0x4338000000000000ull; acci[e] -= 0x4338000000000000ull;
                                accr[e + 8] -= 0x4338000000000000ull; acci[e + 8] -= 0x4338000000000000ull;
                            }
                            pin(accr[e]); pin(acci[e]); pin(accr[e + 8]); pin(acci[e + 8]);
                            if (!SHARED && next < 0) { stage(e); stage(e + 8); }
                            if (next >= 0) {
                                FFT_FENCE();
#pragma unroll
                                for (int q = 0; q < 2; q++)
                                    kb[e / 2][2 * (e & 1) + q] = lane_get(kp + (4 * (e / 2) + 2 * (e & 1) + q) * 64, kl);
                            }
                        }
                    }
                };
                fft_int<FFT_EARLY> first;
                fft_int<8> all;
                fft_int<-1> none;
                if constexpr (!SHARED) {
                    run_piece(fft_int<0>(), first, fft_int<1>());
                    run_piece(fft_int<1>(), first, fft_int<2>());
                    run_piece(fft_int<2>(), first, fft_int<3>());
                    run_piece(fft_int<3>(), first, fft_int<4>());
                    run_piece(fft_int<4>(), first, none);
                } else if constexpr (owner) {
                    run_piece(fft_int<0>(), first, fft_int<1>());
                    run_piece(fft_int<1>(), first, none);
                    const uint32_t flag = sums_done + 4u * (wave ^ 2u);
                    fft_wait(flag, fft_peek(flag), tick);
                    const LDS_AS uint64_t *S = (const LDS_AS uint64_t *)(uintptr_t)(lds + z + (wave ^ 2u) * FFT_BUF);
#pragma unroll
                    for (int e = 0; e < 16; e++) { accr[e] += S[64 * e + lane]; acci[e] += S[1024 + 64 * e + lane]; }
#pragma unroll
                    for (int e = 0; e < 16; e++) stage(e);
                } else {
#pragma unroll
                    for (int e = 0; e < 16; e++) accr[e] = acci[e] = 0;
                    run_piece(fft_int<2>(), all, fft_int<3>());
                    run_piece(fft_int<3>(), first, fft_int<4>());
                    run_piece(fft_int<4>(), first, none);
                    LDS_AS uint64_t *S = (LDS_AS uint64_t *)(uintptr_t)T;
#pragma unroll
                    for (int e = 0; e < 16; e++) { S[64 * e + lane] = accr[e]; S[1024 + 64 * e + lane] = acci[e]; }
                    fft_signal(sums_done + 4u * wave, tick);
                }
            }

            if constexpr (!owner) continue;
            const uint32_t lo = fresh(lane);
            if (A.acc_out) {
                uint64_t *dst = A.acc_out + ((size_t)c * 2 + h) * 2048u;
#pragma unroll
                for (int e = 0; e < 16; e++) { dst[64u * e + lo] = (uint64_t)0 - accr[e]; dst[1024u + 64u * e + lo] = (uint64_t)0 - acci[e]; }
            }
            if (A.lwe_out) {
                uint64_t *dst = A.lwe_out + (size_t)c * 2049u;
                if (h == 0) {
#pragma unroll
                    for (int e = 0; e < 16; e++) {
                        const uint32_t idx = 64u * e + lo;
                        if (idx == 0) dst[0] = (uint64_t)0 - accr[0];
                        else dst[2048u - idx] = accr[e];
                        dst[1024u - idx] = acci[e];
                    }
                } else if (lo == 0) {
                    dst[2048] = (uint64_t)0 - accr[0];
                }
            }
        }
    };
    if constexpr (!SHARED) rotate(fft_int<2>());
    else if ((pair & 1u) == group) rotate(fft_int<0>());
    else rotate(fft_int<1>());
}

// ---- host side ------------------------------------------------------------------------------------------------------

int slz_fft2048_setup() {
    const void *const kernels[] = {(const void *)k_fft_blind_rotate<1>, (const void *)k_fft_blind_rotate<2>};
    for (const void *k : kernels) SLZ_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, FFT_LDS_BYTES));
    if (slz_fft2048_pair_setup() != SLZ_OK) return SLZ_E_HIP;
    return slz_fft2048_team_setup();
}

int slz_fft2048_blind_rotate(slz_ctx *ctx, const uint64_t *lwe_in, const uint64_t *luts, const uint32_t *lut_idx, const void *key,
                             uint32_t n_steps, uint64_t *acc_out, uint64_t *lwe_out, uint32_t batch, hipStream_t s) {
    // Up to one ciphertext per compute unit its eight waves take one together (742 steps: one 7.2 ms against 8.5 with two pairs on it, 256
    // 8.3 against 8.6); from 257 on that needs a second round (301: 14.6 ms against 11.5).
    // Up to 128 ciphertexts two workgroups take each (6.4 to 6.6 us per step against 9.2 to 9.3 with one), unless an overlapping or captured call needs the
    // kernel without memory of its own.  To clear their words, to meet and the launch behind them cost 12 to 16 us: 4 steps take one workgroup / two 44 / 44 us
    // at 1 ciphertext and 46 / 53 at 128, 8 steps 80 / 70 and 82 / 80.
    if (slz_pairs_acquire(ctx, n_steps >= 8 && slz_pairs_fit(batch, s), s))
        return slz_pairs_release(ctx, slz_fft2048_pair(ctx, lwe_in, luts, lut_idx, key, n_steps, acc_out, lwe_out, batch, slz_pairs_grid(batch), SLZ_PAIR_PATIENCE, s), s);
    if (batch <= FFT_TEAM_MAX) return slz_fft2048_team(ctx, lwe_in, luts, lut_idx, key, n_steps, acc_out, lwe_out, batch, s);
    fft_args A;
    A.lwe_in = lwe_in; A.luts = luts; A.lut_idx = lut_idx; A.key = (const d2 *)key; A.tab = (const d2 *)ctx->fft_tab;
    A.acc_out = acc_out; A.lwe_out = lwe_out;
    A.n = ctx->prm.n; A.n_steps = n_steps; A.batch = batch; A.beta = ctx->prm.pbs_base_log;
    for (int q = 0; q < 15; q++)
        for (int t = 0; t < 2; t++) A.f1[q][t] = ctx->fft_f1[q][t];
    const uint32_t grid = slz_fused_grid(batch, 1);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(grid), dim3(FFT_THREADS), FFT_LDS_BYTES, s, A); };
    // From 257 to 512 ciphertexts two pairs share each: 301 11.5 ms against 12.9 with a pair for each (512: 12.2 and 13.1).
    if (batch <= 2 * FFT_TEAM_MAX) launch(k_fft_blind_rotate<2>);
    else launch(k_fft_blind_rotate<1>);
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

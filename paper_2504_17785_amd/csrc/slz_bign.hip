// Blind rotation for large polynomials, N = BS * G with block size BS = 1024 or 2048 and G in {2,4,8,16,32}, k = 1 (the
// 8-bit-precision-shaped parameter sets: N = 32768).  The accumulator (512 KiB per ciphertext at N = 32768) cannot stay
// on chip, so a CMux step is three passes over a per-ciphertext workspace that stays in L2 / Infinity Cache when
// ciphertexts are processed in chunks:
//   P1 "columns, forward":  per accumulator column c (coefficients BS i + c, i < G): rotate, subtract, decompose,
//                           then the first log2(G) transform stages (they pair coefficients BS rows apart, so a
//                           lane holding one column does them in registers), for every level and both primes.
//   P2 "rows":              per prime and block: the remaining forward stages with a wave-level transform (32 or 16
//                           coefficients per lane, block-specific twiddles), multiply-accumulate with the prepared
//                           key over all GGSW rows, the same number of inverse stages.
//   P3 "columns, inverse":  the last log2(G) inverse stages per column, the psi^-j / N twist, CRT lift, accumulate.
#include "slz_bign.h"
#include <vector>

#define BIG_MAX_L 4

// Stores of what the next launch reads, written through the L2: what is left dirty in the L2s is written back after the last workgroup of
// a launch, before the next one may start.
__device__ __forceinline__ void st_through(double *p, double v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_through(uint64_t *p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// ---- P1 ------------------------------------------------------------------------------------------
// BS: block size of the row pass (2048 or 1024); G = N / BS rows of BS columns
template <int G, int BS>
__global__ void __launch_bounds__(256)
k_big_cols_fwd(bign_args A) {
    const uint32_t c = blockIdx.x * 256 + threadIdx.x;          // column, < BS
    const uint32_t b = blockIdx.z;
    const uint32_t comp = blockIdx.y;
    const uint32_t N = A.N, R = 2 * A.l;
    uint32_t logN2 = 1;                                          // log2(2N)
    for (uint32_t g = N; g > 1; g >>= 1) logN2++;
    const uint32_t at = slz_modswitch(A.lwe_in[(size_t)b * (A.n + 1) + A.step], logN2);
    const uint64_t *poly = A.acc + ((size_t)b * 2 + comp) * N;
    uint64_t lam[G];
#pragma unroll
    for (int i = 0; i < G; i++) {
        const uint32_t idx = (uint32_t)BS * i + c;
        lam[i] = slz_rot_coeff([&](uint32_t j) { return poly[j]; }, idx, at, N) - poly[idx];
        lam[i] = slz_round_top_bits(lam[i], A.beta * A.l);
    }
    for (int lev = (int)A.l - 1; lev >= 0; lev--) {              // least significant level first (carries go up)
        double d[G];
#pragma unroll
        for (int i = 0; i < G; i++) d[i] = (double)slz_next_digit(lam[i], A.beta);
        for (int q = 0; q < 2; q++) {
            const slz_mod m = A.mod[q];
            const double *tw = A.tab[q].fwd;
            double y[G];
#pragma unroll
            for (int i = 0; i < G; i++) y[i] = d[i];
            // as cols_fwd, written out: with the call the compiler orders the stages' instructions differently, N = 32768, 256 ciphertexts 506.7 to
            // 507.9 us per step against 504.3 to 507.0, 64: 127.2 to 128.3 against 127.0 to 128.0
#pragma unroll
            for (int half = G / 2, blocks = 1; half >= 1; half >>= 1, blocks <<= 1) {
#pragma unroll
                for (int blk = 0; blk < blocks; blk++) {
                    const double w = tw[blocks + blk];
#pragma unroll
                    for (int j = 0; j < half; j++) bfly(y[blk * 2 * half + j], y[blk * 2 * half + j + half], w, m);
                }
            }
            double *dst = A.X + (((size_t)b * 2 + q) * R + (comp * A.l + lev)) * N + c;
#pragma unroll
            for (int i = 0; i < G; i++) dst[(uint32_t)BS * i] = slz_reduce(y[i], m);
        }
    }
}

// ---- P2 ------------------------------------------------------------------------------------------
// one wave per (ciphertext, prime, 2048-block); four independent waves per workgroup
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_big_rows(bign_args A, uint32_t G, uint32_t n_tasks, int xcd_aware) {
    extern __shared__ double lds[];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Workgroups are dealt round-robin to the 8 XCDs, each with its own 4 MiB L2, and one step's key is as large as
    // one L2.  With xcd_aware the 2G (prime, block) combinations are split between the XCDs, so that an XCD only
    // touches its 1/8 of the key and re-reads it from its L2 for every ciphertext of the chunk.
    uint32_t task = blockIdx.x * 4 + wv;
    if (xcd_aware) {
        const uint32_t cpx = 2 * G / 8;                          // combinations per XCD
        const uint32_t xcd = blockIdx.x & 7u, v = (blockIdx.x >> 3) * 4 + wv;
        task = (v / cpx) * 2 * G + xcd * cpx + v % cpx;
    }
    if (task >= n_tasks) return;                                 // whole wave leaves; no workgroup barriers below
    double *T = lds + wv * TBUF;
    const uint32_t row = task % G, q = (task / G) & 1u, b = task / (2 * G);
    const uint32_t N = A.N, R = 2 * A.l, hh = lane >> 5;
    const slz_mod m = A.mod[q];
    const bign_tabs tb = A.tab[q];
    const double *twA = tb.rowA + (size_t)row * 64, *fwd6 = twA + 32, *fwdB = tb.rowB + (size_t)row * 31 * 64;
    double o0[32], o1[32];
    for (uint32_t r = 0; r < R; r++) {
        int z;
        asm volatile("s_mov_b32 %0, 0" : "=s"(z));              // tables are reloaded per GGSW row (they would spill if hoisted)
        double tw6[16];
#pragma unroll
        for (int mm = 0; mm < 16; mm++) tw6[mm] = ldl(fwd6 + 2 * mm + z, hh * 8u);
        const double *src = A.X + (((size_t)b * 2 + q) * R + r) * N + 2048u * row + z;
        double x[32];
#pragma unroll
        for (int e = 0; e < 32; e++) x[e] = ldl(src + 64 * e, lane * 8u);
        fused_fwd(x, T, tw6, twA, fwdB, m, lane, z);
        // multiply-accumulate with the key polynomials of GGSW row r (both components); spectrum index of x[i] is 2048 row + 32 lane + i:
        // the words of x[i], x[i + 1], x[i + 16] and x[i + 17] are consecutive in the prepared polynomial for even i (slz_prep_pos)
        const double *k0 = A.bskp_step + (((size_t)q * R + r) * 2 + 0) * N + 2048u * row + z;
        const double *k1 = k0 + N;
        const uint32_t key_lane = hh * 1024u + (lane & 31u) * 4u;
#pragma unroll
        for (int g = 0; g < 8; g++) {
            double2 ka[2], kb[2];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                ka[h] = *reinterpret_cast<const double2 *>(k0 + 128 * g + 2 * h + key_lane);
                kb[h] = *reinterpret_cast<const double2 *>(k1 + 128 * g + 2 * h + key_lane);
            }
            const int at[4] = {2 * g, 2 * g + 1, 2 * g + 16, 2 * g + 17};
            const double kk0[4] = {ka[0].x, ka[0].y, ka[1].x, ka[1].y}, kk1[4] = {kb[0].x, kb[0].y, kb[1].x, kb[1].y};
            const double x4[4] = {x[at[0]], x[at[1]], x[at[2]], x[at[3]]};
            double r0[4], r1[4];
            mulmod_k<4>(r0, x4, kk0, m);
            mulmod_k<4>(r1, x4, kk1, m);
#pragma unroll
            for (int u = 0; u < 4; u++) {
                o0[at[u]] = (r == 0) ? r0[u] : o0[at[u]] + r0[u];
                o1[at[u]] = (r == 0) ? r1[u] : o1[at[u]] + r1[u];
            }
        }
        if ((r & 3u) == 3u && r + 1 < R) {                       // more than four rows: keep the running sums below 8 p
#pragma unroll
            for (int g = 0; g < 8; g++) {
                double a4[4], b4[4];
                const double xa[4] = {o0[4 * g], o0[4 * g + 1], o0[4 * g + 2], o0[4 * g + 3]};
                const double xb[4] = {o1[4 * g], o1[4 * g + 1], o1[4 * g + 2], o1[4 * g + 3]};
                reduce_k<4>(a4, xa, m);
                reduce_k<4>(b4, xb, m);
#pragma unroll
                for (int u = 0; u < 4; u++) { o0[4 * g + u] = a4[u]; o1[4 * g + u] = b4[u]; }
            }
        }
        wave_sync();
    }
    // inverse: first 11 stages inside the block, reduce, hand the block to the column pass
    for (int comp = 0; comp < 2; comp++) {
        int z;
        asm volatile("s_mov_b32 %0, 0" : "=s"(z));
        double x[32];
#pragma unroll
        for (int g = 0; g < 4; g++) {
            double r8[8], x8[8];
#pragma unroll
            for (int u = 0; u < 8; u++) x8[u] = comp ? o1[8 * g + u] : o0[8 * g + u];
            reduce_k<8>(r8, x8, m);
#pragma unroll
            for (int u = 0; u < 8; u++) x[8 * g + u] = r8[u];
        }
        fused_inv(x, T, tb.inv, tb.inv, m, lane, z);
        double *dst = A.Y + (((size_t)b * 2 + q) * 2 + comp) * N + 2048u * row;
#pragma unroll
        for (int g = 0; g < 4; g++) {
            double r8[8], x8[8];
#pragma unroll
            for (int u = 0; u < 8; u++) x8[u] = x[8 * g + u];
            reduce_k<8>(r8, x8, m);
#pragma unroll
            for (int u = 0; u < 8; u++) dst[64 * (8 * g + u) + lane] = r8[u];
        }
        wave_sync();
    }
}

// ---- P2 with 1024-blocks -------------------------------------------------------------------------
// One wave per (ciphertext, prime, 1024-block), 16 coefficients per lane: the accumulators of both components, the block
// and the tables fit 256 registers, so two waves share a SIMD and cover each other's memory latency (the 2048-block
// kernel above needs more than 256 and runs one wave per SIMD, 43 % of it waiting for memory).
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_big_rows16(bign_args A, uint32_t G, uint32_t n_tasks, int xcd_aware) {
    extern __shared__ double lds[];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t task = blockIdx.x * 4 + wv;
    if (xcd_aware) {                                             // as above: an XCD keeps to its 1/8 of the (prime, block) pairs
        const uint32_t cpx = 2 * G / 8;
        const uint32_t xcd = blockIdx.x & 7u, v = (blockIdx.x >> 3) * 4 + wv;
        task = (v / cpx) * 2 * G + xcd * cpx + v % cpx;
    }
    if (task >= n_tasks) return;                                 // whole wave leaves; no workgroup barriers below
    double *T = lds + wv * (TBUF16 + 1024u);
    double *twA = T + TBUF16, *twB = twA + 64;                  // this block's forward tables, staged in LDS
    const uint32_t row = task % G, q = (task / G) & 1u, b = task / (2 * G);
    const uint32_t N = A.N, R = 2 * A.l;
    const slz_mod m = A.mod[q];
    const bign_tabs tb = A.tab[q];
    {
        const double *gA = tb.rowA + (size_t)row * 64, *gB = tb.rowB + (size_t)row * 15 * 64;
        twA[lane] = gA[lane];
#pragma unroll
        for (int k = 0; k < 15; k++) twB[64 * k + lane] = gB[64 * k + lane];
        wave_sync();
    }
    // spectrum index of x[i] is 1024 row + 16 lane + i, stored in pairs of registers, lane-minor, from position 1024 row of the prepared polynomial on
    double o0[16], o1[16];
    double xn[16];                                               // the next GGSW row's block, requested one row ahead
    {
        const double *src = A.X + (((size_t)b * 2 + q) * R + 0) * N + 1024u * row;
#pragma unroll
        for (int e = 0; e < 16; e++) xn[e] = ldl(src + 64 * e, lane * 8u);
    }
    for (uint32_t r = 0; r < R; r++) {
        int z;
        asm volatile("s_mov_b32 %0, 0" : "=s"(z));              // tables are reloaded per GGSW row (they would spill if hoisted)
        double x[16];
#pragma unroll
        for (int e = 0; e < 16; e++) x[e] = xn[e];
        // the key words of this row and then the next row's block are requested here (vector memory completes in issue
        // order) and arrive while the transform runs
        const double *k0 = A.bskp_step + (((size_t)q * R + r) * 2 + 0) * N + 1024u * row + z;
        const double *k1 = k0 + N;
        double kk0[16], kk1[16];
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const double2 a = ldl2(k0 + 64 * i, lane * 16u), b = ldl2(k1 + 64 * i, lane * 16u);
            kk0[i] = a.x; kk0[i + 1] = a.y;
            kk1[i] = b.x; kk1[i + 1] = b.y;
        }
        {
            const double *nxt = A.X + (((size_t)b * 2 + q) * R + (r + 1 < R ? r + 1 : r)) * N + 1024u * row + z;
#pragma unroll
            for (int e = 0; e < 16; e++) xn[e] = ldl(nxt + 64 * e, lane * 8u);
        }
        SCHED_FENCE();
        fwd16(x, T, twA, twB, m, lane, z);
        SCHED_FENCE();
#pragma unroll
        for (int g = 0; g < 4; g++) {
            double r0[4], r1[4];
            const double x4[4] = {x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
            const double ka[4] = {kk0[4 * g], kk0[4 * g + 1], kk0[4 * g + 2], kk0[4 * g + 3]};
            mulmod_k<4>(r0, x4, ka, m);
            const double kb[4] = {kk1[4 * g], kk1[4 * g + 1], kk1[4 * g + 2], kk1[4 * g + 3]};
            mulmod_k<4>(r1, x4, kb, m);
#pragma unroll
            for (int u = 0; u < 4; u++) {
                o0[4 * g + u] = (r == 0) ? r0[u] : o0[4 * g + u] + r0[u];
                o1[4 * g + u] = (r == 0) ? r1[u] : o1[4 * g + u] + r1[u];
            }
        }
        if ((r & 3u) == 3u && r + 1 < R) {                       // more than four rows: keep the running sums below 8 p
#pragma unroll
            for (int g = 0; g < 4; g++) {
                double a4[4], b4[4];
                const double xa[4] = {o0[4 * g], o0[4 * g + 1], o0[4 * g + 2], o0[4 * g + 3]};
                const double xb[4] = {o1[4 * g], o1[4 * g + 1], o1[4 * g + 2], o1[4 * g + 3]};
                reduce_k<4>(a4, xa, m);
                reduce_k<4>(b4, xb, m);
#pragma unroll
                for (int u = 0; u < 4; u++) { o0[4 * g + u] = a4[u]; o1[4 * g + u] = b4[u]; }
            }
        }
        wave_sync();
    }
    // inverse: first 10 stages inside the block, reduce, hand the block to the column pass
    for (int comp = 0; comp < 2; comp++) {
        int z;
        asm volatile("s_mov_b32 %0, 0" : "=s"(z));
        double x[16];
#pragma unroll
        for (int g = 0; g < 2; g++) {
            double r8[8], x8[8];
#pragma unroll
            for (int u = 0; u < 8; u++) x8[u] = comp ? o1[8 * g + u] : o0[8 * g + u];
            reduce_k<8>(r8, x8, m);
#pragma unroll
            for (int u = 0; u < 8; u++) x[8 * g + u] = r8[u];
        }
        inv16(x, T, tb.inv, tb.inv, m, lane, z);
        double *dst = A.Y + (((size_t)b * 2 + q) * 2 + comp) * N + 1024u * row;
#pragma unroll
        for (int g = 0; g < 2; g++) {
            double r8[8], x8[8];
#pragma unroll
            for (int u = 0; u < 8; u++) x8[u] = x[8 * g + u];
            reduce_k<8>(r8, x8, m);
#pragma unroll
            for (int u = 0; u < 8; u++) dst[64 * (8 * g + u) + lane] = r8[u];
        }
        wave_sync();
    }
}

// ---- P3 ------------------------------------------------------------------------------------------
template <int G, int BS>
__global__ void __launch_bounds__(256)
k_big_cols_inv(bign_args A) {
    const uint32_t c = blockIdx.x * 256 + threadIdx.x;
    const uint32_t comp = blockIdx.y, b = blockIdx.z;
    const uint32_t N = A.N;
    double res[2][G];
    for (int q = 0; q < 2; q++) {
        const slz_mod m = A.mod[q];
        const double *src = A.Y + (((size_t)b * 2 + q) * 2 + comp) * N + c;
        const double *tw = A.tab[q].inv, *post = A.tab[q].post;
        double y[G];
#pragma unroll
        for (int i = 0; i < G; i++) y[i] = src[(uint32_t)BS * i];
        // stages with half-size t = BS * half: pairs of rows i, i + half; twiddle inv[t + BS (i mod half) + c]
#pragma unroll
        for (int half = 1; half < G; half <<= 1) {
#pragma unroll
            for (int j = 0; j < half; j++) {
                const double w = tw[(uint32_t)BS * half + (uint32_t)BS * j + c];
#pragma unroll
                for (int blk = 0; blk < G / (2 * half); blk++) bfly(y[blk * 2 * half + j], y[blk * 2 * half + j + half], w, m);
            }
        }
#pragma unroll
        for (int i = 0; i < G; i++) res[q][i] = slz_mulmod(y[i], post[(uint32_t)BS * i + c], m);
    }
    uint64_t *poly = A.acc + ((size_t)b * 2 + comp) * N + c;
#pragma unroll
    for (int i = 0; i < G; i++) poly[(uint32_t)BS * i] += slz_crt64(res[0][i], res[1][i], A.mod[1], A.p1inv_mod_p2);
}

// both residues of column c of one component after the mirrored inverse
template <int G>
__device__ __forceinline__ void cols_mirror_both(double (&res)[2][G], const bign_args &A, uint32_t b, uint32_t comp, uint32_t c) {
#pragma unroll
    for (int q = 0; q < 2; q++) {
        const slz_mod m = A.mod[q];
        const double *src = A.Y + (((size_t)b * 2 + q) * 2 + comp) * A.N + c;
        double lo[G / 2], hi[G / 2], ba[G / 2], bb[G / 2];
#pragma unroll
        for (int i = 0; i < G / 2; i++) { lo[i] = src[1024u * i]; hi[i] = src[1024u * (G / 2 + i)]; ba[i] = bb[i] = 0.51; }
        cols_mirror<G / 2>(lo, ba, colI_of(A.tab[q], G), 0, 2, m);
        cols_mirror<G / 2>(hi, bb, colI_of(A.tab[q], G), 1, 2, m);
        lazy_limit(lo, ba, LAZY_MAX / 2, m);
        lazy_limit(hi, bb, LAZY_MAX / 2, m);
#pragma unroll
        for (int i = 0; i < G / 2; i++) {
            cols_mirror_last(lo[i], hi[i], colI_of(A.tab[q], G), m);
            res[q][i] = lo[i];
            res[q][G / 2 + i] = hi[i];
        }
    }
}

// The last column pass of the two-launch steps; acc_in: the accumulator before it (A.acc or the other buffer).
template <int G>
__global__ void __launch_bounds__(256)
k_big_cols_last(bign_args A, const uint64_t *acc_in) {
    const uint32_t c = blockIdx.x * 256 + threadIdx.x;
    const uint32_t comp = blockIdx.y, b = blockIdx.z;
    double res[2][G];
    cols_mirror_both<G>(res, A, b, comp, c);
    const size_t poly = ((size_t)b * 2 + comp) * A.N + c;
#pragma unroll
    for (int i = 0; i < G; i++) A.acc[poly + 1024u * i] = acc_in[poly + 1024u * i] + slz_crt64(res[0][i], res[1][i], A.mod[1], A.p1inv_mod_p2);
}

// k_big_cols_turn (below) for few rows: a thread does a whole column and the rotated one.
template <int G>
__global__ void __launch_bounds__(256)
k_big_cols_turn_short(bign_args A, const uint64_t *__restrict__ acc_in, uint64_t *__restrict__ acc_out) {
    const uint32_t c = blockIdx.x * 256 + threadIdx.x;
    const uint32_t comp = blockIdx.y, b = blockIdx.z;
    const uint32_t N = A.N, R = 2 * A.l;
    uint32_t logN2 = 1;                                          // log2(2N)
    for (uint32_t g = N; g > 1; g >>= 1) logN2++;
    const uint32_t at = slz_modswitch(A.lwe_in[(size_t)b * (A.n + 1) + A.step], logN2);
    const uint32_t u = c + 2 * N - at, urow = u >> 10;           // X^at moves coefficient u (mod 2N, negated from N on) to c
    const size_t poly = ((size_t)b * 2 + comp) * N;
    uint64_t own[G], other[G];
#pragma unroll
    for (int i = 0; i < G; i++) { own[i] = acc_in[poly + c + 1024u * i]; other[i] = acc_in[poly + (u & 1023u) + 1024u * i]; }
    {
        double res[2][G];
        cols_mirror_both<G>(res, A, b, comp, c);
#pragma unroll
        for (int i = 0; i < G; i++) own[i] += slz_crt64(res[0][i], res[1][i], A.mod[1], A.p1inv_mod_p2);
        cols_mirror_both<G>(res, A, b, comp, u & 1023u);
#pragma unroll
        for (int i = 0; i < G; i++) other[i] += slz_crt64(res[0][i], res[1][i], A.mod[1], A.p1inv_mod_p2);
    }
    uint64_t lam[G];
#pragma unroll
    for (int i = 0; i < G; i++) {
        const uint32_t from = (urow + i) & (2 * G - 1);
        uint64_t w = other[0];
#pragma unroll
        for (int k = 1; k < G; k++) w = (from & (G - 1)) == (uint32_t)k ? other[k] : w;
        lam[i] = slz_round_top_bits((from & G ? (uint64_t)0 - w : w) - own[i], A.beta * A.l);
        acc_out[poly + c + 1024u * i] = own[i];
    }
    for (int lev = (int)A.l - 1; lev >= 0; lev--) {              // least significant level first (carries go up)
        double d[G];
#pragma unroll
        for (int i = 0; i < G; i++) d[i] = (double)slz_next_digit(lam[i], A.beta);
#pragma unroll
        for (int q = 0; q < 2; q++) {
            double y[G];
#pragma unroll
            for (int i = 0; i < G; i++) y[i] = d[i];
            cols_fwd<G>(y, A.tab[q].fwd, A.mod[q]);
            double *dst = A.X + (((size_t)b * 2 + q) * R + (comp * A.l + lev)) * N + c;
#pragma unroll
            for (int i = 0; i < G; i++) dst[1024u * i] = slz_reduce(y[i], A.mod[q]);
        }
    }
}

// ---- few ciphertexts: the same step as two launches of more, shorter threads -----------------------------------------
// With few ciphertexts the chip is mostly empty and a step costs the latency of its longest thread and the hand-over between
// dependent launches.  The row pass gives every GGSW row a wave of its own (k_big_rows16_team); the inverse column pass of a step
// and the forward column pass of the next one are one launch (k_big_cols_turn).

// One workgroup of R waves per (ciphertext, prime, 1024-block): wave r transforms GGSW row r and multiplies it with the row's key
// columns; pairs of waves exchange their products through LDS (even waves sum component 0, odd ones component 1), and waves 0 and 1
// collect the sums of the other pairs and run the inverse transforms.  LDS: R transform buffers, which also take the products, and the
// block's forward tables: 45 KiB for four rows, three workgroups per compute unit.
#define TEAM_LDS(R) (((R) * TBUF16 + 1024u) * sizeof(double))
template <int R>
__global__ void __launch_bounds__(64 * R) __attribute__((amdgpu_waves_per_eu(3, 3)))
k_big_rows16_team(bign_args A, uint32_t G) {
    extern __shared__ double lds[];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t task = blockIdx.x;                                  // (ciphertext, prime, block), block fastest
    if (2 * G % 8 == 0) {                                        // an XCD keeps to its 1/8 of the (prime, block) pairs, see k_big_rows
        const uint32_t cpx = 2 * G / 8, xcd = blockIdx.x & 7u, v = blockIdx.x >> 3;
        task = (v / cpx) * 2 * G + xcd * cpx + v % cpx;
    }
    const uint32_t row = task % G, q = (task / G) & 1u, b = task / (2 * G);
    double *T = lds + r * TBUF16, *T_other = lds + (r ^ 1u) * TBUF16;
    double *twA = lds + R * TBUF16, *twB = twA + 64;
    const uint32_t N = A.N;
    const slz_mod m = A.mod[q];
    const bign_tabs tb = A.tab[q];
    int z;
    asm volatile("s_mov_b32 %0, 0" : "=s"(z));
    double x[16], kk[2][16];
    {
        constexpr uint32_t TAB = (1024 + 64 * R - 1) / (64 * R);
        const double *gA = tb.rowA + (size_t)row * 64, *gB = tb.rowB + (size_t)row * 15 * 64;
        double tab[TAB];
#pragma unroll
        for (uint32_t i = 0; i < TAB; i++) {
            const uint32_t t = min(i * 64 * R + threadIdx.x, 1023u);
            tab[i] = t < 64u ? gA[t] : gB[t - 64u];
        }
        const double *src = A.X + (((size_t)b * 2 + q) * R + r) * N + 1024u * row;
#pragma unroll
        for (int e = 0; e < 16; e++) x[e] = ldl(src + 64 * e, lane * 8u);
        const double *key = A.bskp_step + (((size_t)q * R + r) * 2) * N + 1024u * row;
#pragma unroll
        for (int i = 0; i < 16; i += 2)
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const double2 w = ldl2(key + (size_t)c * N + 64 * i, lane * 16u);
                kk[c][i] = w.x;
                kk[c][i + 1] = w.y;
            }
#pragma unroll
        for (uint32_t i = 0; i < TAB; i++) if (i * 64 * R + threadIdx.x < 1024u) twA[i * 64 * R + threadIdx.x] = tab[i];
    }
    __syncthreads();
    SCHED_FENCE();
    fwd16(x, T, twA, twB, m, lane, z);
    wave_sync();
    double o[16];                                                // the component this wave sums: r & 1
#pragma unroll
    for (int g = 0; g < 2; g++) {
        double r0[8], r1[8], x8[8], k0[8], k1[8];
#pragma unroll
        for (int u = 0; u < 8; u++) { x8[u] = x[8 * g + u]; k0[u] = kk[0][8 * g + u]; k1[u] = kk[1][8 * g + u]; }
        mulmod_k<8>(r0, x8, k0, m);
        mulmod_k<8>(r1, x8, k1, m);
#pragma unroll
        for (int u = 0; u < 8; u++) {
            o[8 * g + u] = r & 1u ? r1[u] : r0[u];
            T[64 * (8 * g + u) + lane] = r & 1u ? r0[u] : r1[u];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; i++) o[i] += T_other[64 * i + lane];
    if (R > 2) {
        if (r >= 2) {
#pragma unroll
            for (int i = 0; i < 16; i++) T_other[64 * i + lane] = o[i];         // read by this wave alone before
        }
        __syncthreads();
        if (r >= 2) return;
#pragma unroll
        for (int w = 2; w < R; w += 2) {
            const double *P = lds + (w + (r ^ 1u)) * TBUF16;
#pragma unroll
            for (int i = 0; i < 16; i++) o[i] += P[64 * i + lane];
            if (w == 2 && R > 4) {                                              // at most four products are summed before a reduction
#pragma unroll
                for (int i = 0; i < 16; i++) o[i] = slz_reduce(o[i], m);
            }
        }
    }
    double twi[15];
    const double *gBi = rowBi_of(tb, G) + (size_t)row * 15 * 64;
#pragma unroll
    for (int k = 0; k < 15; k++) twi[k] = ldl(gBi + 64 * k, lane * 8u);
#pragma unroll
    for (int g = 0; g < 2; g++) {
        double r8[8], x8[8];
#pragma unroll
        for (int u = 0; u < 8; u++) x8[u] = o[8 * g + u];
        reduce_k<8>(r8, x8, m);
#pragma unroll
        for (int u = 0; u < 8; u++) o[8 * g + u] = r8[u];
    }
    inv16_mirror(o, T_other, rowAi_of(tb, G) + (size_t)row * 64, twi, m, lane, z);     // this buffer has no other reader any more
    double *dst = A.Y + (((size_t)b * 2 + q) * 2 + r) * N + 1024u * row;
#pragma unroll
    for (int g = 0; g < 2; g++) {
        double r8[8], x8[8];
#pragma unroll
        for (int u = 0; u < 8; u++) x8[u] = o[8 * g + u];
        reduce_k<8>(r8, x8, m);
#pragma unroll
        for (int u = 0; u < 8; u++) st_through(&dst[64 * (8 * g + u) + lane], r8[u]);
    }
}

// Inverse column pass of step A.step - 1 and forward column pass of step A.step for 64 columns of one component.  The forward pass of
// column c needs the new accumulator in columns c and c - a~ (mod 1024), so both are computed (every column twice, which costs less
// than a hand-over between launches).  Eight waves share the work, meeting in LDS: (own or rotated column, prime, half of the rows)
// run the inverse stages inside a half; each then takes a quarter of the row pairs for the last stage, the twist and the lift; an eighth
// of the rows for the differences; and (level, prime, half of the rows) run the forward stages.  Other workgroups read the old
// accumulator, so the new one goes to a second buffer.
template <int G>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4)))
k_big_cols_turn(bign_args A, const uint64_t *__restrict__ acc_in, uint64_t *__restrict__ acc_out) {
    constexpr int H = G / 2, J = H / 4, D = G / 8;
    __shared__ double res[4 * G * 64];                           // [own, rotated][prime][row][column]
    uint64_t *words = reinterpret_cast<uint64_t *>(res);         // afterwards [own, rotated][row][column] ...
    uint64_t *diff = words + 2 * G * 64;                         // ... and [row][column]
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t pairs = 2 * A.batch;
    // (ciphertext, component) and block of columns: with eight pairs and more an XCD keeps to its pairs, so that both readings of a
    // column meet in one L2
    uint32_t pair, x;
    if (pairs >= 8) { pair = (blockIdx.x & 7u) + 8u * (blockIdx.x >> 7); x = (blockIdx.x >> 3) & 15u; }
    else { pair = blockIdx.x >> 4; x = blockIdx.x & 15u; }
    if (pair >= pairs) return;
    const uint32_t comp = pair & 1u, b = pair >> 1, c = 64 * x + lane;
    const uint32_t N = A.N, R = 2 * A.l;
    uint32_t logN2 = 1;                                          // log2(2N)
    for (uint32_t g = N; g > 1; g >>= 1) logN2++;
    const uint32_t at = slz_modswitch(A.lwe_in[(size_t)b * (A.n + 1) + A.step], logN2);
    const uint32_t u = c + 2 * N - at;                           // X^at moves coefficient u (mod 2N, negated from N on) to c
    const uint32_t rot = wave >> 2, col = rot ? u & 1023u : c, urow = u >> 10;
    const size_t poly = (size_t)pair * N;
    const uint32_t j0 = (wave & 3u) * J;                         // this wave's row pairs (j, j + H) of the lift
    uint64_t lo[J], hi[J];
    {
        const uint32_t q = (wave >> 1) & 1u, part = wave & 1u;
        const slz_mod m = A.mod[q];
        double y[H], bd[H];
        const double *src = A.Y + (((size_t)b * 2 + q) * 2 + comp) * N + 1024u * part * H + col;
#pragma unroll
        for (int i = 0; i < H; i++) { y[i] = src[1024u * i]; bd[i] = 0.51; }
        cols_mirror<H>(y, bd, colI_of(A.tab[q], G), part, 2, m);
        lazy_limit(y, bd, LAZY_MAX / 2, m);
#pragma unroll
        for (int i = 0; i < H; i++) res[((rot * 2 + q) * G + part * H + i) * 64 + lane] = y[i];
#pragma unroll
        for (int k = 0; k < J; k++) {
            lo[k] = acc_in[poly + col + 1024u * (j0 + k)];
            hi[k] = acc_in[poly + col + 1024u * (H + j0 + k)];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < J; k++) {
        double r[2][2];
#pragma unroll
        for (int p = 0; p < 2; p++) {
            r[0][p] = res[((rot * 2 + p) * G + j0 + k) * 64 + lane];
            r[1][p] = res[((rot * 2 + p) * G + H + j0 + k) * 64 + lane];
            cols_mirror_last(r[0][p], r[1][p], colI_of(A.tab[p], G), A.mod[p]);
        }
        lo[k] += slz_crt64(r[0][0], r[0][1], A.mod[1], A.p1inv_mod_p2);
        hi[k] += slz_crt64(r[1][0], r[1][1], A.mod[1], A.p1inv_mod_p2);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < J; k++) {
        words[(rot * G + j0 + k) * 64 + lane] = lo[k];
        words[(rot * G + H + j0 + k) * 64 + lane] = hi[k];
        if (!rot) {
            st_through(&acc_out[poly + c + 1024u * (j0 + k)], lo[k]);
            st_through(&acc_out[poly + c + 1024u * (H + j0 + k)], hi[k]);
        }
    }
    __syncthreads();
    // Differences, rounded to beta l bits, plus half a base in every digit: the digit of a level is then a bit field minus half a base.
    uint64_t offset = 0;
    for (uint32_t k = 0; k < A.l; k++) offset += 1ull << (A.beta * k + A.beta - 1);
#pragma unroll
    for (int k = 0; k < D; k++) {
        const uint32_t i = wave * D + k, from = (urow + i) & (2 * G - 1);
        const uint64_t w = words[(G + (from & (G - 1))) * 64 + lane];
        diff[i * 64 + lane] = slz_round_top_bits((from & G ? (uint64_t)0 - w : w) - words[i * 64 + lane], A.beta * A.l) + offset;
    }
    __syncthreads();
    const uint32_t mask = (1u << A.beta) - 1u, mid = 1u << (A.beta - 1);
    for (uint32_t t = wave; t < 4 * A.l; t += 8) {
        const uint32_t half = t & 1u, q = (t >> 1) & 1u, lev = t >> 2, shift = A.beta * (A.l - 1 - lev);
        const slz_mod m = A.mod[q];
        const double *tw = A.tab[q].fwd;
        auto digit = [&](int i) { return (double)(int32_t)(((uint32_t)(diff[i * 64 + lane] >> shift) & mask) - mid); };
        double y[H];
#pragma unroll
        for (int j = 0; j < H; j++) {
            const double a = digit(j), v = slz_mulmod(digit(j + H), tw[1], m);
            y[j] = half ? a - v : a + v;
        }
#pragma unroll
        for (int d = H / 2, blocks = 1; d >= 1; d >>= 1, blocks <<= 1) {
#pragma unroll
            for (int blk = 0; blk < blocks; blk++) {
                const double w = tw[2 * blocks + half * blocks + blk];
#pragma unroll
                for (int j = 0; j < d; j++) bfly(y[blk * 2 * d + j], y[blk * 2 * d + j + d], w, m);
            }
        }
        double *dst = A.X + (((size_t)b * 2 + q) * R + (comp * A.l + lev)) * N + 1024u * half * H + c;
#pragma unroll
        for (int i = 0; i < H; i++) st_through(&dst[1024u * i], slz_reduce(y[i], m));
    }
}

// ---- host ------------------------------------------------------------------------------------------

int slz_bign_supported(const slz_params *p) {
    if (p->k != 1 || p->pbs_level > BIG_MAX_L) return 0;
    for (uint32_t G = 2; G <= 32; G <<= 1)
        if (p->N == 2048u * G || p->N == 1024u * G) return 1;
    return 0;
}

static bool block_fits(uint32_t N, uint32_t BS) {
    const uint32_t G = N / BS;
    return N % BS == 0 && G >= 2 && G <= 32 && (G & (G - 1)) == 0;
}

// Block-specific forward tables of one prime for blocks of BS = 64 * E coefficients (E = 32 or 16 per lane), ra [G][64] and
// rb [G][E - 1][64], or with `inverse` the inverses of their entries: fwd[x] = psi^bitrev(x), so 1 / fwd[x] = -psi^(N - bitrev(x)).
static double inverse_entry(const std::vector<double> &nat, uint32_t x) {
    const uint32_t N = (uint32_t)nat.size();
    auto bitrev = [&](uint32_t v) {
        uint32_t r = 0;
        for (uint32_t h = N >> 1, b = 1; h; h >>= 1, b <<= 1) r |= v & h ? b : 0;
        return r;
    };
    return x ? -nat[bitrev(N - bitrev(x))] : 1.0;
}
static void fill_block_tables(const std::vector<double> &nat, uint32_t BS, bool inverse, double *ra, double *rb) {
    const uint32_t G = (uint32_t)nat.size() / BS, E = BS / 64;
    int late = 0;                                   // stages done after the transposition: log2 E
    for (uint32_t e = E; e > 1; e >>= 1) late++;
    auto entry = [&](size_t x) { return inverse ? inverse_entry(nat, (uint32_t)x) : nat[x]; };
    for (uint32_t row = 0; row < G; row++, ra += 64) {
        // block `row` continues the transform with sub-block counts m' = 1, 2, ..., BS / 2; its sub-block blk at that
        // stage is block (G + row) m' + blk of the whole transform: table entry fwd[(G + row) m' + blk]
        ra[0] = 1.0;
        for (uint32_t x = 1; x < 64; x++) {
            uint32_t mp = 1;
            while (mp * 2 <= x) mp *= 2;
            ra[x] = entry((size_t)(G + row) * mp + (x - mp));
        }
        for (int s = 0; s < late; s++) {
            const uint32_t t = (E / 2) >> s, mp = BS / (2 * t);
            for (uint32_t blk = 0; blk < (1u << s); blk++, rb += 64)
                for (uint32_t l = 0; l < 64; l++) rb[l] = entry((size_t)(G + row) * mp + (E * l) / (2 * t) + blk);
        }
    }
}
int slz_build_block_tables(slz_ctx *ctx, uint32_t BS, double **dA, double **dB) {
    const uint32_t N = ctx->prm.N, G = N / BS, nB = BS / 64 - 1;
    std::vector<double> nat(N), rowA((size_t)2 * G * 64), rowB((size_t)2 * G * nB * 64);
    for (size_t q = 0; q < 2; q++) {
        SLZ_HIP(hipMemcpy(nat.data(), ctx->tab[q].fwd, (size_t)N * sizeof(double), hipMemcpyDeviceToHost));
        fill_block_tables(nat, BS, false, &rowA[q * G * 64], &rowB[q * G * nB * 64]);
    }
    SLZ_HIP(hipMalloc((void **)dA, rowA.size() * sizeof(double)));
    SLZ_HIP(hipMalloc((void **)dB, rowB.size() * sizeof(double)));
    SLZ_HIP(hipMemcpy(*dA, rowA.data(), rowA.size() * sizeof(double), hipMemcpyHostToDevice));
    SLZ_HIP(hipMemcpy(*dB, rowB.data(), rowB.size() * sizeof(double), hipMemcpyHostToDevice));
    return SLZ_OK;
}

// The tables of the 1024-block kernels in one piece of device memory, per prime: rowA [G][64], rowB [G][15][64], their inverses, and the
// column constants of the mirrored inverse [32].
static int build_tables16(slz_ctx *ctx) {
    const uint32_t N = ctx->prm.N, G = N / 1024;
    std::vector<double> nat(N), t(2 * BIG16_TAB(G), 0.0);
    for (int q = 0; q < 2; q++) {
        double *o = &t[q * BIG16_TAB(G)], *col = o + (size_t)G * 64 * 32;
        SLZ_HIP(hipMemcpy(nat.data(), ctx->tab[q].fwd, (size_t)N * sizeof(double), hipMemcpyDeviceToHost));
        fill_block_tables(nat, 1024, false, o, o + (size_t)G * 64);
        fill_block_tables(nat, 1024, true, o + (size_t)G * 64 * 16, o + (size_t)G * 64 * 17);
        for (uint32_t x = 0; x < 2; x++) col[x] = ctx->mirror_last[q][x];
        for (uint32_t x = 2; x < G; x++) col[x] = inverse_entry(nat, x);
    }
    SLZ_HIP(hipMalloc((void **)&ctx->bign16_tab, t.size() * sizeof(double)));
    SLZ_HIP(hipMemcpy(ctx->bign16_tab, t.data(), t.size() * sizeof(double), hipMemcpyHostToDevice));
    return SLZ_OK;
}

// worst-case bounds (units of p) of one block size: column stages start from digits, rows from reduced values
static bool bounds_ok(uint32_t N, uint32_t BS) {
    const uint32_t G = N / BS;
    double a = 1e-6;
    for (uint32_t g = G; g > 1; g >>= 1) a += slz_mulmod_bound(a);
    if (a > 7.5) return false;
    a = 0.5 + 1e-9;
    for (int s = 0; s < 6; s++) a += slz_mulmod_bound(a);        // block stages 1..6, then the reduction inside the wave transform
    if (a > 7.5) return false;
    a = 0.5 + 1e-9;
    for (int s = 0; s < (BS == 2048 ? 5 : 4); s++) a += slz_mulmod_bound(a);
    // sums over the GGSW rows are reduced after every fourth row
    if (0.5 + 4.0 * slz_mulmod_bound(a) > 7.5) return false;
    a = 0.5 + 1e-9;
    for (uint32_t g = G; g > 1; g >>= 1) a += slz_mulmod_bound(a);
    if (slz_mulmod_bound(a) > 1.95) return false;
    // 1024-blocks: the mirrored inverse counts products by a constant form of the bound (slz_wave_ntt.h)
    for (double s = 0.5; BS == 1024 && s < LAZY_MAX; s += 0.1)
        if (slz_mulmod_bound(s) > LAZY_PRODUCT(s)) return false;
    return true;
}

int slz_bign_init(slz_ctx *ctx) {
    const uint32_t N = ctx->prm.N;
    ctx->has_bign16 = 0;
    ctx->bign_block = 0;
    ctx->bign_lanes = 2;
    ctx->bign_latency = 1;
    bool any = false;
    if (block_fits(N, 2048) && bounds_ok(N, 2048)) {
        int rc = slz_build_block_tables(ctx, 2048, &ctx->bign_rowA, &ctx->bign_rowB);
        if (rc != SLZ_OK) return rc;
        SLZ_HIP(hipFuncSetAttribute((const void *)k_big_rows, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * TBUF * sizeof(double)));
        ctx->bign_block = 2048;
        any = true;
    }
    if (block_fits(N, 1024) && bounds_ok(N, 1024)) {
        int rc = build_tables16(ctx);
        if (rc != SLZ_OK) return rc;
        SLZ_HIP(hipFuncSetAttribute((const void *)k_big_rows16, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * (TBUF16 + 1024) * sizeof(double)));
        const struct { const void *kernel; uint32_t rows; } team[] = {{(const void *)k_big_rows16_team<2>, 2}, {(const void *)k_big_rows16_team<4>, 4},
                                                                      {(const void *)k_big_rows16_team<6>, 6}, {(const void *)k_big_rows16_team<8>, 8}};
        for (const auto &t : team) SLZ_HIP(hipFuncSetAttribute(t.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)TEAM_LDS(t.rows)));
        if (slz_bign_xcd_setup() != SLZ_OK) return SLZ_E_HIP;
        ctx->has_bign16 = 1;
        ctx->bign_block = 1024;                                  // preferred: two waves per SIMD in the row pass
        any = true;
    }
    return any ? SLZ_OK : SLZ_E_UNSUPPORTED;
}

void slz_bign_destroy(slz_ctx *ctx) {
    if (ctx->bign_rowA) (void)hipFree(ctx->bign_rowA);
    if (ctx->bign_rowB) (void)hipFree(ctx->bign_rowB);
    if (ctx->bign16_tab) (void)hipFree(ctx->bign16_tab);
    if (ctx->bign_spare) (void)hipFree(ctx->bign_spare);
    ctx->bign_rowA = ctx->bign_rowB = ctx->bign16_tab = nullptr;
    ctx->bign_spare = nullptr;
    for (int j = 0; j < 2; j++) {
        if (ctx->bign_lane_stream[j]) (void)hipStreamDestroy((hipStream_t)ctx->bign_lane_stream[j]);
        if (ctx->bign_lane_done[j]) (void)hipEventDestroy((hipEvent_t)ctx->bign_lane_done[j]);
        ctx->bign_lane_stream[j] = ctx->bign_lane_done[j] = nullptr;
    }
    if (ctx->bign_fork) (void)hipEventDestroy((hipEvent_t)ctx->bign_fork);
    ctx->bign_fork = nullptr;
}

template <int G, int BS>
static void launch_cols(bool fwd, const bign_args &A, uint32_t batch, hipStream_t s) {
    const dim3 grid(BS / 256, 2, batch);
    if (fwd) hipLaunchKernelGGL((k_big_cols_fwd<G, BS>), grid, dim3(256), 0, s, A);
    else hipLaunchKernelGGL((k_big_cols_inv<G, BS>), grid, dim3(256), 0, s, A);
}

static void launch_cols_any(bool fwd, uint32_t G, uint32_t BS, const bign_args &A, uint32_t batch, hipStream_t s) {
    if (BS == 2048) {
        switch (G) {
            case 2: launch_cols<2, 2048>(fwd, A, batch, s); break;
            case 4: launch_cols<4, 2048>(fwd, A, batch, s); break;
            case 8: launch_cols<8, 2048>(fwd, A, batch, s); break;
            case 16: launch_cols<16, 2048>(fwd, A, batch, s); break;
            default: launch_cols<32, 2048>(fwd, A, batch, s); break;
        }
    } else {
        switch (G) {
            case 2: launch_cols<2, 1024>(fwd, A, batch, s); break;
            case 4: launch_cols<4, 1024>(fwd, A, batch, s); break;
            case 8: launch_cols<8, 1024>(fwd, A, batch, s); break;
            case 16: launch_cols<16, 1024>(fwd, A, batch, s); break;
            default: launch_cols<32, 1024>(fwd, A, batch, s); break;
        }
    }
}

// One step of the latency-oriented kernels (1024-blocks): first / turn between two steps / last column pass around the row pass.
// The accumulator alternates between the caller's buffer and `spare`; the last pass leaves it in the caller's.
template <int G>
static void launch_step_lat(const bign_args &A, uint64_t *spare, uint32_t n_steps, hipStream_t s) {
    uint64_t *cur = A.step & 1u ? spare : A.acc, *prev = A.step & 1u ? A.acc : spare;    // the accumulator after A.step steps, and before the last of them
    if (A.step == 0) hipLaunchKernelGGL((k_big_cols_fwd<G, 1024>), dim3(4, 2, A.batch), dim3(256), 0, s, A);
    // one thread per column below eight rows: eight waves for 64 columns would have one row pair each (us per step at N = 2048, l = 2, 256
    // ciphertexts 68 against 38, at N = 4096, l = 2, 64: 30 against 27; at N = 8192 eight waves are faster, one ciphertext 14.7 against 18.0)
    else if constexpr (G <= 4) hipLaunchKernelGGL((k_big_cols_turn_short<G>), dim3(4, 2, A.batch), dim3(256), 0, s, A, (const uint64_t *)prev, cur);
    else hipLaunchKernelGGL((k_big_cols_turn<G>), dim3((2 * A.batch >= 8 ? (2 * A.batch + 7) / 8 * 8 : 2 * A.batch) * 16), dim3(512), 0, s, A, (const uint64_t *)prev, cur);
    const dim3 tasks(A.batch * 2 * G);
    if (A.l == 1) hipLaunchKernelGGL(k_big_rows16_team<2>, tasks, dim3(128), TEAM_LDS(2), s, A, (uint32_t)G);
    else if (A.l == 2) hipLaunchKernelGGL(k_big_rows16_team<4>, tasks, dim3(256), TEAM_LDS(4), s, A, (uint32_t)G);
    else if (A.l == 3) hipLaunchKernelGGL(k_big_rows16_team<6>, tasks, dim3(384), TEAM_LDS(6), s, A, (uint32_t)G);
    else hipLaunchKernelGGL(k_big_rows16_team<8>, tasks, dim3(512), TEAM_LDS(8), s, A, (uint32_t)G);
    if (A.step + 1 == n_steps)
        hipLaunchKernelGGL((k_big_cols_last<G>), dim3(4, 2, A.batch), dim3(256), 0, s, A, (const uint64_t *)cur);
}
static void launch_step_lat_any(uint32_t G, const bign_args &A, uint64_t *spare, uint32_t n_steps, hipStream_t s) {
    switch (G) {
        case 2: launch_step_lat<2>(A, spare, n_steps, s); break;
        case 4: launch_step_lat<4>(A, spare, n_steps, s); break;
        case 8: launch_step_lat<8>(A, spare, n_steps, s); break;
        case 16: launch_step_lat<16>(A, spare, n_steps, s); break;
        default: launch_step_lat<32>(A, spare, n_steps, s); break;
    }
}

// Streams and events of the concurrent lanes (created at the first use, default priority; also while the caller's stream is being
// captured, which records nothing: a graph gets its two lanes whether or not the context has used them before).
static int ensure_lanes(slz_ctx *ctx) {
    if (ctx->bign_lane_stream[0]) return SLZ_OK;
    for (int j = 0; j < 2; j++) {
        hipStream_t st;
        hipEvent_t ev;
        if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) return SLZ_E_HIP;
        ctx->bign_lane_stream[j] = st;
        if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) return SLZ_E_HIP;
        ctx->bign_lane_done[j] = ev;
    }
    hipEvent_t ev;
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) return SLZ_E_HIP;
    ctx->bign_fork = ev;
    return SLZ_OK;
}

// Ciphertexts up to which a step runs as the two launches above.  us per CMux step, three launches per step (as they were: with kernels of their
// own for few ciphertexts, up to 512 / G) -> two; l = 2:
//   N = 32768: 1: 34 -> 22, 4: 39 -> 25, 8: 41 -> 33, 16: 53 -> 44, 24: 73 -> 56, 32: 78 -> 70, 48: 101 -> 103 (most of these run as one launch: slz_bign_xcd_takes)
//   N = 16384: 8: 34 -> 21, 32: 50 -> 40, 48: 61 -> 53, 56: 63 -> 59, 64: 68 -> 69     N = 8192: 64: 50 -> 41, 96: 57 -> 56, 112: 60 -> 64
//   N = 4096: 64: 32 -> 27, 128: 48 -> 38     N = 2048: 256: 50 -> 38
// Past that the column work done twice costs more than the launch and the accumulator's traffic that it saves.
// l = 1: N = 32768: 32: 61 -> 50     N = 16384: 48: 47 -> 43, 49: 47 -> 43, 50: 46.4 -> 46.1 (three of today: 44.8 to 46.5), 56: 47.5 -> 48     N = 8192: 96: 46 -> 42.5, 112: 48 -> 49
// l = 3, 4: a workgroup of the row pass is six or eight waves, of which a compute unit takes two or one, so the step grows by rounds of 512 or 256
// workgroups, 2 G per ciphertext.  G <= 8: one round of l = 3 and three of l = 4 win, three launches of today / two:
//   l = 3: N = 2048: 192: 43.9 / 46.1     N = 4096: 64: 44.9 / 35.3, 96: 46.3 / 47.0     N = 8192: 32: 45.9 / 38.0, 40: 46.4 / 48.2, 64: 49.8 / 62.9
//   l = 4: N = 2048: 192: 51.7 / 52.6, 224: 53.5 / 64.7     N = 4096: 96: 54.8 / 53.1, 104: 56.3 / 64.9     N = 8192: 48: 55.7 / 54.7, 52: 56.1 / 67.0
// G >= 16:
//   l = 3: N = 16384: 24: 52 / 50, 32: 55 / 61, 33: 70.5 / 62, 40: 72.6 / 71.9, 42: 73 / 80     N = 32768: 16: 70 / 67, 20: 88 / 84, 22: 87 / 85, 24: 88 / 92
//   l = 4: N = 16384: 24: 61 / 56, 32: 64 / 70, 33: 84 / 76, 40: 86 / 83, 42: 87 / 91     N = 32768: 16: 81 / 77, 20: 99 / 94, 22: 102.5 / 99.7, 24: 104 / 106
uint32_t slz_bign_latency_max_batch(uint32_t G, uint32_t l) {
    if (l <= 2) return G >= 32 ? 32u : G == 16 ? (l == 1 ? 49u : 56u) : G == 8 ? 96u : 512u / G;
    if (G >= 16) return G == 16 ? 40u : 22u;
    return (l == 3 ? 256u : 384u) / G;
}
// From more than this many on they run as two even halves on the two lanes: N = 32768: 16: 44 either way, 24: 60 -> 57, 32: 75 -> 71;
// N = 16384: 32: 40 either way, 48: 54 -> 53; N = 8192: 64: 41 -> 43.
static uint32_t latency_one_lane_max(uint32_t G) { return G >= 16 ? 512u / G : 0xffffffffu; }
// Ciphertexts of the first of two lanes of the three-launch steps (1024-blocks); 0: the lanes take chunks of `half`, or one
// lane takes all, as up to 512 / G ciphertexts always (1024 row tasks, a wave for every SIMD).  `half` ciphertexts are 2048 row tasks or more: alone on the chip they fill it, so a smaller batch leaves the chip idle at
// every hand-over between its launches, which a second lane fills; a batch a little larger would be a full lane and a small rest.  From a
// quarter above `half` on (G = 2: an eighth) the rest is large enough to hide its launches behind the full lane, while two even halves are
// one and a half rounds of row tasks each; G >= 16 and the upper part of G = 8 move so much memory per ciphertext that even lanes win.
// us per CMux step, one lane or full lane and rest -> even lanes:
//   G = 2, l = 2: 260 ciphertexts 52 -> 47, 520: 74 -> 65, 640: 79 -> 80     G = 4, l = 2: 140: 54 -> 50, 288: 76 -> 73, 384: 88 -> 94
//   G = 8, l = 2: 110: 63.6 -> 60.3, 152: 81 -> 77, 176: 83 -> 88, 208: 101 -> 98; l = 1: 66: 43.5 -> 40.4, 88: 45.0 -> 45.7, 112: 49.6 -> 47.7
//   G = 16, l = 2: 38: 65 -> 59, 92: 94 -> 91     G = 32, l = 2: 24: 76 -> 73, 33: 94 -> 86, 48: 103 -> 101, 64: 129 -> 129
// The cut leaves the second lane, and the first where the batch allows, a count that the XCD-aware order of the row pass takes (16 / G
// ciphertexts at G = 4 and 8): 132 at G = 4 51 -> 48.5, 66 at G = 8, l = 2 54 -> 51.
uint32_t slz_bign_first_of_even_lanes(uint32_t G, uint32_t batch, uint32_t half) {
    const bool even = batch <= half + half / (G == 2 ? 8 : 4) || G >= 16 || (G == 8 && batch >= half + half * 5 / 8);
    const uint32_t unit = G == 4 || G == 8 ? 16 / G : 1;
    return even && batch > 512 / G && batch <= 2 * half ? batch - batch / 2 / unit * unit : 0;
}

// The second accumulator of the two-launch steps, and behind it the control words of the one launch, asked for with the first scratch of a
// context and never again: a later call allocates nothing, whatever its batch, and may be captured.  Without them a step runs as three launches at every batch size.
void slz_bign_scratch(slz_ctx *ctx) {
    if (!ctx->has_bign16 || ctx->bign_spare_asked) return;
    ctx->bign_spare_asked = 1;
    const uint32_t lat_max = slz_bign_latency_max_batch(ctx->prm.N / 1024, ctx->prm.pbs_level);
    const size_t cts = ctx->max_batch < lat_max ? ctx->max_batch : lat_max;
    void *buf = nullptr;
    if (slz_scratch_alloc(&buf, cts * 2 * ctx->prm.N * sizeof(uint64_t) + slz_bign_xcd_ctl_bytes()) != SLZ_OK) return;
    ctx->bign_spare = (uint64_t *)buf;
    ctx->bign_ctl = (uint32_t *)(ctx->bign_spare + cts * 2 * ctx->prm.N);
}

// Arguments of the kernels for `batch` ciphertexts whose workspace starts `first` ciphertexts into the context's; step and key are the caller's.
static bign_args args_of(const slz_ctx *ctx, uint32_t BS, const uint64_t *lwe_in, uint64_t *acc, size_t first, uint32_t batch) {
    const slz_params &p = ctx->prm;
    const uint32_t N = p.N, G = N / BS, R = 2 * p.pbs_level;
    bign_args a;
    a.lwe_in = lwe_in;
    a.acc = acc;
    a.X = ctx->xhat + first * 2 * R * N;
    a.Y = ctx->outhat + first * 2 * 2 * N;
    a.bskp_step = nullptr;
    a.n = p.n; a.step = 0; a.N = N; a.pad = 0; a.beta = p.pbs_base_log; a.l = p.pbs_level; a.batch = batch;
    for (int q = 0; q < 2; q++) {
        a.tab[q].fwd = ctx->tab[q].fwd;
        if (BS == 2048) {
            a.tab[q].rowA = ctx->bign_rowA + (size_t)q * G * 64;
            a.tab[q].rowB = ctx->bign_rowB + (size_t)q * G * 31 * 64;
        } else {
            const double *t = ctx->bign16_tab + q * BIG16_TAB(G);
            a.tab[q].rowA = t;
            a.tab[q].rowB = t + (size_t)G * 64;
        }
        a.tab[q].inv = ctx->tab[q].inv;
        a.tab[q].post = ctx->tab[q].post;
        a.mod[q] = ctx->mod[q];
    }
    a.p1inv_mod_p2 = ctx->p1inv_mod_p2;
    return a;
}

// Batches that run all steps in one launch (slz_bign_xcd.hip): N = 32768 with two levels, rounds of eight ciphertexts, 15.7 (1024 steps) to 16.8 us (256
// steps) per step and round whether it is full or not.  us per step of the launches below it (two up to 32 ciphertexts, then three): 1: 21.7, 4: 25, 8: 31.5,
// 9: 37.9, 16: 42.9, 17: 41.4, 18: 48.4, 20: 47.6, 21: 47.9, 24: 52.7, 25: 54.8, 28: 62, 32: 67.6, 33: 81, 36: 85.4, 40: 85.5, 48: 94.9, 64: 121: they win at the
// beginning of the third and fourth round and from the sixth on.
uint32_t slz_bign_xcd_takes(uint32_t G, uint32_t l, uint32_t batch) {
    if (G != 32 || l != 2) return 0;
    return batch <= 16 || (batch >= 22 && batch <= 24) || (batch >= 31 && batch <= 40);
}

// The one launch on `workgroups` workgroups; any number of them goes through all steps (tests run fewer), SLZ_XCD_WORKGROUPS are one per slot.  patience:
// slz_bign_xcd.hip; tests take less than SLZ_XCD_PATIENCE.
int slz_bign_xcd_run(slz_ctx *ctx, const uint64_t *lwe_in, const double *bskp, uint32_t n_steps, uint64_t *acc, uint32_t batch, uint32_t workgroups,
                     hipStream_t s) {
    return slz_bign_xcd_run(ctx, lwe_in, bskp, n_steps, acc, batch, workgroups, SLZ_XCD_PATIENCE, s);
}
int slz_bign_xcd_run(slz_ctx *ctx, const uint64_t *lwe_in, const double *bskp, uint32_t n_steps, uint64_t *acc, uint32_t batch, uint32_t workgroups,
                     uint32_t patience, hipStream_t s) {
    bign_args a = args_of(ctx, 1024, lwe_in, acc, 0, batch);
    a.bskp_step = bskp;
    return slz_bign_xcd_launch(a, ctx->bign_ctl, n_steps, workgroups, patience, s);
}

// Runs steps [0, n_steps) on accumulators that the caller has initialised in `acc` ([batch][2][N]).
int slz_bign_cmux_steps(slz_ctx *ctx, const uint64_t *lwe_in, const double *bskp, uint32_t n_steps, uint64_t *acc,
                        uint32_t batch, hipStream_t s) {
    const slz_params &p = ctx->prm;
    const uint32_t N = p.N, BS = (uint32_t)ctx->bign_block, G = N / BS, R = 2 * p.pbs_level;
    if (n_steps == 0) return SLZ_OK;
    // (on a stream limited to some compute units the workgroups that run do the others' tasks in turn, where the launches below deal theirs evenly: 12 steps on
    // 128 of 256 compute units, us in one launch / below: 1 ciphertext 697 / 284, 8: 716 / 528, 24: 2080 / 773)
    if (ctx->bign_latency && BS == 1024 && ctx->bign_ctl && slz_bign_xcd_takes(G, p.pbs_level, batch) && slz_compute_units(s) >= SLZ_XCD_WORKGROUPS)
        return slz_bign_xcd_run(ctx, lwe_in, bskp, n_steps, acc, batch, SLZ_XCD_WORKGROUPS, s);
    // few ciphertexts otherwise: every step in two launches (1024-blocks only, and where there was room for the second accumulator)
    const bool lat = ctx->bign_latency && BS == 1024 && batch <= slz_bign_latency_max_batch(G, p.pbs_level) && ctx->bign_spare;
    // Ciphertexts go through all steps in chunks whose workspace (X, Y, accumulators: (2R + 4 + 2) N doubles each) stays
    // in the 256 MB Infinity Cache; the key (read once per chunk and step) streams from HBM.
    const size_t per_ct = (size_t)(2 * R + 4 + 2) * N * 8;
    uint32_t chunk = (uint32_t)((size_t)224 * 1024 * 1024 / per_ct);
    const uint32_t slots = BS == 2048 ? 1024u : 2048u;              // resident row-pass waves: one or two per SIMD
    const uint32_t fill = slots / (2 * G) ? slots / (2 * G) : 1;     // ciphertexts whose row tasks fill the chip once
    chunk = chunk / fill * fill;
    if (chunk < fill) chunk = fill;
    // Two lanes: the chunk is cut in two halves that run on two streams, so that the row pass of one half (bound by
    // arithmetic) overlaps the column passes of the other (bound by memory).  Measured at N = 32768: 5 % faster than one
    // lane; three or four lanes of the same size overflow the Infinity Cache and are slower.
    uint32_t lanes = (uint32_t)ctx->bign_lanes;
    if (lat) {
        if (batch <= latency_one_lane_max(G)) lanes = 1;
        chunk = lanes >= 2 ? (batch + 1) / 2 : batch;
    } else if (lanes >= 2) {
        uint32_t half = chunk / 2 / fill * fill;
        if (half < fill) half = fill;
        const uint32_t first = BS == 1024 ? slz_bign_first_of_even_lanes(G, batch, half) : 0;
        if (first) chunk = first;
        else if (batch > half) chunk = half;
        else lanes = 1;
    }
    if (chunk > batch) chunk = batch;
    if (lanes >= 2) {
        int rc = ensure_lanes(ctx);                                 // only where they are used: idle queues cost a lone stream 3 % of its launches
        if (rc != SLZ_OK) return rc;
        SLZ_HIP(hipEventRecord((hipEvent_t)ctx->bign_fork, s));
        for (uint32_t j = 0; j < lanes; j++) SLZ_HIP(hipStreamWaitEvent((hipStream_t)ctx->bign_lane_stream[j], (hipEvent_t)ctx->bign_fork, 0));
    }
    for (uint32_t g0 = 0; g0 < batch; g0 += lanes * chunk) {
        bign_args A[2];
        hipStream_t st[2];
        uint32_t n_tasks[2], nbs[2], used = 0;
        for (uint32_t j = 0; j < lanes; j++) {
            const uint32_t c0 = g0 + j * chunk;
            if (c0 >= batch) break;
            const uint32_t nb = (batch - c0 < chunk) ? batch - c0 : chunk;
            A[j] = args_of(ctx, BS, lwe_in + (size_t)c0 * (p.n + 1), acc + (size_t)c0 * 2 * N, (size_t)j * chunk, nb);
            n_tasks[j] = nb * 2 * G;
            nbs[j] = nb;
            st[j] = lanes >= 2 ? (hipStream_t)ctx->bign_lane_stream[j] : s;
            used = j + 1;
        }
        for (uint32_t step = 0; step < n_steps; step++) {
            for (uint32_t j = 0; j < used; j++) {
                bign_args &a = A[j];
                a.step = step;
                a.bskp_step = bskp + (size_t)step * 2 * R * 2 * N;
                if (lat) {
                    launch_step_lat_any(G, a, ctx->bign_spare + (a.acc - acc), n_steps, st[j]);
                    continue;
                }
                launch_cols_any(true, G, BS, a, nbs[j], st[j]);
                // the XCD-aware order needs the task count to split evenly over 8 XCDs x 4 waves x (2G/8) combinations
                const int xcd_aware = (2 * G) % 8 == 0 && n_tasks[j] % 32 == 0 && (n_tasks[j] / 8) % (2 * G / 8) == 0;
                if (BS == 2048)
                    hipLaunchKernelGGL(k_big_rows, dim3((n_tasks[j] + 3) / 4), dim3(256), 4 * TBUF * sizeof(double), st[j], a, G,
                                       n_tasks[j], xcd_aware);
                else
                    hipLaunchKernelGGL(k_big_rows16, dim3((n_tasks[j] + 3) / 4), dim3(256), 4 * (TBUF16 + 1024) * sizeof(double), st[j], a,
                                       G, n_tasks[j], xcd_aware);
                launch_cols_any(false, G, BS, a, nbs[j], st[j]);
            }
        }
    }
    if (lanes >= 2) {
        for (uint32_t j = 0; j < lanes; j++) {
            SLZ_HIP(hipEventRecord((hipEvent_t)ctx->bign_lane_done[j], (hipStream_t)ctx->bign_lane_stream[j]));
            SLZ_HIP(hipStreamWaitEvent(s, (hipEvent_t)ctx->bign_lane_done[j], 0));
        }
    }
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

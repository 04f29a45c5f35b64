// Device helpers of the large-N kernels (slz_bign.hip: passes as launches, slz_bign_xcd.hip: passes inside one launch).
#pragma once
#include "slz_internal.h"
#include "slz_modarith.h"
#include "slz_wave_ntt.h"

struct bign_tabs {                 // per prime
    const double *fwd;             // natural forward table of the full transform (fwd[m + blk])
    const double *rowA;            // [G][64]      block-specific twiddles of stages with 1..32 sub-blocks (uniform per wave)
    const double *rowB;            // [G][31][64]  block-specific per-lane twiddles of the last five forward stages (1024-blocks: [G][15][64], four)
    const double *inv;             // natural inverse table
    const double *post;            // natural twist table
};

struct bign_args {
    const uint64_t *lwe_in;
    uint64_t *acc;                 // [batch][2][N]
    double *X;                     // [batch][2 primes][R][N]
    double *Y;                     // [batch][2 primes][2][N]
    const double *bskp_step;       // prepared GGSW of this step: [2][R][2][N]
    uint32_t n, step, N, pad, beta, l, batch;    // pad: not read.  Without it the arguments are 184 bytes and 8 ciphertexts of N = 32768 (1024 steps)
                                   // take 33.76 ms, in every order of these words tried, against 33.59; with a word more (200 bytes) 33.87
    bign_tabs tab[2];
    slz_mod mod[2];
    double p1inv_mod_p2;
};

// forward column stages (strides N/2 .. BS) on a column of G rows: pairs of rows, twiddle by block of rows (uniform)
template <int G>
__device__ __forceinline__ void cols_fwd(double (&y)[G], const double *tw, slz_mod m) {
#pragma unroll
    for (int half = G / 2, blocks = 1; half >= 1; half >>= 1, blocks <<= 1) {
#pragma unroll
        for (int blk = 0; blk < blocks; blk++) {
            const double w = tw[blocks + blk];
#pragma unroll
            for (int j = 0; j < half; j++) bfly(y[blk * 2 * half + j], y[blk * 2 * half + j + half], w, m);
        }
    }
}

// 1024-blocks: the tables of the mirrored inverse follow rowA [G][64] and rowB [G][15][64] in memory (BIG16_TAB), one allocation
// and one copy for all: inverses of rowA and of rowB, and the column stages' [32]: inverses of fwd[2 .. G - 1], [0] = 1 / N,
// [1] = 1 / (N fwd[1])
#define BIG16_TAB(G) ((size_t)(G) * 64 * 32 + 32)
__device__ __forceinline__ const double *rowAi_of(const bign_tabs &t, uint32_t G) { return t.rowA + (size_t)G * 64 * 16; }
__device__ __forceinline__ const double *rowBi_of(const bign_tabs &t, uint32_t G) { return t.rowA + (size_t)G * 64 * 17; }
__device__ __forceinline__ const double *colI_of(const bign_tabs &t, uint32_t G) { return t.rowA + (size_t)G * 64 * 32; }

// Column stages of the mirrored inverse inside a part of K rows (1024-blocks): block `first` .. of the forward stage with
// the same strides.  bd: bounds in units of p.
template <int K>
__device__ __forceinline__ void cols_mirror(double (&x)[K], double (&bd)[K], const double *colI, uint32_t part, uint32_t parts, slz_mod m) {
#pragma unroll
    for (int half = 1; half < K; half <<= 1) {
#pragma unroll
        for (int blk = 0; blk < K / (2 * half); blk++) {
            const double w = colI[(parts + part) * (K / (2 * half)) + blk];
#pragma unroll
            for (int j = 0; j < half; j++) {
                double *pa[1] = {&x[blk * 2 * half + j]}, *pb[1] = {&x[blk * 2 * half + j + half]};
                double *ua[1] = {&bd[blk * 2 * half + j]}, *ub[1] = {&bd[blk * 2 * half + j + half]};
                const double pw[1] = {w};
                gs_k<1>(pa, pb, ua, ub, pw, m);
            }
        }
    }
}
// the last stage with the factor 1 / N: f, g <- (f + g) / N, (f - g) / (N w)
__device__ __forceinline__ void cols_mirror_last(double &f, double &g, const double *colI, slz_mod m) {
    const double s = f + g, d = f - g;
    f = slz_mulmod(s, colI[0], m);
    g = slz_mulmod(d, colI[1], m);
}

// slz_bign_xcd.hip: all CMux steps of a batch in one launch.  a.acc [batch][2][N] initialised, a.X for min(batch, 8) ciphertexts, a.bskp_step the key of step 0,
// ctl slz_bign_xcd_ctl_bytes() bytes
#define SLZ_XCD_WORKGROUPS 256u
#define SLZ_XCD_PATIENCE (1u << 22)      // looks at the L2 of half a microsecond and more: seconds, where a phase takes microseconds
int slz_bign_xcd_setup();
size_t slz_bign_xcd_ctl_bytes();
int slz_bign_xcd_launch(const bign_args &a, uint32_t *ctl, uint32_t n_steps, uint32_t workgroups, uint32_t patience, hipStream_t s);

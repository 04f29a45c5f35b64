// Host side and key preparation of the floating-point transform path (see slz_fft.h): error bound, tables, key spectra.
#include "slz_xcd.h"
#include "slz_fft.h"
#include <cmath>
#include <cstring>
#include <vector>

// ---- the error bound ------------------------------------------------------------------------------------------------
// u = 2^-53.  All constants are multiples of u; M = N / 2 points; d = all digits of a row, K = a piece (2-norms over the N
// real coefficients, which are the 2-norms of the M folded complex ones).
//  Tables: a twiddle is computed in long double (64-bit significand) and rounded once.  Its angle is pi times an exact number below 3,
//  off by at most 2 * 3 pi * 2^-64 (pi itself and the product); cosine, sine and their quotient err by at most 2^-63 together, and
//  rounding to double after rounding to long double adds at most 2^-64 per component: below 26 * 2^-64 = 0.013 u; a quarter turn given
//  the cosine 2^-60 has that as its only error, 0.008 u.  TABLE = 0.02 u stands for this below, once per use of a twiddle.
//  Forward (radix-4 butterflies, each a0 + v^2 a2 +- (v a1 + v^3 a3) and a0 - v^2 a2 +- i (v a1 - v^3 a3)): a complex product
//  of two multiplications and two fused multiply-adds errs by at most 2 u |w| |a|, the rounding of the twiddle's two
//  components adds sqrt(1/2) u and TABLE, the two layers of additions u each: 4.73 u per butterfly relative to the 2-norm, five
//  layers of butterflies for M = 1024.  So ||dX||_2 <= 23.7 u ||X||_2 = 23.7 u sqrt(M) ||d||_2.
//  Products: S = D0 K0 + D1 K1 as a chain of four fused multiply-adds per component: partial results are at most
//  |D0 K0| (twice), |D0 K0| + |D1 K1| (twice), so the error is at most u (4 |D0 K0| + 2 |D1 K1|); the key spectrum is a
//  correctly rounded value of a double-double transform: another u |D K| (1.05 u with the transform's own error).
//  Inverse (decimation in time): every output is (1 / M) sum_k S_k with unit weights, so it is bounded along paths, relative
//  to (1 / M) sum |S_k| <= ||d||_2 ||K||_2: half-sizes 1 and 2 only add (u each); half-size 4 adds, multiplies by sqrt(1/2)
//  inside the second addition (u + 0.61 u + u, 0.61 u being the constant's rounding); half-sizes 8 to 256 are o = a +- wr (b -+ tau i b) with w = wr (1 + i tau): rounding of
//  wr and tau at most 2 u |b|, of the bracket u |b|, of the result u |o|, together 4 u; half-size 512 with the twist is the
//  same with a already multiplied by a plain complex factor (2.71 u, not above the 3 u of the other operand), and the second
//  half of its outputs is turned by 45 degrees: an addition and the constant sqrt(1/2) (1.61 u; the product itself is inside the
//  fused rounding add).  1 + 1 + 2.61 + 6 * 4 + 4 + 1.61 = 34.22 u, and TABLE for each of the seven stages with table twiddles.
//  With eight waves per ciphertext (slz_fft2048_team.hip) the forward layers are the same, and half-sizes 4 and 8 are one radix-4 layer
//  (on a path one product, 2.7072 u and TABLE, and two additions): 1 + 1 + 4.7072 + 6 * 4 + 1.61 = 32.32 u and seven times TABLE, below.
//  Second-order terms are covered by the factor 1 + 2^-40.
// Every row r contributes ||d_r|| ||K_(r,j)||.  The chain of four constants above is for two rows.
// N = 1024, M = 512: the forward layers are radix-2 butterflies of the inverse's form, at most 4 u and TABLE each relative to the 2-norm
// (final rounding u |o|, the rest 3 u |b|, and the two outputs' norm is at least sqrt(2) |b|): nine of them; the inverse
// has one stage less: 30.22 u and six times TABLE.
// N = 512, M = 256: eight forward layers; half-size 4 is a butterfly like the others, 27.61 u and six times TABLE; four rows, so the
// chain of fused multiply-adds gives (8 + 6 + 4 + 2) u |D K|, 5 u per row.
// N = 4096, M = 2048: the first forward layer is radix 2 with the constant (1 + i) / sqrt(2) on integers, whose sums p = b.x -+ b.y are
// exact: the constant's rounding 0.61 u and the result's u.  Then radix 4 (4.7072 u and TABLE), two radix-8 layers (a product 2.7072 u
// and TABLE, two additions u each, and a third whose odd part may be a sum, rounded u, times sqrt(1/2), 0.61 u, inside the addition that
// rounds u: 7.3172 u and TABLE) and radix 4.  Inverse: half-sizes 1, 2, 4 as above (4.61 u); twice a radix-4 layer (on a path one product,
// 2.7072 u and TABLE, and two additions) and a radix-2 one (4 u and TABLE); 512, 1024 with the twist, the turn (9.61 u and TABLE twice):
// 31.6344 u and six times TABLE.
double slz_fft_error_bound(uint32_t N, uint32_t rows, uint32_t beta) {
    const double u = std::ldexp(1.0, -53), key = 1.05, table = 0.02;
    double fwd, inv;
    int bits = SLZ_FFT_PIECE_BITS;
    if (N == 2048 && rows == 2) { fwd = 5 * (4.7072 + table); inv = 34.22 + 7 * table; }
    else if (N == 1024 && rows == 2) { fwd = 9 * (4.0 + table); inv = 30.22 + 6 * table; }
    else if (N == 512 && rows == 4) { fwd = 8 * (4.0 + table); inv = 27.61 + 6 * table; bits = F9_PIECE_BITS; }
    else if (N == 4096 && rows == 2) { fwd = 1.61 + 2 * (4.7072 + table) + 2 * (7.3172 + table); inv = 4.61 + 2 * (4.7072 + 4.0) + 9.61 + 6 * table; }
    else return 1e300;
    const double norm_d = std::ldexp(std::sqrt((double)N), (int)beta - 1);
    const double norm_k = std::ldexp(std::sqrt((double)N), bits - 1);
    // products: 3 u per row for two rows at equal bounds, 5 u for four
    return (fwd + rows + 1.0 + key + inv) * u * (double)rows * norm_d * norm_k * (1.0 + std::ldexp(1.0, -40));
}

int slz_fft_supported(const slz_params *p) {                        // N = 4096: slz_fft4096_supported
    return p->N != 4096 && p->k == 1 && p->pbs_base_log <= 30 && slz_fft_error_bound(p->N, 2 * p->pbs_level, p->pbs_base_log) < 0.499;
}

// ---- tables ---------------------------------------------------------------------------------------------------------
static const long double PI_L = 3.14159265358979323846264338327950288L;
struct cpl { double r, i; };

// angle of W(m, blk), in units of pi: the constant of the root is i (1/2), W halves it, the children of a block have +-W
static long double node_angle(uint32_t m, uint32_t blk) {
    long double phi = 0.5L;                                        // constant of the root block
    uint32_t bits = 0;
    while ((1u << bits) < m) bits++;
    for (uint32_t s = 0; s < bits; s++) {
        const uint32_t right = (blk >> (bits - 1 - s)) & 1u;
        phi = phi / 2 + (right ? 1.0L : 0.0L);
    }
    return phi / 2;
}
static cpl unit(long double a) { return {(double)cosl(PI_L * a), (double)sinl(PI_L * a)}; }
// (cos, tan) of an angle in units of pi; a quarter turn gets a tiny cosine instead of zero, so that cos * tan = +-1 exactly
// and the error is 2^-60
static cpl cos_tan(long double a) {
    long double c = cosl(PI_L * a), s = sinl(PI_L * a);
    if (fabsl(c) < 1e-15L) return {std::ldexp(1.0, -60), s > 0 ? std::ldexp(1.0, 60) : -std::ldexp(1.0, 60)};
    return {(double)c, (double)(s / c)};
}
static void three(cpl *out, size_t stride, uint32_t m, uint32_t blk) {
    const long double v = node_angle(2 * m, 2 * blk);
    for (int q = 0; q < 3; q++) out[q * stride] = unit((q + 1) * v);
}

static void build_2048(std::vector<cpl> &t, double (&f1_out)[15][2]) {
    const uint32_t M = 1024;
    t.resize(FFT_TAB_LEN);
    for (uint32_t x = 0; x < 16; x++) {
        three(&t[FFT_F2_OFF + x], 16, 16, x);
        for (uint32_t q = 0; q < 4; q++) three(&t[FFT_F2_OFF + (3 + 3 * q) * 16 + x], 16, 64, 4 * x + q);
    }
    for (uint32_t g = 0; g < 2; g++)
        for (uint32_t l = 0; l < 64; l++)
            for (uint32_t b = 0; b < 2; b++) three(&t[FFT_F3_OFF + (g * 6 + 3 * b) * 64 + l], 64, 256, g * 128 + 2 * l + b);
    for (uint32_t l = 0; l < 8; l++) {
        cpl *o = &t[FFT_I2_OFF + l];
        o[0] = cos_tan(-(long double)l / 8);
        o[8] = cos_tan(-(long double)l / 16);
        for (uint32_t q = 0; q < 2; q++) o[8 * (2 + q)] = cos_tan(-(long double)(8 * q + l) / 32);
        for (uint32_t q = 0; q < 4; q++) o[8 * (4 + q)] = cos_tan(-(long double)(8 * q + l) / 64);
    }
    for (uint32_t l = 0; l < 64; l++) {
        cpl *o = &t[FFT_I3_OFF + l];
        o[0] = cos_tan(-(long double)l / 128);
        for (uint32_t q = 0; q < 2; q++) o[64 * (1 + q)] = cos_tan(-(long double)(64 * q + l) / 256);
        for (uint32_t q = 0; q < 8; q++) {
            const long double j = 64 * q + l;
            o[64 * (3 + 2 * q)] = unit(-j / (2 * M));
            o[64 * (4 + 2 * q)] = cos_tan(-j / (2 * M) - j / 512);
        }
    }
    cpl *tt = &t[FFT_T_OFF];                                        // eight waves per ciphertext
    for (uint32_t l = 0; l < 4; l++)
        for (uint32_t q = 0; q < 3; q++) tt[FFT_T2_OFF + 4 * q + l] = unit(-(long double)((q + 1) * l) / 8);
    for (uint32_t q = 0; q < 2; q++) {
        for (uint32_t l = 0; l < 16; l++) tt[FFT_T3_OFF + 16 * q + l] = cos_tan(-(long double)l / (16 << q));
        for (uint32_t l = 0; l < 64; l++) tt[FFT_T4_OFF + 64 * q + l] = cos_tan(-(long double)l / (64 << q));
    }
    for (uint32_t l = 0; l < 256; l++) {
        cpl *o = tt + FFT_T5_OFF + l;
        o[0] = cos_tan(-(long double)l / 256);
        for (uint32_t q = 0; q < 2; q++) {
            const long double j = 256 * q + l;
            o[256 * (1 + 2 * q)] = unit(-j / (2 * M));
            o[256 * (2 + 2 * q)] = cos_tan(-j / (2 * M) - j / 512);
        }
    }
    cpl f1[15];
    three(f1, 1, 1, 0);
    for (uint32_t q = 0; q < 4; q++) three(f1 + 3 + 3 * q, 1, 4, q);
    for (int q = 0; q < 15; q++) { f1_out[q][0] = f1[q].r; f1_out[q][1] = f1[q].i; }
}

// the four twiddles of three layers that begin with m blocks, for block `blk` of the first
static void four(cpl *out, size_t stride, uint32_t m, uint32_t blk) {
    out[0] = cos_tan(node_angle(m, blk));
    out[stride] = cos_tan(node_angle(2 * m, 2 * blk));
    for (uint32_t q = 0; q < 2; q++) out[(2 + q) * stride] = cos_tan(node_angle(4 * m, 4 * blk + 2 * q));
}
static void build_1024(std::vector<cpl> &t, double (&f1_out)[15][2]) {
    const uint32_t M = 512;
    t.resize(F10_TAB_LEN);
    for (uint32_t x = 0; x < 8; x++) four(&t[F10_F2_OFF + x], 8, 8, x);
    for (uint32_t l = 0; l < 64; l++) four(&t[F10_F3_OFF + l], 64, 64, l);
    for (uint32_t l = 0; l < 8; l++) {
        cpl *o = &t[F10_I2_OFF + l];
        o[0] = cos_tan(-(long double)l / 8);
        o[8] = cos_tan(-(long double)l / 16);
        for (uint32_t q = 0; q < 2; q++) o[8 * (2 + q)] = cos_tan(-(long double)(8 * q + l) / 32);
    }
    for (uint32_t l = 0; l < 64; l++) {
        cpl *o = &t[F10_I3_OFF + l];
        o[0] = cos_tan(-(long double)l / 64);
        o[64] = cos_tan(-(long double)l / 128);
        for (uint32_t q = 0; q < 4; q++) {
            const long double j = 64 * q + l;
            o[64 * (2 + 2 * q)] = unit(-j / (2 * M));
            o[64 * (3 + 2 * q)] = cos_tan(-j / (2 * M) - j / 256);
        }
    }
    cpl f1[4];
    four(f1, 1, 1, 0);
    for (int q = 0; q < 4; q++) { f1_out[q][0] = f1[q].r; f1_out[q][1] = f1[q].i; }
}

static void build_512(std::vector<cpl> &t, double (&f1_out)[15][2]) {
    const uint32_t M = 256;
    t.resize(F9_TAB_LEN);
    for (uint32_t x = 0; x < 8; x++) four(&t[F9_F2_OFF + x], 8, 8, x);
    for (uint32_t l = 0; l < 64; l++) {
        t[F9_F3_OFF + l] = cos_tan(node_angle(64, l));
        t[F9_F3_OFF + 64 + l] = cos_tan(node_angle(128, 2 * l));
    }
    for (uint32_t l = 0; l < 4; l++) {
        cpl *o = &t[F9_I2_OFF + l];
        o[0] = cos_tan(-(long double)l / 4);
        o[4] = cos_tan(-(long double)l / 8);
        for (uint32_t q = 0; q < 2; q++) o[4 * (2 + q)] = cos_tan(-(long double)(4 * q + l) / 16);
    }
    for (uint32_t l = 0; l < 32; l++) {
        cpl *o = &t[F9_I3_OFF + l];
        o[0] = cos_tan(-(long double)l / 32);
        o[32] = cos_tan(-(long double)l / 64);
        for (uint32_t q = 0; q < 4; q++) {
            const long double j = 32 * q + l;
            o[32 * (2 + 2 * q)] = unit(-j / (2 * M));
            o[32 * (3 + 2 * q)] = cos_tan(-j / (2 * M) - j / 128);
        }
    }
    cpl f1[4];
    four(f1, 1, 1, 0);
    for (int q = 0; q < 4; q++) { f1_out[q][0] = f1[q].r; f1_out[q][1] = f1[q].i; }
}

// the powers 1 .. 7 of the twiddle of a radix-8 layer that begins with m blocks, for block `blk`; the angle is reduced exactly
static void eight(cpl *out, size_t stride, uint32_t m, uint32_t blk) {
    const long double v = node_angle(4 * m, 4 * blk);
    for (int q = 0; q < 7; q++) out[q * stride] = unit(fmodl((q + 1) * v, 2.0L));
}
static void build_4096(std::vector<cpl> &t, double (&f1_out)[15][2]) {
    const uint32_t M = 2048;
    t.resize(F12_TAB_LEN);
    for (uint32_t x = 0; x < 8; x++) eight(&t[F12_F2_OFF + x], 8, 8, x);
    for (uint32_t x = 0; x < 64; x++) eight(&t[F12_F3_OFF + x], 64, 64, x);
    for (uint32_t g = 0; g < 4; g++)
        for (uint32_t l = 0; l < 64; l++)
            for (uint32_t b = 0; b < 2; b++) three(&t[F12_F4_OFF + (g * 6 + 3 * b) * 64 + l], 64, 512, (g * 64 + l) * 2 + b);
    auto inverse = [&](cpl *o, uint32_t stride, uint32_t half) {      // half-sizes half and 2 half as (v, v^2, v^3), 4 half as (cos, tan)
        for (uint32_t l = 0; l < half; l++) {
            for (uint32_t q = 0; q < 3; q++) o[q * stride + l] = unit(-(long double)((q + 1) * l) / (2 * half));
            for (uint32_t q = 0; q < 2; q++) o[(3 + q) * stride + l] = cos_tan(-(long double)(half * q + l) / (4 * half));
        }
    };
    inverse(&t[F12_I2_OFF], 8, 8);
    inverse(&t[F12_I3_OFF], 64, 64);
    for (uint32_t l = 0; l < 256; l++) {
        cpl *o = &t[F12_I4_OFF + l];
        o[0] = cos_tan(-(long double)l / 512);
        for (uint32_t q = 0; q < 4; q++) {
            const long double j = 256 * q + l;
            o[256 * (1 + 2 * q)] = unit(-j / (2 * M));
            o[256 * (2 + 2 * q)] = cos_tan(-j / (2 * M) - j / 1024);
        }
    }
    cpl f1[6];
    for (uint32_t b = 0; b < 2; b++) three(f1 + 3 * b, 1, 2, b);
    for (int q = 0; q < 6; q++) { f1_out[q][0] = f1[q].r; f1_out[q][1] = f1[q].i; }
}

// Host copies of the tables of one size, built by the first context that needs them (a millisecond of long-double functions).
struct host_tables {
    std::vector<cpl> t;
    double f1[15][2];
    std::vector<double> w;                                         // twiddles of the key preparation as double-doubles: W(m, blk) at m + blk
};
static host_tables build(uint32_t N) {
    host_tables r{};
    const uint32_t M = N / 2;
    if (N == 4096) build_4096(r.t, r.f1);
    else if (N == 2048) build_2048(r.t, r.f1);
    else if (N == 1024) build_1024(r.t, r.f1);
    else build_512(r.t, r.f1);
    r.w.resize(4 * (size_t)M);
    for (uint32_t x = 1; x < M; x++) {
        uint32_t m = 1;
        while (2 * m <= x) m *= 2;
        const long double a = PI_L * node_angle(m, x - m), c = cosl(a), s = sinl(a);
        r.w[4 * x] = (double)c; r.w[4 * x + 1] = (double)(c - (long double)(double)c);
        r.w[4 * x + 2] = (double)s; r.w[4 * x + 3] = (double)(s - (long double)(double)s);
    }
    return r;
}
static const host_tables &tables(uint32_t N) {
    if (N == 4096) { static const host_tables t4096 = build(4096); return t4096; }
    if (N == 2048) { static const host_tables t2048 = build(2048); return t2048; }
    if (N == 1024) { static const host_tables t1024 = build(1024); return t1024; }
    static const host_tables t512 = build(512);
    return t512;
}

// ---- pairs of workgroups (slz_xcd.h) ------------------------------------------------------------------------------------

static bool in_capture(hipStream_t s) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess) (void)hipGetLastError();
    return capture != hipStreamCaptureStatusNone;
}
// While a stream is being captured, the runtime refuses allocations and queries of events to every thread that does not allow them itself.  What is
// asked for here has nothing to do with what is being captured.
struct beside_captures {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    beside_captures() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~beside_captures() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// Their words and mail: 32 bytes per coefficient and pair, for as many pairs as a launch makes; asked for once, by the context's first
// call outside a capture, whatever its batch: later ones allocate nothing.  A context without them (no room) runs every batch with one workgroup per ciphertext.
static void pairs_scratch(slz_ctx *ctx) {
    __atomic_store_n(&ctx->pair_asked, 1, __ATOMIC_RELAXED);
    const uint32_t pairs = slz_pairs_most(ctx) / 2;
    const size_t words = (SLZ_PAIR_WORDS * sizeof(uint32_t) + 255) & ~(size_t)255;
    void *buf = nullptr;
    hipEvent_t ev;
    if (slz_scratch_alloc(&buf, words + (size_t)pairs * 2 * 2 * (ctx->prm.N / 2) * 16) != SLZ_OK) return;
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess) { (void)hipGetLastError(); (void)hipFree(buf); return; }
    ctx->pair_ctl = (uint32_t *)buf;
    ctx->pair_mail = (char *)buf + words;
    ctx->pair_done = ev;
}

// Whether pairs for `batch` ciphertexts all find a place at once, two compute units each; otherwise one workgroup on each is faster.  100 steps of N = 2048, us with
// one workgroup / pairs: on 64 compute units 32 ciphertexts 943 / 675, 64: 945 / 1325; on 240 compute units 128: 949 / 1321; on 8 (one of each XCD,
// where a pair has no place) 1: 939 / 2950.
int slz_pairs_fit(uint32_t batch, hipStream_t s) { return batch <= SLZ_PAIR_MAX && slz_pairs_grid(batch) <= slz_compute_units(s); }

static int pairs_free(slz_ctx *ctx, int wanted, hipStream_t s) {
    beside_captures allowed;
    if (!ctx->pair_asked) pairs_scratch(ctx);
    if (!wanted || !ctx->pair_ctl) return 0;
    if (!ctx->pair_used) return 1;
    // the same stream's earlier launches come first anyway, unless the handle has passed on to a new stream
    const bool done = ctx->pair_stream == s || hipEventQuery((hipEvent_t)ctx->pair_done) == hipSuccess;
    if (done && hipStreamWaitEvent(s, (hipEvent_t)ctx->pair_done, 0) == hipSuccess) return 1;
    (void)hipGetLastError();
    return 0;
}
// The context's words and mail for a launch on s (where it wants them), or 0: calls of one context on several streams may overlap, and a captured call may be
// replayed at any time, so those that could meet an earlier launch's use of them keep to the kernels that need none; so does a call that comes while
// another thread's has them in hand, between here and slz_pairs_release.
int slz_pairs_acquire(slz_ctx *ctx, int wanted, hipStream_t s) {
    if (!wanted && __atomic_load_n(&ctx->pair_asked, __ATOMIC_RELAXED)) return 0;
    if (in_capture(s) || __atomic_exchange_n(&ctx->pair_held, 1, __ATOMIC_ACQUIRE)) return 0;
    if (pairs_free(ctx, wanted, s)) return 1;
    __atomic_store_n(&ctx->pair_held, 0, __ATOMIC_RELEASE);
    return 0;
}
// rc: of the launches.  Where one of them or the event behind them failed, nothing tells when the memory is free again: it stays held, and the
// context runs without pairs from then on.
int slz_pairs_release(slz_ctx *ctx, int rc, hipStream_t s) {
    if (rc != SLZ_OK) return rc;
    SLZ_HIP(hipEventRecord((hipEvent_t)ctx->pair_done, s));
    ctx->pair_used = 1;
    ctx->pair_stream = s;
    __atomic_store_n(&ctx->pair_held, 0, __ATOMIC_RELEASE);
    return SLZ_OK;
}
__global__ void __launch_bounds__(256) k_pairs_clear(uint32_t *ctl) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < SLZ_PAIR_WORDS) ctl[i] = 0;
}
void slz_pairs_clear(slz_ctx *ctx, hipStream_t s) {
    hipLaunchKernelGGL(k_pairs_clear, dim3((SLZ_PAIR_WORDS + 255) / 256), dim3(256), 0, s, ctx->pair_ctl);
}

int slz_fft_init(slz_ctx *ctx) {
    const host_tables &h = tables(ctx->prm.N);
    std::memcpy(ctx->fft_f1, h.f1, sizeof(h.f1));
    SLZ_HIP(hipMalloc((void **)&ctx->fft_tab, h.t.size() * sizeof(cpl)));
    SLZ_HIP(hipMalloc((void **)&ctx->fft_prep_tab, h.w.size() * sizeof(double)));
    SLZ_HIP(hipMemcpy(ctx->fft_tab, h.t.data(), h.t.size() * sizeof(cpl), hipMemcpyHostToDevice));
    SLZ_HIP(hipMemcpy(ctx->fft_prep_tab, h.w.data(), h.w.size() * sizeof(double), hipMemcpyHostToDevice));
    return ctx->prm.N == 4096 ? slz_fft4096_setup() : ctx->prm.N == 2048 ? slz_fft2048_setup() : ctx->prm.N == 1024 ? slz_fft1024_setup() : slz_fft512_setup();
}

void slz_fft_destroy(slz_ctx *ctx) {
    if (ctx->pair_done) (void)hipEventDestroy((hipEvent_t)ctx->pair_done);
    if (ctx->pair_ctl) (void)hipFree(ctx->pair_ctl);
    ctx->pair_done = ctx->pair_mail = nullptr;
    ctx->pair_ctl = nullptr;
    if (ctx->fft_tab) (void)hipFree(ctx->fft_tab);
    if (ctx->fft_prep_tab) (void)hipFree(ctx->fft_prep_tab);
    ctx->fft_tab = nullptr;
    ctx->fft_prep_tab = nullptr;
}

size_t slz_fft_key_bytes(const slz_params *p) {
    if (slz_fft4096_supported(p)) return (size_t)p->n * F12_KEY_STEP * 16;
    return slz_fft_supported(p) ? (size_t)p->n * (p->N == 2048 ? FFT_KEY_STEP : p->N == 1024 ? F10_KEY_STEP : F9_KEY_STEP) * 16 : 0;
}

// ---- key spectra ----------------------------------------------------------------------------------------------------
// Double-double arithmetic (error-free sums and products; the build contracts nothing by itself).
struct dd { double h, l; };
__device__ __forceinline__ dd dd_norm(double a, double b) { const double s = a + b; return {s, b - (s - a)}; }      // |a| >= |b|
__device__ __forceinline__ dd dd_add(dd a, dd b) {
    const double s = a.h + b.h, t = s - a.h;
    const double e = (a.h - (s - t)) + (b.h - t);
    return dd_norm(s, e + (a.l + b.l));
}
__device__ __forceinline__ dd dd_neg(dd a) { return {-a.h, -a.l}; }
__device__ __forceinline__ dd dd_mul(dd a, dd b) {
    const double p = a.h * b.h;
    return dd_norm(p, __builtin_fma(a.h, b.h, -p) + (a.h * b.l + a.l * b.h));
}

// One workgroup per (key polynomial, piece): the forward transform of the piece in double-double, times -1 / M, rounded (the
// kernel keeps its accumulator negated).
// Step layout [piece][half g][k][row, component][lane]: K points per lane, M / (64 K) halves.
template <uint32_t M, uint32_t ROWS, uint32_t K, int PIECES, int BITS>
__global__ void __launch_bounds__(256)
k_fft_prepare(const uint64_t *__restrict__ bsk, const double *__restrict__ wtab, double2 *__restrict__ dst) {
    __shared__ double rh[M], rl[M], ih[M], il[M];
    const uint32_t poly = blockIdx.x, piece = blockIdx.y;          // poly = (step * ROWS + row) * 2 + component
    const uint64_t *src = bsk + (size_t)poly * (2 * M);
    auto digit = [&](uint64_t w) {
        int64_t v = (int64_t)w, d = 0;
        for (uint32_t j = 0; j <= piece; j++) {
            const int bits = j == PIECES - 1 ? 64 - BITS * (PIECES - 1) : BITS;
            d = (int64_t)((uint64_t)v << (64 - bits)) >> (64 - bits);
            v = (int64_t)((uint64_t)v - (uint64_t)d) >> BITS;
        }
        return (double)d;
    };
    for (uint32_t x = threadIdx.x; x < M; x += 256) {
        rh[x] = digit(src[x]);
        ih[x] = digit(src[x + M]);
        rl[x] = il[x] = 0.0;
    }
    __syncthreads();
    for (uint32_t m = 1, half = M / 2; m < M; m *= 2, half /= 2) {
        for (uint32_t b = threadIdx.x; b < M / 2; b += 256) {
            const uint32_t blk = b / half, x = blk * 2 * half + b % half, y = x + half;
            const double *w = wtab + 4 * (size_t)(m + blk);
            const dd wr = {w[0], w[1]}, wi = {w[2], w[3]}, ar = {rh[x], rl[x]}, ai = {ih[x], il[x]}, br = {rh[y], rl[y]}, bi = {ih[y], il[y]};
            const dd tr = dd_add(dd_mul(br, wr), dd_neg(dd_mul(bi, wi))), ti = dd_add(dd_mul(br, wi), dd_mul(bi, wr));
            const dd pr = dd_add(ar, tr), pi = dd_add(ai, ti), qr = dd_add(ar, dd_neg(tr)), qi = dd_add(ai, dd_neg(ti));
            rh[x] = pr.h; rl[x] = pr.l; ih[x] = pi.h; il[x] = pi.l;
            rh[y] = qr.h; rl[y] = qr.l; ih[y] = qi.h; il[y] = qi.l;
        }
        __syncthreads();
    }
    constexpr uint32_t RC = 2 * ROWS, halves = M / (64 * K), step_len = PIECES * M * RC;
    const uint32_t step = poly / RC, rc = poly % RC;
    for (uint32_t x = threadIdx.x; x < M; x += 256) {
        const uint32_t g = x / (64 * K), lane = (x / K) & 63u, k = x % K;
        double2 v;
        v.x = rh[x] * (-1.0 / M);
        v.y = ih[x] * (-1.0 / M);
        dst[(size_t)step * step_len + (((piece * halves + g) * K + k) * RC + rc) * 64 + lane] = v;
    }
}

int slz_fft_prepare(slz_ctx *ctx, const uint64_t *bsk, void *dst, hipStream_t s) {
    const uint32_t polys = ctx->prm.n * 4 * ctx->prm.pbs_level;
    auto launch = [&](auto kernel, uint32_t pieces) {
        hipLaunchKernelGGL(kernel, dim3(polys, pieces), dim3(256), 0, s, bsk, ctx->fft_prep_tab, (double2 *)dst);
    };
    if (ctx->prm.N == 4096) launch(k_fft_prepare<2048, 2, 8, SLZ_FFT_PIECES, SLZ_FFT_PIECE_BITS>, SLZ_FFT_PIECES);
    else if (ctx->prm.N == 2048) launch(k_fft_prepare<1024, 2, 8, SLZ_FFT_PIECES, SLZ_FFT_PIECE_BITS>, SLZ_FFT_PIECES);
    else if (ctx->prm.N == 1024) launch(k_fft_prepare<512, 2, 8, SLZ_FFT_PIECES, SLZ_FFT_PIECE_BITS>, SLZ_FFT_PIECES);
    else launch(k_fft_prepare<256, 4, 4, F9_PIECES, F9_PIECE_BITS>, F9_PIECES);
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

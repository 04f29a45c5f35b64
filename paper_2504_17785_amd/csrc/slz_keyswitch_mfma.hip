// LWE key switching as an int8 matrix-core contraction (gfx950 v_mfma_i32_32x32x32_i8).
//
// out[c][x] -= sum_rho d_rho(c) * KSK_rho[x] (mod 2^64) is a dense product of the digit matrix (ciphertexts x key rows,
// digits in [-B/2, B/2), one byte each when B <= 2^8) with the key matrix (key rows x output words).  A 64-bit key word w
// is recoded into eight signed bytes s_p in [-128, 128) with w = sum_p s_p 2^(8p) (mod 2^64): s_p is byte p of
// (w + 0x80..80) with its top bit flipped.  Each byte plane is one int8 x int8 -> int32 contraction; the eight plane sums
// are recombined with shifts at the end.  Products are at most 2^14 in magnitude, so an int32 accumulator is exact for
// fewer than 2^17 key rows; the host keeps every segment of the row index below that, and a workgroup that takes a range
// adds its sums to the output before it gets there.
//
// Row order inside the contraction is level-major, rho = j * kN + i, so that 16 consecutive rows are 16 consecutive mask
// words at one level (kN must be a multiple of 32).
#include "slz_internal.h"
#include "slz_modarith.h"
#include "slz_mfma_i8.h"

#define KM_WAVES 8                      // waves per workgroup = 32-ciphertext tiles per workgroup
#define KM_THREADS (64 * KM_WAVES)
#define KM_IT_KB (KM_WAVES / 2)         // 32-row blocks per iteration: each thread brings in 8 rows of one output word
#define KM_TARGET_WGS 768               // workgroups aimed for when the row index is cut into segments (three per CU)
#define KM_RANGES_GROUPS_PREP 16        // ciphertext groups up to which workgroups take ranges of rows across x tiles: operand form,
#define KM_RANGES_GROUPS_STD 8          // standard key
#define KM_ROUND_BLOCKS 20              // a further round of workgroups (first loads, sums) in blocks of a workgroup's work
#define KM_BUF_V4 (KM_IT_KB * 2 * 8 * 32)   // 16-byte slots per LDS buffer: [block][half][plane][x]

// ---- digits --------------------------------------------------------------------------------------------------------
// dig[tile][kb][lane] (16 bytes): the A operand of lane `lane` for 32-row block kb of 32-ciphertext tile `tile`:
// ciphertext 32 tile + lane % 32, rows 32 kb + 16 (lane / 32) + t for byte t.  Ciphertexts past the batch get zero digits.
// Signed digits without a carry chain: with H = sum_j (B/2) B^(l-j), digit j of v is ((v + H) >> beta (l-j)) mod B - B/2.
// A workgroup takes 32 ciphertexts x 128 mask words: every wave reads whole 512-byte runs of a ciphertext, the digit bytes
// are turned through LDS (rows of 128 + 16 bytes: the 16-byte reads of 8 neighbouring lanes then cover all banks), and
// every store instruction writes one 1 KiB operand block.
// init: where the contraction adds its segments up, the output's (0, b') is written here as well, a run of the tile's 32 (n + 1) consecutive words by
// each workgroup of it (a launch of its own took 5 us of 110 at 1024 ciphertexts of kN = 2048, n = 742; as a part of every ciphertext's
// words, 26 of 801 at kN = 4096, 33 ciphertexts of that size took 42.2 us against 42.0 with the launch, now 40.1, and 4096 675 against 665, now 670;
// 1024 of kN = 2048, n = 742: 107.1 against 108.9, now 106.2).
#define KD_WORDS 128
#define KD_PITCH (KD_WORDS + 16)
#define KD_LEVELS 8                     // levels turned through LDS at a time
__global__ void __launch_bounds__(256)
k_ksm_digits(const uint64_t *__restrict__ lwe_in, v4i *__restrict__ dig, uint32_t kN, uint32_t beta, uint32_t l, uint32_t batch,
             uint32_t n_kb, uint64_t *__restrict__ init, uint32_t n) {
    __shared__ __attribute__((aligned(16))) unsigned char L[KD_LEVELS * 32 * KD_PITCH];
    const uint32_t lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const uint32_t w0 = blockIdx.x * KD_WORDS, tile = blockIdx.y;
    const uint32_t n_blk = min((kN - w0) / 32u, (uint32_t)KD_WORDS / 32u);    // 32-word blocks of this workgroup (kN % 32 == 0)
    const uint32_t bits = beta * l;
    const uint32_t half_b = 1u << (beta - 1), half = 0x01010101u * half_b;
    uint64_t H = 0;
    for (uint32_t j = 0; j < l; j++) H |= (uint64_t)half_b << (beta * j);
    // wave `wave` reads ciphertexts 8 wave .. 8 wave + 7 of the tile, a half-wave 128 words of one, four of a lane.  Unconditional, of the nearest words
    // that exist, and all before the first is used; four digits are one LDS store.  With two words of a lane per ciphertext, behind conditions, and a store per
    // digit, the keyswitch took, kN = 2048, n = 742, 24 ciphertexts 20.9 us, now 20.5, 1024: 88.9, now 87.4; kN = 1024, 256: 29.8, now 29.1.
    const uint32_t c0 = 8 * wave + lane / 32, wl = 4 * (lane % 32);
    uint64_t v[4][4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const uint64_t *src = lwe_in + (size_t)min(tile * 32 + c0 + 2 * q, batch - 1) * (kN + 1) + min(w0 + wl, kN - 4);
#pragma unroll
        for (int h = 0; h < 4; h++) v[q][h] = src[h];
    }
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
        for (int h = 0; h < 4; h++) v[q][h] = slz_round_top_bits(tile * 32 + c0 + 2 * q < batch ? v[q][h] : 0ull, bits) + H;
    if (init) {
        const uint32_t width = n + 1, total = min(32u, batch - 32 * tile) * width, part = (total + gridDim.x - 1) / gridDim.x;
        const uint32_t end = min(total, (blockIdx.x + 1) * part);
        uint64_t *dst = init + (size_t)tile * 32 * width;
        uint32_t c = blockIdx.x * part / width, x = blockIdx.x * part - c * width + threadIdx.x;
        for (uint32_t i = blockIdx.x * part + threadIdx.x; i < end; i += 256, x += 256) {
            while (x >= width) { x -= width; c++; }
            dst[i] = x == n ? lwe_in[(size_t)(32 * tile + c) * (kN + 1) + kN] : 0ull;
        }
    }
    for (uint32_t j0 = 0; j0 < l; j0 += KD_LEVELS) {
        const uint32_t nj = min(l - j0, (uint32_t)KD_LEVELS);
        if (j0) __syncthreads();                                    // the previous group has been read
        for (uint32_t jj = 0; jj < nj; jj++) {                     // level j0 + jj + 1, most significant first
            const uint32_t sh = beta * (l - 1 - (j0 + jj));
#pragma unroll
            for (int q = 0; q < 4; q++) {
                uint32_t u = 0;
#pragma unroll
                for (int h = 0; h < 4; h++) u |= ((uint32_t)(v[q][h] >> sh) & (2 * half_b - 1)) << 8 * h;
                // u - B/2 in each byte: no borrow leaves a byte whose top bit is set and made right afterwards
                u = ((u | 0x80808080u) - (half & 0x7f7f7f7fu)) ^ ((u ^ ~half) & 0x80808080u);
                *reinterpret_cast<uint32_t *>(&L[(jj * 32 + c0 + 2 * q) * KD_PITCH + wl]) = u;
            }
        }
        __syncthreads();
        // operand blocks (level, 32-word block) of this group, dealt to the waves; lane = ciphertext + 32 half
        for (uint32_t ob = wave; ob < nj * n_blk; ob += 4) {
            const uint32_t jj = ob / n_blk, kbl = ob % n_blk;
            const v4i o = *reinterpret_cast<const v4i *>(&L[(jj * 32 + lane % 32) * KD_PITCH + 32 * kbl + 16 * (lane / 32)]);
            const uint32_t kb = ((j0 + jj) * kN + w0) / 32 + kbl;
            dig[((size_t)tile * n_kb + kb) * 64 + lane] = o;
        }
    }
}

// ---- key in operand form ----------------------------------------------------------------------------------------------
// The contraction's B operands, ready to be copied into LDS: P[x tile][block kb][half][plane p][x in tile] (16 bytes):
// byte t = signed byte p of the key word of row 32 kb + 16 half + t, output word 32 (x tile) + x.  Words past n and
// blocks past the last row (the block count is padded to a multiple of 2 KM_IT_KB) are zero.  One iteration of a
// workgroup (KM_IT_KB blocks of one x tile) is KM_BUF_V4 consecutive entries, in the order of its LDS buffer.
#define KM_KB_PAD (2 * KM_IT_KB)
__host__ __device__ static inline uint32_t ksm_padded_blocks(uint32_t n_kb) { return (n_kb + KM_KB_PAD - 1) / KM_KB_PAD * KM_KB_PAD; }

__global__ void __launch_bounds__(256)
k_ksk_prepare(const uint64_t *__restrict__ ksk, v4i *__restrict__ out, uint32_t kN, uint32_t n, uint32_t l, uint32_t n_kb,
              uint32_t n_kb_pad, uint32_t x_tiles) {
    const uint32_t xl = threadIdx.x % 32, half = (threadIdx.x / 32) % 2;
    const uint32_t kb = blockIdx.x * 4 + threadIdx.x / 64, xt = blockIdx.y;
    if (kb >= n_kb_pad) return;
    const uint32_t x = xt * 32 + xl, width = n + 1;
    uint64_t w[16];
#pragma unroll
    for (int t = 0; t < 16; t++) {
        const uint32_t rho = 32 * kb + 16 * half + t;             // level-major row: rho = j kN + i
        const uint32_t j = rho / kN, i = rho % kN;
        w[t] = (kb < n_kb && x < width) ? slz_signed_bytes(ksk[((size_t)i * l + j) * width + x]) : 0ull;
    }
    uint64_t lo[8], hi[8], pl[8], ph[8];
#pragma unroll
    for (int t = 0; t < 8; t++) { lo[t] = w[t]; hi[t] = w[8 + t]; }
    slz_byte_planes(lo, pl);
    slz_byte_planes(hi, ph);
    v4i *dst = out + (((size_t)xt * n_kb_pad + kb) * 2 + half) * 8 * 32 + xl;
#pragma unroll
    for (int p = 0; p < 8; p++) {
        v4i o = {(int)(uint32_t)pl[p], (int)(uint32_t)(pl[p] >> 32), (int)(uint32_t)ph[p], (int)(uint32_t)(ph[p] >> 32)};
        dst[p * 32] = o;
    }
}

// ---- contraction ---------------------------------------------------------------------------------------------------
struct ksm_args {
    const uint64_t *ksk;
    const v4i *kskp;        // prepared key (k_ksk_prepare) or null
    const v4i *dig;
    const uint64_t *lwe_in; // this chunk's input ciphertexts (for the bodies when direct)
    uint64_t *out;
    uint32_t direct;        // one segment: a workgroup owns its output words and stores (0, b') - sum itself; otherwise
                            // `out` already holds (0, b') and the segments are combined with atomics
    uint32_t kN, n, l, batch;
    uint32_t n_tiles;       // 32-ciphertext tiles in dig
    uint32_t n_kb;          // 32-row blocks in total (l kN / 32)
    uint32_t kb_cap;        // most blocks between two flushes of the accumulators (int32)
    uint32_t x_tiles, ct_groups;
    // Which blocks of which x tile a workgroup takes, as a range of positions x tile * padded blocks + block (multiples of 2 KM_IT_KB):
    // by segments, work items (segment, x tile, ciphertext group), group fastest;
    uint32_t kb_per_seg, total, per_xcd;
    // by ranges: the positions are cut into 8 ranges_per_xcd equal ones, each taken by ct_groups workgroups
    uint32_t ranges_per_xcd, range;
};

// PREP: the key comes in operand form (A.kskp) and goes from global memory to LDS as it is; otherwise every thread recodes
// eight words of the standard key per iteration.
template <bool PREP, bool RANGES>
__global__ void __launch_bounds__(KM_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_ksm_main(ksm_args A) {
    __shared__ v4i lds[2 * KM_BUF_V4];                              // 64 KiB
    const uint32_t kb_pad = ksm_padded_blocks(A.n_kb);
    uint32_t cg, begin, end;
    if (RANGES) {
        // The workgroups of an XCD take consecutive ranges, ct_groups of them the same one: they read the same key words at the same time, and the digits
        // of a range are read by the x tiles that share it.
        const uint32_t r = blockIdx.x / 8, range = (blockIdx.x % 8) * A.ranges_per_xcd + r / A.ct_groups;
        cg = r % A.ct_groups;
        begin = range * A.range;
        end = min(begin + A.range, A.x_tiles * kb_pad);
        if (begin >= end) return;
    } else {
        // work items are dealt so that one XCD (workgroups b, b+8, ...) walks a contiguous range: the workgroups resident on
        // it share a segment of the key and neighbouring output words, which its L2 then serves
        const uint32_t item = (blockIdx.x % 8) * A.per_xcd + blockIdx.x / 8;
        if (blockIdx.x / 8 >= A.per_xcd || item >= A.total) return;
        // inside a segment the order is (block of 8 ciphertext groups, x tile, group in the block): the 64 workgroups resident on
        // an XCD are then about 8 groups x 8 x tiles, and its L2 sees each of their digit and key streams once instead of the
        // digits of 64 groups against one x tile (the digit operands are the larger stream)
        const uint32_t per_seg = A.ct_groups * A.x_tiles;
        const uint32_t seg = item / per_seg, r = item % per_seg;
        const uint32_t n_full = A.ct_groups / 8, blk = 8 * A.x_tiles;
        uint32_t xt;
        if (r < n_full * blk) {
            cg = (r / blk) * 8 + r % 8;
            xt = (r % blk) / 8;
        } else {                                                    // the last, narrower block
            const uint32_t rr = r - n_full * blk, w = A.ct_groups - n_full * 8;
            cg = n_full * 8 + rr % w;
            xt = rr / w;
        }
        begin = xt * kb_pad + seg * A.kb_per_seg;
        end = min(begin + A.kb_per_seg, (xt + 1) * kb_pad);
    }
    const uint32_t lane = threadIdx.x % 64;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const uint32_t tile = cg * KM_WAVES + wave;
    const bool tile_ok = tile < A.n_tiles;
    const uint32_t width = A.n + 1;

    // key-loading role: output word x, rows 8 oct .. 8 oct + 7 of the iteration's 32 KM_IT_KB rows
    const uint32_t xl = lane % 32;
    const uint32_t oct = 2 * wave + lane / 32;
    const size_t row_stride = (size_t)A.l * width;                  // words between consecutive mask indices at one level
    // where the next requests are: x tile and block, level j and mask index i of this thread's first row; they advance by 32 KM_IT_KB rows per
    // iteration, from the last block of an x tile to the first of the next one
    uint32_t req_at = begin, req_xt = begin / kb_pad, req_kb = begin % kb_pad;
    const uint32_t req_end = RANGES ? A.n_kb : min(A.n_kb, req_kb + (end - begin));
    bool req_ok = req_xt * 32 + xl < width;
    uint32_t j = (req_kb * 32 + 8 * oct) / A.kN, i = (req_kb * 32 + 8 * oct) % A.kN;
    const uint32_t lds_w = ((((oct / 4) * 2 + (oct / 2) % 2) * 8) * 32 + xl) * 2 + (oct & 1);   // in 8-byte units, plane 0

    // Two register stages of key words and digit operands: what iteration t consumes was requested during iteration t-2,
    // so a load has two iterations of MFMAs to arrive.  Loads are unconditional (rows or words out of range read a valid
    // address and are replaced by zero when consumed), which keeps the wait counts static.
    uint64_t kw0[8], kw1[8];
    bool ok0, ok1;
    v4i an0[KM_IT_KB], an1[KM_IT_KB];
    // operand form: the iteration's KM_BUF_V4 entries are consecutive; a thread moves entries tid + KM_THREADS u (the same
    // eight registers hold them as four 16-byte values)
    uint32_t dig_kb;                                                // block of the last key request: its digits are requested next
    auto load_key = [&](uint64_t (&kw)[8], bool &ok) {
        dig_kb = req_kb;
        if (PREP) {
            // blocks up to the padded count exist (zero past the last row)
            const uint32_t kbc = RANGES ? req_kb : min(req_kb, kb_pad - KM_IT_KB);
            const v4i *src = A.kskp + ((size_t)req_xt * kb_pad + kbc) * (2 * 8 * 32) + threadIdx.x;
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const v4i v = src[u * KM_THREADS];
                kw[2 * u] = (uint64_t)(uint32_t)v[0] | ((uint64_t)(uint32_t)v[1] << 32);
                kw[2 * u + 1] = (uint64_t)(uint32_t)v[2] | ((uint64_t)(uint32_t)v[3] << 32);
            }
            ok = true;
        } else {
            ok = req_ok && req_kb + oct / 4 < req_end;
            const uint64_t *src = A.ksk + (ok ? ((size_t)i * A.l + j) * width + req_xt * 32 + xl : (size_t)0);
#pragma unroll
            for (int t = 0; t < 8; t++) kw[t] = src[(size_t)t * row_stride];
            i += 32 * KM_IT_KB;
            while (i >= A.kN) { i -= A.kN; j++; }
        }
        if (!RANGES) {                                              // past the end: clamped, or one line, and unused
            req_kb += KM_IT_KB;
            return;
        }
        req_at += KM_IT_KB;
        if (req_at >= end) {                                        // past the end: the last entries, or one line, again
            req_ok = false;
            return;
        }
        req_kb += KM_IT_KB;
        if (req_kb == kb_pad) {
            req_kb = 0;
            req_xt++;
            req_ok = req_xt * 32 + xl < width;
            j = 8 * oct / A.kN;
            i = 8 * oct % A.kN;
        }
    };
    const size_t dig_base = (size_t)(tile_ok ? tile : 0) * A.n_kb;
    auto load_dig = [&](v4i (&an)[KM_IT_KB]) {
        // blocks past the last row meet zero key bytes, so their digits need no masking
#pragma unroll
        for (int q = 0; q < KM_IT_KB; q++) an[q] = A.dig[(dig_base + min(dig_kb + q, A.n_kb - 1)) * 64 + lane];
    };

    v16i acc[8];
#pragma unroll
    for (int p = 0; p < 8; p++)
#pragma unroll
        for (int r = 0; r < 16; r++) acc[p][r] = 0;

    uint32_t buf = 0;
    auto body = [&](uint64_t (&kw)[8], bool &ok, v4i (&an)[KM_IT_KB]) {
        // recode to signed bytes, transpose 8 rows x 8 planes, park the plane operands in LDS
        if (PREP) {
            uint64_t *dst = reinterpret_cast<uint64_t *>(lds + buf * KM_BUF_V4 + threadIdx.x);
#pragma unroll
            for (int u = 0; u < 4; u++) {
                dst[u * KM_THREADS * 2] = kw[2 * u];
                dst[u * KM_THREADS * 2 + 1] = kw[2 * u + 1];
            }
        } else {
            uint64_t w[8], plane[8];
#pragma unroll
            for (int t = 0; t < 8; t++) w[t] = ok ? slz_signed_bytes(kw[t]) : 0ull;
            slz_byte_planes(w, plane);
            uint64_t *dst = reinterpret_cast<uint64_t *>(lds + buf * KM_BUF_V4) + lds_w;
#pragma unroll
            for (int p = 0; p < 8; p++) dst[(size_t)p * 64] = plane[p];
        }
        load_key(kw, ok);
        __syncthreads();
        // one barrier per iteration is enough with two buffers: a wave reaches the barrier of iteration t only after it
        // has read everything of iteration t-1, and buffer (t+1)%2 is not written before that barrier
        if (tile_ok) {
            // the plane operands of the next half block are read from LDS while four MFMAs run
            const v4i *src = lds + buf * KM_BUF_V4 + (lane / 32) * (8 * 32) + xl;
            v4i bb[2][4];
#pragma unroll
            for (int p = 0; p < 4; p++) bb[0][p] = src[p * 32];
#pragma unroll
            for (int g = 0; g < 2 * KM_IT_KB; g++) {               // half block g: block g/2, planes 4 (g%2) .. +3
                if (g + 1 < 2 * KM_IT_KB) {
#pragma unroll
                    for (int p = 0; p < 4; p++) bb[(g + 1) & 1][p] = src[(((g + 1) / 2) * 2 * 8 + 4 * ((g + 1) % 2) + p) * 32];
                }
                __builtin_amdgcn_sched_barrier(0);      // keep the reads above the MFMAs they overlap with
#pragma unroll
                for (int p = 0; p < 4; p++)
                    acc[4 * (g % 2) + p] = __builtin_amdgcn_mfma_i32_32x32x32_i8(an[g / 2], bb[g & 1][p], acc[4 * (g % 2) + p], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        load_dig(an);
        buf ^= 1;
    };
    load_key(kw0, ok0);
    load_dig(an0);
    load_key(kw1, ok1);
    load_dig(an1);
    auto add_up = [&](uint32_t xt) {
        uint32_t ln = lane;
        if (RANGES) asm volatile("" : "+v"(ln));                    // the addresses below are made here and not kept through the iterations
        const uint32_t x = xt * 32 + ln % 32;
        if (!tile_ok || x >= width) return;
        // accumulator register r of a lane is ciphertext 8 (r / 4) + 4 (lane / 32) + r % 4 of the tile, output word x
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const uint32_t c = tile * 32 + 8 * (r / 4) + 4 * (ln / 32) + (r % 4);
            if (c < A.batch) {
                uint64_t val = 0;
#pragma unroll
                for (int p = 0; p < 8; p++) val += (uint64_t)(int64_t)acc[p][r] << (8 * p);
                if (!RANGES && A.direct) {
                    const uint64_t base = x == A.n ? A.lwe_in[(size_t)c * (A.kN + 1) + A.kN] : 0ull;
                    A.out[(size_t)c * width + x] = base - val;
                } else {
                    atomicAdd((unsigned long long *)&A.out[(size_t)c * width + x], (unsigned long long)(0 - val));
                }
            }
        }
    };
    uint32_t xt = begin / kb_pad, kb = begin % kb_pad, summed = 0;
    for (uint32_t at = begin; at < end; at += 2 * KM_IT_KB) {
        body(kw0, ok0, an0);
        body(kw1, ok1, an1);
        if (!RANGES) continue;
        kb += 2 * KM_IT_KB;
        summed += 2 * KM_IT_KB;
        if (kb < kb_pad && at + 2 * KM_IT_KB < end && summed < A.kb_cap) continue;
        // the sums of this x tile so far go out; what the next iterations need is on its way
        add_up(xt);
#pragma unroll
        for (int p = 0; p < 8; p++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[p][r] = 0;
        summed = 0;
        if (kb == kb_pad) { kb = 0; xt++; }
    }
    if (!RANGES) add_up(xt);
}

int slz_ksm_supported(const slz_params *p) {
    return p->ks_base_log <= 8 && ((uint64_t)p->k * p->N) % 32 == 0;
}

void slz_ksm_destroy(slz_ctx *ctx) {
    if (ctx->ks_dig) (void)hipFree(ctx->ks_dig);
    ctx->ks_dig = nullptr;
}

// How the contraction of `batch` ciphertexts is cut, into A: its grid by segments, or, with A.ranges_per_xcd not 0, by ranges.
static int ksm_plan(const slz_params &p, uint32_t batch, bool prepared, ksm_args &A, uint32_t &grid) {
    const uint32_t kN = p.k * p.N;
    const uint32_t n_kb = (uint32_t)((uint64_t)p.ks_level * kN / 32);
    A.kN = kN; A.n = p.n; A.l = p.ks_level;
    A.n_kb = n_kb;
    A.x_tiles = (p.n + 1 + 31) / 32;
    A.batch = batch;
    A.n_tiles = (batch + 31) / 32;
    A.ct_groups = (A.n_tiles + KM_WAVES - 1) / KM_WAVES;
    // int32 accumulators: 32 kb_per_seg rows of |digit * byte| <= 2^(beta-1) * 2^7 must stay strictly below 2^31
    A.kb_cap = (1u << (20 - p.ks_base_log)) - 2 * KM_IT_KB;
    // segments of the row index: enough workgroups for three rounds over the 256 CUs (a workgroup spends about half
    // its time outside the MFMA loop at ten iterations, so fewer, longer segments with idle CUs measured no better)
    uint32_t segs = (KM_TARGET_WGS + A.x_tiles * A.ct_groups - 1) / (A.x_tiles * A.ct_groups);
    segs = max(1u, min(segs, (n_kb + 7) / 8));
    uint32_t kbs = ((n_kb + segs - 1) / segs + 2 * KM_IT_KB - 1) / (2 * KM_IT_KB) * (2 * KM_IT_KB);
    kbs = min(kbs, A.kb_cap);
    segs = (n_kb + kbs - 1) / kbs;
    A.kb_per_seg = kbs;
    const uint64_t total = (uint64_t)segs * A.x_tiles * A.ct_groups;
    if (total > (1u << 30)) return SLZ_E_UNSUPPORTED;
    A.total = (uint32_t)total;
    A.per_xcd = (A.total + 7) / 8;
    A.direct = segs == 1;
    A.ranges_per_xcd = A.range = 0;
    grid = A.per_xcd * 8;
    // Ranges of rows across x tiles, one per resident workgroup, instead of three rounds of segments: a workgroup's first loads and the
    // sums it adds to the output come once (or twice, at the end of an x tile) and not three times.  us, segments / ranges, standard
    // (prepared) key, kN = 2048, n = 742: 64 ciphertexts 27.9 / 23.3 (25.3 / 20.9), 512: 79 / 55 (74 / 51), 1024: 112 / 86 (104 / 79),
    // 2048: 171 / 148 (160 / 133), 4096: 294 / 287 (272 / 253); kN = 1024, 777: 73 / 46 (67 / 42); kN = 4096, 1024: 210 / 161
    // (196 / 145); kN = 32768, n = 1024, 24: 320 / 339 (293 / 241), 256: 518 / 527 (472 / 413).  Past 16 groups half of the workgroups
    // would be left out; past 8 the recoding of a standard key, done by each of the groups, wants the third workgroup of a CU's queue.
    // A standard key past the 256 MB of the memory-side cache comes from memory in rows of 8 (n + 1) bytes, of which the workgroups of
    // an XCD read the whole width together only by segments.
    const bool from_memory = !prepared && (uint64_t)kN * p.ks_level * (p.n + 1) * 8 > (256u << 20);
    if (segs == 1 || A.ct_groups > (prepared ? KM_RANGES_GROUPS_PREP : KM_RANGES_GROUPS_STD) || from_memory) return SLZ_OK;
    // Whether they are the shorter way, counted in blocks.  They are not where a number of groups that does not divide 32 leaves workgroups out and the
    // segments come out even (kN = 4096, n = 800, prepared key, blocks by segments / ranges: 11 groups 4 x 216 / 1040, 419 / 437 us, 13: 452 / 478;
    // 9: 4 x 160 / 696, 336 / 320, 14: 5 x 216 / 1040, 533 / 498; kN = 32768, 7: 4 x 1280 / 5280, 2514 / 2687), nor where the segments are one round and no
    // range is longer than one of them (kN = 2048, n = 300, l = 3, 256 ciphertexts, standard key: 24.2 / 27.3).
    const uint32_t per_xcd = 32 / A.ct_groups, unit = 2 * KM_IT_KB, positions = A.x_tiles * ksm_padded_blocks(n_kb);
    const uint32_t range = ((positions + 8 * per_xcd - 1) / (8 * per_xcd) + unit - 1) / unit * unit;
    const uint64_t rounds = (A.total + 255) / 256;
    if (range >= rounds * kbs + KM_ROUND_BLOCKS * (rounds - 1)) return SLZ_OK;
    A.ranges_per_xcd = per_xcd;
    A.range = range;
    grid = 8 * per_xcd * A.ct_groups;
    return SLZ_OK;
}
// tested on the host
int slz_ksm_takes_ranges(const slz_params *p, uint32_t batch, int prepared) {
    ksm_args A;
    uint32_t grid;
    return ksm_plan(*p, batch, prepared, A, grid) == SLZ_OK && A.ranges_per_xcd;
}

// The launches of one keyswitch given its digit scratch (`dig`: room for max_tiles 32-ciphertext tiles).
static int ksm_run(const slz_params &p, void *dig, uint32_t max_tiles, const uint64_t *lwe_in, const uint64_t *ksk, const void *kskp,
                   uint64_t *lwe_out, uint32_t batch, hipStream_t s) {
    const uint32_t kN = p.k * p.N;
    ksm_args A;
    A.ksk = ksk;
    A.kskp = (const v4i *)kskp;
    A.dig = (const v4i *)dig;
    for (uint32_t c0 = 0; c0 < batch; c0 += max_tiles * 32) {
        uint32_t grid;
        const int rc = ksm_plan(p, min(batch - c0, max_tiles * 32), kskp, A, grid);
        if (rc != SLZ_OK) return rc;
        A.out = lwe_out + (size_t)c0 * (p.n + 1);
        A.lwe_in = lwe_in + (size_t)c0 * (kN + 1);
        hipLaunchKernelGGL(k_ksm_digits, dim3((kN + KD_WORDS - 1) / KD_WORDS, A.n_tiles), dim3(256), 0, s, A.lwe_in, (v4i *)dig, kN, p.ks_base_log,
                           p.ks_level, A.batch, A.n_kb, A.direct ? nullptr : A.out, p.n);
        auto *kernel = kskp ? A.ranges_per_xcd ? k_ksm_main<true, true> : k_ksm_main<true, false>
                            : A.ranges_per_xcd ? k_ksm_main<false, true> : k_ksm_main<false, false>;
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(KM_THREADS), 0, s, A);
    }
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

// Size of the key in operand form, 0 when the parameter set does not use the matrix cores.
size_t slz_ksm_prepared_bytes(const slz_params *p) {
    if (!slz_ksm_supported(p)) return 0;
    const uint64_t n_kb64 = (uint64_t)p->ks_level * p->k * p->N / 32;
    if (n_kb64 > (1u << 26)) return 0;
    const size_t x_tiles = (p->n + 1 + 31) / 32;
    return x_tiles * ksm_padded_blocks((uint32_t)n_kb64) * (2 * 8 * 32) * sizeof(v4i);
}

int slz_ksm_prepare(slz_ctx *ctx, const uint64_t *ksk, void *dst, hipStream_t s) {
    const slz_params &p = ctx->prm;
    const uint32_t kN = p.k * p.N, n_kb = (uint32_t)((uint64_t)p.ks_level * kN / 32), n_kb_pad = ksm_padded_blocks(n_kb);
    const uint32_t x_tiles = (p.n + 1 + 31) / 32;
    hipLaunchKernelGGL(k_ksk_prepare, dim3((n_kb_pad + 3) / 4, x_tiles), dim3(256), 0, s, ksk, (v4i *)dst, kN, p.n, p.ks_level, n_kb,
                       n_kb_pad, x_tiles);
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

// Exactly one of ksk (standard form) and kskp (operand form) is given.  Writes every word of lwe_out.
int slz_ksm_launch(slz_ctx *ctx, const uint64_t *lwe_in, const uint64_t *ksk, const void *kskp, uint64_t *lwe_out, uint32_t batch,
                   hipStream_t s) {
    const slz_params &p = ctx->prm;
    const uint64_t n_kb64 = (uint64_t)p.ks_level * p.k * p.N / 32;
    if (n_kb64 > (1u << 26)) return SLZ_E_UNSUPPORTED;
    const uint32_t max_tiles = min((ctx->max_batch + 31) / 32, 32768u);
    if (!ctx->ks_dig) {     // digit scratch, sized for max_batch (larger batches go through in chunks)
        if (slz_scratch_alloc(&ctx->ks_dig, (size_t)max_tiles * n_kb64 * 1024) != SLZ_OK) return SLZ_E_NOMEM;
    }
    return ksm_run(p, ctx->ks_dig, max_tiles, lwe_in, ksk, kskp, lwe_out, batch, s);
}

// ---- the variant that allocates nothing ------------------------------------------------------------------------------
// Digit scratch for callers that cannot allocate: a file-scope device array (every device the library runs on holds its
// own copy until the process ends).  Host code never passes the array's name to a kernel: the device address is looked
// up once per device and kept in scratch_ptr.
#define SLZ_KS_STATIC_MAX_DEVICES 64
static __device__ __align__(256) unsigned char scratch[SLZ_KS_STATIC_SCRATCH_BYTES];
static void *scratch_ptr[SLZ_KS_STATIC_MAX_DEVICES];

extern "C" int slz_keyswitch_batch_static(slz_ctx *ctx, const uint64_t *lwe_in_dev, const uint64_t *ksk_dev, uint64_t *lwe_out_dev,
                                          uint32_t batch, void *hip_stream) {
    if (!ctx || !lwe_in_dev || !ksk_dev || !lwe_out_dev || batch == 0) return SLZ_E_INVALID_ARG;
    if (((uintptr_t)lwe_in_dev & 7u) || ((uintptr_t)ksk_dev & 15u) || ((uintptr_t)lwe_out_dev & 7u)) return SLZ_E_INVALID_ARG;
    const slz_params &p = ctx->prm;
    if (!slz_ksm_supported(&p)) return SLZ_E_UNSUPPORTED;
    const uint64_t n_kb64 = (uint64_t)p.ks_level * p.k * p.N / 32;
    if (n_kb64 > (1u << 26)) return SLZ_E_UNSUPPORTED;
    const uint64_t tiles = ((uint64_t)batch + 31) / 32;
    if (tiles * n_kb64 * 1024 > (uint64_t)SLZ_KS_STATIC_SCRATCH_BYTES) return SLZ_E_TOO_LARGE;
    int dev = -1;
    SLZ_HIP(hipGetDevice(&dev));
    if (dev != ctx->device || dev < 0 || dev >= SLZ_KS_STATIC_MAX_DEVICES) return SLZ_E_INVALID_ARG;
    if (!scratch_ptr[dev]) {
        void *ptr = nullptr;
        SLZ_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return SLZ_E_HIP;
        scratch_ptr[dev] = ptr;
    }
    hipStream_t s = (hipStream_t)hip_stream;
    // every digit slot of the tiles in use is rewritten by k_ksm_digits (ciphertexts past the batch get zeros), so the
    // contents the previous call left behind are never read
    return ksm_run(p, scratch_ptr[dev], (uint32_t)tiles, lwe_in_dev, ksk_dev, nullptr, lwe_out_dev, batch, s);
}

// Blind rotation for N = 32768 (32 blocks of 1024, k = 1, two levels; no other set) as one launch whose workgroups go through all CMux steps
// together.  A team of 32 workgroups, one per compute unit of an XCD, takes one ciphertext at a time: accumulator and transforms (2.5 MiB at
// N = 32768) stay in that XCD's 4 MiB L2, where the passes as launches of their own (slz_bign.hip) write them back to the memory-side
// cache at the end of every launch and read them from there; what an XCD reads past its L2 is the key, 4 MiB per step.
//
// us per step, the two launches of slz_bign.hip -> here: 1 ciphertext 21.7 -> 15.4, 4: 25 -> 15.5, 8: 32.5 -> 16.2.  A step is 38 k cycles: rows 20 k (14 k of
// them FP64 issue on the SIMDs), turn 8 k, lift 6 k, and three times 1.5 k from the last store of a phase to the first load of the next.  Measured
// on the way: key words in 256-byte runs N / 4 apart, requested with the row's inputs 24.0; during the arithmetic, in 8 KiB runs 17.3;
// two teams per compute unit (128 registers) 19.4 per ciphertext, and two ciphertexts that take turns in one workgroup 17.2: beyond 4 MiB both
// read their transforms past the L2 again; with the inputs and results left out (nothing but phases, LDS and the key from the L2) 10.
//
// Memory order.  The vector L1 caches are not coherent; an XCD's L2 is shared by all its compute units.  What a phase writes goes to the
// L2 by plain stores (the L1 writes through; s_waitcnt vmcnt(0) waits for the L2's acknowledgement before the task is reported done), what it reads of
// other tasks comes by agent-scope loads, which pass the L1.  This holds only inside one XCD, so a list of ciphertexts has an owner:
// the first workgroup to come writes the XCC_ID that it runs on, and workgroups of other XCDs leave the list alone.
//
// Every wait ends.  A slot (1 / XCD_SLOTS of every phase's tasks) belongs to the workgroup that joined with its number, or is claimed phase by
// phase by a workgroup that has done its own part of the phase; a claim is only made by a workgroup that runs, and waits only for tasks of
// earlier phases.  So the first unfinished phase always has all its tasks either claimed by running workgroups that wait for nothing, or claimed next by
// one of them; nothing depends on how many workgroups are resident, or on which XCDs the launch was dealt to.  That holds for control words that this
// launch alone writes.  A call that overlaps another one on its context, which its caller has to prevent, clears them under it: accumulators and transforms are
// lost then, as in the other kernels, and a wait would have no end.  So a wait gives up after `patience` looks, and so do all behind it; what a
// workgroup reads and writes does not go out of range by that, as no address is taken from another's results.
#include "slz_bign.h"
#include "slz_xcd.h"

#define XCD_LISTS 8u             // one per XCD
#define XCD_SLOTS 32u
static_assert(SLZ_XCD_WORKGROUPS == XCD_LISTS * XCD_SLOTS, "one workgroup per slot");
#define XCD_OWNED 0x80000000u
// control words of a list (uint32_t), in lines of their own
#define XCD_CTL 256u
#define XCD_OWNER 0u
#define XCD_JOINED 32u
#define XCD_DONE 64u
#define XCD_SLOT 96u

struct xcd_args {
    bign_args a;                 // X [list][2][R][N], acc [batch][2][N]; bskp_step: the key of step 0; step: not used
    uint32_t *ctl;               // [lists][XCD_CTL], zero
    uint32_t lists, n_steps;
    uint32_t patience;           // looks of a wait until it gives up, one at least
};

__device__ __forceinline__ double ld_l2(const double *uniform_base, uint32_t lane_byte_off) {
    return __hip_atomic_load(reinterpret_cast<const double *>(reinterpret_cast<const char *>(uniform_base) + lane_byte_off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_l2(const uint64_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// The lane, opaque: what depends on it is computed in the phase that uses it.  Otherwise the addresses of every phase are kept for the whole
// launch, and spilled: 20 reloads from memory a step, half as long as the step.
__device__ __forceinline__ uint32_t xcd_lane() {
    uint32_t lane = threadIdx.x & 63u;
    asm volatile("" : "+v"(lane));
    return lane;
}

// done[slot]: how many of the list's phases the slot's tasks are done of.  Words of one line that 32 workgroups store to and 32 lanes of a
// wave read at once: a counter instead, 32 atomic additions to one word: 17.0 us per step against 16.2.
// All slots' tasks of the phases before `phase` are done, or this was the last of `patience` looks (see above): then every wait after it takes one.
__device__ __forceinline__ void xcd_wait(const uint32_t *done, uint32_t phase, uint32_t wave, uint32_t &patience) {
    if (wave == 0) {
        uint32_t left = patience;
        while (__builtin_amdgcn_ballot_w64(__hip_atomic_load(done + (threadIdx.x & (XCD_SLOTS - 1u)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < phase))
            if (--left == 0) { patience = left = 1; break; }
    }
    __syncthreads();
}
__device__ __forceinline__ void xcd_finish(uint32_t *done, uint32_t slot, uint32_t phase) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // this wave's stores have reached the L2
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(done + slot, phase + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A step is three phases of 32 tasks:
//   turn:  rotate, subtract, decompose and forward column stages for 64 columns of one component
//   rows:  blocks i and G - 1 - i of one prime: the forward stages inside the block, products with the key, the inverse stages
//   lift:  inverse column stages, lift and accumulation for 64 columns of one component
struct xcd_ct {                  // the ciphertext at hand
    uint64_t *acc;               // [2][N]
    double *X;                   // [2][R][N]; after the rows components 0 and 1 of a prime are in place of its rows 0 and 1
    const uint64_t *lwe;
};

// Lift, columns 64 (task >> 1) .. of component task & 1.  (prime, quarter of the rows) run the inverse stages inside a
// quarter; each wave then takes an eighth of the row quadruples (j, j + G / 4, ..) for the last two stages, both primes, and the lift.
template <int G>
__device__ __forceinline__ void xcd_lift(const xcd_args &K, const xcd_ct &ct, double *res, uint32_t wave, uint32_t task, const uint32_t *done, uint32_t phase, uint32_t &patience) {
    constexpr int Q = G / 4, J = Q / 8;
    static_assert(J >= 1, "eight waves share the quadruples");
    const bign_args &A = K.a;
    const uint32_t lane = xcd_lane();
    const uint32_t comp = task & 1u, c = 64 * (task >> 1) + lane;
    const uint32_t N = 1024u * G;
    uint64_t *acc = ct.acc + (size_t)comp * N;
    xcd_wait(done, phase, wave, patience);
    const uint32_t j0 = wave * J;
    uint64_t w[J][4];
    {
        const uint32_t q = wave >> 2, part = wave & 3u;
        const slz_mod m = A.mod[q];
        double y[Q], bd[Q];
        const double *src = ct.X + ((size_t)q * 4 + comp) * N + 1024u * part * Q;
#pragma unroll
        for (int i = 0; i < Q; i++) { y[i] = ld_l2(src + 1024u * i, c * 8u); bd[i] = 0.51; }
#pragma unroll
        for (int k = 0; k < J; k++)
#pragma unroll
            for (int i = 0; i < 4; i++) w[k][i] = ld_l2(&acc[1024u * (j0 + k + Q * i) + c]);
        cols_mirror<Q>(y, bd, colI_of(A.tab[q], G), part, 4, m);
        lazy_limit(y, bd, LAZY_MAX / 4, m);
#pragma unroll
        for (int i = 0; i < Q; i++) res[(q * G + part * Q + i) * 64 + lane] = y[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < J; k++) {
        double r[2][4];
#pragma unroll
        for (int p = 0; p < 2; p++) {
            const slz_mod m = A.mod[p];
            const double *colI = colI_of(A.tab[p], G);
#pragma unroll
            for (int i = 0; i < 4; i++) r[p][i] = res[(p * G + j0 + k + Q * i) * 64 + lane];
#pragma unroll
            for (int h = 0; h < 4; h += 2) {                     // the last stage but one: rows Q apart, block h / 2 of 2
                const double s = r[p][h] + r[p][h + 1], d = r[p][h] - r[p][h + 1];
                r[p][h] = s;
                r[p][h + 1] = slz_mulmod(d, colI[2 + h / 2], m);
            }
            cols_mirror_last(r[p][0], r[p][2], colI, m);
            cols_mirror_last(r[p][1], r[p][3], colI, m);
        }
#pragma unroll
        for (int i = 0; i < 4; i++) acc[1024u * (j0 + k + Q * i) + c] = w[k][i] + slz_crt64(r[0][i], r[1][i], A.mod[1], A.p1inv_mod_p2);
    }
}

// Non-temporal: the key streams through the L2 and should not drive out what the team passes on in it.
typedef double xcd_two __attribute__((ext_vector_type(2)));
// Key words FROM .. TO - 1 of both components that this wave multiplies with; key: its row of the block (xcd_key).
template <int FROM, int TO>
__device__ __forceinline__ void xcd_key_load(double (&kk)[2][16], const double *key, uint32_t N) {
    const uint32_t lane = xcd_lane();
    SCHED_FENCE();
#pragma unroll
    for (int i = FROM; i < TO; i += 2)
#pragma unroll
        for (int c = 0; c < 2; c++) {
            const xcd_two w = __builtin_nontemporal_load(reinterpret_cast<const xcd_two *>(reinterpret_cast<const char *>(key + (size_t)c * N + 64 * i) + lane * 16u));
            kk[c][i] = w.x;
            kk[c][i + 1] = w.y;
        }
    SCHED_FENCE();
}
// Task `slot` of the rows: four waves, one per GGSW row, on block slot / 2 and four on block G - 1 - slot / 2, prime slot & 1.
template <int G> __device__ __forceinline__ uint32_t xcd_block(uint32_t slot, uint32_t wave) { return wave >> 2 ? G - 1u - (slot >> 1) : slot >> 1; }
template <int G>
__device__ __forceinline__ const double *xcd_key(const xcd_args &K, uint32_t wave, uint32_t slot, uint32_t step) {
    return K.a.bskp_step + (((size_t)step * 2 + (slot & 1u)) * 4 + (wave & 3u)) * 2 * 1024u * G + 1024u * xcd_block<G>(slot, wave);
}
// Of the waves with the same component of a prime one collects the sums and runs the inverse transform: waves 0, 1 and 6, 7, one per SIMD.
__device__ __forceinline__ bool xcd_collects(uint32_t wave) { return ((wave >> 1) & 1u) == wave >> 2; }

// Turn, columns 64 (task >> 1) .. of component task & 1.  An eighth of the rows per wave for the digits; then (level, prime,
// half of the rows) run the forward stages.
template <int G>
__device__ __forceinline__ void xcd_turn(const xcd_args &K, const xcd_ct &ct, int32_t *digits, uint32_t wave,
                                         uint32_t task, uint32_t at, const uint32_t *done, uint32_t phase, uint32_t &patience) {
    constexpr int H = G / 2, D = G / 8;
    constexpr uint32_t N = 1024u * G;
    const bign_args &A = K.a;
    const uint32_t lane = xcd_lane();
    const uint32_t comp = task & 1u, c = 64 * (task >> 1) + lane;
    const uint32_t u = c + 2 * N - at, urow = u >> 10;           // X^at moves coefficient u (mod 2N, negated from N on) to c
    const uint64_t *acc = ct.acc + (size_t)comp * N;
    xcd_wait(done, phase, wave, patience);
    uint64_t own[D], other[D];
#pragma unroll
    for (int k = 0; k < D; k++) {
        const uint32_t from = (urow + wave * D + k) & (G - 1);
        own[k] = ld_l2(&acc[1024u * (wave * D + k) + c]);
        other[k] = ld_l2(&acc[1024u * from + (u & 1023u)]);
    }
#pragma unroll
    for (int k = 0; k < D; k++) {
        const uint32_t i = wave * D + k, from = urow + i;
        uint64_t v = slz_round_top_bits((from & G ? (uint64_t)0 - other[k] : other[k]) - own[k], A.beta * 2);
        digits[(G + i) * 64 + lane] = slz_next_digit(v, A.beta);
        digits[i * 64 + lane] = slz_next_digit(v, A.beta);
    }
    __syncthreads();
    {
        const uint32_t half = wave & 1u, q = (wave >> 1) & 1u, lev = wave >> 2;
        const slz_mod m = A.mod[q];
        const double *tw = A.tab[q].fwd;
        const int32_t *dig = digits + lev * G * 64 + lane;
        double y[H];
#pragma unroll
        for (int j = 0; j < H; j++) {
            const double a = (double)dig[j * 64], v = slz_mulmod((double)dig[(j + H) * 64], tw[1], m);
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
        double *dst = ct.X + ((size_t)q * 4 + (comp * 2 + lev)) * N + 1024u * half * H + c;
#pragma unroll
        for (int i = 0; i < H; i++) dst[1024u * i] = slz_reduce(y[i], m);
    }
}

// Rows, see k_big_rows16_team.  tabs: the two blocks' forward tables in LDS, [64] and [15][64] each; the one's are the other's inverse ones,
// read backwards (inv16_mirror).  key, next: the wave's key words of this step and of the one after.
// 128 KiB of key words per step and compute unit come from beyond the L2 at 11 to 13 bytes per clock, in order with every other load of the
// compute unit, and a wave that asks for more than a few at once waits to issue: so they are asked for a few at a time during the arithmetic,
// half of them from the sums of the step before on (kk_half: done), half during the forward stages.
template <int G>
__device__ __forceinline__ void xcd_rows(const xcd_args &K, const xcd_ct &ct, double (&kk)[2][16], bool kk_half, const uint64_t *ahead, uint64_t &ahead_word, const double *key, const double *next, double *lds, const double *tabs, uint32_t wave,
                                         uint32_t slot, const uint32_t *done, uint32_t phase, uint32_t &patience) {
    constexpr uint32_t R = 4, N = 1024u * G;
    const bign_args &A = K.a;
    const uint32_t lane = xcd_lane();
    const uint32_t q = slot & 1u, h = wave >> 2, r = wave & 3u, row = xcd_block<G>(slot, wave);
    const slz_mod m = A.mod[q];
    double *T = lds + wave * 1024u, *T_other = lds + (wave ^ 1u) * 1024u;
    const double *twA = tabs + h * 1024u, *twB = twA + 64, *mirror = tabs + (h ^ 1u) * 1024u;
    int z;
    asm volatile("s_mov_b32 %0, 0" : "=s"(z));
    double x[16];
    if (!kk_half) xcd_key_load<0, 8>(kk, key, N);
    xcd_wait(done, phase, wave, patience);
    {
        const double *src = ct.X + ((size_t)q * R + r) * N + 1024u * row;
#pragma unroll
        for (int e = 0; e < 16; e++) x[e] = ld_l2(src + 64 * e, lane * 8u);
    }
    ahead_word = *ahead;                                         // mask word of the step after: here its way from memory costs nothing
    SCHED_FENCE();
    fwd16<false, true>(x, T, twA, twB, m, lane, z, [&](int s) {
        if (s == 0) xcd_key_load<8, 10>(kk, key, N);
        if (s == 1) xcd_key_load<10, 12>(kk, key, N);
        if (s == 2) xcd_key_load<12, 14>(kk, key, N);
        if (s == 3) xcd_key_load<14, 16>(kk, key, N);
    });
    wave_sync();
    asm volatile("" : "+v"(ahead_word));
    double o[16];                                                // the component this wave sums: r & 1
#pragma unroll
    for (int g = 0; g < 4; g++) {
        double r0[4], r1[4], x4[4], k0[4], k1[4];
#pragma unroll
        for (int u = 0; u < 4; u++) { x4[u] = x[4 * g + u]; k0[u] = kk[0][4 * g + u]; k1[u] = kk[1][4 * g + u]; }
        mulmod_k<4>(r0, x4, k0, m);
        mulmod_k<4>(r1, x4, k1, m);
#pragma unroll
        for (int u = 0; u < 4; u++) {
            o[4 * g + u] = r & 1u ? r1[u] : r0[u];
            T[64 * (4 * g + u) + lane] = r & 1u ? r0[u] : r1[u];
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; i++) o[i] += T_other[64 * i + lane];
    const bool collects = xcd_collects(wave);                    // of the pairs of waves 2 r' and 2 r' + 1 one hands its sums to the other
    if (!collects) {
#pragma unroll
        for (int i = 0; i < 16; i++) T_other[64 * i + lane] = o[i];             // read by this wave alone before
    }
    __syncthreads();
    if (!collects) xcd_key_load<0, 8>(kk, next, N);
    if (collects) {
        double twi[15];
#pragma unroll
        for (int t = 1; t < 16; t <<= 1)
#pragma unroll
            for (int k = 0; k < t; k++) twi[t - 1 + k] = mirror[64 * (2 * t - 1 - k) + 63u - lane];      // entry 2 t - 2 - k of [15][64] behind [64]
        const double *P = lds + (wave ^ 3u) * 1024u;             // where the wave of the other pair with the same component has put its sums
#pragma unroll
        for (int i = 0; i < 16; i++) o[i] += P[64 * i + lane];
#pragma unroll
        for (int g = 0; g < 2; g++) {
            double r8[8], x8[8];
#pragma unroll
            for (int u = 0; u < 8; u++) x8[u] = o[8 * g + u];
            reduce_k<8>(r8, x8, m);
#pragma unroll
            for (int u = 0; u < 8; u++) o[8 * g + u] = r8[u];
        }
        // T_other has no other reader any more
        inv16_mirror<true>(o, T_other, mirror, twi, m, lane, z, [&](int s) {
            if (s == 0) xcd_key_load<0, 2>(kk, next, N);
            if (s == 1) xcd_key_load<2, 4>(kk, next, N);
            if (s == 2) xcd_key_load<4, 6>(kk, next, N);
            if (s == 3) xcd_key_load<6, 8>(kk, next, N);
        });
        double *dst = ct.X + ((size_t)q * R + (r & 1u)) * N + 1024u * row;     // the four waves have read the block
#pragma unroll
        for (int g = 0; g < 2; g++) {
            double r8[8], x8[8];
#pragma unroll
            for (int u = 0; u < 8; u++) x8[u] = o[8 * g + u];
            reduce_k<8>(r8, x8, m);
#pragma unroll
            for (int u = 0; u < 8; u++) dst[64 * (8 * g + u) + lane] = r8[u];
        }
    }
}

// LDS: a transform buffer per wave, then the tables of two blocks, whose first entry nobody reads: in it a workgroup's first wave tells the
// others what it has found.
#define XCD_LDS ((8 * 1024 + 2048) * sizeof(double))
template <int G>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_big_xcd(xcd_args K) {
    static_assert(G == 32, "a slot is one task of every phase; 2 N = 2^16");
    constexpr uint32_t N = 1024u * G;
    extern __shared__ double lds[];
    double *tabs = lds + 8 * 1024;
    uint32_t *told = reinterpret_cast<uint32_t *>(tabs);
    const bign_args &A = K.a;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t xcc = slz_xcc_id();
    double kk[2][16];
    const double *kk_of = nullptr;                               // the block and step whose first half of the key words kk holds
    uint32_t tab_slot = ~0u;
    uint32_t patience = K.patience;
    auto broadcast = [&](uint32_t v) -> uint32_t {               // thread 0's value to all
        __syncthreads();
        if (threadIdx.x == 0) *told = v;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(*told);
    };
    for (uint32_t k = 0; k < K.lists; k++) {
        const uint32_t list = (xcc + k) % K.lists;
        uint32_t *ctl = K.ctl + list * XCD_CTL, *done = ctl + XCD_DONE;
        uint32_t rank = XCD_OWNED;
        if (threadIdx.x == 0) {
            uint32_t owner = 0;
            __hip_atomic_compare_exchange_strong(ctl + XCD_OWNER, &owner, xcc + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (owner == 0 || owner == xcc + 1) rank = __hip_atomic_fetch_add(ctl + XCD_JOINED, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        rank = broadcast(rank);
        if (rank == XCD_OWNED) continue;                         // another XCD's list
        if (rank >= XCD_SLOTS) return;                           // every slot has a workgroup that runs
        const uint32_t rounds = (A.batch - list + K.lists - 1) / K.lists, total = rounds * K.n_steps;
        xcd_ct ct;
        auto choose = [&](uint32_t round) {
            const size_t b = min(list + round * K.lists, A.batch - 1);      // past the last one: chosen, not used
            ct.acc = A.acc + b * 2 * N;
            ct.lwe = A.lwe_in + b * (A.n + 1);
            ct.X = A.X + (size_t)list * 2 * 4 * N;
        };
        // phase 0, 1, 2 of the list's step p
        uint64_t mask_word;                                      // of the step
        auto turn = [&](uint32_t slot, uint32_t p) {
            xcd_turn<G>(K, ct, reinterpret_cast<int32_t *>(lds), wave, slot, slz_modswitch(mask_word, 16), done, 3 * p, patience);
            xcd_finish(done, slot, 3 * p);
        };
        auto rows = [&](uint32_t slot, uint32_t p, uint32_t step, const uint64_t *ahead, uint64_t &ahead_word) {
            if (tab_slot != slot) {
                const bign_tabs &tb = A.tab[slot & 1u];
                for (uint32_t t = 1 + threadIdx.x; t < 2048u; t += 512u) {
                    const uint32_t block = xcd_block<G>(slot, t >> 8), i = t & 1023u;
                    tabs[t] = i < 64u ? tb.rowA[block * 64 + i] : tb.rowB[block * 15 * 64 + i - 64];
                }
                tab_slot = slot;                                 // read behind the barriers of xcd_wait
            }
            const double *key = xcd_key<G>(K, wave, slot, step), *next = xcd_key<G>(K, wave, slot, step + 1 < K.n_steps ? step + 1 : 0);
            xcd_rows<G>(K, ct, kk, kk_of == key, ahead, ahead_word, key, next, lds, tabs, wave, slot, done, 3 * p + 1, patience);
            kk_of = next;
            xcd_finish(done, slot, 3 * p + 1);
        };
        auto lift = [&](uint32_t slot, uint32_t p) {
            xcd_lift<G>(K, ct, lds, wave, slot, done, 3 * p + 2, patience);
            xcd_finish(done, slot, 3 * p + 2);
        };
        // the slot of this workgroup's number is its own from the first phase on that nobody has claimed it for
        uint32_t first = 0;
        if (threadIdx.x == 0) first = __hip_atomic_fetch_or(ctl + XCD_SLOT + rank, XCD_OWNED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        first = broadcast(first);
        kk_of = nullptr;
        uint32_t p = first / 3, kind = first % 3, step = p % K.n_steps, round = p / K.n_steps;
        choose(round);
        // while there are slots that no workgroup has joined for: each phase's tasks of those go to whoever claims them first
        for (bool full = false; p < total && !(full && kind == 0);) {
            uint32_t slot = rank;
            for (;;) {
                mask_word = ct.lwe[step];
                uint64_t unused;
                if (kind == 0) turn(slot, p);
                else if (kind == 1) rows(slot, p, step, ct.lwe, unused);
                else lift(slot, p);
                if (slot == rank) {
                    slot = broadcast(threadIdx.x == 0 ? __hip_atomic_load(ctl + XCD_JOINED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u);
                    full = slot >= XCD_SLOTS;
                } else {
                    slot++;
                }
                for (; slot < XCD_SLOTS; slot++) {
                    uint32_t seen = 3 * p + kind;
                    if (threadIdx.x == 0) __hip_atomic_compare_exchange_strong(ctl + XCD_SLOT + slot, &seen, 3 * p + kind + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (broadcast(seen) == 3 * p + kind) break;
                }
                if (slot >= XCD_SLOTS) break;
            }
            if (++kind == 3) {
                kind = 0;
                p++;
                if (++step == K.n_steps) { step = 0; choose(++round); }
            }
        }
        mask_word = ct.lwe[step];
        for (; p < total; p++) {
            uint64_t ahead_word;
            turn(rank, p);
            rows(rank, p, step, step + 1 < K.n_steps ? ct.lwe + step + 1 : A.lwe_in + (size_t)min(list + (round + 1) * K.lists, A.batch - 1) * (A.n + 1), ahead_word);
            lift(rank, p);
            mask_word = ahead_word;
            if (++step == K.n_steps) { step = 0; choose(++round); }
        }
    }
}

__global__ void __launch_bounds__(256) k_xcd_clear(uint32_t *ctl, uint32_t words) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i < words) ctl[i] = 0;
}

int slz_bign_xcd_setup() {
    SLZ_HIP(hipFuncSetAttribute((const void *)k_big_xcd<32>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)XCD_LDS));
    return SLZ_OK;
}

size_t slz_bign_xcd_ctl_bytes() { return XCD_LISTS * XCD_CTL * sizeof(uint32_t); }

int slz_bign_xcd_launch(const bign_args &a, uint32_t *ctl, uint32_t n_steps, uint32_t workgroups, uint32_t patience, hipStream_t s) {
    xcd_args K;
    K.a = a;
    K.ctl = ctl;
    K.lists = a.batch < XCD_LISTS ? a.batch : XCD_LISTS;
    K.n_steps = n_steps;
    K.patience = patience;
    hipLaunchKernelGGL(k_xcd_clear, dim3(K.lists * XCD_CTL / 256), dim3(256), 0, s, ctl, K.lists * XCD_CTL);
    hipLaunchKernelGGL(k_big_xcd<32>, dim3(workgroups), dim3(512), XCD_LDS, s, K);
    SLZ_HIP(hipGetLastError());
    return SLZ_OK;
}

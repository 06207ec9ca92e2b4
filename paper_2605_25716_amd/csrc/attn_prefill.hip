// Prefill-shaped partial attention (Section 4.1, per-node local computation) for 16-bit storage: many query rows
// per head against one KV shard.  Bound by the matrix pipe at the clock the chip sustains on real operand data plus
// the part of the softmax's vector work that does not overlap it.  Vector instructions overlap matrix instructions
// best inside one wave (in the shadow of that wave's own MFMAs), so each wave software-pipelines across key tiles:
// in iteration t it computes S^T(t) = K'(t) Q'^T and then issues the MFMAs of O^T += V'(t-1)^T P(t-1)^T together with
// the online softmax of tile t.
//   * one workgroup = 8 or 4 waves x 32 query rows of one (sequence, query head); the launch chooses (see below);
//   * K'/V' tiles of 64 keys are shared by the waves through LDS (two slots each), filled by LDS-direct global
//     loads one iteration ahead (no staging registers), one workgroup barrier per iteration;
//   * LDS tiles are unpadded (LDS-direct loads write 64 consecutive 16-byte slots per wave); bank conflicts are
//     avoided by XOR-swizzling the 16-byte chunk index with the row;
//   * both products are computed transposed, S^T = K' Q'^T and O^T = V'^T P^T (32x32x16 MFMA), so the fp32 score
//     tile already sits in the lane layout the second product wants for P^T: probabilities never cross lanes.
//     K' operands are 16-byte LDS reads; V'^T operands come from the row-major V' tile through the transposing LDS
//     read (ds_read_b64_tr_b16), so V' is never transposed in memory or in registers;
//   * workgroups that share a KV head are placed on the same XCD (shared L2);
//   * QB = 8 or 4: K', V' arrive as the transport codec's codes (Section 7.5).  The LDS-direct loads are replaced by
//     ordinary loads of the codes and of the rows' (scale, lo) one iteration ahead; each thread rebuilds its 8-element
//     chunk exactly as the dequantise call would (fp32 fma, one narrowing) and writes it to the same swizzled LDS slot,
//     so everything downstream is unchanged and consumes the same values as dequantise-then-attend.
#include <type_traits>

#include "fedrag_device.h"
#include "fedrag_host.h"

namespace fedrag {

#ifndef FEDRAG_PRE_PD
#define FEDRAG_PRE_PD 4
#endif
constexpr int kPrePD = FEDRAG_PRE_PD;         // MFMA operands are read from LDS this many MFMAs ahead

// CAUSAL: the queries are the last Lq of the L tokens whose K'/V' are given, and query i sees keys 0 .. i + (L - Lq)
// (Section 5.3: the Inquirer's own part of a decoder layer's attention).  That call works on plaintext V, whose
// outlier channels are not spread by a scrambling matrix (|v| of several tens), so a probability rounded once to the
// storage type (relative error 2^-9 in bf16) would move an output by more than the 16-bit output tolerance.  The
// CAUSAL instantiation therefore feeds the second product P = P_hi + P_lo, two storage-type terms (about 16
// significant bits), at the price of twice the MFMAs of that product.
// WALK: several shards whose query tiles alone cover the chip.  A workgroup visits the shards one after the other and carries
// its maximum, sum and output along: no partials and no aggregation.  The probabilities of a shard are rounded against the
// shard's own running maximum, as they are in a launch of its own: its first tile starts the maximum anew, 2^32 below the
// weight collected so far, and the output takes the fp32 factor between the two, which may be as large as that, or less where it
// would carry outputs beyond 2^120, so that values are as free as in a launch per shard.  (What stays
// below is nothing beside fp32 sums.  With the maximum carried along the weight between shards sat in the 16 bits of the
// probabilities: an error of 3.6e-4 against 64 bits where this, like a partial per shard, has 3.3e-4.)
// KG = 2: the waves form two groups that share the workgroup's query rows and halve its keys, each with tile slots of its own;
// their outputs are aggregated through LDS.  For launches of few workgroups: the same rows and keys on as many waves with half
// the query rows a workgroup, so half the runs, and half the fp32 partials to write and fold, or none.
template <class T, int D, bool CAUSAL, int QB, int NW, bool WALK, int KG>
FEDRAG_KERNEL __launch_bounds__(NW * kWave, D == 64 && NW == 4 ? 3 : 2) void prefill_attn_kernel(const typename T::elem* __restrict__ Q,
                                                                      const KeyRuns runs,
                                                                      const float* __restrict__ Kprm,
                                                                      const float* __restrict__ Vprm, int Hq,
                                                                      FastDiv by_heads, FastDiv by_group,
                                                                      FastDiv by_tiles, FastDiv by_unit,
                                                                      FastDiv by_inner, int run_by_run, int64_t Lq,
                                                                      const int32_t* __restrict__ kv_lens,
                                                                      const int32_t* __restrict__ q_lens, int n_units, int fold,
                                                                      int together, int past_l2,
                                                                      float scale_log2,
                                                                      float* __restrict__ O, float* __restrict__ lse) {
    typedef typename T::elem elem;
    typedef typename T::vec8 vec8;
    constexpr int NWG = NW / KG;             // waves of a key group
    constexpr int kThreads = NWG * kWave;
    constexpr int kQTile = NWG * kPreQ;  // query rows per workgroup
    constexpr int ROWB = D * 2;             // bytes per tile row in LDS (no padding)
    constexpr int SLOT = kPreK * ROWB;      // bytes per tile slot
    constexpr int KS = D / 16;              // contraction steps of S^T
    constexpr int MT = D / 32;              // 32-row tiles of O^T
    constexpr int CH = D / 8;               // 16-byte chunks per row
    constexpr int LPT = (kPreK * CH) / kThreads;  // LDS-direct loads (QB: 8-element chunks) per thread per tile
    static_assert(!WALK || (!CAUSAL && QB == 0), "several shards: the plain form");
    static_assert(KG == 1 || (KG == 2 && NW == 8 && QB == 0 && !CAUSAL && !WALK), "two groups of four waves: the plain form");
    static_assert(QB == 0 || QB == 8 || QB == 4, "16-bit values, or 8- / 4-bit codes");
    static_assert(QB == 0 || !CAUSAL, "codes are what travels to the Compute Node; the Inquirer's own K, V are plain");
    constexpr int CROWB = QB ? D * QB / 8 : ROWB;  // bytes per row of K' / V' as stored (values, or codes)

    // One array per tile slot: distinct objects let the compiler see that the LDS-direct load filling one slot
    // does not alias the LDS reads of another, so it does not make those reads wait for the load.
    __shared__ __attribute__((aligned(16))) char ks0_all[KG * SLOT], ks1_all[KG * SLOT], vs0_all[KG * SLOT], vs1_all[KG * SLOT];

    // XCD-aware placement: consecutive workgroup ids are dealt round-robin to the 8 XCDs (one L2 each);
    // give every XCD whole (sequence, KV head) units so that the workgroups sharing K'/V' share an L2.
    // With more than one run (several shards, or few query tiles and many keys; not CAUSAL) there is one workgroup
    // per (query tile, run) and O / lse are [n_runs][rows] partials that the Section 4.1 aggregation folds afterwards.
    // The launch chooses which of the two varies faster inside a unit (by_inner: the number of runs, or of query tiles).
    // The arguments are one trip to memory, not one per branch and division that reads them: short causal calls 4..6 % (117 rows
    // of 32 heads of 128: 8.9 -> 8.4 us), long ones 0..2 %.  The form on 8-bit codes with four waves has no register
    // to spare for them.
    if constexpr (!(QB != 0 && D == 64 && NW == 4)) {
        FEDRAG_HAVE_HERE(FEDRAG_S3(by_unit), FEDRAG_S3(by_inner), FEDRAG_S3(by_tiles), FEDRAG_S3(by_group), FEDRAG_S3(by_heads),
                         FEDRAG_S(run_by_run), FEDRAG_S(n_units), FEDRAG_S(Lq), FEDRAG_S(kv_lens), FEDRAG_S(q_lens), FEDRAG_S(Q),
                         FEDRAG_S(O), FEDRAG_S(lse), FEDRAG_S(Hq), FEDRAG_S(fold), FEDRAG_S(together), FEDRAG_S(runs.n_shards),
                         FEDRAG_S(runs.n_runs));
    }
    const int G = (int)by_group.d;
    const int n_runs = runs.n_runs;
    const int xcd = blockIdx.x % 8;
    const int slot = blockIdx.x / 8;
    // by_unit: the workgroups of a unit, G * q_tiles * n_runs, or (CAUSAL only: together) the units of an XCD, which then
    // advance side by side: the long tiles of all of them first, as below
    const int outer_slot = (int)by_unit.div(slot), inner_slot = slot - outer_slot * (int)by_unit.d;
    const int unit_slot = CAUSAL && together ? inner_slot : outer_slot;
    const int unit = xcd + 8 * unit_slot;
    if (unit >= n_units) return;
    const int in_unit = CAUSAL && together ? outer_slot : inner_slot;
    const int outer = (int)by_inner.div(in_unit), inner = in_unit - outer * (int)by_inner.d;
    const int w_in_unit = run_by_run ? inner : outer;
    const int run = run_by_run ? outer : inner;
    int split = 0;
    const KeyShard shard = WALK ? runs.s[0] : runs.shard_of(run, &split);
    FEDRAG_HAVE_HERE(FEDRAG_S(shard.K), FEDRAG_S(shard.V), FEDRAG_S(shard.L), FEDRAG_S(shard.per));
    const elem* K = (const elem*)shard.K;
    const elem* V = (const elem*)shard.V;
    const int64_t L_stride = shard.L;
    const int64_t keys_per_run = shard.per;
    // CAUSAL: later query tiles visit more keys.  Hand out the last tile of every head of the group first, then the
    // one before it, and so on: workgroups are started in index order as compute units free up, so every compute
    // unit ends up with a long tile followed by short ones and the launch does not wait on a late long tile.
    const int hg = CAUSAL ? (int)by_group.mod(w_in_unit) : (int)by_tiles.div(w_in_unit);
    int qt = (int)by_tiles.mod(w_in_unit);
    if (CAUSAL) {
        const int pos = (int)by_group.div(w_in_unit);
        const int folded = fold ? (int)(by_tiles.d + 1) / 2 : (int)by_tiles.d;  // first part: last tile first
        qt = pos < folded ? (int)by_tiles.d - 1 - pos : pos - folded;
    }
    const int b = (int)by_heads.div(unit);
    const int g = (int)by_heads.mod(unit);
    const int h = g * G + hg;

    const int tid = threadIdx.x;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid / kWave);  // wave-uniform
    const int grp = KG == 1 ? 0 : wave_all / NWG;
    const int wave = KG == 1 ? wave_all : wave_all % NWG;  // in its group
    char* const ks0 = ks0_all + grp * SLOT;
    char* const ks1 = ks1_all + grp * SLOT;
    char* const vs0 = vs0_all + grp * SLOT;
    char* const vs1 = vs1_all + grp * SLOT;
    const int lane = tid % kWave;
    const int li = lane % 32;
    const int lh = lane / 32;

    const elem* Qh = Q + ((int64_t)b * Hq + h) * Lq * D;
    const char* Kg = (const char*)K + (int64_t)unit * L_stride * CROWB;
    const char* Vg = (const char*)V + (int64_t)unit * L_stride * CROWB;
    const float* Kpg = QB ? Kprm + (int64_t)unit * L_stride * 2 : nullptr;  // (scale, lo) per key row
    const float* Vpg = QB ? Vprm + (int64_t)unit * L_stride * 2 : nullptr;
    // keys of this sequence: all L_stride rows, or the first kv_lens[b] of them (padded batch of unequal sequences)
    int64_t L = L_stride;
    // query rows of this sequence that exist (padded batch): rows past them are neither computed nor written
    int64_t Lq_rows = Lq;
    if (kv_lens || q_lens) {  // both asked for at once
        const int nk = (kv_lens ? kv_lens : q_lens)[b], nq = (q_lens ? q_lens : kv_lens)[b];
        asm volatile("" ::"v"(nk), "v"(nq));
        if (kv_lens) L = nk < 0 ? 0 : (nk < L_stride ? nk : L_stride);
        if (q_lens) Lq_rows = nq < 0 ? 0 : (nq < Lq ? nq : Lq);
    }
    if ((int64_t)qt * kQTile >= Lq_rows) return;  // workgroup-uniform, before any barrier
    const int64_t part_row0 = (int64_t)run * n_units * G * Lq;  // n_units * G * Lq = rows of one partial
    float* Oh = O + (part_row0 + ((int64_t)b * Hq + h) * Lq) * D;
    float* Lh = lse + part_row0 + ((int64_t)b * Hq + h) * Lq;
    if (!CAUSAL && !WALK && n_runs > 1) {  // this workgroup's run of keys; a run past the end is empty
        const int64_t k_begin = (int64_t)split * keys_per_run;
        const int64_t k_end = k_begin + keys_per_run < L ? k_begin + keys_per_run : L;
        L = k_end > k_begin ? k_end - k_begin : 0;
        Kg += k_begin * CROWB;
        Vg += k_begin * CROWB;
        if (QB) {
            Kpg += k_begin * 2;
            Vpg += k_begin * 2;
        }
    }

    const int64_t q_row = (int64_t)qt * kQTile + wave * kPreQ + li;  // this lane's query row
    if (L == 0) {  // no keys (workgroup-uniform, before any barrier): O = 0, lse = -inf
        if (q_row < Lq_rows) {
            for (int c = lh * (D / 2); c < (lh + 1) * (D / 2); c += 4) *(f32x4_t*)(Oh + q_row * D + c) = zero_vec<f32x4_t>();
            if (lh == 0) Lh[q_row] = -INFINITY;
        }
        return;
    }
    f32x16_t acc_o[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) acc_o[i] = zero_vec<f32x16_t>();
    // CAUSAL: the running maximum starts at the lowest finite value: a row may see no key of the first tiles that its
    // workgroup visits, and -inf - m_run has to be -inf then.  KG = 2: so may the second group's.
    float m_run = CAUSAL || KG == 2 ? -__FLT_MAX__ : -INFINITY, l_run = 0.f;

    // ---- global -> LDS (direct buffer loads).  One wave-wide load fills 64 consecutive 16-byte slots = 64 / CH
    // tile rows.  LDS slot p of row r holds global chunk p ^ swz(r): K' swz(r) = r % CH, V' swz(r) = (4 (r % 4)) % CH;
    // both depend on r only through r % 16, which is the same for every load of a thread.  The buffer resource
    // starts at the tile and covers the rest of the shard, so rows past the end of the shard arrive as zeros; tile -1 and
    // tiles past the end, which the loops ask for behind their last one, read nothing.
    constexpr int RPW = kWave / CH;  // rows per wave-wide load
    const int ld_r = wave * RPW + lane / CH;  // row within a set of NWG * RPW rows
    const int ld_p = lane % CH;               // slot within the row
    const int ld_voff_k = ld_r * ROWB + ((ld_p ^ (ld_r % CH)) << 4);
    const int ld_voff_v = ld_r * ROWB + ((ld_p ^ ((4 * (ld_r % 4)) % CH)) << 4);
    static_assert((NWG * RPW) % 16 == 0, "swizzle must not depend on the load index");
    auto load_tile = [&](const char* G_, char* slot_base, int tile, bool is_k) {
        const int64_t byte0 = (int64_t)tile * SLOT;
        const int64_t left = L * ROWB - byte0;
        const bool none = CAUSAL ? tile < 0 : left < 0;
        const int n_rec = none ? 0 : (int)(left < 0x7fffffff ? left : 0x7fffffff);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(G_ + byte0), 0, n_rec, 0x00020000);
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            char* lp = slot_base + (j * NWG + wave) * (RPW * ROWB);  // wave-uniform LDS base
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (void __attribute__((address_space(3)))*)lp, 16,
                                                     is_k ? ld_voff_k : ld_voff_v, j * (NWG * RPW * ROWB), 0, 0);
        }
    };

    // ---- QB: codes -> registers one iteration ahead, then -> LDS.  Chunk j of a thread is row (j * kThreads + tid)
    // / CH of the tile, 8 channels from 8 (tid % CH); reads past the end of the shard return zeros (code 0, scale 0,
    // lo 0: the row dequantises to zeros, as rows past the end arrive in the 16-bit path).
    struct CodeChunk {
        uint32_t c[QB == 8 ? 2 : 1];
        u32x2_t prm;
    };
    CodeChunk kst[QB ? LPT : 1], vst[QB ? LPT : 1];
    const int cq_row = tid / CH, cq_c = tid % CH;
    auto fetch_codes = [&](const char* G_, const float* Pg_, int tile, CodeChunk (&st)[QB ? LPT : 1]) {
        const int64_t row0 = (int64_t)tile * kPreK;
        const int64_t left_rows = L - row0 > 0 ? L - row0 : 0;
        const int64_t lc = left_rows * CROWB, lp = left_rows * 8;
        const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(G_ + row0 * CROWB), 0, (int)(lc < 0x7fffffff ? lc : 0x7fffffff), 0x00020000);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(Pg_ + row0 * 2), 0, (int)(lp < 0x7fffffff ? lp : 0x7fffffff), 0x00020000);
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            const int r = j * (kThreads / CH) + cq_row;
            if constexpr (QB == 8) {
                const u32x2_t w = __builtin_amdgcn_raw_buffer_load_b64(rc, r * CROWB + cq_c * 8, 0, 0);
                st[j].c[0] = w[0];
                st[j].c[1] = w[1];
            } else {
                st[j].c[0] = __builtin_amdgcn_raw_buffer_load_b32(rc, r * CROWB + cq_c * 4, 0, 0);
            }
            st[j].prm = __builtin_amdgcn_raw_buffer_load_b64(rp, r * 8, 0, 0);
        }
    };
    auto store_codes = [&](char* slot_base, const CodeChunk (&st)[QB ? LPT : 1], bool is_k) {
#pragma unroll
        for (int j = 0; j < LPT; ++j) {
            const int r = j * (kThreads / CH) + cq_row;
            const uint32_t sb = st[j].prm[0], lb = st[j].prm[1];
            const float scale = __builtin_bit_cast(float, sb), lo = __builtin_bit_cast(float, lb);
            vec8 out;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t code = QB == 8 ? (st[j].c[e / 4] >> (8 * (e % 4))) & 255u : (st[j].c[0] >> (4 * e)) & 15u;
                float x = __builtin_fmaf((float)code, scale, lo);
                pin_here(x);  // the dequantised value is the fp32 result narrowed afterwards: two roundings, not one
                out[e] = T::from_float(x);
            }
            const int swz = is_k ? r % CH : (4 * (r % 4)) % CH;
            *(vec8*)(slot_base + r * ROWB + ((cq_c ^ swz) << 4)) = out;
        }
    };

    // ---- per-lane LDS read offsets
    // K' operand (row 32 mt + li, elements 16 ks + 8 lh): chunk (2 ks + lh) ^ (li % CH)
    int k_off[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) k_off[ks] = li * ROWB + ((((2 * ks + lh) % CH) ^ (li % CH)) << 4);
    // V'^T operand through the transposing read: 16-lane group gq covers d-rows 16 (gq % 2) .. +16 of the 32-row
    // tile i; lane s of the group points at key row 4 lh + s / 4 (+8 for the second read), elements
    // 32 i + 16 (gq % 2) + 4 (s % 4) .. +4, i.e. chunk 4 i + 2 (gq % 2) + (s % 4) / 2, byte 8 ((s % 4) % 2) in it
    const int s16 = lane % 16;
    const int gq = lane / 16;
    int v_off[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        const int chunk = 4 * i + 2 * (gq % 2) + (s16 % 4) / 2;
        const int swz = (4 * ((s16 / 4) % 4)) % CH;
        v_off[i] = (4 * lh + s16 / 4) * ROWB + (((chunk % CH) ^ swz) << 4) + 8 * ((s16 % 4) % 2);
    }

    // keys this workgroup has to visit, and the first tile in which some key is hidden from some row of the
    // workgroup (past the end of the shard, or - CAUSAL - after the row's own position)
    const int64_t off = L - Lq;
    const int64_t q_first = (int64_t)qt * kQTile;
    const int64_t q_last = (q_first + kQTile < Lq ? q_first + kQTile : Lq) - 1;
    const int64_t wg_keys = CAUSAL ? (q_last + off + 1 < L ? q_last + off + 1 : L) : L;
    int n_tiles = (int)((wg_keys + kPreK - 1) / kPreK);
    int t_mask0 = (int)((CAUSAL ? (q_first + off + 1 < L ? q_first + off + 1 : L) : L) / kPreK);
    int key_lim = (int)(CAUSAL ? (q_row + off + 1 < L ? q_row + off + 1 : L) : L);  // this lane's row sees keys < key_lim
    if constexpr (KG == 2) {
        // The second group begins half-way.  Both take the same number of tiles and of masked ones (barriers are common): where the
        // count is odd the second group's last tile lies behind its keys and is masked as a whole.
        const int half = (n_tiles + 1) / 2, first = grp * half;
        n_tiles = half;
        t_mask0 = t_mask0 > half ? t_mask0 - half : 0;
        Kg += (int64_t)first * SLOT;
        Vg += (int64_t)first * SLOT;
        L -= (int64_t)first * kPreK;
        key_lim -= first * kPreK;
    }
    // prologue: K' of the first tile to visit is fetched first, Q' behind it
    int tile = CAUSAL ? n_tiles - 1 : 0;
    if constexpr (QB == 0) load_tile(Kg, ks0, tile, true);
    else fetch_codes(Kg, Kpg, tile, kst);
    const int64_t q_ld = q_row < Lq ? q_row : Lq - 1;
    vec8 qop[KS];  // Q'^T operands: column li, contraction slice 16 ks + 8 lh
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qop[ks] = *(const vec8*)(Qh + q_ld * D + ks * 16 + lh * 8);

    f32x16_t S0;      // S^T of the current tile, keys 0..31
    f32x16_t S1[2];   // S1[t & 1]: S^T of tile t, keys 32..63 (kept one iteration longer, see below)
    vec8 P[2][4];     // P[t & 1]: P^T operands of tile t, one per 16-key step
    constexpr bool SPLIT = CAUSAL;           // second storage-type term of every probability (see above)
    vec8 Plo[SPLIT ? 2 : 1][SPLIT ? 4 : 1];  // Plo[t & 1]: P - P as stored in P[t & 1], narrowed
    auto put_p = [&](int par, int kk, int e, float pe) {
        const elem hi = T::from_float(pe);
        P[par][kk][e] = hi;
        if constexpr (SPLIT) Plo[par][kk][e] = T::from_float(pe - T::to_float(hi));
    };
    // SPLIT: the first narrowing of a pair stays in its slice, as its sum does; left to the scheduler it moved behind the phase,
    // where no product hides it: 2 to 6 % of every masked call (2048 tokens x 32 heads of 128 61.2 us and 59.1, 4 x as many of 64
    // 125.6 and 122.4).  The second term is as well off where the compiler puts it, and the plain form loses nothing.
    auto pin_p = [&](int par, int kk, int w) {
        if constexpr (SPLIT) {
            u32x4_t v = __builtin_bit_cast(u32x4_t, P[par][kk]);
            uint32_t x = v[w];
            pin_here(x);
            v[w] = x;
            P[par][kk] = __builtin_bit_cast(vec8, v);
        }
    };
    float alph[2];    // alph[t & 1]: rescale factor of the running output that goes with P(t)
    int drop = 0;      // WALK: what the first tile of a shard takes off the maximum it finds

    auto read_vop = [&](const char* vt, int kk, int i) -> vec8 {
        const char* p = vt + kk * 16 * ROWB + v_off[i];
        const u32x2_t lo = lds_read_tr16(p);
        const u32x2_t hi = lds_read_tr16(p + 8 * ROWB);
        u32x4_t w;
        w[0] = lo[0]; w[1] = lo[1]; w[2] = hi[0]; w[3] = hi[1];
        return __builtin_bit_cast(vec8, w);
    };

    // One pipeline iteration t, in two MFMA phases with vector work in their shadow:
    //   A(t)   = S^T(t) = K'(t) Q'^T                     together with  B2(t-1) = probabilities of keys 32..63 of
    //                                                                   tile t-1 (its maximum is already known);
    //   C(t-1) = O^T += V'(t-1)^T P(t-1)^T               together with  B1(t) = row maximum of tile t, new running
    //                                                                   maximum, rescale factor, probabilities of
    //                                                                   keys 0..31 of tile t.
    // Splitting the softmax of a tile over two phases gives both MFMA phases about the same vector load.
    // `par` carries t % 2 as a compile-time constant so that the double-buffered register sets are addressed
    // statically.  m_run is the running maximum after tile t-1 until B1(t) replaces it.
    // t counts the visits of the pipelined part: t = 0 is its first tile and has no C, t = n is nothing but B2 and C of
    // tile n - 1, all between run both phases on tiles that every row sees whole.  Only the kFirst form masks; a masked
    // tile is one kFirst and one kLast by itself, outside the pipeline.  (A tail of masked tiles behind the steady loop, its
    // stages switched by runtime flags, spilled its registers: 9000 cycles per tile against 1300 to 2600, most of the time
    // of a segment of a few hundred tokens; masking in the steady loop made that loop 15 % slower.)
    // The order of the tiles decides which probabilities are exact (those of the keys that raise the maximum) and so the
    // bits of the result.  Plain: first to last, the one ragged tile at the end.  CAUSAL, whose two terms of P leave no such
    // error: last to first, so that the pipeline starts with the last of the tiles on the diagonal.
    // `next` is the tile after this one, whose K' is fetched meanwhile (ldK).
    enum { kFirst, kSteady, kLast };
    auto iteration = [&](int tile, int next, auto par, auto stage, bool ldK) {
        constexpr int p = decltype(par)::value;  // t & 1
        constexpr int q = 1 - p;                 // (t - 1) & 1 == (t + 1) & 1
        constexpr int kind = decltype(stage)::value;
        constexpr bool doC = kind != kFirst;
        constexpr bool doAB = kind != kLast;
        constexpr int NM = 4 * MT;
        static_assert(NM == 16 || NM == 8, "slice plans assume d = 128 or 64");
        if constexpr (QB == 0) {
            if (ldK) load_tile(Kg, q ? ks1 : ks0, next, true);  // K'(t+1) -> slot (t+1) & 1 (last read by A(t-1))
            if constexpr (doAB) load_tile(Vg, p ? vs1 : vs0, tile, false);  // V'(t) -> slot t & 1 (last read by C(t-2))
        } else {  // the codes of the same two tiles into registers; they reach their (free) slots between the phases
            if (ldK) fetch_codes(Kg, Kpg, next, kst);
            if constexpr (doAB) fetch_codes(Vg, Vpg, tile, vst);
        }

        // --- A(t) and B2(t-1).  Lane gets query li and, per 32-key half, keys 8 (r / 4) + 4 lh + r % 4, r = 0..15.
        // Contraction element e of step kk of the second product <-> key 16 kk + 8 (e / 4) + 4 lh + e % 4, so
        // register r of half 1 goes to step 2 + r / 8, element r % 8.
        const char* kt = p ? ks1 : ks0;
        if constexpr (doAB) {
            constexpr int NA = 2 * KS;  // MFMAs of A: slice j -> half j % 2, contraction step j / 2
            vec8 kop[NA];
#pragma unroll
            for (int j = 0; j < kPrePD; ++j) kop[j] = *(const vec8*)(kt + (j % 2) * 32 * ROWB + k_off[j / 2]);
            S0 = zero_vec<f32x16_t>();
            S1[p] = zero_vec<f32x16_t>();
            float psum = 0.f;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NA; ++j) {
                if (j + kPrePD < NA) kop[j + kPrePD] = *(const vec8*)(kt + ((j + kPrePD) % 2) * 32 * ROWB + k_off[(j + kPrePD) / 2]);
                if (j % 2 == 0) S0 = T::mfma32(kop[j], qop[j / 2], S0);
                else S1[p] = T::mfma32(kop[j], qop[j / 2], S1[p]);
                if constexpr (doC) {
                    const int r0 = (j * 16) / NA, r1 = ((j + 1) * 16) / NA;  // registers of half 1 handled here
#pragma unroll
                    for (int r = r0; r < r1; ++r) {
                        const float pe = fast_exp2(__builtin_fmaf(S1[q][r], scale_log2, -m_run));
                        psum += pe;
                        put_p(q, 2 + r / 8, r % 8, pe);
                        if (r % 2) pin_p(q, 2 + r / 8, (r % 8) / 2);
                    }
                    pin_here(psum);  // the slice's vector work stays in the slice
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            l_run += psum;
            if (kind == kFirst && tile >= t_mask0) {  // the ragged end, or a tile that reaches past a row's own position
                const int key0 = tile * kPreK + 4 * lh;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = key0 + 8 * (r / 4) + (r % 4);
                    if (key >= key_lim) S0[r] = -INFINITY;
                    if (key + 32 >= key_lim) S1[p][r] = -INFINITY;  // also seen by B2(t) later
                }
            }
        } else {  // B2(t-1)
            float psum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float pe = fast_exp2(__builtin_fmaf(S1[q][r], scale_log2, -m_run));
                psum += pe;
                put_p(q, 2 + r / 8, r % 8, pe);
            }
            l_run += psum;
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (QB != 0) {
            if (ldK) store_codes(q ? ks1 : ks0, kst, true);
            __builtin_amdgcn_sched_barrier(0);
        }
        const char* vt = q ? vs1 : vs0;
        if constexpr (doC) {
            if (__builtin_amdgcn_ballot_w64(alph[q] != 1.0f) != 0) {  // wave-uniform: skip when no maximum moved
#pragma unroll
                for (int i = 0; i < MT; ++i) acc_o[i] *= alph[q];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // --- C(t-1) and B1(t)
        {
            // 4 MT slices of one MFMA each, with scheduling fences between slices: a slice holds the MFMA, its
            // share of B1 and the transposing reads of the operand four MFMAs ahead.  Shares: slices 0-1 the row
            // maximum, slice 2 the new running maximum and the rescale factor, slices 2.. the 16 probabilities.
            constexpr int FIRST = 2;  // first slice that produces probabilities
            vec8 vop[NM];
            if constexpr (doC) {
#pragma unroll
                for (int j = 0; j < kPrePD; ++j) vop[j] = read_vop(vt, j / MT, j % MT);
            }
            float mx = S0[0];
            float m_new = 0.f, psum = 0.f;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NM; ++j) {
                if constexpr (doC) {
                    if (j + kPrePD < NM) vop[j + kPrePD] = read_vop(vt, (j + kPrePD) / MT, (j + kPrePD) % MT);
                    acc_o[j % MT] = T::mfma32(vop[j], P[q][j / MT], acc_o[j % MT]);
                    if constexpr (SPLIT) acc_o[j % MT] = T::mfma32(vop[j], Plo[q][j / MT], acc_o[j % MT]);
                }
                if constexpr (doAB) {
                    if (j == 0) {
#pragma unroll
                        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, S0[r]);
                    }
                    if (j == 1) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, S1[p][r]);
                    }
                    if (j == FIRST) {
                        mx = xor32_max(mx);
                        // scale > 0: max commutes with the scaling
                        const float low = WALK && kind == kFirst ? m_run - (float)drop : m_run;
                        m_new = fmaxf(low, mx * scale_log2);
                        alph[p] = exp2_diff(m_run, m_new);
                        // m_run - drop is low and what rounding took off it, far more than a rounding of a small m_run and, of a
                        // very large one, all of drop: the two are exact (Knuth's sum of two numbers), their factors one by one
                        if (WALK && kind == kFirst && m_new == low && drop != 0) {
                            const float d = (float)drop, back = low - m_run, err = (m_run - (low - back)) - (d + back);
                            alph[p] = ldexpf(fast_exp2(err), drop);
                        }
                    }
                    if (j >= FIRST) {
                        constexpr int NS = NM - FIRST;
                        const int r0 = ((j - FIRST) * 16) / NS, r1 = ((j - FIRST + 1) * 16) / NS;
#pragma unroll
                        for (int r = r0; r < r1; ++r) {
                            const float pe = fast_exp2(__builtin_fmaf(S0[r], scale_log2, -m_new));
                            psum += pe;
                            put_p(p, r / 8, r % 8, pe);
                            if (r % 2) pin_p(p, r / 8, (r % 8) / 2);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (doAB) {
                l_run = l_run * alph[p] + psum;
                m_run = m_new;
            }
        }
        if constexpr (doAB) {
            if constexpr (QB != 0) store_codes(p ? vs1 : vs0, vst, false);
            // keep this iteration's results above the barrier that follows (they are consumed in the next iteration)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                u32x4_t w = __builtin_bit_cast(u32x4_t, P[p][kk]);
                pin_here(w);
                P[p][kk] = __builtin_bit_cast(vec8, w);
                if constexpr (SPLIT) {
                    u32x4_t wl = __builtin_bit_cast(u32x4_t, Plo[p][kk]);
                    pin_here(wl);
                    Plo[p][kk] = __builtin_bit_cast(vec8, wl);
                }
            }
            pin_here(l_run);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    std::integral_constant<int, 0> even;
    std::integral_constant<int, 1> odd;
    std::integral_constant<int, kFirst> first;
    std::integral_constant<int, kSteady> steady;
    std::integral_constant<int, kLast> last;

    // Barrier that makes the tiles in flight visible to the workgroup: every wave waits for its own LDS-direct loads first.
    // (Left to the compiler the wait is missing where a loop's back edge leads to the barrier.)
    auto tile_barrier = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), the other counters untouched
        __syncthreads();
    };
    // WALK: the next shard's first K' tile is fetched behind the last step of this one, which reads no K' (slot 0 was last read
    // before the barrier ahead of it)
    auto next_shard = [&](int sh) {
        if constexpr (WALK) {
            if (sh + 1 == runs.n_shards) return;
            const KeyShard next = runs.s[sh + 1];
            L = next.L;
            Kg = (const char*)next.K + (int64_t)unit * L * CROWB;
            Vg = (const char*)next.V + (int64_t)unit * L * CROWB;
            load_tile(Kg, ks0, 0, true);
        }
    };
    if constexpr (QB != 0) store_codes(ks0, kst, true);
    alph[0] = alph[1] = 1.0f;
    tile_barrier();
    if constexpr (CAUSAL) {
        // masked tiles are finished one by one, except the last of them, which the pipeline starts with; it takes an odd
        // number of tiles
        while (tile > t_mask0 || (tile & 1)) {
            iteration(tile, 0, even, first, false);
            tile_barrier();
            --tile;
            load_tile(Kg, ks0, tile, true);
            iteration(0, 0, odd, last, false);
            tile_barrier();
        }
        iteration(tile, tile - 1, even, first, true);
        tile_barrier();
        for (; tile > 0; tile -= 2) {
            iteration(tile - 1, tile - 2, odd, steady, true);
            tile_barrier();
            iteration(tile - 2, tile - 3, even, steady, true);
            tile_barrier();
        }
        iteration(0, 0, odd, last, false);
    } else for (int sh = 0;;) {
        // the pipeline takes the largest odd number of whole tiles (tile 0 in any case); what is left, a whole tile, the
        // ragged one or both, is finished one by one behind it.  Their K' arrives in the slot of odd tiles, where the
        // pipeline's last iteration has put the next one.
        const int n_pipe = t_mask0 <= 2 ? 1 : t_mask0 - 1 + (t_mask0 & 1);
        iteration(0, 1, even, first, true);
        drop = 0;
        tile_barrier();
        for (tile = 1; tile < n_pipe; tile += 2) {
            iteration(tile, tile + 1, odd, steady, true);
            tile_barrier();
            iteration(tile + 1, tile + 2, even, steady, true);
            tile_barrier();
        }
        if (n_pipe == n_tiles) next_shard(sh);
        iteration(0, 0, odd, last, false);
        for (tile = n_pipe; tile < n_tiles;) {
            iteration(tile, 0, odd, first, false);
            tile_barrier();
            const bool more = ++tile < n_tiles;
            if (more) {
                if constexpr (QB == 0) load_tile(Kg, ks1, tile, true);
                else fetch_codes(Kg, Kpg, tile, kst);
            } else {
                next_shard(sh);
            }
            iteration(0, 0, even, last, false);
            if (!more) break;
            if constexpr (QB != 0) store_codes(ks1, kst, true);
            tile_barrier();
        }
        if (!WALK || ++sh == runs.n_shards) break;
        tile = 0;
        n_tiles = (int)((L + kPreK - 1) / kPreK);
        t_mask0 = (int)(L / kPreK);
        key_lim = (int)L;
        float top = 0.f;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) top = fmaxf(top, fabsf(acc_o[i][r]));
        const int down = 32 - __builtin_amdgcn_frexp_expf(xor32_sum(l_run)), room = 120 - __builtin_amdgcn_frexp_expf(xor32_max(top));
        drop = down < room ? down : room;
        tile_barrier();
    }

    // epilogue: lane holds query li and rows d = 32 i + 8 (r / 4) + 4 lh + r % 4 of O^T.  The rows go out through LDS
    // (the tiles are dead; every wave has its share of them), so that a store covers whole 128-byte lines: straight from
    // the accumulators it would cover 32 bytes of each of 32 rows, 4 us for a 256-row workgroup.  The 16-byte chunk
    // index is XORed with the row against bank conflicts.
    float l_tot = xor32_sum(l_run);
    __syncthreads();
    constexpr int WB = 4 * SLOT / NWG;         // bytes per wave
    constexpr int OC = D / KG;                 // output columns that are this wave's to store
    constexpr int PC = WB / (kPreQ * 4) < OC ? WB / (kPreQ * 4) : OC;  // columns per pass
    constexpr int PCH = PC / 4;                // 16-byte chunks per row and pass
    static_assert(PC % 32 == 0 && OC % PC == 0, "a pass is whole 32-column tiles");
    const int slot_w = wave_all * 4 / NW;
    char* mine = (slot_w == 0 ? ks0_all : slot_w == 1 ? ks1_all : slot_w == 2 ? vs0_all : vs1_all) + (wave_all % (NW / 4)) * WB;
    f32x16_t out[OC / 32];
    if constexpr (KG == 1) {
#pragma unroll
        for (int i = 0; i < MT; ++i) out[i] = acc_o[i];
    } else {
        // The other group's wave holds the same rows over the other keys: each gives away half of the columns, with its maximum and
        // sum, and finishes the other half (Section 4.1 aggregation, in base 2).
        constexpr int HT = MT / 2;
        auto give = [&](int i0) {
#pragma unroll
            for (int i = 0; i < HT; ++i)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    f32x4_t o;
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[r] = acc_o[i0 + i][4 * r4 + r];
                    *(f32x4_t*)(mine + (i * 4 + r4) * (kWave * 16) + lane * 16) = o;
                }
        };
        if (grp == 0) give(HT);
        else give(0);
        f32x2_t ml;
        ml[0] = m_run; ml[1] = l_tot;
        *(f32x2_t*)(mine + HT * 4 * (kWave * 16) + lane * 8) = ml;
#pragma unroll
        for (int i = 0; i < HT; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float lo = acc_o[i][r], hi = acc_o[HT + i][r];
                out[i][r] = grp == 0 ? lo : hi;
            }
        __syncthreads();
        const int peer = wave_all < NWG ? wave_all + NWG : wave_all - NWG, slot_p = peer * 4 / NW;
        const char* theirs = (slot_p == 0 ? ks0_all : slot_p == 1 ? ks1_all : slot_p == 2 ? vs0_all : vs1_all) + (peer % (NW / 4)) * WB;
        ml = *(const f32x2_t*)(theirs + HT * 4 * (kWave * 16) + lane * 8);
        const float m_all = fmaxf(m_run, ml[0]);
        const float a = fast_exp2(m_run - m_all), b = fast_exp2(ml[0] - m_all);
        l_tot = l_tot * a + ml[1] * b;
        m_run = m_all;
#pragma unroll
        for (int i = 0; i < HT; ++i)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const f32x4_t o = *(const f32x4_t*)(theirs + (i * 4 + r4) * (kWave * 16) + lane * 16);
#pragma unroll
                for (int r = 0; r < 4; ++r) out[i][4 * r4 + r] = out[i][4 * r4 + r] * a + o[r] * b;
            }
        __syncthreads();
    }
    const float inv = (l_tot > 0.f) ? 1.0f / l_tot : 0.f;
    const int64_t row0 = (int64_t)qt * kQTile + wave * kPreQ;
    const int col0 = grp * OC;
#pragma unroll
    for (int c0 = 0; c0 < OC; c0 += PC) {
#pragma unroll
        for (int i = c0 / 32; i < (c0 + PC) / 32; ++i)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                f32x4_t o;
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = out[i][4 * r4 + r] * inv;
                const int chunk = 8 * (i - c0 / 32) + 2 * r4 + lh;
                *(f32x4_t*)(mine + li * (PC * 4) + ((chunk ^ (li % PCH)) << 4)) = o;
            }
        wave_lds_fence();
        auto store = [&](auto nontemporal) {
#pragma unroll
            for (int u = 0; u < kPreQ * PCH / kWave; ++u) {
                const int e = u * kWave + lane;
                const int row = e / PCH, chunk = e % PCH;
                const f32x4_t o = *(const f32x4_t*)(mine + row * (PC * 4) + ((chunk ^ (row % PCH)) << 4));
                f32x4_t* to = (f32x4_t*)(Oh + (row0 + row) * D + col0 + c0 + chunk * 4);
                if (row0 + row < Lq_rows) {
                    if constexpr (decltype(nontemporal)::value) {
                        __builtin_nontemporal_store(o, to);
                        asm volatile("");  // (two stores that differ in the hint alone would be merged into one without it)
                    } else {
                        *to = o;
                    }
                }
            }
        };
        if (past_l2) store(std::true_type{});
        else store(std::false_type{});
        wave_lds_fence();
    }
    if constexpr (WALK) {  // a sum of up to 2^32 against a maximum as far down: its exponent goes to the maximum, where it is exact
        const int e = __builtin_amdgcn_frexp_expf(l_tot);
        m_run += (float)e;
        l_tot = ldexpf(l_tot, -e);
    }
    if (grp == 0 && lh == 0 && q_row < Lq_rows) Lh[q_row] = (l_tot > 0.f) ? (m_run + fast_log2(l_tot)) * kLn2 : -INFINITY;
}

// Waves per workgroup.  Eight share a K'/V' tile between 256 query rows, one workgroup per compute unit: the best rate
// when the launch is whole rounds of them (2048 x 16384 x 32 heads of 128: 478 us, against 508 with four).  Four (128 rows) sit
// two to a compute unit, three at d = 64, fill and drain it independently and waste less of a ragged end.  q of them per unit
// take a + b q rounds of the larger form, fitted to launches of 1 to 15 per unit: b is half a round at d = 128, less where three
// overlap, more on codes, whose tiles are rebuilt for half the rows (2 x 1347 tokens x 16 heads on 8-bit codes of 64: 39 us with
// four, 35 with eight; of 128 63 and 53; 2500 x 4 x 32 heads of 64 in 16 bits 258 and 290).  Where there are several rounds a
// workgroup's start and end, some four tiles (two on codes), are half hidden behind its neighbours with four waves (4096 x 64
// rows of 128 x 500 keys: 88 us, 101 with eight).
// Always four with a mask, whose tiles are unequal (2048-token segment 62 against 79 us, 300 tokens 12 against 17), and for 16-bit
// batches with query counts, whose workgroups are fewer than the padded shape says (the 10-pair re-rank batch 29 against 42;
// where every sequence is as long as the padding, 2 to 6 % slower).  On codes such a batch goes by its padded shape.
struct PrefillCost {
    float c8, c4;  // in tiles of the larger form, for the launch with workgroups of eight and of four waves
    bool four() const { return c4 < c8; }
    float least() const { return c4 < c8 ? c4 : c8; }
};
static PrefillCost prefill_cost(int64_t wgs8, int64_t wgs4, float tiles, float ends, int D, bool codes) {
    const int64_t cus = attn_target_wgs();
    const int64_t q8 = (wgs8 + cus - 1) / cus, q4 = (wgs4 + cus - 1) / cus;
    const float a = D == 64 ? (codes ? 0.20f : 0.15f) : codes ? 0.08f : 0.05f;
    const float b = D == 64 ? (codes ? 0.465f : 0.445f) : codes ? 0.55f : 0.51f;
    return PrefillCost{(float)q8 * (tiles + ends), (a + b * (float)q4) * (tiles + 0.5f * ends)};
}
// What the choice between the forms needs in microseconds: a key tile of the larger form, and the fold of n partials of `rows`
// rows, at 7.5 bytes per ns.
static float prefill_tile_us(int D) { return D == 64 ? 1.19f : 1.77f; }
static float prefill_fold_us(int n, int64_t rows, int D) {
    return n > 1 ? 3.0f + (float)n * (float)rows * (float)(D + 1) * 4.0f / 7.5e6f : 0.0f;
}
static bool prefill_wants_4_waves(int64_t wgs8, int64_t wgs4, int64_t tiles, int D, bool codes) {
    const float ends = wgs8 <= attn_target_wgs() ? 0.0f : codes ? 2.0f : 4.0f;
    return prefill_cost(wgs8, wgs4, (float)tiles, ends, D, codes).four();
}

// Several shards: whether a workgroup visits them all (WALK), by the same cost.  Either way a workgroup's start and end take
// four tiles; a shard's end inside a walk takes one, runs of unequal length end unevenly, and the fold reads a partial per run.
// At d = 64 the walking form is itself 5 % slower.
// Only from query tiles for a whole round on: below that shards side by side fill the chip (1500 x 32 heads x 2 x 5000 keys
// 252 us, 253 to 283 walked; 1100 x 32 x 8 x 5000 714 and 960).  4096 x 64 rows of 128 x 8 x 8192 keys: 7.44 ms walked, 7.76 with
// partials; 2048 x 32 x 8 x 2048 515 and 605 us, x 8 x 512 139 and 217, x (8000 + 500) 252 and 418; 4096 x 64 of 64 x 2 x 300 62
// and 99.  Where the rounds come out uneven it is the other way: 1100 x 64 x 4 x 3000 549 and 454.
static bool prefill_walks(const AttnProblem& p, const KeyRuns& runs, int64_t heads, int64_t tiles8, int64_t tiles4, bool* four) {
    const int D = p.D;
    if (heads * tiles8 < attn_target_wgs()) return false;
    int n = 0;
    float total = 0.0f, longest = 0.0f;
    for (int i = 0; i < p.n_shards; ++i) {
        if (runs.s[i].L <= 0) continue;
        const float tiles = (float)((runs.s[i].L + kPreK - 1) / kPreK);
        total += tiles;
        longest = tiles > longest ? tiles : longest;
        ++n;
    }
    if (n < 2 || runs.n_runs != n) return false;
    const float mean = total / (float)n;
    const float side_by_side = prefill_cost(heads * tiles8 * n, heads * tiles4 * n, mean, 4.0f, D, false).least() +
                               0.5f * (longest - mean) + prefill_fold_us(n, (int64_t)p.B * p.Hq * p.Lq, D) / prefill_tile_us(D);
    const PrefillCost walked = prefill_cost(heads * tiles8, heads * tiles4, total + (float)(n - 1), 4.0f, D, false);
    *four = walked.four();
    return walked.least() * (D == 64 ? 1.05f : 1.0f) < side_by_side;
}

// Few workgroups and runs at will: whether two groups of four waves share 128 query rows and halve their keys (KG = 2), with the
// runs re-cut for that, twice as long, by cost as above.  Half the runs are half the partials to write and fold (500 x
// 32 x 1000 keys of 128 31.6 us against 27.8), or none (2 x 958 x 16 x 933 35.6 and 25.2, 487 x 64 x 2255 of 64 39.1 and 28.5), and shards
// whose runs fitted no round fit one (123 x 32 x (6278 + 971 + 4650) 49.6 and 40.6).  Each group stages tiles of its own, which
// at d = 128, where LDS is the busier side, costs a tenth (1024 x 16 x 8192 76.7 and 78.2: stays as it was), and a launch that
// does not half fill the chip gains nothing (11 x 16 x 385 of 64 8.5 and 9.1).
// Where the other form has more workgroups than one round they even out, and its cost is that of its mean run, not of its longest
// (2 x 86 x 32 x (449 + 6900 + 2725 + 550) of 64, 0.90 by the longest, 1.04 by the mean: 34.3 us and 41.6 with two groups).
// Not where a workgroup takes all keys by rule (a mask, counts per sequence): up to 1.5 workgroups a compute unit two groups are
// 7 to 15 % faster (2048 x 16 heads with a mask 51.2 us and 46.5), but from two on 10 % slower, and a sequence's outputs would
// then depend on how many others are in its batch.
static bool prefill_two_groups(KeyRuns* runs, int64_t wgs8, int64_t wgs4, int64_t rows, int D) {
    const int64_t cus = attn_target_wgs();
    int64_t total = 0, tiles = 0, tiles1 = 0;  // tiles1: of the longest run
    int shards = 0;
    for (int i = 0; i < runs->n_shards; ++i) {
        const int64_t L = runs->s[i].L, run = L < runs->s[i].per ? L : runs->s[i].per;
        total += L;
        tiles += (L + kPreK - 1) / kPreK;
        shards += L > 0 ? 1 : 0;
        tiles1 = (run + kPreK - 1) / kPreK > tiles1 ? (run + kPreK - 1) / kPreK : tiles1;
    }
    if (wgs4 < 1 || wgs8 * 2 > cus || shards * wgs4 > cus) return false;
    const int64_t want = cus / wgs4;
    int64_t pairs = ((total + kPrePair - 1) / kPrePair + want - 1) / want;
    if (pairs < kPreMinTilesPerSplit) pairs = kPreMinTilesPerSplit;
    KeyRuns two = *runs;
    attn_cut_runs(two, prefill_least_run(two, pairs * kPrePair, want), kPrePair);
    const int64_t wgs = two.n_runs * wgs4;
    if (two.n_runs > runs->n_runs || wgs > cus || wgs * 2 < cus) return false;
    int64_t steps = 0;
    for (int i = 0; i < two.n_shards; ++i) {
        const int64_t run = two.s[i].L < two.s[i].per ? two.s[i].L : two.s[i].per;
        steps = (run + kPrePair - 1) / kPrePair > steps ? (run + kPrePair - 1) / kPrePair : steps;
    }
    const float tile_us = prefill_tile_us(D);
    const bool one_round = wgs8 * runs->n_runs <= cus;
    const float one = prefill_cost(wgs8 * runs->n_runs, wgs4 * runs->n_runs, one_round ? (float)tiles1 : (float)tiles / (float)runs->n_runs,
                                   one_round ? 0.0f : 4.0f, D, false).least() * tile_us + prefill_fold_us(runs->n_runs, rows, D);
    const float both = ((float)steps * (D == 64 ? 1.0f : 1.1f) + 0.33f) * tile_us + prefill_fold_us(two.n_runs, rows, D);
    if (both >= one) return false;
    *runs = two;
    return true;
}

// The least run, in whole pairs of key tiles and of at least `from` keys, that leaves at most `most` runs.  A longer run never
// leaves more of them, so it is found by halving; no less than one run a shard is asked for.  (Tried one pair after the other, 16
// shards, the longest of 131072 keys, took 156 us of a call's host time.)
int64_t prefill_least_run(const KeyRuns& shards, int64_t from, int64_t most) {
    int64_t longest = 0;
    for (int i = 0; i < shards.n_shards; ++i) longest = shards.s[i].L > longest ? shards.s[i].L : longest;
    int64_t lo = from / kPrePair, hi = (longest + kPrePair - 1) / kPrePair;
    if (hi < lo) hi = lo;  // a run a shard already
    KeyRuns cut = shards;
    attn_cut_runs(cut, lo * kPrePair, kPrePair);
    if (cut.n_runs <= most) return lo * kPrePair;
    while (hi - lo > 1) {  // lo leaves too many
        const int64_t mid = lo + (hi - lo) / 2;
        attn_cut_runs(cut, mid * kPrePair, kPrePair);
        if (cut.n_runs <= most) hi = mid;
        else lo = mid;
    }
    return hi * kPrePair;
}

bool prefill_stores_past_l2(const AttnProblem& p, const PrefillForm& f) {
    const int64_t bytes = (int64_t)p.B * p.Hq * p.Lq * f.runs.n_runs * (4 * p.D);
    const int64_t most = p.D == 64 ? kPastL2Partials64 : f.runs.n_runs == 2 ? kPastL2TwoPartials : kPastL2Partials;
    return bytes >= kPastL2Bytes && (f.runs.n_runs == 1 || bytes < most);
}

// What a launch does, decided from the sizes alone.
PrefillForm prefill_form(const AttnProblem& p) {
    PrefillForm f;
    // Without a mask or per-sequence query counts a row's position in its head means nothing, and the query heads of
    // a KV head are contiguous in Q, O and lse: the kernel then sees one head of G * Lq rows per KV head, so that
    // short segments fill their 256-row tiles (128 queries x 4 heads: 2 full tiles instead of 4 half-empty ones).
    const bool pack_group = !p.causal && !p.q_lens;
    f.Hq = pack_group ? p.Hkv : p.Hq;
    f.Lq = pack_group ? (int64_t)(p.Hq / p.Hkv) * p.Lq : p.Lq;
    f.kind = PrefillForm::kPlain;
    f.four = false;
    f.runs = attn_runs_of(p);
    // several runs: only the plain call (every key of every sequence, every query row, no mask) takes them
    const bool one_run_only = p.causal || p.kv_lens || p.q_lens;
    if (one_run_only) {
        if (p.n_shards > 1) f.runs.n_runs = 0;  // refused
        else {
            f.runs.s[0].per = f.runs.s[0].L > 0 ? ((f.runs.s[0].L + kPreK - 1) / kPreK) * kPreK : kPreK;
            f.runs.first[1] = 1;
            f.runs.n_runs = 1;
            f.runs.by_runs = FastDiv(1);
        }
    }
    if (f.runs.n_runs < 1) return f;
    const int64_t tiles8 = (f.Lq + 8 * kPreQ - 1) / (8 * kPreQ), tiles4 = (f.Lq + 4 * kPreQ - 1) / (4 * kPreQ);
    const int64_t heads = (int64_t)p.B * f.Hq;
    if (!p.causal && p.quant_bits == 0) {
        if (p.n_shards > 1 && prefill_walks(p, f.runs, heads, tiles8, tiles4, &f.four)) {  // writes O, lse; no partials
            const KeyRuns runs = f.runs;
            f.runs.n_shards = 0;
            for (int i = 0; i < p.n_shards; ++i)
                if (runs.s[i].L > 0) f.runs.s[f.runs.n_shards++] = runs.s[i];
            f.runs.n_runs = 1;
            f.runs.by_runs = FastDiv(1);
            f.kind = PrefillForm::kWalk;
            return f;
        }
        // (no more partials than the plan that the workspace is sized for has)
        if (!one_run_only && prefill_two_groups(&f.runs, heads * tiles8, heads * tiles4, (int64_t)p.B * p.Hq * p.Lq, p.D)) {
            f.kind = PrefillForm::kTwoGroups;
            return f;
        }
    }
    int64_t key_tiles = 1;  // of the longest run
    for (int i = 0; i < f.runs.n_shards; ++i) {
        const int64_t keys = f.runs.s[i].L < f.runs.s[i].per ? f.runs.s[i].L : f.runs.s[i].per;
        if ((keys + kPreK - 1) / kPreK > key_tiles) key_tiles = (keys + kPreK - 1) / kPreK;
    }
    f.four = p.causal || (p.q_lens && p.quant_bits == 0 && p.B > 1) ||
             prefill_wants_4_waves(heads * f.runs.n_runs * tiles8, heads * f.runs.n_runs * tiles4, key_tiles, p.D, p.quant_bits != 0);
    return f;
}

// Order of a unit's workgroups when there are several runs.  The runs of a query tile side by side, unless one run's
// workgroups fill the chip by themselves and a unit's keys are several times an XCD's 4 MiB of L2: then run by run, so that
// the workgroups at work share the keys of one shard (8 shards of 8192 keys, 4096 x 64 query rows: 7.97 ms, 8.24 side by
// side, 8.02 with a launch per shard; at 8 MB of keys both orders take the same time, at 3 MB run by run is 5 % slower).
constexpr int64_t kPreRunByRunBytes = 16 << 20;
constexpr int64_t kPreTogetherBytes = 8 << 20;  // K and V of an XCD's units, whose L2 is 4 MiB

template <class T, int D, bool CAUSAL, int QB, int NW, bool WALK, int KG = 1>
static hipError_t launch_prefill_nw(const AttnProblem& p, const PrefillForm& f, float* Odst, float* Ldst, hipStream_t stream) {
    typedef typename T::elem elem;
    const KeyRuns& runs = f.runs;
    const int n_units = p.B * p.Hkv;
    constexpr int kRows = NW / KG * kPreQ;
    const int64_t q_tiles = (f.Lq + kRows - 1) / kRows;
    const int64_t tiles_of_unit = (int64_t)(f.Hq / p.Hkv) * q_tiles;
    const int64_t per_unit = tiles_of_unit * runs.n_runs;
    const int64_t grid = (int64_t)8 * ((n_units + 7) / 8) * per_unit;
    if (!grid_fits(grid, NW * kWave)) return hipErrorInvalidValue;
    int64_t keys = 0;
    for (int i = 0; i < runs.n_shards; ++i) keys += runs.s[i].L;
    const bool run_by_run = n_units * tiles_of_unit >= attn_target_wgs() && keys * (4 * D) > kPreRunByRunBytes;
    // With every workgroup resident at once (two per compute unit, started in index order) the second half goes beside
    // the first: the shortest tile to the longest, and all compute units end together (2048 tokens: 65 -> 60 us).
    const int fold = CAUSAL && grid <= 2 * (int64_t)attn_target_wgs() ? 1 : 0;
    // With a mask the units of an XCD advance together, unless their keys are many times its L2: 2 x 4096 tokens x 16 heads
    // of 64 one unit after the other 143 us, together 126; 2 x 2048 of 128 83 and 62; 4 x 4096 of 128 (8 MiB) 415 and 386, but
    // 8 x 4096 (16 MiB) 1524 and 1567.
    const int64_t units_per_xcd = (n_units + 7) / 8;
    const int together = CAUSAL && units_per_xcd * keys * (4 * D) <= kPreTogetherBytes ? 1 : 0;
    const int past_l2 = prefill_stores_past_l2(p, f) ? 1 : 0;
    hipLaunchKernelGGL((prefill_attn_kernel<T, D, CAUSAL, QB, NW, WALK, KG>), dim3((unsigned)grid), dim3(NW * kWave), 0, stream,
                       (const elem*)p.Q, runs, p.K_params, p.V_params, f.Hq, FastDiv(p.Hkv), FastDiv(f.Hq / p.Hkv),
                       FastDiv(q_tiles), FastDiv(together ? units_per_xcd : per_unit), FastDiv(run_by_run ? tiles_of_unit : runs.n_runs),
                       run_by_run ? 1 : 0, f.Lq, p.kv_lens, p.q_lens, n_units, fold, together, past_l2,
                       p.scale * kLog2e, Odst, Ldst);
    return hipGetLastError();
}

template <class T, int D, bool CAUSAL, int QB = 0>
static hipError_t launch_prefill_t(const AttnProblem& p, const PrefillForm& f, hipStream_t stream) {
    if (QB != 0 && (p.n_shards > 1 || !p.K_params || !p.V_params)) return hipErrorInvalidValue;
    const int64_t rows = (int64_t)p.B * p.Hq * p.Lq;
    const int n = f.runs.n_runs;
    float* Odst = p.O;
    float* Ldst = p.lse;
    if (n > 1) {  // partials
        if (!p.workspace || p.workspace_bytes < (size_t)n * rows * (D + 1) * sizeof(float)) return hipErrorInvalidValue;
        Odst = (float*)p.workspace;
        Ldst = Odst + (size_t)n * rows * D;
    }
    hipError_t e = hipErrorInvalidValue;
    if constexpr (CAUSAL) {
        e = launch_prefill_nw<T, D, true, 0, 4, false>(p, f, Odst, Ldst, stream);
    } else {
        if constexpr (QB == 0) {
            if (f.kind == PrefillForm::kWalk)
                e = f.four ? launch_prefill_nw<T, D, false, 0, 4, true>(p, f, Odst, Ldst, stream)
                           : launch_prefill_nw<T, D, false, 0, 8, true>(p, f, Odst, Ldst, stream);
            if (f.kind == PrefillForm::kTwoGroups) e = launch_prefill_nw<T, D, false, 0, 8, false, 2>(p, f, Odst, Ldst, stream);
        }
        if (f.kind == PrefillForm::kPlain)
            e = f.four ? launch_prefill_nw<T, D, false, QB, 4, false>(p, f, Odst, Ldst, stream)
                       : launch_prefill_nw<T, D, false, QB, 8, false>(p, f, Odst, Ldst, stream);
    }
    if (e != hipSuccess || n == 1) return e;
    return launch_lse_merge(Odst, Ldst, n, rows, D, p.O, p.lse, stream);
}

template <class T>
static hipError_t launch_prefill_d(const AttnProblem& p, hipStream_t stream) {
    const PrefillForm f = prefill_form(p);
    if (f.runs.n_runs < 1) return hipErrorInvalidValue;
    if (p.quant_bits != 0) {  // K', V' as transport codes (never with the mask: the Inquirer's own K, V are plain)
        if (p.causal || (p.quant_bits != 8 && p.quant_bits != 4)) return hipErrorInvalidValue;
        if (p.quant_bits == 8)
            return p.D == 128 ? launch_prefill_t<T, 128, false, 8>(p, f, stream) : launch_prefill_t<T, 64, false, 8>(p, f, stream);
        return p.D == 128 ? launch_prefill_t<T, 128, false, 4>(p, f, stream) : launch_prefill_t<T, 64, false, 4>(p, f, stream);
    }
    if (p.causal)
        return p.D == 128 ? launch_prefill_t<T, 128, true>(p, f, stream) : launch_prefill_t<T, 64, true>(p, f, stream);
    return p.D == 128 ? launch_prefill_t<T, 128, false>(p, f, stream) : launch_prefill_t<T, 64, false>(p, f, stream);
}

hipError_t launch_prefill_attn(const AttnProblem& p, hipStream_t stream) {
    return p.dtype == FEDRAG_BF16 ? launch_prefill_d<BF16>(p, stream) : launch_prefill_d<F16>(p, stream);
}

}  // namespace fedrag

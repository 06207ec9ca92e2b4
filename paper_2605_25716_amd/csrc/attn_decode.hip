// Decode-shaped partial attention (Section 4.1, per-node local computation) for 16-bit storage:
// at most 16 query rows per (sequence, KV head) unit, i.e. the GQA group packed into one MFMA column tile.
// HBM-bound: every K'/V' byte of the shard is read exactly once and nothing is reused, so the kernel is built around keeping
// whole rows in flight.
//
// One workgroup = one unit x one split of the shard's keys; its four (two, eight) waves take 32-key tiles round-robin.
// Lane l of a wave: lr = l % 16, lq = l / 16.
//   S^T tile (32 keys x 16 queries) = K'(32 x d) . Q'^T(d x 16): two 16-key MFMA tiles; this lane ends up with
//   query lr and keys {16 mt + 4 lq + r}.  Those eight keys are also this lane's contraction slice of
//   O^T(d x 16) += V'^T(d x 32) . P^T(32 x 16).
// 16-bit values reach their operands through LDS, in tiles that belong to one wave and need no barrier.  A K' operand straight
// from memory takes 64 bytes of each of 16 rows a load, 16 of them from each of 16 consecutive lanes, and a compute unit takes
// 256 KB of such loads in twice the time of whole rows (9.7 us and 5.0 on 32 workgroups), which was what a launch that does not
// fill the chip waited for: one sequence of 8192 keys x 8 heads of 128 16.8 us and 13.4 now (call with its aggregation), 512 keys
// 9.9 and 7.8, of 64 10.9 and 9.3, 5.9 and 4.8; launches at the rate of memory gain 0 to 4 %.  What is in flight holds no registers.
// Transport codes, whose rebuilding is the bound, and 16-bit values of 128 columns in whole rounds of long runs (kDecLongRun) are
// loaded straight into registers as operands, and the d-rows of O^T are assigned d = DCH * i + j (tile j, row i) so that lane
// (i = lr) needs exactly the DCH contiguous elements [DCH*lr, DCH*lr + DCH) of each of its eight keys: an in-register 8 x DCH
// transpose.  Past the end of a run the register form reads the last key again and the LDS form reads nothing; both mask it.
// P is split into two storage-type terms (hi + lo) so that the probabilities enter the second product with
// ~16 significant bits; the matrix pipe is idle most of the time anyway.
// Splits are normalised partials (O, lse) in the caller's workspace and are folded by the Section 4.1
// aggregation kernel (merge.hip).
#include <type_traits>

#include "fedrag_device.h"
#include "fedrag_host.h"

namespace fedrag {

// Transpose 8 rows of NC 16-bit elements: in[e] holds NC elements (NC/2 words), out[c] holds 8 (4 words).
template <int NC>
__device__ __forceinline__ void transpose_keys_b16(const uint32_t (&in)[8][NC / 2], u32x4_t (&out)[NC]) {
#pragma unroll
    for (int c2 = 0; c2 < NC / 2; ++c2) {
#pragma unroll
        for (int r2 = 0; r2 < 4; ++r2) {
            const uint32_t a = in[2 * r2][c2];
            const uint32_t b = in[2 * r2 + 1][c2];
            out[2 * c2][r2] = __builtin_amdgcn_perm(b, a, 0x05040100u);      // {a.lo, b.lo}
            out[2 * c2 + 1][r2] = __builtin_amdgcn_perm(b, a, 0x07060302u);  // {a.hi, b.hi}
        }
    }
}

// One 32-key tile in registers.  QB = 0: K' rows as MFMA operands, V' rows as loaded.  QB = 8 or 4: the transport
// codec's codes of the same elements (Section 7.5) plus the (scale, lo) of the rows this lane touches.
template <class T, int D, int QB>
struct DecTile {
    typename T::vec8 k[2][D / 32];
    uint32_t v[8][D / 32];
};
template <class T, int D>
struct DecTile<T, D, 8> {
    u32x4_t kc[2][D / 64];  // 16 codes per (16-key tile, pair of contraction steps): one 16-byte load each
    u32x2_t vc[8];          // 8 codes per key (D = 128: DCH = 8 elements per lane and key)
    u32x2_t kp[2];          // (scale, lo) as bits, of key rows 16 mt + lr
    u32x2_t vp[8];          // of this lane's eight keys
};
template <class T, int D>
struct DecTile<T, D, 4> {
    u32x4_t kc[2];          // 32 codes per 16-key tile (all four contraction steps): one 16-byte load
    uint32_t vc[8];
    u32x2_t kp[2];
    u32x2_t vp[8];
};

// 8 codes -> 8 storage-type values, exactly as dequantize_rows_kernel produces them: fma(code, scale, lo) in fp32,
// narrowed once.  (The fp32 value is pinned so that the two roundings are not folded into one.)
//
// The kernel is bound by these instructions, so a 4-bit code is not converted to a float first: its bits, masked in place,
// are read as an fp16 subnormal - code * 2^-24, or code * 2^-20 four bits further up - by an fma that takes an fp16 operand
// from either half of a register, and the row's scale carries the power of two.  Both scalings are exact, so the product
// the fma rounds is the same.  A scale from 2^100 up (rows whose range is beyond any activation) would overflow and takes
// the plain conversions: a wave-uniform branch before each operand's part of a step, so that the check of the V' scales does
// not wait for them before the first product.
struct RowScale {
    float scale, lo, scale24, scale20;
};
__device__ __forceinline__ RowScale row_scale(u32x2_t prm) {
    const uint32_t scale_bits = prm[0], lo_bits = prm[1];  // (bit-casting a vector element in place picks element 0)
    const float scale = __builtin_bit_cast(float, scale_bits), lo = __builtin_bit_cast(float, lo_bits);
    return RowScale{scale, lo, scale * 16777216.0f, scale * 1048576.0f};
}
constexpr float kPlainScale = 1.2676506e30f;  // 2^100
template <int N>
__device__ __forceinline__ bool any_plain_scale(const u32x2_t (&prm)[N]) {
    float top = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) top = fmaxf(top, fabsf(row_scale(prm[i]).scale));
    return __builtin_amdgcn_ballot_w64(!(top < kPlainScale)) != 0;
}
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float fma_half(uint32_t w, int half, float scale, float lo) {
    const f16x2_t h = __builtin_bit_cast(f16x2_t, w);
    float x = __builtin_fmaf((float)h[half], scale, lo);
    pin_here(x);
    return x;
}
template <class T>
__device__ __forceinline__ typename T::vec8 dequant8(u32x2_t w, const RowScale& r, std::true_type) {  // 8-bit codes
    // a byte converts with one instruction wherever it sits, which leaves the masks nothing to save (56 us per shard of
    // the decode workload against 64 by way of the subnormals)
    typename T::vec8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float x = __builtin_fmaf((float)((w[e / 4] >> (8 * (e % 4))) & 255u), r.scale, r.lo);
        pin_here(x);
        out[e] = T::from_float(x);
    }
    return out;
}
template <class T, bool PLAIN>
__device__ __forceinline__ typename T::vec8 dequant8(uint32_t w, const RowScale& r, std::bool_constant<PLAIN>) {  // 4-bit
    typename T::vec8 out;
    if constexpr (PLAIN) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float x = __builtin_fmaf((float)((w >> (4 * e)) & 15u), r.scale, r.lo);
            pin_here(x);
            out[e] = T::from_float(x);
        }
        return out;
    }
    const uint32_t up = w >> 8;
    const uint32_t a = w & 0x000f000fu, b = w & 0x00f000f0u;    // codes 0, 4 and (times 16) 1, 5
    const uint32_t c = up & 0x000f000fu, d = up & 0x00f000f0u;  // codes 2, 6 and (times 16) 3, 7
    out[0] = T::from_float(fma_half(a, 0, r.scale24, r.lo));
    out[1] = T::from_float(fma_half(b, 0, r.scale20, r.lo));
    out[2] = T::from_float(fma_half(c, 0, r.scale24, r.lo));
    out[3] = T::from_float(fma_half(d, 0, r.scale20, r.lo));
    out[4] = T::from_float(fma_half(a, 1, r.scale24, r.lo));
    out[5] = T::from_float(fma_half(b, 1, r.scale20, r.lo));
    out[6] = T::from_float(fma_half(c, 1, r.scale24, r.lo));
    out[7] = T::from_float(fma_half(d, 1, r.scale20, r.lo));
    return out;
}

// On codes the kernel is bound by its own instruction stream (rebuilding every element costs more than fetching
// it).  At 4 bits it runs with one register tile set per wave and kDecCodesOcc workgroups per compute unit instead
// of one workgroup with a ring of two: the other workgroup's waves fill the issue slots a wave leaves while it
// waits (measured 61 -> 56 us per shard of the decode workload; at 8 bits the ring of two stayed ahead, 60 vs 62).
#ifndef FEDRAG_DEC_NBUF_Q8
#define FEDRAG_DEC_NBUF_Q8 2
#endif
#ifndef FEDRAG_DEC_NBUF_Q4
#define FEDRAG_DEC_NBUF_Q4 1
#endif
#ifndef FEDRAG_DEC_AUX
#define FEDRAG_DEC_AUX 2    // cache-policy bits of the streaming loads: non-temporal (K'/V' are read once)
#endif

// 16-bit values: NS tiles of K' and V' per wave in LDS.  Two, 128 KiB of LDS at d = 128 and half of that at d = 64, so one or two
// workgroups to a compute unit.  One, and twice the workgroups, where there are more of them than compute units and their runs are so
// short that start and end are what they spend their time on, which a neighbour then hides: 64 sequences x 8 heads of 128 x 100
// keys 7.3 us against 10.4 (8.5 before), 400 keys 20.0 and 22.4, 1000 44.6 and 45.4; beyond that two tiles are 0 to 1 % ahead.  At
// d = 64 100 keys 5.4 and 5.9, 256 8.1 either way, 400 11.5 and 11.3.  Also where a wave has one tile: 128 keys x 8 heads 3.7 and 4.3.
constexpr int64_t dec_single_tile_run(int d) { return d == 128 ? 1024 : 256; }  // keys of the longest run up to which it is one

// 16-bit values of 128 columns in whole rounds of long runs stay in registers: at the rate of memory the LDS form is 1 to 4 % behind
// where the units lie powers of two apart (64 sequences x 8 heads x 32768 keys 1189 us and 1217, x 8192 301 and 310, 16 x 8192 75.4
// and 78.4), for whatever reason - not the order in which a tile's rows or a run's tiles are asked for - and within 1.5 % of it
// elsewhere (64 x 3000 122 and 120, 32 x 4000 80.5 and 82).  At d = 64 both take the same time.  Where a round is partly empty,
// for its number of workgroups or for shorter ones, what counts is again what a compute unit takes by itself (33 x 4096 131 us and 116).
constexpr int64_t kDecLongRun = 2048;

// PARTS: a run is summed part by part, `part` tiles of a wave at a time (attn_runs_of).  A form of its own, as putting a part aside
// takes some 0.3 us: 0 to 3 % of cut launches on 16-bit values and most on 8-bit codes (9 x 2000 keys 16.8 -> 17.7 us), on 4-bit
// codes 2 to 8 % (9 x 8192 keys 26.7 -> 27.7 us, uncut 31.5; 11 x 1400 12.0 -> 12.9, uncut 13.3).  Put aside in LDS instead, codes
// took another 2 to 6 %.
template <class T, int D, int QB, int NS, int WAVES, bool PARTS>
FEDRAG_KERNEL __launch_bounds__(WAVES * kWave, QB == 4 ? kDecCodesOcc : NS * D > 0 && NS * D <= 128 ? 2 : 1) void decode_attn_kernel(const typename T::elem* __restrict__ Q,
                                                                     const KeyRuns runs,
                                                                     const float* __restrict__ Kprm,
                                                                     const float* __restrict__ Vprm, int R,
                                                                     float scale_log2, float* __restrict__ O,
                                                                     float* __restrict__ lse, int64_t total_rows,
                                                                     const int32_t* __restrict__ kv_lens,
                                                                     const int32_t* __restrict__ q_lens, int Lq,
                                                                     FastDiv by_hkv, int part) {
    typedef typename T::elem elem;
    typedef typename T::vec8 vec8;
    typedef DecTile<T, D, QB> Tile;
    static_assert(QB == 0 || (D == 128 && NS == 0), "the quantised path is laid out for d = 128, in registers");
    constexpr int KS = D / 32;   // contraction steps of the first product
    constexpr int DCH = D / 16;  // elements per lane per key of V' (= number of 16-row tiles of O^T)
    constexpr int NW = DCH / 2;  // 32-bit words of that
    constexpr int ROWB = QB ? D * QB / 8 : D * 2;  // bytes per row of K' / V' as stored (values, or codes)
    constexpr int TILEB = kDecTile * ROWB;
    constexpr bool LDS = NS > 0;  // tiles go to LDS; otherwise to registers
    constexpr int NBUF = QB == 0 ? 2 : QB == 8 ? FEDRAG_DEC_NBUF_Q8 : FEDRAG_DEC_NBUF_Q4;
    constexpr int AUX = FEDRAG_DEC_AUX;

    // LDS: NS slots per wave for the tiles, an array each, so that the compiler sees that the fill of one does not alias the
    // reads of another.  At the end the waves' outputs take their place: 8 rows in the first slot of K', 8 in that of V'.
    constexpr int OROW = (D + 4) * 4;  // bytes
    constexpr int SLOT = LDS ? TILEB : 8 * OROW;
    static_assert(SLOT >= 8 * OROW, "eight rows of outputs fit a slot");
    __shared__ __attribute__((aligned(16))) char ks0[WAVES][SLOT], vs0[WAVES][SLOT];
    __shared__ __attribute__((aligned(16))) char ks1[WAVES][NS == 2 ? SLOT : 16], vs1[WAVES][NS == 2 ? SLOT : 16];
    __shared__ float sm_m[WAVES][16];
    __shared__ float sm_l[WAVES][16];
    auto out_row = [&](int w, int n) { return (float*)((n < 8 ? ks0[w] : vs0[w]) + n % 8 * OROW); };

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);  // wave-uniform: keeps the tile loop scalar
    const int lane = tid % kWave;
    const int lr = lane % 16;
    const int lq = lane / 16;
    // The arguments are one trip to memory and the shard a second one, where branches and addresses made five of them: a token's
    // attention in a request over 32 layers, 24.9 -> 24.4 us a layer; 128 keys 3.72 -> 3.66 us; long runs even.
    FEDRAG_HAVE_HERE(FEDRAG_S3(runs.by_runs), FEDRAG_S(runs.n_shards), FEDRAG_S(Q), FEDRAG_S(R), FEDRAG_S(scale_log2), FEDRAG_S(O),
                     FEDRAG_S(lse), FEDRAG_S(total_rows), FEDRAG_S(kv_lens), FEDRAG_S(q_lens), FEDRAG_S(Lq), FEDRAG_S3(by_hkv));
    if constexpr (PARTS) FEDRAG_HAVE_HERE(FEDRAG_S(part));
    const int64_t unit = runs.by_runs.div(blockIdx.x);
    const int run = (int)runs.by_runs.mod(blockIdx.x);  // index of this workgroup's partial
    int split;
    const KeyShard shard = runs.shard_of(run, &split);
    FEDRAG_HAVE_HERE(FEDRAG_S(shard.K), FEDRAG_S(shard.V), FEDRAG_S(shard.L), FEDRAG_S(shard.per));
    const void* K = shard.K;
    const void* V = shard.V;
    const int64_t L = shard.L;
    const int64_t keys_per_split = shard.per;
    const int64_t k_begin = (int64_t)split * keys_per_split;
    // keys of this unit's sequence: all L rows, or the first kv_lens[b] of them (padded batch of unequal sequences);
    // a split that starts past them is empty and returns O = 0, lse = -inf like an empty shard
    int64_t L_seq = L;
    int q_len = 0;
    if (kv_lens || q_lens) {  // both asked for at once
        const uint32_t b = by_hkv.div((uint32_t)unit);
        const int nk = (kv_lens ? kv_lens : q_lens)[b], nq = (q_lens ? q_lens : kv_lens)[b];
        asm volatile("" ::"v"(nk), "v"(nq));
        const int64_t v = __builtin_amdgcn_readfirstlane(nk);
        if (kv_lens) L_seq = v < 0 ? 0 : (v < L ? v : L);
        q_len = __builtin_amdgcn_readfirstlane(nq);
    }
    int64_t k_end = k_begin + keys_per_split;
    if (k_end > L_seq) k_end = L_seq;
    if (k_end < k_begin) k_end = k_begin;

    const elem* Qu = Q + unit * R * D;
    const char* Kb = (const char*)K + unit * L * ROWB;
    const char* Vb = (const char*)V + unit * L * ROWB;

    // Q'^T operands: column lr (query), contraction slice 32 ks + 8 lq; padding queries lie past the end of the
    // buffer and arrive as zeros
    // Which 8 channels lane group lq contracts in step ks is free as long as Q' and K' agree.  16-bit K': 32 ks + 8 lq.  Codes: every
    // lane fetches 16 bytes of its row at once - 16 codes = steps 2h, 2h+1 (8 bits) or 32 codes = all four steps (4 bits) - so that a
    // load still covers 64 contiguous bytes per row; with 8- or 4-byte loads the kernel was bound by the number of rows a load
    // instruction touches, not by bytes.
    auto chan0 = [&](int ks) -> int {
        return QB == 0 ? ks * 32 + lq * 8 : (QB == 8 ? 16 * lq + 64 * (ks / 2) + 8 * (ks % 2) : 32 * lq + 8 * ks);
    };
    vec8 qop[KS];
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc((void*)Qu, 0, R * D * 2, 0x00020000);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        qop[ks] = __builtin_bit_cast(vec8, __builtin_amdgcn_raw_buffer_load_b128(rq, (lr * D + chan0(ks)) * 2, 0, 0));

    f32x4_t acc_o[DCH];
#pragma unroll
    for (int i = 0; i < DCH; ++i) acc_o[i] = zero_vec<f32x4_t>();
    float m_run = -INFINITY, l_run = 0.f;
    // PARTS: what a wave has put aside, outputs, sums and their maximum.  Every addition to it halves what is there, by a maximum above
    // both, so that the parts together pass fp32's range no sooner than one of them.
    f32x4_t part_o[PARTS ? DCH : 1];
    float m_part = -INFINITY, l_part = 0.f;
    int part_end = part;
#pragma unroll
    for (int i = 0; i < (PARTS ? DCH : 1); ++i) part_o[i] = zero_vec<f32x4_t>();
    auto put_aside = [&]() {
        if constexpr (PARTS) {
            const float M = fmaxf(m_part, m_run) + 1.0f;
            const float a = exp2_diff(m_part, M), b = exp2_diff(m_run, M);
#pragma unroll
            for (int i = 0; i < DCH; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    part_o[i][e] = __builtin_fmaf(acc_o[i][e], b, part_o[i][e] * a);
                    acc_o[i][e] = 0.f;
                }
            l_part = __builtin_fmaf(l_run, b, l_part * a);
            m_part = M;
            l_run = 0.f;
            m_run = -INFINITY;
            part_end += part;
        }
    };

    const int64_t split_bytes = (k_end - k_begin) * ROWB;  // < 2^31, guaranteed by the split planner
    // Registers: per-lane byte offsets inside a 32-key tile, and buffer resources based at the split's first key: the address is
    // (scalar resource base) + (scalar tile offset) + (per-lane 32-bit offset), one VGPR per lane in total.
    constexpr int EB = QB ? QB : 16;  // bits per stored element
    const uint32_t koff = (uint32_t)(lr * ROWB + lq * EB);          // 8 elements per lane and contraction step
    const uint32_t kqoff = (uint32_t)(lr * ROWB + lq * 16);         // codes: 16 bytes per lane
    const uint32_t voff = (uint32_t)(lq * 4 * ROWB + lr * DCH * EB / 8);
    const __amdgpu_buffer_rsrc_t rk =
        __builtin_amdgcn_make_buffer_rsrc((void*)(Kb + k_begin * ROWB), 0, (int)split_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rv =
        __builtin_amdgcn_make_buffer_rsrc((void*)(Vb + k_begin * ROWB), 0, (int)split_bytes, 0x00020000);
    // quantised path: the (scale, lo) pairs of the split's rows, 8 bytes per key
    const int64_t n_split_keys = k_end - k_begin;
    const __amdgpu_buffer_rsrc_t rkp = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(QB ? Kprm + (unit * L + k_begin) * 2 : nullptr), 0, QB ? (int)(n_split_keys * 8) : 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rvp = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(QB ? Vprm + (unit * L + k_begin) * 2 : nullptr), 0, QB ? (int)(n_split_keys * 8) : 0, 0x00020000);
    // LDS: a tile arrives in whole rows, 1 KiB of them a load.  Slot p of row r holds chunk p ^ swz(r), so that the 16 rows
    // of a K' operand, and the 16 of a transposing read of V', fall on different banks.  The resource starts at the tile and ends
    // with the run: rows past the end (with per-sequence key counts they are padding that may hold anything), and tiles behind it,
    // are not read and arrive as zeros.
    constexpr int CH = D / 8;               // 16-byte chunks per row
    constexpr int RPW = kWave / CH;         // rows per load
    constexpr int KL = kDecTile / RPW;      // loads per tile of K' or V'
    auto swz_k = [&](int r) { return D == 128 ? r % 16 : r / 2 % 8; };
    auto swz_v = [&](int r) { return D == 128 ? r % 4 * 4 + r / 4 % 2 * 2 : r / 2 % 4 * 2; };
    auto fill = [&](int tile, char* slot, bool is_k) {
        const int left = (int)split_bytes - tile * TILEB;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void*)((is_k ? Kb : Vb) + k_begin * ROWB + (int64_t)tile * TILEB), 0, left > 0 ? left : 0, 0x00020000);
#pragma unroll
        for (int j = 0; j < KL; ++j) {
            const int r = lane / CH + j * RPW;
            const int off = r * ROWB + (((lane % CH) ^ (is_k ? swz_k(r) : swz_v(r))) << 4);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (void __attribute__((address_space(3)))*)(slot + j * (kWave * 16)), 16, off,
                                                     0, 0, AUX);
        }
    };
    auto load_k = [&](int tile, Tile& t) {  // tile index inside the split; all 32 keys exist
        const int soff = tile * TILEB;
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            if constexpr (QB == 0) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const int off = (int)koff + mt * 16 * ROWB + ks * 4 * EB;
                    t.k[mt][ks] = __builtin_bit_cast(vec8, __builtin_amdgcn_raw_buffer_load_b128(rk, off, soff, AUX));
                }
            } else if constexpr (QB == 8) {
#pragma unroll
                for (int h = 0; h < KS / 2; ++h)
                    t.kc[mt][h] = __builtin_amdgcn_raw_buffer_load_b128(rk, (int)kqoff + mt * 16 * ROWB + 64 * h, soff, AUX);
            } else {
                t.kc[mt] = __builtin_amdgcn_raw_buffer_load_b128(rk, (int)kqoff + mt * 16 * ROWB, soff, AUX);
            }
            if constexpr (QB != 0)
                t.kp[mt] = __builtin_amdgcn_raw_buffer_load_b64(rkp, (mt * 16 + lr) * 8, tile * kDecTile * 8, 0);
        }
    };
    auto load_v = [&](int tile, Tile& t) {
        const int soff = tile * TILEB;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int off = (int)voff + ((e / 4) * 16 + (e % 4)) * ROWB;
            if constexpr (QB != 0) {
                if constexpr (QB == 8) t.vc[e] = __builtin_amdgcn_raw_buffer_load_b64(rv, off, soff, AUX);
                else t.vc[e] = __builtin_amdgcn_raw_buffer_load_b32(rv, off, soff, AUX);
                t.vp[e] = __builtin_amdgcn_raw_buffer_load_b64(rvp, ((e / 4) * 16 + (e % 4) + lq * 4) * 8,
                                                               tile * kDecTile * 8, 0);
            } else if constexpr (NW == 4) {
                const u32x4_t w = __builtin_amdgcn_raw_buffer_load_b128(rv, off, soff, AUX);
                t.v[e][0] = w[0]; t.v[e][1] = w[1]; t.v[e][2] = w[2]; t.v[e][3] = w[3];
            } else {
                const u32x2_t w = __builtin_amdgcn_raw_buffer_load_b64(rv, off, soff, AUX);
                t.v[e][0] = w[0]; t.v[e][1] = w[1];
            }
        }
    };
    // ragged last tile: rows past the end of the run re-read its last key, k_end - 1 (the tail exists, so
    // k_end > k_begin).  Rows past k_end are never touched: with per-sequence key counts they are padding that may
    // hold anything, and a NaN there would survive the multiplication by a zero probability.
    auto load_clamped = [&](int64_t key0, Tile& t) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            int64_t key = key0 + mt * 16 + lr;
            if (key >= k_end) key = k_end - 1;
            if constexpr (QB == 0) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) t.k[mt][ks] = *(const vec8*)(Kb + key * ROWB + ks * 4 * EB + lq * EB);
            } else if constexpr (QB == 8) {
#pragma unroll
                for (int h = 0; h < KS / 2; ++h) t.kc[mt][h] = *(const u32x4_t*)(Kb + key * ROWB + lq * 16 + 64 * h);
            } else {
                t.kc[mt] = *(const u32x4_t*)(Kb + key * ROWB + lq * 16);
            }
            if constexpr (QB != 0) t.kp[mt] = *(const u32x2_t*)(Kprm + (unit * L + key) * 2);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            int64_t key = key0 + (e / 4) * 16 + lq * 4 + (e % 4);
            if (key >= k_end) key = k_end - 1;
            const char* p = Vb + key * ROWB + lr * DCH * EB / 8;
            if constexpr (QB == 0) {
#pragma unroll
                for (int w = 0; w < NW; ++w) t.v[e][w] = ((const uint32_t*)p)[w];
            } else {
                if constexpr (QB == 8) t.vc[e] = *(const u32x2_t*)p;
                else t.vc[e] = *(const uint32_t*)p;
                t.vp[e] = *(const u32x2_t*)(Vprm + (unit * L + key) * 2);
            }
        }
    };

    // all loads done but the N asked for last (LDS-direct loads are waited for by hand)
    auto wait_loads = [&](auto n) {
        constexpr int N = decltype(n)::value;
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
        __builtin_amdgcn_sched_barrier(0);
    };
    // One 32-key tile.  `reload` refills its slots or registers with tile `next_tile` as soon as each half has been consumed (K'
    // after the first product, V' after the second, or after the in-register transpose), so that the loads fly behind the
    // softmax, the second product and the other set's step.  younger: loads asked for after this tile's V' when it is used.
    auto step = [&](Tile& t, int64_t key0, bool masked, bool reload, int next_tile, char* kslot, char* vslot, auto younger) {
        f32x4_t s[2];
        auto score = [&](auto plain) {
            RowScale krow[2];
            if constexpr (QB != 0) {
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) krow[mt] = row_scale(t.kp[mt]);
            }
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                s[mt] = zero_vec<f32x4_t>();
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    vec8 kop;
                    if constexpr (LDS)
                        kop = *(const vec8*)(kslot + (mt * 16 + lr) * ROWB + (((4 * ks + lq) ^ swz_k(lr)) << 4));
                    else if constexpr (QB == 0) kop = t.k[mt][ks];
                    else if constexpr (QB == 8) {
                        const u32x4_t w = t.kc[mt][ks / 2];
                        u32x2_t c;  // (vector elements are copied out one by one before use)
                        const uint32_t c0 = w[2 * (ks % 2)], c1 = w[2 * (ks % 2) + 1];
                        c[0] = c0;
                        c[1] = c1;
                        kop = dequant8<T>(c, krow[mt], plain);
                    } else {
                        const uint32_t c = t.kc[mt][ks];
                        kop = dequant8<T>(c, krow[mt], plain);
                    }
                    s[mt] = T::mfma16(kop, qop[ks], s[mt]);
                }
            }
        };
        if constexpr (QB == 4) {
            if (any_plain_scale(t.kp)) score(std::true_type{});
            else score(std::false_type{});
        } else {
            score(std::true_type{});
        }
        if (reload) {
            if constexpr (LDS) {
                __builtin_amdgcn_sched_barrier(0);
                fill(next_tile, kslot, true);
                __builtin_amdgcn_sched_barrier(0);
            } else {
                load_k(next_tile, t);
            }
        }
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = s[e / 4][e % 4] * scale_log2;
        if (masked) {  // the ragged end of the run
            const int left = (int)(k_end - key0) - lq * 4;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if ((e / 4) * 16 + e % 4 >= left) p[e] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, p[e]);
        mx = xor32_max(xor16_max(mx));
        const float m_new = fmaxf(m_run, mx);  // finite: the tile's first key exists
        const float alpha = exp2_diff(m_run, m_new);
        if (masked) {  // a key alone has the probability 1
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] -= m_new;
        } else {  // one rounding of the exponent's argument: scores of some hundreds leave 2^-15 in a product rounded first
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = __builtin_fmaf(s[e / 4][e % 4], scale_log2, -m_new);
        }
        float psum = 0.f;
        vec8 ph, pl;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float pe = fast_exp2(p[e]);
            psum += pe;
            ph[e] = T::from_float(pe);
            pl[e] = T::from_float(pe - T::to_float(ph[e]));
        }
        l_run = l_run * alpha + psum;
        m_run = m_new;
        // second product in two halves of the d-rows to keep the transposed operands short-lived
        u32x4_t vt[DCH];
        if constexpr (LDS) {
            wait_loads(younger);
#pragma unroll
            for (int i = 0; i < DCH; ++i)
#pragma unroll
                for (int mt = 0; mt < 2; ++mt) {
                    const int r = mt * 16 + lq * 4 + lr / 4;
                    const u32x2_t w = lds_read_tr16(vslot + r * ROWB + (((2 * i + lr % 4 / 2) ^ swz_v(r)) << 4) + lr % 2 * 8);
                    vt[i][2 * mt] = w[0];
                    vt[i][2 * mt + 1] = w[1];
                }
        } else if constexpr (QB == 0) {
            transpose_keys_b16<DCH>(t.v, vt);
        } else {
            uint32_t v16[8][DCH / 2];  // the eight keys' rows in the storage type, as the unquantised path loads them
            auto rebuild = [&](auto plain) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const u32x4_t w = __builtin_bit_cast(u32x4_t, dequant8<T>(t.vc[e], row_scale(t.vp[e]), plain));
#pragma unroll
                    for (int c = 0; c < DCH / 2; ++c) v16[e][c] = w[c];
                }
            };
            if constexpr (QB == 4) {
                if (any_plain_scale(t.vp)) rebuild(std::true_type{});
                else rebuild(std::false_type{});
            } else {
                rebuild(std::true_type{});
            }
            transpose_keys_b16<DCH>(v16, vt);
        }
        if constexpr (!LDS) {
            if (reload) load_v(next_tile, t);
        }
#pragma unroll
        for (int i = 0; i < DCH; ++i) {
            acc_o[i] *= alpha;
            const vec8 vop = __builtin_bit_cast(vec8, vt[i]);
            acc_o[i] = T::mfma16(vop, ph, acc_o[i]);
            acc_o[i] = T::mfma16(vop, pl, acc_o[i]);
        }
        if constexpr (LDS) {
            if (reload) {
                __builtin_amdgcn_sched_barrier(0);
                fill(next_tile, vslot, false);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    // Wave w owns tiles w, w + WAVES, ... of the split.  NS sets of slots (codes: NBUF register tile sets) form a ring: a set is refilled with
    // the tile NBUF steps ahead as soon as it has been consumed.  In the steady-state loop every refill is
    // unconditional, so the in-order load counter can be waited on precisely (oldest tile only).
    if constexpr (LDS) {
        const int64_t n_keys = k_end - k_begin;
        const int n_tiles = (int)((n_keys + kDecTile - 1) / kDecTile);  // the ragged one among them
        const int n_mine = n_tiles > wave ? (n_tiles - wave + WAVES - 1) / WAVES : 0;
        const int ragged = n_keys % kDecTile ? n_tiles - 1 : -1;  // rows past its end arrive as zeros and are masked
        char *k0 = ks0[wave], *v0 = vs0[wave], *k1 = ks1[wave], *v1 = vs1[wave];
        // i-th tile of this wave out of a set of slots, with `others` sets asked for after it
        auto turn = [&](int i, auto set, auto others, auto reload) {
            constexpr int N = 2 * KL * decltype(others)::value;
            constexpr bool more = decltype(reload)::value;
            const int tile = wave + i * WAVES;
            Tile none;
            wait_loads(std::integral_constant<int, N + KL>{});
            step(none, k_begin + (int64_t)tile * kDecTile, tile == ragged, more, tile + NS * WAVES,
                 decltype(set)::value ? k1 : k0, decltype(set)::value ? v1 : v0, std::integral_constant<int, N + (more ? KL : 0)>{});
        };
        std::integral_constant<int, 0> c0;
        std::integral_constant<int, 1> c1;
        std::true_type refill;
        std::false_type done;
        if (n_mine > 0) {
            fill(wave, k0, true);
            fill(wave, v0, false);
            if constexpr (NS == 2) {
                fill(wave + WAVES, k1, true);  // (nothing if there is none)
                fill(wave + WAVES, v1, false);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {  // waited for here: ahead of a loop the compiler waits for all in flight
                u32x4_t w = __builtin_bit_cast(u32x4_t, qop[ks]);
                pin_here(w);
                qop[ks] = __builtin_bit_cast(vec8, w);
            }
            if constexpr (NS == 1) {
                for (int i = 0; i + 1 < n_mine; ++i) turn(i, c0, c0, refill);
                turn(n_mine - 1, c0, c0, done);
            } else {
                int i = 0;
                for (; i + 4 <= n_mine; i += 2) {
                    turn(i, c0, c1, refill);
                    turn(i + 1, c1, c1, refill);
                    if (PARTS && i + 2 >= part_end) put_aside();
                }
                if (n_mine - i == 3) {
                    turn(i, c0, c1, refill);
                    turn(i + 1, c1, c1, done);
                    turn(i + 2, c0, c0, done);
                } else {
                    turn(i, c0, c1, done);
                    if (n_mine - i == 2) turn(i + 1, c1, c0, done);
                }
            }
            wait_loads(c0);  // (a second tile that is not there)
        }
    } else {
        const int64_t n_keys = k_end - k_begin;
        const int n_full_all = (int)(n_keys / kDecTile);  // full tiles in the split
        const int n_mine = (n_full_all > wave) ? (n_full_all - wave + WAVES - 1) / WAVES : 0;
        auto tile_of = [&](int i) { return wave + i * WAVES; };  // i-th tile of this wave
        auto tile_key = [&](int i) { return k_begin + (int64_t)tile_of(i) * kDecTile; };
        Tile t[NBUF];
#pragma unroll
        for (int j = 0; j < NBUF; ++j)
            if (j < n_mine) { load_k(tile_of(j), t[j]); load_v(tile_of(j), t[j]); }
        int i = 0;
        for (; i + 2 * NBUF <= n_mine; i += NBUF) {
#pragma unroll
            for (int j = 0; j < NBUF; ++j) {
                step(t[j], tile_key(i + j), false, true, tile_of(i + j + NBUF), nullptr, nullptr, 0);
            }
            if (PARTS && i + NBUF >= part_end) put_aside();
        }
        // fewer than 2*NBUF tiles left: refills become conditional, then the ring drains
#pragma unroll
        for (int j = 0; j < NBUF; ++j) {
            if (i + j < n_mine) {
                if (i + j + NBUF < n_mine) step(t[j], tile_key(i + j), false, true, tile_of(i + j + NBUF), nullptr, nullptr, 0);
                else step(t[j], tile_key(i + j), false, false, 0, nullptr, nullptr, 0);
            }
        }
#pragma unroll
        for (int j = 0; j < NBUF; ++j)
            if (i + NBUF + j < n_mine) step(t[j], tile_key(i + NBUF + j), false, false, 0, nullptr, nullptr, 0);
        // ragged tail of the split (fewer than 32 keys): the wave whose turn it is takes it
        const int rem = (int)(n_keys % kDecTile);
        if (rem > 0 && (n_full_all % WAVES) == wave) {
            const int64_t key0 = k_begin + (int64_t)n_full_all * kDecTile;
            load_clamped(key0, t[0]);
            step(t[0], key0, true, false, 0, nullptr, nullptr, 0);
        }
    }

    if constexpr (PARTS) {
        put_aside();
#pragma unroll
        for (int i = 0; i < DCH; ++i) acc_o[i] = part_o[i];
        m_run = m_part;
        l_run = l_part;
    }
    // fold the four waves (Section 4.1 aggregation, in base 2); a thread finishes 4 columns of a row, so that the
    // fold of a short launch is one pass of 16-byte LDS reads
    const float l_tot = xor32_sum(xor16_sum(l_run));
    if (lq == 0) {
        sm_m[wave][lr] = m_run;
        sm_l[wave][lr] = l_tot;
    }
    if (lr < R) {
        if constexpr (LDS) {
#pragma unroll
            for (int i = 0; i < DCH; ++i) *(f32x4_t*)(out_row(wave, lr) + 16 * i + 4 * lq) = acc_o[i];
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < DCH; i += 4) {
                    f32x4_t o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = acc_o[i + e][r];
                    *(f32x4_t*)(out_row(wave, lr) + DCH * (4 * lq + r) + i) = o;
                }
        }
    }
    __syncthreads();
    float* Oout = O + ((int64_t)run * total_rows + unit * R) * D;
    float* Lout = lse + (int64_t)run * total_rows + unit * R;
    // padded batch with per-sequence query counts: row n of the unit is query n % Lq of its head; rows past the
    // sequence's count are padding and are not written
    int q_rows = Lq;
    if (q_lens) {
        const int v = q_len;
        q_rows = v < 0 ? 0 : (v < Lq ? v : Lq);
    }
    for (int idx = tid; idx < R * (D / 4); idx += WAVES * kWave) {
        const int n = idx / (D / 4);
        const int d = idx % (D / 4) * 4;
        if (q_lens && n % Lq >= q_rows) continue;
        float M = sm_m[0][n];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) M = fmaxf(M, sm_m[w][n]);
        f32x4_t num = zero_vec<f32x4_t>();
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float a = exp2_diff(sm_m[w][n], M);
            const f32x4_t o = *(const f32x4_t*)(out_row(w, n) + d);
#pragma unroll
            for (int e = 0; e < 4; ++e) num[e] = __builtin_fmaf(a, o[e], num[e]);
            den = __builtin_fmaf(a, sm_l[w][n], den);
        }
        const bool any = den > 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] = any ? num[e] / den : 0.f;
        *(f32x4_t*)(Oout + n * D + d) = num;
        if (d == 0) Lout[n] = any ? (M + fast_log2(den)) * kLn2 : -INFINITY;
    }
}

template <class T, int D, int QB>
static hipError_t launch_decode_t(const AttnProblem& p, hipStream_t stream) {
    typedef typename T::elem elem;
    const float scale_log2 = p.scale * kLog2e;
    const int64_t rows = (int64_t)p.B * p.Hq * p.Lq;
    int64_t part_keys;
    const KeyRuns runs = attn_runs_of(p, &part_keys);
    const int splits = runs.n_runs;
    if (splits < 1) return hipErrorInvalidValue;
    if (QB != 0 && p.n_shards > 1) return hipErrorInvalidValue;
    for (int i = 0; i < kMaxShards; ++i)  // a run is addressed with 32-bit byte offsets
        if (runs.s[i].L > 0 && runs.s[i].per * (int64_t)(QB ? D * QB / 8 : D * 2) > 0x7fffffffLL) return hipErrorInvalidValue;
    const int R = (int)((p.Hq / p.Hkv) * p.Lq);
    const int64_t units = (int64_t)p.B * p.Hkv;
    float* Odst = p.O;
    float* Ldst = p.lse;
    if (splits > 1) {
        if (!p.workspace || p.workspace_bytes < (size_t)splits * rows * (D + 1) * sizeof(float)) return hipErrorInvalidValue;
        Odst = (float*)p.workspace;
        Ldst = Odst + (size_t)splits * rows * D;
    }
    int64_t longest = 0, total = 0;
    for (int i = 0; i < runs.n_shards; ++i) {
        total += runs.s[i].L;
        const int64_t keys = runs.s[i].L < runs.s[i].per ? runs.s[i].L : runs.s[i].per;
        longest = keys > longest ? keys : longest;
    }
    int tiles = 0;  // per wave in LDS
    if (QB == 0) {
        const int64_t wgs = units * splits, cus = attn_target_wgs(), rounds = (wgs + cus - 1) / cus;
        // One tile also where such runs fill one round, from some 300 keys of 128 on (32 x 8 x 400 keys 11.7 us and 12.2 with two, 777 19.6
        // and 20.2, 1024 24.4 and 25.3 - 24.6 from registers -, 300 9.5 either way; of 64 two: 512 8.2 and 7.7).  (Parts need two.)
        const bool whole = D == 128 && part_keys == 0 && wgs * 10 >= cus * 9 && longest > 3 * kDecStride;
        tiles = longest <= kDecStride || ((wgs > cus || whole) && longest <= dec_single_tile_run(D)) ? 1 : 2;
        if (D == 128 && longest >= kDecLongRun && units * total * 10 >= rounds * cus * longest * 9) tiles = 0;
    }
    constexpr int kRegisters = QB == 0 && D == 64 ? 2 : 0;  // (16 bits of 64 columns have no such form)
    const int part = (int)((part_keys + kDecStride - 1) / kDecStride) & ~1;  // a wave's tiles of it, which are taken in pairs
    auto kernel = part_keys ? decode_attn_kernel<T, D, QB, kRegisters, kDecWaves, true> : decode_attn_kernel<T, D, QB, kRegisters, kDecWaves, false>;
    int threads = kDecThreads;
    if constexpr (QB == 0) {
        if (tiles == 1) kernel = decode_attn_kernel<T, D, 0, 1, kDecWaves, false>;  // (runs that were not cut anew)
        if (tiles == 2) kernel = part_keys ? decode_attn_kernel<T, D, 0, 2, kDecWaves, true> : decode_attn_kernel<T, D, 0, 2, kDecWaves, false>;
        // Two tiles in all: two waves and half of the LDS, so twice the workgroups to a compute unit (2048 units of 5, 20, 33, 48, 64 keys of
        // 64 4.9, 5.6, 6.7, 7.5, 8.6 us against 6.6, 7.3, 8.1, 8.8, 9.7, 8192 units 12.6 and 20.5, 26.3 and 28.9; of 128 2048 x 5 8.8 and 12.3;
        // a handful 1 to 3 %).  The waves left out had nothing.
        if (tiles == 1 && longest <= 2 * kDecTile) {
            kernel = decode_attn_kernel<T, D, 0, 1, kDecWaves / 2, false>;
            threads = kDecThreads / 2;
        }
        // Two tiles a wave and no more, on compute units of their own: eight waves with one tile each instead, whose loads are out at
        // once and whose chain of products is half as long (129 keys x 8 heads 4.8 -> 4.3 us, 192 4.9 -> 4.3, 256 5.5 -> 5.2, 1000 in
        // four runs 7.9 -> 7.65).  From some 300 keys on the two are within 1 %, at d = 64, whose tiles are half the bytes, this loses 2 to 5 %.
        if constexpr (D == 128)
            if (tiles == 2 && longest <= 2 * kDecStride) {
                kernel = decode_attn_kernel<T, D, 0, 1, 2 * kDecWaves, false>;
                threads = 2 * kDecThreads;
            }
    }
    if (!grid_fits(units * splits, kDecThreads)) return hipErrorInvalidValue;  // (eight waves are one round at most)
    hipLaunchKernelGGL(kernel, dim3((unsigned)(units * splits)), dim3(threads), 0, stream, (const elem*)p.Q, runs,
                       p.K_params, p.V_params, R, scale_log2, Odst, Ldst, rows, p.kv_lens, p.q_lens, (int)p.Lq, FastDiv(p.Hkv), part > 2 ? part : 2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || splits == 1) return e;
    return launch_lse_merge(Odst, Ldst, splits, rows, D, p.O, p.lse, stream, p.q_lens, p.Lq, (int64_t)p.Hq * p.Lq);
}

hipError_t launch_decode_attn(const AttnProblem& p, hipStream_t stream) {
    if (p.quant_bits != 0) {  // codes of the transport codec in place of K', V' (d = 128, checked by the caller)
        if (p.D != 128) return hipErrorInvalidValue;
        if (p.dtype == FEDRAG_BF16)
            return p.quant_bits == 8 ? launch_decode_t<BF16, 128, 8>(p, stream) : launch_decode_t<BF16, 128, 4>(p, stream);
        return p.quant_bits == 8 ? launch_decode_t<F16, 128, 8>(p, stream) : launch_decode_t<F16, 128, 4>(p, stream);
    }
    if (p.dtype == FEDRAG_BF16)
        return p.D == 128 ? launch_decode_t<BF16, 128, 0>(p, stream) : launch_decode_t<BF16, 64, 0>(p, stream);
    return p.D == 128 ? launch_decode_t<F16, 128, 0>(p, stream) : launch_decode_t<F16, 64, 0>(p, stream);
}

}  // namespace fedrag

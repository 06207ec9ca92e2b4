// Enc / Dec row transforms (Section 4.2, scrambled attention protocol, steps 1 and 3):
//   gather form   Y[j,:]       = X[perm[j],:] . Phi      (feature scramble + token permutation)
//   scatter form  Y[perm[i],:] = X[i,:] . Phi            (descramble + inverse permutation)
// One d x d matrix per KV head, shared by the G query heads of its group.
//
// 16-bit storage path: HBM-bound (each row is read once and written once, 2*d^2 flop per 4*d bytes), so the
// d x d product runs on MFMA only to stay far below the memory time.  A wave owns 16 rows at a time:
// rows are fetched with full-row coalesced 16-byte loads, staged through a wave-private LDS tile into the
// MFMA operand layout, multiplied against Phi^T held in registers for the whole kernel, and the fp32
// results are narrowed once (RNE), transposed back through the same LDS tile and stored as full rows.
#include <type_traits>

#include "fedrag_device.h"
#include "fedrag_host.h"

namespace fedrag {

// Two shapes of the tiled kernel.  Plain rows (QB = 0): 4 waves per workgroup, one per SIMD, Phi^T in 128 registers
// per wave for the whole kernel - the wave does little besides moving rows, and memory time hides it.  Rows that
// leave through the transport codec (QB = 8, 4): the codec's arithmetic needs a second wave per SIMD to hide behind the
// other wave's memory time, and two waves only fit when Phi^T stays in LDS and its operands are read per tile (32 KiB of
// LDS reads per 8 KiB of rows: a few per cent of the LDS rate).
// The codec shape was bound by its vector instructions while every 8-element chunk of a row, on its way out through LDS,
// had its own range reduction and divisions: 16 x 8111 tokens x 8 heads of 128 to 8 bits (fp16) 190 us, to 4 bits 205.  Coded
// from the accumulators (encode_row: some 190 instructions per 32 elements, 430 before) they take 159 and 146, near the
// memory's rate (5.1 TB/s).
constexpr int scr_waves(int qb) { return qb ? 8 : 4; }
constexpr int kScrPad = 8;    // elements of row padding in LDS (16 bytes: keeps 16-byte alignment, breaks bank stride)
constexpr int kScrRows = 32;  // rows per wave step (two 16-row MFMA column tiles)
// Register row-tile sets per wave (ring).  Plain, d = 128: three.  d = 64, where three only lengthen the start and the end of a
// short slab: two (16000 tokens x 8 heads 14.4 us against 15.1; 16 x 8192 as fast).  The codec's two waves per SIMD cover one
// another: at d = 128 the code around a second set costs more than it hides (4 x 7000 tokens x 4 heads 21.5 us against 25.7,
// 16 x 8192 159 against 165); at d = 64 two (16 x 8192 to 4 bits 70 against 76).
constexpr int scr_ring(int qb, int d) { return qb ? (d == 128 ? 1 : 2) : (d == 128 ? 3 : 2); }
#ifndef FEDRAG_SCR_WGS
#define FEDRAG_SCR_WGS 256    // workgroups to aim for over the whole launch (one per CU)
#endif
constexpr int kNonTemporal = 2;  // cache-policy bits of a buffer store

struct ScrambleJob {
    const void* X;
    const void* Phi;       // dense form: [Hkv, D, D]
    void* Y;
    // structured form (Section 4.2, Phi = S1 P1 H P2 S2), [Hkv, D] each; see structured_entry()
    const float* s_in;
    const int32_t* p_in;
    const int32_t* p_out;
    const float* s_out;
    // quantised output (transport codec of Section 7.5 applied to the narrowed rows): Y holds the codes, params the
    // per-row (scale, lo)
    float* params;
};

// Entry (k, n) of S1 P1 Hs P2 with the permutations as gathers and Hs the +-1 Sylvester matrix:
//   x S1 P1 Hs P2 = sum_k x[k] s_in[k] Hs[p_in^{-1}(k)][p_out[n]],   Hs[i][m] = (-1)^popcount(i & m).
// The 1/sqrt(d) of the normalised Hadamard matrix and S2 are applied to the fp32 sums afterwards, so that every
// product in the sums is x[k] times +-s_in[k] and nothing is rounded before the accumulation.
__device__ __forceinline__ float structured_entry(float s_in_k, int p_in_inv_k, int p_out_n) {
    return (__builtin_popcount(p_in_inv_k & p_out_n) & 1) ? -s_in_k : s_in_k;
}

// blockIdx.x = (head * members + member) * b_groups + bg; blockIdx.y selects the job (K or V).
// The `members` workgroups of one (job, head) share that head's Phi and sweep the sequences b = 0..B-1 together:
// every [L, d] slab is cut into 128-row groups dealt round-robin to the members, and the 4 waves of a member take
// the 32-row tiles of its group.  So at any moment the members of a (job, head) write one contiguous window that
// moves down the slab, the windows of all jobs and heads sit at the same offset inside their slabs (measured: a few
// per cent faster than one contiguous part per member, and than windows at staggered offsets), and Phi is staged
// once per workgroup for all sequences.  (When the slabs are too
// short to occupy the chip that way - decode queries - the sequences are dealt to b_groups workgroups instead.)
// A ring of NBUF register tile sets keeps gathered tiles (8 KiB each) in flight per wave behind the LDS
// staging and the MFMAs (it runs straight through the slab boundaries); the gather indices of a tile are fetched
// one step before its rows.  Tiles that start past the end of a slab are computed on clamped rows and not stored.
// QB = 0: rows leave in the storage type.  QB = 8 or 4: each narrowed row goes through the transport codec instead
// (same arithmetic as quantize_rows_kernel on the stored row) and leaves as codes plus (scale, lo).
template <class T, int D, bool ST, int QB>
FEDRAG_KERNEL __launch_bounds__(scr_waves(QB) * kWave, 1) void scramble_rows_kernel(ScrambleJob job0, ScrambleJob job1,
                                                                       const int32_t* __restrict__ perm,
                                                                       int64_t perm_batch_stride,  // 0 or L
                                                                       int B, int H, int G, int64_t L, int members,
                                                                       FastDiv by_slab, int b_groups) {
    typedef typename T::elem elem;
    typedef typename T::vec8 vec8;
    typedef typename T::vec4 vec4;
    constexpr int LDP = D + kScrPad;
    constexpr int CH = D / 8;              // 16-byte chunks per row
    constexpr int RPI = kWave / CH;        // rows covered by one wave-wide 16-byte load
    constexpr int NI = kScrRows / RPI;     // wave-wide loads per 32-row tile
    constexpr int KS = D / 32;             // contraction steps
    constexpr int MT = D / 16;             // output-column tiles
    constexpr int kScrWaves = scr_waves(QB);
    constexpr int kScrThreads = kScrWaves * kWave;
    constexpr bool kScrPhiLds = QB != 0;
    constexpr int NBUF = scr_ring(QB, D);
    constexpr int kPhiElems = D * LDP;
    constexpr int kTileElems = kScrWaves * kScrRows * LDP;
    // Codec shape: which output column row i of operand tile mt stands for is free, and is chosen so that a lane ends with whole
    // runs of 4 kMG columns of a row: 16 code bytes, or a quarter of the row where that is less.
    constexpr int kMG = QB == 8 ? 4 : MT;
    auto column = [](int mt, int i) {
        return QB == 0 ? mt * 16 + i : mt / kMG * (16 * kMG) + i / 4 * (4 * kMG) + mt % kMG * 4 + i % 4;
    };
    constexpr int kLdsElems = kScrPhiLds ? kPhiElems + kTileElems : (kPhiElems > kTileElems ? kPhiElems : kTileElems);

    // The staged matrix and the per-wave row tiles share one buffer when the operands are copied into registers (it is
    // then only needed until every wave has done so); with kScrPhiLds Phi^T stays and the row tiles follow it.
    __shared__ __attribute__((aligned(16))) elem lds[kLdsElems];

    const ScrambleJob job = blockIdx.y == 0 ? job0 : job1;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);  // wave-uniform
    const int lane = tid % kWave;
    const int h = blockIdx.x / (members * b_groups);
    const int member = (blockIdx.x / b_groups) % members;
    const int bg = blockIdx.x % b_groups;  // this workgroup takes sequences bg, bg + b_groups, ...

    const int ld_row = lane / CH;        // row within one wave-wide load
    const int ld_col = (lane % CH) * 8;  // element offset of this lane's 16 bytes

    // tile i of this wave: sequence b = i / tiles per slab, k-th tile of the wave inside this member's part
    const int n_mine = ((B - bg + b_groups - 1) / b_groups) * (int)by_slab.d;
    auto tile_b = [&](int i) { return bg + (int)by_slab.div((uint32_t)i) * b_groups; };
    auto tile_row0 = [&](int i) {
        const int k = (int)by_slab.mod((uint32_t)i);
        return ((int64_t)(k * members + member) * kScrWaves + wave) * kScrRows;
    };
    auto slab_off = [&](int i) { return ((int64_t)tile_b(i) * H + h) * L * D; };
    const elem* Xj = (const elem*)job.X;

    // Gather indices of a tile: lane l (< 32) holds the source row of tile row l; rows past the end re-read row L-1
    // (computed, never stored).  Memory operations are counted in order: the wait for one is a wait for all that were
    // issued before it, and what hides behind a branch cannot be counted, so that a wait past it is one for nearly everything
    // in flight.  Hence buffer accesses, which drop what is out of range, for the indices and for the stores.
    auto load_idx = [&](int i) -> int32_t {
        if (i >= n_mine) i = n_mine - 1;  // the index prefetch runs one tile past the end
        const int64_t row0 = tile_row0(i), first = row0 < L ? row0 : L - 1;
        const int last = (int)(L - 1 - first < kScrRows ? L - 1 - first : kScrRows);
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(perm + (int64_t)tile_b(i) * perm_batch_stride + first), 0, perm ? kScrRows * 4 : 0, 0x00020000);
        return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(rp, (lane % kScrRows < last ? lane % kScrRows : last) * 4, 0, 0);
    };
    auto load_rows = [&](int i, int32_t idx, vec8 (&buf)[NI]) {
        const elem* X = Xj + slab_off(i);
        if (!perm) {
            const int64_t j = tile_row0(i) + lane % kScrRows;
            idx = (int32_t)(j < L ? j : L - 1);
        }
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            const int64_t src = __shfl(idx, k * RPI + ld_row);
            buf[k] = __builtin_nontemporal_load((const vec8*)(X + src * D + ld_col));
        }
    };

    // ---- Phi^T operands (once per workgroup): phi operand (mt, ks) of a lane is Phi^T[16 mt + lane%16][32 ks + 8 (lane/16)
    // .. +8].  A structured key is multiplied out as Phi^T; a dense Phi goes to LDS row by row as it is stored and the
    // transposing LDS read hands out the operands.  (Transposed on the way in, two bytes at a time, this took longer than a
    // short slab's rows: a 117-token segment of 32 heads 12.2 -> 7.9 us, Enc of a 4096-token shard 13.2 -> 10.6 us.)
    const int lr = lane % 16;
    const int lq = lane / 16;
    // codec shape: Phi^T stays in front, a dense Phi is staged in the row tiles' place behind it
    elem* stage = lds + (kScrPhiLds && !ST ? kPhiElems : 0);
    auto phi_operand = [&](int mt, int ks) -> vec8 {
        if constexpr (ST) return *(const vec8*)(&lds[(mt * 16 + lr) * LDP + ks * 32 + lq * 8]);
        // two 4 x 16 blocks of Phi
        const char* p = (const char*)&stage[(ks * 32 + lq * 8 + lr / 4) * LDP + column(mt, lr % 4 * 4)];
        const u32x2_t lo = lds_read_tr16(p), hi = lds_read_tr16(p + 4 * LDP * (int)sizeof(elem));
        u32x4_t w;
        w[0] = lo[0]; w[1] = lo[1]; w[2] = hi[0]; w[3] = hi[1];
        return __builtin_bit_cast(vec8, w);
    };
    __shared__ __attribute__((aligned(16))) int32_t p_in_inv[ST ? D : 4];
    if (ST) {
        // structured form: the matrix is S1 P1 Hs P2, generated here from the key (entries +-s_in[k], which the
        // storage type holds exactly by the caller's contract); indices are masked into range
        const int32_t* g1 = job.p_in + (int64_t)(h / G) * D;
        for (int k = tid; k < D; k += kScrThreads) p_in_inv[g1[k] & (D - 1)] = k;
        __syncthreads();
        const float* a = job.s_in + (int64_t)(h / G) * D;
        const int32_t* g2 = job.p_out + (int64_t)(h / G) * D;
        // a thread keeps its 8 rows k0 .. k0+7 of Phi and walks the columns
        static_assert(kScrThreads % CH == 0, "k0 is the same in every pass");
        const int k0 = (tid % CH) * 8;
        float ak[8];
        int inv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            ak[e] = a[k0 + e];
            inv[e] = p_in_inv[k0 + e];
        }
#pragma unroll
        for (int n = tid / CH; n < D; n += kScrThreads / CH) {
            const int m = g2[column(n / 16, n % 16)] & (D - 1);
            vec8 v;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = T::from_float(structured_entry(ak[e], inv[e], m));
            *(vec8*)&lds[n * LDP + k0] = v;
        }
    } else {
        const elem* P = (const elem*)job.Phi + (int64_t)(h / G) * D * D;
#pragma unroll
        for (int c = tid; c < D * CH; c += kScrThreads)
            *(vec8*)&stage[c / CH * LDP + (c % CH) * 8] = *(const vec8*)(P + (int64_t)c * 8);
    }
    __syncthreads();
    vec8 phi[kScrPhiLds ? 1 : MT][kScrPhiLds ? 1 : KS];
    if constexpr (!kScrPhiLds) {  // in registers for the whole kernel
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) phi[mt][ks] = phi_operand(mt, ks);
        __syncthreads();  // the matrix in LDS is dead from here on; the buffer becomes the row tiles
    } else if constexpr (!ST) {  // to LDS, so that an operand is one 16-byte read from here on
        static_assert(MT * KS % kScrWaves == 0, "the operands divide evenly over the waves");
#pragma unroll
        for (int u = 0; u < MT * KS / kScrWaves; ++u) {
            const int op = wave + u * kScrWaves;
            *(vec8*)&lds[(op / KS * 16 + lr) * LDP + op % KS * 32 + lq * 8] = phi_operand(op / KS, op % KS);
        }
        __syncthreads();
    }
    const elem* phi_lds = &lds[lr * LDP + lq * 8];  // kScrPhiLds: operand (mt, ks) at + mt * 16 * LDP + ks * 32
    // structured form: S2 and the Hadamard normalisation, for this lane's output columns 16 mt + 4 lq + r
    // (codec shape: in LDS, in that order, to be read once a row)
    f32x4_t post[ST && QB == 0 ? MT : 1];
    __shared__ __attribute__((aligned(16))) float post_lds[ST && QB != 0 ? D : 4];
    if (ST) {
        const float* b = job.s_out + (int64_t)(h / G) * D;
        const float norm = D == 128 ? 0.08838834764831845f : 0.125f;  // 1 / sqrt(D)
        if constexpr (QB == 0) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) post[mt][r] = b[mt * 16 + lq * 4 + r] * norm;
        } else {
            if (tid < D) post_lds[tid] = b[column(tid / 16, tid % 16)] * norm;
            __syncthreads();
        }
    }

    elem* my = lds + (kScrPhiLds ? kPhiElems : 0) + wave * (kScrRows * LDP);

    // One row of the codec shape, a quarter of it in each of the lanes lr + 16 lq, straight from the accumulators: the range of
    // the narrowed row is the narrowed range of the sums (rounding is monotonic), the two divisions are done once a lane, and
    // the codes leave as 16 bytes a lane with no trip through LDS.
    float one = 1.0f;  // unknown to the compiler: x * one - lo takes x in 16 bits as it is, and is x - lo
    if constexpr (QB != 0) pin_here(one);
    auto encode_row = [&](f32x4_t (&y)[MT], int row, __amdgpu_buffer_rsrc_t ry, __amdgpu_buffer_rsrc_t rprm) {
        constexpr int LEVELS = (1 << (QB ? QB : 1)) - 1;
        if constexpr (ST) {
            int off = 0;
            pin_here(off);  // as for Phi^T below: read here, not kept
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                y[mt] *= *(const f32x4_t*)&post_lds[off + mt * 16 + lq * 4];
                pin_here(y[mt]);  // the product is rounded before it is narrowed, as in the plain form
            }
        }
        float lo = y[0][0], hi = y[0][0];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) { lo = fminf(lo, y[mt][r]); hi = fmaxf(hi, y[mt][r]); }
        lo = xor32_min(xor16_min(lo));
        hi = xor32_max(xor16_max(hi));
        lo = T::to_float(T::from_float(lo));
        hi = T::to_float(T::from_float(hi));
        const float range = hi - lo;
        const float scale = range / (float)LEVELS;
        // x - lo >= 0, so the sum is >= 1/2: converting to unsigned truncates = floors, and the lower clamp takes only NaN;
        // a constant row (range 0) gets steps 0, hence code 0
        const float steps = range > 0.0f ? (float)LEVELS / range : 0.0f;
        // 8 bits: the sum is below 256 (x - lo <= range, and range * steps rounds to 255 or one unit above it), so
        // the truncated byte is the code; an infinite sum (a range too small for 255 / range) truncates to 255,
        // the upper clamp of the definition, and a NaN (0 times that) to 0
        auto code = [&](int c) {  // c-th of this lane's columns
            const typename T::elem x = T::from_float(y[c / 4][c % 4]);
            const float t = __builtin_fmaf(__builtin_fmaf(T::to_float(x), one, -lo), steps, 0.5f);
            return QB == 8 ? t : clamp_code(t, (float)LEVELS);
        };
        uint32_t w[D * QB / 128 ? D * QB / 128 : 1];
#pragma unroll
        for (int k = 0; k < D / 64; ++k) {  // 16 columns a turn
            float t[16];
            uint32_t q[4];
#pragma unroll
            for (int e = 0; e < 16; ++e)  // 4 bits: the even columns of 8 in one word of bytes, the odd ones in the next
                t[e] = code(16 * k + (QB == 8 ? e : e / 8 * 8 + e % 4 * 2 + e / 4 % 2));
            bytes_of(t, q);
            if constexpr (QB == 8) {
#pragma unroll
                for (int e = 0; e < 4; ++e) w[4 * k + e] = q[e];
            } else {
                w[2 * k] = q[0] | q[1] << 4;
                w[2 * k + 1] = q[2] | q[3] << 4;
            }
        }
        constexpr int OUTB = D * QB / 8;
        if constexpr (D * QB == 256) {
            u32x2_t v;
            v[0] = w[0]; v[1] = w[1];
            __builtin_amdgcn_raw_buffer_store_b64(v, ry, row * OUTB + lq * 8, 0, kNonTemporal);
        } else {
#pragma unroll
            for (int k = 0; k < D * QB / 512; ++k) {
                u32x4_t v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = w[4 * k + e];
                __builtin_amdgcn_raw_buffer_store_b128(v, ry, row * OUTB + lq * 16, k * 64, kNonTemporal);
            }
        }
        u32x2_t prm;
        prm[0] = __builtin_bit_cast(uint32_t, scale);
        prm[1] = __builtin_bit_cast(uint32_t, lo);
        // one lane of a row stores them: the offset of the others is out of range
        __builtin_amdgcn_raw_buffer_store_b64(prm, rprm, lq == 0 ? row * 8 : 0x40000000, 0, 0);
    };

    auto step = [&](vec8 (&buf)[NI], int i, bool reload, int32_t& idx_next) {
        const int64_t row0 = tile_row0(i);
        const int64_t slab_row0 = ((int64_t)tile_b(i) * H + h) * L;
        // rows of the tile that exist, as stored
        constexpr int OUTB = QB ? D * QB / 8 : D * 2;
        const int n_out = (int)(L - row0 < 0 ? 0 : L - row0 < kScrRows ? L - row0 : kScrRows);
        const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((char*)job.Y + (slab_row0 + row0) * OUTB, 0,
                                                                            n_out * OUTB, 0x00020000);
        // rows -> LDS tile
#pragma unroll
        for (int k = 0; k < NI; ++k) *(vec8*)(&my[(k * RPI + ld_row) * LDP + ld_col]) = buf[k];
        wave_lds_fence();
        // Refill this register set with the tile NBUF steps ahead and fetch the indices of the one after it: in the codec shape
        // ahead of those rows, so that they are not waited for with them.  (Plain rows, at the rate of a copy, are up to 3 %
        // slower with that much more in flight: 64 x 2048 tokens x 8 heads of 64 93.6 us against 89.)
        if (reload) {
            const int32_t idx = idx_next;
            if (QB != 0) idx_next = load_idx(i + NBUF + 1);
            load_rows(i + NBUF, idx, buf);
            if (QB == 0) idx_next = load_idx(i + NBUF + 1);
        }
        if constexpr (QB == 0) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                // X^T operands: column = row (16 half + lane%16) of the tile, contraction slice 32 ks + 8 (lane/16)
                vec8 xop[KS];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    xop[ks] = *(const vec8*)(&my[(half * 16 + lr) * LDP + ks * 32 + lq * 8]);
                // Y^T tile (d x 16 rows) = Phi^T . X^T : lane holds tile row lane%16, output columns 16 mt + 4 lq + r
                f32x4_t acc[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    acc[mt] = zero_vec<f32x4_t>();
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) acc[mt] = T::mfma16(phi[mt][ks], xop[ks], acc[mt]);
                }
                // the 16 rows of this half are only read by the operand loads above (same wave, in order):
                // overwrite them with the narrowed results
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    vec4 o;
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[r] = T::from_float(ST ? acc[mt][r] * post[mt][r] : acc[mt][r]);
                    *(vec4*)(&my[(half * 16 + lr) * LDP + mt * 16 + lq * 4]) = o;
                }
            }
            wave_lds_fence();
            // full-row stores
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                const vec8 v = *(const vec8*)(&my[(k * RPI + ld_row) * LDP + ld_col]);
                const int64_t j = row0 + k * RPI + ld_row;
                if constexpr (D == 128) {  // (1 to 2 % faster from 16 x 8192 tokens on than the form below)
                    if (j < L) __builtin_nontemporal_store(v, (vec8*)((elem*)job.Y + (slab_row0 + j) * D + ld_col));
                } else {
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), ry,
                                                           (k * RPI + ld_row) * OUTB + ld_col * 2, 0, kNonTemporal);
                }
            }
        } else {
            // Both halves share an operand read.  The offset is one the compiler cannot see through (always 0), so that the
            // Phi^T operand reads stay with the MFMAs that use them instead of being hoisted into 128 registers.
            const __amdgpu_buffer_rsrc_t rprm =
                __builtin_amdgcn_make_buffer_rsrc(job.params + 2 * (slab_row0 + row0), 0, n_out * 8, 0x00020000);
            int phi_off = 0;
            pin_here(phi_off);
            const elem* phi_t = phi_lds + phi_off;
            vec8 xop[2][KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int half = 0; half < 2; ++half)
                    xop[half][ks] = *(const vec8*)(&my[(half * 16 + lr) * LDP + ks * 32 + lq * 8]);
            f32x4_t acc[2][MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                acc[0][mt] = acc[1][mt] = zero_vec<f32x4_t>();
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const vec8 op = *(const vec8*)(phi_t + mt * 16 * LDP + ks * 32);
#pragma unroll
                    for (int half = 0; half < 2; ++half) acc[half][mt] = T::mfma16(op, xop[half][ks], acc[half][mt]);
                }
            }
#pragma unroll
            for (int half = 0; half < 2; ++half) encode_row(acc[half], half * 16 + lr, ry, rprm);
        }
        wave_lds_fence();  // reads of the output tile done before the next tile's rows land
    };

    vec8 buf[NBUF][NI];
    int32_t idx_next = 0;
#pragma unroll
    for (int j = 0; j < NBUF; ++j)
        if (j < n_mine) load_rows(j, load_idx(j), buf[j]);
    if (NBUF < n_mine) idx_next = load_idx(NBUF);
    int i = 0;
    // steady state: tiles i+NBUF .. exist for every set, index prefetch may run one tile past the end (clamped)
    for (; i + 2 * NBUF <= n_mine; i += NBUF) {
#pragma unroll
        for (int j = 0; j < NBUF; ++j) step(buf[j], i + j, true, idx_next);
    }
#pragma unroll
    for (int j = 0; j < NBUF; ++j) {
        if (i + j < n_mine) {
            if (i + j + NBUF < n_mine) step(buf[j], i + j, true, idx_next);
            else step(buf[j], i + j, false, idx_next);
        }
    }
#pragma unroll
    for (int j = 0; j < NBUF; ++j)
        if (i + NBUF + j < n_mine) step(buf[j], i + NBUF + j, false, idx_next);
}

// A handful of rows per head (the decoding step: its queries, and Dec of its result): the tiled kernels stage a whole matrix
// per workgroup through LDS and registers for one or two rows.  Here a workgroup takes one (sequence, head) slab of at most
// kFewRows rows, and what counts is the number of trips to memory one after the other and of instructions fetched once.  Every
// thread asks for its share of the matrix, the rows, and what the aggregation needs of the first outputs, before it waits for
// anything: two columns of every 32 (d = 128) or 8 contraction steps, whole rows of the matrix to a wave.  Sums of a share are
// formed in its wave, the shares are added through LDS in order, the fp32 sum is narrowed once.
// With a whole column of the matrix a thread, 128 loads behind the rows', 64 sequences of 32 heads took 10.4 us and Dec 22.7, now
// 4.8 and 10.2.
// CS: workgroups that a slab's columns are split over, of 256 / CS threads; sums are formed as without, in the same order.  What one
// compute unit can fetch is then no longer the bound of a launch with few slabs, nor its LDS that of several rows.  d = 128, 32
// slabs, calls back to back, CS = 1 and 4: a decoded token's queries 2.65 and 2.41 us (fp32 3.33, 2.54), Dec of its result 3.20, 2.56, with
// the aggregation 3.57, 2.90; 4 rows 3.37, 3.08 (4.27, 3.21), 3.99, 3.24 and 4.53, 3.64; 16 rows 6.0, 5.3 (7.4, 5.9), 7.3, 6.3 and 9.4, 8.6.
// With up to kSplitRows rows, whose staging needs an eighth of the loads and registers, it is worth it for any number of slabs:
// 2048 x 4 rows of 128 7.7, 7.2 (16.3, 13.4), Dec 11.9, 11.9; at d = 64, whose workgroups of four columns' share are small, CS = 2
// from kSplitSlabs on (2048 x 1: 3.5, CS = 4 4.0, CS = 2 3.2; 512 x 4: 2.8, 2.85, 2.75).  More rows: from kSplitSlabs on CS = 1 (512 x 8
// of 128: 5.0, 5.1; fp32 7.9, 11.1; 128 x 8: 4.35, 4.23; 5.6, 4.7).
//   SCATTER == false: Y[j] = X[perm[j]] . Phi ; SCATTER == true (fp32): Y[perm[i]] = X[i] . Phi
constexpr int kFewRows = 16;
constexpr int kSplitRows = 4;
constexpr int64_t kSplitSlabs = 128;
// Of the form that sums in 64 bits, whose LDS is twice as much a row: at d = 64 eight rows of it leave room for four workgroups
// a compute unit, where 16 left two (64 x 32 slabs of 1, 5, 8 rows 4.8, 6.9, 8.6 us against 6.4, 9.7, 11.5).
constexpr int wide_rows(int d) { return d == 64 ? kFewRows / 2 : kFewRows; }
constexpr int kF32Threads = 256;  // workgroup size of the plain-FMA kernels

// fp32 storage in the terms of the 16-bit types
struct F32 {
    typedef float elem;
    static __device__ __forceinline__ elem from_float(float x) { return x; }
    static __device__ __forceinline__ float to_float(elem x) { return x; }
};

// The Section 4.1 aggregation of two partials of a row, in the arithmetic and order of lse_merge_kernel.
struct RowWeights {
    float a, b, inv;  // a, b < 0: weight zero, the partial takes no part
};
__device__ __forceinline__ RowWeights weights_of_two(float la, float lb, float* lse) {
    const float M = fmaxf(fmaxf(-INFINITY, la), lb);
    RowWeights w{-1.f, -1.f, 0.f};
    float den = 0.f;
    if (M != -INFINITY) {
        if (la != -INFINITY) den += w.a = expf(la - M);
        if (lb != -INFINITY) den += w.b = expf(lb - M);
        w.inv = 1.0f / den;
    }
    *lse = (M == -INFINITY) ? -INFINITY : M + logf(den);
    return w;
}
__device__ __forceinline__ float merge_two(const RowWeights& w, float mine, float other) {
    float o = 0.f;
    if (w.a != -1.f) o = __builtin_fmaf(w.a, mine, o);
    if (w.b != -1.f) o = __builtin_fmaf(w.b, other, o);
    return w.a != -1.f || w.b != -1.f ? o * w.inv : 0.f;
}

template <class T, int D, bool SCATTER, bool ST, bool WIDE, int CS, int ROWS>
__device__ __forceinline__ void few_rows(const ScrambleJob& job0, const ScrambleJob& job1, const int32_t* __restrict__ perm,
                                         int64_t perm_batch_stride, FastDiv by_h, FastDiv by_g, int L, const RowsMerge& mg) {
    typedef typename T::elem elem;
    constexpr bool kF32 = sizeof(elem) == 4;
    static_assert(!SCATTER || (kF32 && !ST), "Dec is fp32, and by a matrix here");
    constexpr bool kMerge = SCATTER;  // may be asked for the aggregation as well
    static_assert(CS == 1 || !ST, "the key's factors are for all columns");
    constexpr int kThreads = kF32Threads / CS;
    constexpr int COLS = D / CS;            // columns of this workgroup
    constexpr int LPK = COLS / 2;           // lanes per row of the matrix, two columns each
    constexpr int KG = kThreads / LPK;      // shares of the contraction, as many whatever CS
    constexpr int KPG = D / KG;             // steps of a share
    constexpr int kRows = WIDE && ROWS > wide_rows(D) ? wide_rows(D) : ROWS;  // at most
    constexpr int EPC = 16 / (int)sizeof(elem);              // row elements per 16-byte load
    constexpr int XC = (kRows * D / EPC + kThreads - 1) / kThreads;  // such loads per thread, at most
    typedef elem chunk_t __attribute__((ext_vector_type(EPC)));
    typedef elem pair_t __attribute__((ext_vector_type(2)));
    // WIDE (fp32 storage): the rounding of the queries comes back multiplied by the scores, and there is time for sums in 64 bits
    // (4 rows x 512 keys, outputs against 64 bits: 1.0e-6 with fp32 sums one after the other, 0.8e-6; log-sum-exps 1.0e-7, 0.6e-7)
    static_assert(!WIDE || (kF32 && !SCATTER), "queries in fp32 storage");
    typedef typename std::conditional<WIDE, double, float>::type acc_t;
    typedef acc_t acc4_t __attribute__((ext_vector_type(4)));
    typedef acc_t acc2_t __attribute__((ext_vector_type(2)));
    __shared__ __attribute__((aligned(16))) acc_t xs[kRows * D];
    __shared__ __attribute__((aligned(16))) acc_t part[KG][kRows * COLS];
    __shared__ int32_t p_in_inv[ST ? D : 1];
    __shared__ float s_in[ST ? D : 1];
    const ScrambleJob job = blockIdx.y == 0 ? job0 : job1;
    FEDRAG_HAVE_HERE(FEDRAG_S(job.X), FEDRAG_S(job.Y), FEDRAG_S(perm), FEDRAG_S(perm_batch_stride), FEDRAG_S3(by_h), FEDRAG_S3(by_g),
                     FEDRAG_S(L));
    // (of a key's pointers only in fp32: 16 rows of K and V of 8 heads of 64 in 16 bits took 4.25 us with them, 4.01 without, of 128 6.3
    // and 6.1; in fp32 4.09 and 4.24)
    if constexpr (ST && kF32) FEDRAG_HAVE_HERE(FEDRAG_S(job.s_in), FEDRAG_S(job.p_in), FEDRAG_S(job.p_out), FEDRAG_S(job.s_out));
    if constexpr (!ST) FEDRAG_HAVE_HERE(FEDRAG_S(job.Phi));
    if constexpr (kMerge)
        FEDRAG_HAVE_HERE(FEDRAG_S(mg.lse_in), FEDRAG_S(mg.O_other), FEDRAG_S(mg.lse_other), FEDRAG_S(mg.lse_out));
    const int tid = threadIdx.x;
    const int cl = 2 * (tid % LPK);  // first of this thread's two columns
    const int kg = tid / LPK;
    const int bh = blockIdx.x;
    const int b = (int)by_h.div((uint32_t)bh);
    const int hk = (int)by_g.div(by_h.mod((uint32_t)bh));  // the head's matrix
    const int c0 = CS > 1 ? (int)blockIdx.z * COLS : 0;
    const elem* X = (const elem*)job.X + (int64_t)bh * L * D;
    elem* Y = (elem*)job.Y + (int64_t)bh * L * D;
    const int32_t* pm = perm ? perm + (int64_t)b * perm_batch_stride : nullptr;
    const int n_out = L * COLS;

    // where the rows come from (those past the end re-read the last one and are left out)
    int src[XC];
#pragma unroll
    for (int u = 0; u < XC; ++u) {
        const int j = (tid + u * kThreads) / (D / EPC);
        src[u] = j < L ? j : L - 1;
    }
    if (!SCATTER && pm) {
#pragma unroll
        for (int u = 0; u < XC; ++u) src[u] = pm[src[u]];
    }
    // and where this thread's first output goes: asked for ahead of the matrix, which a wait for it would be a wait for otherwise
    auto row_of = [&](int e) { return e < n_out ? e / COLS : L - 1; };
    int first_dst = row_of(tid);
    if (SCATTER && pm) first_dst = pm[first_dst];
    // the matrix
    pair_t phi_in[ST ? 1 : KPG];
    if constexpr (!ST) {
        const elem* P = (const elem*)job.Phi + (int64_t)hk * D * D + (int64_t)kg * KPG * D + c0 + cl;
#pragma unroll
        for (int i = 0; i < KPG; ++i) phi_in[i] = *(const pair_t*)(P + i * D);
    }
    int32_t key_inv = 0, key_out0 = 0, key_out1 = 0;
    float key_in = 0.f, post0 = 1.f, post1 = 1.f;  // post: fp32 of columns cl, cl + 1; 16 bits (post0) of column tid % D
    if constexpr (ST) {
        const int64_t at = (int64_t)hk * D;
        if (tid < D) {
            key_inv = job.p_in[at + tid];
            key_in = job.s_in[at + tid];
        }
        key_out0 = job.p_out[at + cl];
        key_out1 = job.p_out[at + cl + 1];
        post0 = job.s_out[at + (kF32 ? cl : tid % D)];
        post1 = job.s_out[at + cl + 1];
    }
    // the rows
    chunk_t x_in[XC];
#pragma unroll
    for (int u = 0; u < XC; ++u)
        x_in[u] = *(const chunk_t*)(X + (int64_t)src[u] * D + (tid + u * kThreads) % (D / EPC) * EPC);
    // outputs e = tid, tid + 256, ... : row and what the aggregation reads of it
    struct Out {
        int64_t dst;
        float la, lb, other;
    };
    auto out_of = [&](int e, int dst) {
        Out o{dst, 0.f, 0.f, 0.f};
        if (kMerge && mg.lse_in) {
            o.la = mg.lse_in[(int64_t)bh * L + row_of(e)];
            o.lb = mg.lse_other[(int64_t)bh * L + dst];
            o.other = mg.O_other[((int64_t)bh * L + dst) * D + c0 + e % COLS];
        }
        return o;
    };
    Out next = out_of(tid, first_dst);

#pragma unroll
    for (int u = 0; u < XC; ++u)
#pragma unroll
        for (int q = 0; q < EPC; ++q)
            if (XC > 1 || tid < kRows * D / EPC) xs[(tid + u * kThreads) * EPC + q] = T::to_float(x_in[u][q]);
    if constexpr (ST) {
        if (tid < D) {
            p_in_inv[key_inv & (D - 1)] = tid;
            // 16 bits: the matrix entries are +-scale_in narrowed to the storage type, as in the tiled kernel
            s_in[tid] = T::to_float(T::from_float(key_in));
        }
        post0 *= D == 128 ? 0.08838834764831845f : 0.125f;  // 1 / sqrt(D)
        post1 *= D == 128 ? 0.08838834764831845f : 0.125f;
    }
    __syncthreads();
    acc_t phi[KPG][2];
#pragma unroll
    for (int i = 0; i < KPG; ++i) {
        if constexpr (ST) {
            const int k = kg * KPG + i;
            phi[i][0] = structured_entry(s_in[k], p_in_inv[k], key_out0 & (D - 1));
            phi[i][1] = structured_entry(s_in[k], p_in_inv[k], key_out1 & (D - 1));
            if (kF32) { phi[i][0] *= post0; phi[i][1] *= post1; }  // fp32: as the tiled fp32 kernel; 16 bits: after the sum
        } else {
            phi[i][0] = T::to_float(phi_in[i][0]);
            phi[i][1] = T::to_float(phi_in[i][1]);
        }
    }
#pragma unroll 1
    for (int r = 0; r < L; ++r) {
        acc2_t a;
        a[0] = a[1] = 0;
#pragma unroll
        for (int i4 = 0; i4 < KPG; i4 += 4) {
            const acc4_t x = *(const acc4_t*)(&xs[r * D + kg * KPG + i4]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    if constexpr (sizeof(acc_t) == 8) a[c] = __builtin_fma(x[e], phi[i4 + e][c], a[c]);
                    else a[c] = __builtin_fmaf(x[e], phi[i4 + e][c], a[c]);
                }
        }
        *(acc2_t*)(&part[kg][r * COLS + cl]) = a;
    }
    __syncthreads();
#pragma unroll 1
    for (int e = tid; e < n_out; e += kThreads) {
        const Out o = next;
        if (e + kThreads < n_out) {
            const int row = row_of(e + kThreads);
            next = out_of(e + kThreads, SCATTER && pm ? pm[row] : row);
        }
        acc_t sum = part[0][e];
#pragma unroll
        for (int g = 1; g < KG; ++g) sum += part[g][e];
        float v = (float)sum;
        if (ST && !kF32) {
            v *= post0;
            pin_here(v);  // narrowed afterwards, as in the tiled kernel: in one operation a zero would lose its sign
        }
        if (kMerge && mg.lse_in) {
            float l;
            v = merge_two(weights_of_two(o.la, o.lb, &l), v, o.other);
            if (c0 + e % COLS == 0) mg.lse_out[(int64_t)bh * L + o.dst] = l;
        }
        Y[o.dst * D + c0 + e % COLS] = T::from_float(v);
    }
}

template <class T, int D, bool SCATTER, bool ST, bool WIDE>
FEDRAG_KERNEL __launch_bounds__(kF32Threads) void few_rows_kernel(ScrambleJob job0, ScrambleJob job1,
                                                               const int32_t* __restrict__ perm,
                                                               int64_t perm_batch_stride, FastDiv by_h, FastDiv by_g, int L,
                                                               RowsMerge mg) {
    few_rows<T, D, SCATTER, ST, WIDE, 1, kFewRows>(job0, job1, perm, perm_batch_stride, by_h, by_g, L, mg);
}

template <class T, int D, bool SCATTER, bool WIDE, int CS, int ROWS>
FEDRAG_KERNEL __launch_bounds__(kF32Threads / CS) void few_rows_of_few_columns_kernel(ScrambleJob job0, ScrambleJob job1,
                                                                                   const int32_t* __restrict__ perm,
                                                                                   int64_t perm_batch_stride, FastDiv by_h,
                                                                                   FastDiv by_g, int L, RowsMerge mg) {
    few_rows<T, D, SCATTER, false, WIDE, CS, ROWS>(job0, job1, perm, perm_batch_stride, by_h, by_g, L, mg);
}

// fp32 rows times fp32 matrix (fp32 storage path of Enc, and Dec for every storage type) on the fp32 matrix cores, for slabs
// of more rows than the kernel above takes.  mg.lse_in != NULL (scatter form only): the transformed row is one of two partials
// of Section 4.1 and is aggregated with the other one, which is already in destination order, before it is stored.
// What bounds it below some hundred rows is the chain of trips to memory, so the rows, their destinations and what the
// aggregation needs of them are asked for ahead of the matrix, or of the product of the step before, and a row's weights are
// evaluated once, by one thread, not by each of its columns' (Dec of 117 rows of 32 heads of 128 7.4 -> 5.8 us, with the aggregation
// 12.8 -> 6.7; 4096 rows 60 -> 48 and 132 -> 60; 40 rows, with plain FMAs and a column of the matrix a thread, 13.7, now 5.6).
// v_mfma_f32_32x32x2_f32: A 32 x 2 (lane: row lane % 32, k = lane / 32), B 2 x 32 (lane: column lane % 32, k = lane / 32),
// C 32 x 32 (lane: column lane % 32, register r: row 8 (r / 4) + 4 (lane / 32) + r % 4).  Wave w of the 4 owns the
// 32-column slice w % (D / 32) of the output and keeps that slice of Phi in registers as B operands (D / 2 of them);
// the rows of a step (32 for D = 128, two tiles of 32 for D = 64) are staged once in LDS, coalesced, and every wave
// reads its tile's rows from there 16 bytes at a time: the 4 floats are the A operands of 4 steps, contraction index
// 8 j + 4 (lane / 32) + e for read j, element e.  The next step's rows are fetched into registers before the MFMAs
// of the current one and go to the other LDS buffer after them: one barrier per step.
// RT: 32-row tiles per step.  One at d = 128; two at d = 64, but one, with half the waves, for slabs of at most 32 rows, where the
// second tile's waves had nothing to do and held their place: 64 x 32 slabs of 17, 24, 32 rows 11.5, 12.2, 12.7 us against 15.0, 15.3,
// 15.6 (a plain-FMA kernel 11.9, 13.7, 15.8), structured 10.0, 10.8, 11.6 against 15.1, 15.5, 16.2.
constexpr int mf_threads(int d, int rt) { return d / 32 * rt * kWave; }
template <int D, bool SCATTER, bool ST, bool MERGE, int RT>
FEDRAG_KERNEL __launch_bounds__(mf_threads(D, RT)) void rows_times_matrix_mfma_f32_kernel(ScrambleJob job0, ScrambleJob job1,
                                                                                 const int32_t* __restrict__ perm,
                                                                                 int64_t perm_batch_stride, FastDiv by_h,
                                                                                 FastDiv by_g, int64_t L, FastDiv by_chunks,
                                                                                 int steps_per_wg, RowsMerge mg) {
    constexpr int SL = D / 32;         // 32-column slices of the output
    constexpr int kThreads = mf_threads(D, RT);
    constexpr int TR = 32 * RT;        // rows per step
    constexpr int LDP = D + 4;         // padded LDS row, floats: 16-byte reads of 8 rows cover all banks once
    constexpr int NJ = D / 8;          // 16-byte operand reads per row
    constexpr int CPR = D / 4;         // 16-byte chunks per row
    constexpr int CPT = TR * CPR / kThreads;  // chunks per thread per step
    static_assert(CPT * kThreads == TR * CPR, "a step's rows divide evenly over the threads");
    __shared__ __attribute__((aligned(16))) float xs[2][TR * LDP];
    __shared__ int32_t p_in_inv[ST ? D : 1];
    __shared__ float s_in[ST ? D : 1];
    // scatter form: where the rows of a step go and their weights, looked up and evaluated once a row
    __shared__ int32_t row_dst[SCATTER ? 2 : 1][SCATTER ? TR : 1];
    __shared__ RowWeights row_w[MERGE ? 2 : 1][MERGE ? TR : 1];
    static_assert(!SCATTER || !ST, "Dec by a key's factors is not a product");
    static_assert(!MERGE || SCATTER, "the aggregation is part of Dec");

    const ScrambleJob job = blockIdx.y == 0 ? job0 : job1;
    // one trip to memory, and heads without divisions: 1 to 7 % of launches of up to some 30 us, 2.5 % on average over 114
    FEDRAG_HAVE_HERE(FEDRAG_S(job.X), FEDRAG_S(job.Y), FEDRAG_S(perm), FEDRAG_S(perm_batch_stride), FEDRAG_S3(by_h), FEDRAG_S3(by_g),
                     FEDRAG_S(L), FEDRAG_S3(by_chunks), FEDRAG_S(steps_per_wg));
    if constexpr (ST) FEDRAG_HAVE_HERE(FEDRAG_S(job.s_in), FEDRAG_S(job.p_in), FEDRAG_S(job.p_out), FEDRAG_S(job.s_out));
    else FEDRAG_HAVE_HERE(FEDRAG_S(job.Phi));
    if constexpr (MERGE)
        FEDRAG_HAVE_HERE(FEDRAG_S(mg.lse_in), FEDRAG_S(mg.O_other), FEDRAG_S(mg.lse_other), FEDRAG_S(mg.lse_out));
    const int tid = threadIdx.x;
    const int wave = tid / kWave;
    const int lane = tid % kWave;
    const int n = lane % 32;
    const int kk = lane / 32;
    const int slice = wave % SL;
    const int rt = wave / SL;
    const int bh = (int)by_chunks.div(blockIdx.x);
    const int chunk = (int)by_chunks.mod(blockIdx.x);
    const int b = (int)by_h.div((uint32_t)bh);
    const int hk = (int)by_g.div(by_h.mod((uint32_t)bh));  // the head's matrix
    const int64_t first_row = (int64_t)chunk * steps_per_wg * TR;
    if (first_row >= L) return;  // workgroup-uniform, before any barrier
    int n_steps = (int)((L - first_row + TR - 1) / TR);
    if (n_steps > steps_per_wg) n_steps = steps_per_wg;

    const float* X = (const float*)job.X + (int64_t)bh * L * D;
    float* Y = (float*)job.Y + (int64_t)bh * L * D;
    const int32_t* pm = perm ? perm + (int64_t)b * perm_batch_stride : nullptr;

    // gather form: a step's source rows.  A wait for one load is one for all before it, so the first step's indices are asked for
    // ahead of the matrix, and the rows they lead to behind it; asked for in one go ahead of it, the matrix waited for the
    // indices (16 x 64 rows x 32 heads of 128 16.6 us, 17.3 so, 16.2 now; 4 x 500 structured 17.1, 17.8, 16.2).  Structured keys of
    // 64 columns have no registers to spare for the indices meanwhile: a fourth workgroup a compute unit would be lost.
    constexpr bool kSrcAhead = !(D == 64 && ST);
    int32_t src[SCATTER ? 1 : CPT];
    auto fetch_src = [&](int64_t row0) {
        if constexpr (!SCATTER) {
#pragma unroll
            for (int q = 0; q < CPT; ++q) {
                int64_t j = row0 + (tid + q * kThreads) / CPR;
                if (j >= L) j = L - 1;  // rows past the end: computed on a real row, never stored
                src[q] = pm ? pm[j] : (int32_t)j;
            }
        }
    };
    auto fetch = [&](int64_t row0, f32x4_t (&buf)[CPT]) {
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            const int e = tid + q * kThreads;
            int64_t j = row0 + e / CPR;
            if (j >= L) j = L - 1;
            if constexpr (!SCATTER) j = src[q];
            buf[q] = *(const f32x4_t*)(X + j * D + (e % CPR) * 4);
        }
    };
    // thread t < TR: row t of a step
    int32_t next_dst = 0;
    float next_la = 0.f, next_lb = 0.f;
    auto fetch_row = [&](int64_t row0) {
        if (!SCATTER || tid >= TR) return;
        const int64_t j = row0 + tid < L ? row0 + tid : L - 1;
        next_dst = pm ? pm[j] : (int32_t)j;
        if constexpr (MERGE) {
            next_la = mg.lse_in[(int64_t)bh * L + j];
            next_lb = mg.lse_other[(int64_t)bh * L + next_dst];
        }
    };
    // asked for ahead of the matrix
    f32x4_t buf[CPT];
    if constexpr (SCATTER) fetch(first_row, buf);
    else if constexpr (kSrcAhead) fetch_src(first_row);
    fetch_row(first_row);

    const int col = 32 * slice + n;  // this lane's output column
    float phi[NJ][4];
    if (ST) {  // column `col` of S1 P1 H P2 S2, generated from the key
        const int32_t* g1 = job.p_in + (int64_t)hk * D;
        for (int k = tid; k < D; k += kThreads) {
            p_in_inv[g1[k] & (D - 1)] = k;
            s_in[k] = job.s_in[(int64_t)hk * D + k];
        }
        __syncthreads();
        const int m = job.p_out[(int64_t)hk * D + col] & (D - 1);
        const float post = job.s_out[(int64_t)hk * D + col] * (D == 128 ? 0.08838834764831845f : 0.125f);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = 8 * j + 4 * kk + e;
                phi[j][e] = structured_entry(s_in[k], p_in_inv[k], m) * post;
            }
    } else {
        const float* P = (const float*)job.Phi + (int64_t)hk * D * D;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) phi[j][e] = P[(8 * j + 4 * kk + e) * D + col];
    }

    auto stash = [&](int slot, const f32x4_t (&buf)[CPT]) {
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            const int e = tid + q * kThreads;
            *(f32x4_t*)(&xs[slot][(e / CPR) * LDP + (e % CPR) * 4]) = buf[q];
        }
    };

    auto stash_row = [&](int slot, int64_t row0) {
        if (!SCATTER || tid >= TR) return;
        row_dst[slot][tid] = next_dst;
        if constexpr (MERGE) {
            float l;
            row_w[slot][tid] = weights_of_two(next_la, next_lb, &l);
            if (row0 + tid < L) mg.lse_out[(int64_t)bh * L + next_dst] = l;
        }
    };

    if constexpr (!SCATTER) {
        if constexpr (!kSrcAhead) fetch_src(first_row);
        fetch(first_row, buf);
    }
    stash(0, buf);
    stash_row(0, first_row);
    __syncthreads();
    for (int s_ = 0; s_ < n_steps; ++s_) {
        const int64_t row0 = first_row + (int64_t)s_ * TR;
        const bool more = s_ + 1 < n_steps;
        if (more) {
            fetch_src(row0 + TR);
            fetch(row0 + TR, buf);
            fetch_row(row0 + TR);
        }
        auto row_of = [&](int r) { return 32 * rt + 8 * (r / 4) + 4 * kk + (r % 4); };  // of the step, accumulator register r
        if (row0 + 32 * rt < L) {  // (d = 64: the second tile of a step may be past the end)
            float other[MERGE ? 16 : 1];
            if constexpr (MERGE) {  // the other partial's elements are on their way behind the product
#pragma unroll
                for (int r = 0; r < 16; ++r) other[r] = mg.O_other[((int64_t)bh * L + row_dst[s_ & 1][row_of(r)]) * D + col];
            }
            const float* xr = &xs[s_ & 1][(32 * rt + n) * LDP + 4 * kk];
            f32x16_t acc = zero_vec<f32x16_t>();
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const f32x4_t a = *(const f32x4_t*)(xr + 8 * j);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], phi[j][e], acc, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t j = row0 + row_of(r);
                if (j >= L) continue;
                float v = acc[r];
                if constexpr (SCATTER) {
                    if constexpr (MERGE) v = merge_two(row_w[s_ & 1][row_of(r)], v, other[r]);
                    Y[(int64_t)row_dst[s_ & 1][row_of(r)] * D + col] = v;
                } else {
                    Y[j * D + col] = v;
                }
            }
        }
        if (more) {
            stash((s_ + 1) & 1, buf);
            stash_row((s_ + 1) & 1, row0 + TR);
        }
        __syncthreads();
    }
}

// Rows times a structured key, factor by factor: the scales and the channel gathers are what they are, and the Hadamard matrix is
// seven (d = 64: six) steps of additions and subtractions, in place of a product with a matrix that every workgroup multiplies out.
// 16 lanes hold a row, D / 16 values each: a lane's own values are combined in registers, those of different lanes by
// data-parallel moves; the two gathers go through LDS, within a wave.  Every load but those of rows that wait for their indices is
// asked for at once.
// Dec, always: the fp32 product was bound by the fp32 matrix pipe or, for few rows, by its chain of waits; this is bound by memory
// or by the launch, whose arguments are one trip to memory (117 rows 3.2 -> 3.05 us).  Its sums of 128 are seven roundings deep.
//   32 heads, us, product -> factors    1 row        16           117          1000         4096
//   of 128                              3.3 -> 2.9   7.1 -> 2.9   6.4 -> 3.2   17.2 -> 7.5  47 -> 23
//   of 64                               2.5 -> 2.4   4.4 -> 2.6   5.0 -> 2.7   7.8 -> 4.9   20.3 -> 12.0
// Queries in 16 bits: heads of at most kHadSlab rows, where a tile of the product is mostly padding or its matrix is all it does,
// or at most kHadTotal rows in all.  Beyond that the product is hidden by memory and this is not.  Only 129 to 160 rows a head
// would gain again (256 x 32 x 129 rows of 128 151 and 124, 64 x 32 x 160 42.7 and 32.9; of 64 65.9 and 65.2, 21.4 and 19.3), as the
// product begins a second pass of 128 rows there; it has no rule of its own.
//   32 heads, us, product, factors      4 rows       16           117          1000         1500         2048         4096
//   of 128                              3.8, 3.0     6.3, 3.0     6.0, 3.2     7.4, 6.3     10.3, 9.0    11.1, 11.0   15.5, 16.9
//   of 64                               3.0, 2.5     4.2, 2.6     4.2, 2.7     4.6, 4.3     6.0, 5.1     6.9, 6.5     10.6, 10.5
//   x 256 sequences                     32 rows      64           80           96           112          128          256
//   of 128                              69.6, 26.1   72.9, 47.4   76.5, 69.8   82.4, 83.4   87.8, 97.5   92.2, 109    183, 223
//   of 64                               30.4, 16.6   33.1, 27.9   35.5, 33.5   38.9, 39.4   42.0, 45.2   46.7, 52.0   91, 134
//   x 32                                48           64           80           96           112          128          256
//   of 128                              14.8, 10.8   14.8, 11.5   14.2, 13.9   14.2, 14.0   14.4, 16.5   15.3, 17.3   27.4, 27.5
//   of 64                               7.8, 6.2     8.1, 6.5     8.7, 8.1     9.0, 8.6     9.5, 10.5    9.7, 10.4    15.7, 16.3
// Enc of K and V, which its coded form equals bit for bit, keeps the product at every size.
//   SCATTER == false: Y[j] = X[perm[j]] . Phi ; SCATTER == true (fp32): Y[perm[i]] = X[i] . Phi
constexpr int64_t kHadSlab = 96, kHadTotal = 48 << 10;
constexpr int64_t kHadWgsPerUnit = 8;  // workgroups a compute unit has from where on one takes several steps
constexpr int kHadRows = 16;        // rows per workgroup step
constexpr int kHadThreads = 16 * kHadRows;
constexpr float kHadLeast = 0x1p-100f;  // terms of sums above it have all their bits that count
template <class T, int D, bool SCATTER>
FEDRAG_KERNEL __launch_bounds__(kHadThreads) void hadamard_rows_kernel(ScrambleJob job, const int32_t* __restrict__ perm,
                                                                       int64_t perm_batch_stride, FastDiv by_chunks, FastDiv by_heads,
                                                                       FastDiv by_group, int64_t L, int steps_per_wg, int first_slab) {
    typedef typename T::elem elem;
    static_assert(!SCATTER || sizeof(elem) == 4, "Dec is fp32");
    constexpr int E = D / 16;                                            // values per lane
    constexpr int EPC = E * (int)sizeof(elem) > 16 ? 16 / (int)sizeof(elem) : E;  // values per load, a lane's loads 16 lanes apart
    constexpr int NC = E / EPC;
    constexpr int LDP = D + 4;
    typedef elem chunk_t __attribute__((ext_vector_type(EPC)));
    typedef int32_t keys_t __attribute__((ext_vector_type(4), aligned(4)));  // key arrays are dword-aligned
    __shared__ __attribute__((aligned(16))) float rows[kHadRows][LDP];
    FEDRAG_HAVE_HERE(FEDRAG_S(job.X), FEDRAG_S(job.Y), FEDRAG_S(job.s_in), FEDRAG_S(job.p_in), FEDRAG_S(job.p_out), FEDRAG_S(job.s_out),
                     FEDRAG_S(perm), FEDRAG_S(perm_batch_stride), FEDRAG_S3(by_chunks), FEDRAG_S3(by_heads), FEDRAG_S3(by_group), FEDRAG_S(L),
                     FEDRAG_S(steps_per_wg), FEDRAG_S(first_slab));
    const int tid = threadIdx.x, rl = tid / 16, l = tid % 16;
    const int slab = (int)by_chunks.div(blockIdx.x), chunk = (int)blockIdx.x - slab * (int)by_chunks.d;
    const int bh = first_slab + slab;
    const int b = (int)by_heads.div(bh), h = bh - b * (int)by_heads.d;
    const int64_t at = (int64_t)by_group.div(h) * D;
    const int32_t* pm = perm ? perm + (int64_t)b * perm_batch_stride : nullptr;
    const elem* X = (const elem*)job.X + (int64_t)bh * L * D;
    elem* Y = (elem*)job.Y + (int64_t)bh * L * D;
    float* my = rows[rl];
    const int64_t row0 = (int64_t)chunk * steps_per_wg * kHadRows + rl;
    int n_steps = (int)((L - (int64_t)chunk * steps_per_wg * kHadRows + kHadRows - 1) / kHadRows);
    if (n_steps > steps_per_wg) n_steps = steps_per_wg;

    auto natural = [&](int c) { return (c * 16 + l) * EPC; };  // first channel of this lane's load c
    auto row_of = [&](int s) { const int64_t j = row0 + (int64_t)s * kHadRows; return j < L ? j : L - 1; };
    // Which block of E positions of the Hadamard product lane l holds: the moves flip bit 0, bit 1, bits 0 to 2 and bit 3 of a lane's
    // number, and block a is where the set of these that leads there from lane 0 is a.
    const int a = l ^ (l & 4 ? 3 : 0);

    int32_t idx = pm ? pm[row_of(0)] : (int32_t)row_of(0);
    auto load = [&](int64_t j, chunk_t (&x)[NC]) {
#pragma unroll
        for (int c = 0; c < NC; ++c) x[c] = *(const chunk_t*)(X + j * D + natural(c));
    };
    chunk_t x[NC];
    if constexpr (SCATTER) load(row_of(0), x);
    float s_in[E], post[E];
    int g_in[E], g_out[E];  // the gathers, as channels
    auto load_key = [&](const void* p, int (&v)[E], bool in_place) {
#pragma unroll
        for (int q = 0; q < E / 4; ++q) {
            const int n = in_place ? E * a + 4 * q : EPC < 8 ? natural(q) : natural(0) + 4 * q;
            const keys_t w = *(const keys_t*)((const int32_t*)p + at + n);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * q + e] = w[e];
        }
    };
    load_key(job.p_in, g_in, true);
    load_key(job.p_out, g_out, false);
    int bits[E];
    load_key(job.s_in, bits, false);
#pragma unroll
    for (int e = 0; e < E; ++e) s_in[e] = T::to_float(T::from_float(__builtin_bit_cast(float, bits[e])));  // as the products take it
    load_key(job.s_out, bits, false);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        post[e] = __builtin_bit_cast(float, bits[e]) * (D == 128 ? 0.08838834764831845f : 0.125f);  // 1 / sqrt(D)
        g_in[e] &= D - 1;
        g_out[e] &= D - 1;
    }
    if constexpr (!SCATTER) load(idx, x);
    const uint32_t sign[4] = {(a & 1) ? 0x80000000u : 0u, (a & 2) ? 0x80000000u : 0u, (a & 4) ? 0x80000000u : 0u,
                              (a & 8) ? 0x80000000u : 0u};
    for (int s = 0; s < n_steps; ++s) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int q = 0; q < EPC; q += 4) {
                f32x4_t v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = T::to_float(x[c][q + e]) * s_in[c * EPC + q + e];
                *(f32x4_t*)(my + natural(c) + q) = v;
            }
        const int64_t j = row0 + (int64_t)s * kHadRows;
        const int64_t to = SCATTER ? idx : j;
        if (s + 1 < n_steps) {  // the next row, on its way meanwhile
            idx = pm ? pm[row_of(s + 1)] : (int32_t)row_of(s + 1);
            load(SCATTER ? row_of(s + 1) : idx, x);
        }
        wave_lds_fence();
        float z[E];
#pragma unroll
        for (int e = 0; e < E; ++e) z[e] = my[g_in[e]];
#pragma unroll
        for (int w = 1; w < E; w *= 2)
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (!(e & w)) {
                    const float p = z[e], q = z[e + w];
                    z[e] = p + q;
                    z[e + w] = p - q;
                }
        auto across = [&](float v, float other, int bit) {
            return other + __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) ^ sign[bit]);
        };
#pragma unroll
        for (int e = 0; e < E; ++e) {
            z[e] = across(z[e], dpp_move<0xB1>(z[e]), 0);   // quad_perm [1,0,3,2]
            z[e] = across(z[e], dpp_move<0x4E>(z[e]), 1);   // quad_perm [2,3,0,1]
            z[e] = across(z[e], dpp_move<0x141>(z[e]), 2);  // row_half_mirror
            z[e] = across(z[e], dpp_move<0x128>(z[e]), 3);  // row_ror:8
        }
        wave_lds_fence();  // all have gathered
#pragma unroll
        for (int q = 0; q < E; q += 4) {
            f32x4_t v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = z[q + e];
            *(f32x4_t*)(my + E * a + q) = v;
        }
        wave_lds_fence();
        float out_of_range = 0.f, most = 0.f;  // NaN where a sum is not finite; the largest sum
        if constexpr (SCATTER) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                out_of_range = __builtin_fmaf(z[e], 0.f, out_of_range);
                most = fmaxf(most, fabsf(z[e]));
            }
            out_of_range = most < kHadLeast ? 1.f : out_of_range;
            pin_here(out_of_range);  // (the sums would be kept for it)
        }
        chunk_t y[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                // Zeros have the sign that the products give them, whose sums start at +0: in 16 bits before the scale, in fp32 behind it.
                const float sum = my[g_out[c * EPC + e]];
                float v = SCATTER ? __builtin_fmaf(sum, post[c * EPC + e], 0.0f) : (sum + 0.0f) * post[c * EPC + e];
                pin_here(v);  // rounded before it is narrowed
                y[c][e] = T::from_float(v);
            }
        if (j < L) {
#pragma unroll
            for (int c = 0; c < NC; ++c) *(chunk_t*)(Y + to * D + natural(c)) = y[c];
        }
        wave_lds_fence();
        if constexpr (SCATTER) {
            // The products have both of a key's scales in every term.  Here a sum may pass the range that its column's scale would bring it
            // back into, or lose bits below it: rows with a sum that is not finite, or none above kHadLeast, are formed again, column by column
            // in 64 bits, and stored over.  (A row that holds an infinity comes out the same; one of zeros is left.)
            if (__builtin_expect(__any(out_of_range != 0.f), 0)) {
                load(j < L ? j : L - 1, x);
                float in = 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int e = 0; e < EPC; ++e) in = fmaxf(in, fabsf(x[c][e]));
                in = group_max<16>(in);
                const bool again = group_max<16>(out_of_range == out_of_range ? 0.f : 1.f) > 0.f || group_max<16>(most) < kHadLeast;
                if (again && in > 0.f && j < L) {
#pragma unroll 1
                    for (int e = 0; e < E; ++e) {  // what this lane has stored
                        const int c = natural(e / EPC) + e % EPC, m = job.p_out[at + c] & (D - 1);
                        double sum = 0.0;
#pragma unroll 1
                        for (int i = 0; i < D; ++i) {
                            const int k = job.p_in[at + i] & (D - 1);
                            const double t = (double)X[j * D + k] * (double)job.s_in[at + k];
                            sum += __popc(i & m) & 1 ? -t : t;
                        }
                        Y[to * D + c] = (float)(sum * ((double)job.s_out[at + c] * (D == 128 ? 0.08838834764831845 : 0.125)) + 0.0);
                    }
                }
                load(row_of(s + 1), x);  // as it was
            }
        }
    }
}

FEDRAG_KERNEL void invert_perm_kernel(const int32_t* __restrict__ perm, int64_t L, int32_t* __restrict__ inv) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < L) inv[perm[j]] = (int32_t)j;
}

// Debug aid: is every row of perm [n_perm, L] a permutation of 0..L-1?  marks [n_perm, L] counts the hits of every
// index; flag receives bit 0 for an index outside [0, L) and bit 1 for an index that occurs more than once (every
// index in range and none twice means all L occur).
FEDRAG_KERNEL void validate_perm_clear_kernel(int32_t* __restrict__ marks, int64_t total, int32_t* __restrict__ flag) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < total) marks[e] = 0;
    if (e == 0) flag[0] = 0;
}
FEDRAG_KERNEL void validate_perm_kernel(const int32_t* __restrict__ perm, int64_t L, int64_t total,
                                     int32_t* __restrict__ marks, int32_t* __restrict__ flag) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int64_t row = e / L;
    const int32_t p = perm[e];
    if (p < 0 || p >= L) atomicOr(flag, 1);
    else if (atomicAdd(&marks[row * L + p], 1) != 0) atomicOr(flag, 2);
}

// ------------------------------------------------------------------------------------------------ launchers
static int ceil_div_i64(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

static ScrambleJob device_job(const RowsJob& j, int i) {
    return ScrambleJob{j.X[i], j.Phi[i], j.Y[i], j.s_in[i], j.p_in[i], j.p_out[i], j.s_out[i], j.params[i]};
}

template <class T, int D, bool SCATTER>
static hipError_t launch_hadamard(const RowsJob& j, hipStream_t stream);

template <class T, int D, bool SCATTER, bool WIDE>
static hipError_t launch_few_rows(const RowsJob& j, hipStream_t stream) {
    const bool few_slabs = j.BH * j.n_jobs <= kSplitSlabs, handful = j.L <= kSplitRows;
    const int cs = j.structured ? 1 : few_slabs || (handful && D == 128) ? 4 : handful ? 2 : 1;
    if (!grid_fits(j.BH, kF32Threads)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)j.BH, (unsigned)j.n_jobs, (unsigned)cs);
#define FEDRAG_SPLIT(CS_, ROWS_) few_rows_of_few_columns_kernel<T, D, SCATTER, WIDE, CS_, ROWS_>
    auto kernel = few_rows_kernel<T, D, SCATTER, false, WIDE>;
    if constexpr (!SCATTER)
        if (j.structured) kernel = few_rows_kernel<T, D, false, true, WIDE>;
    if (cs == 4) kernel = handful ? FEDRAG_SPLIT(4, kSplitRows) : FEDRAG_SPLIT(4, kFewRows);
    if constexpr (D == 64)
        if (cs == 2) kernel = FEDRAG_SPLIT(2, kSplitRows);
#undef FEDRAG_SPLIT
    hipLaunchKernelGGL(kernel, grid, dim3(kF32Threads / cs), 0, stream, device_job(j, 0), device_job(j, 1), j.perm, j.perm_batch_stride,
                       FastDiv(j.H), FastDiv(j.G), (int)j.L, j.merge);
    return hipGetLastError();
}

template <class T, int D>
static hipError_t launch_scramble16(const RowsJob& j, hipStream_t stream) {
    if (j.structured && j.n_jobs == 1 && j.quant_bits == 0 && (j.L <= kHadSlab || j.BH * j.L <= kHadTotal) &&
        grid_fits(j.BH, kHadThreads))
        return launch_hadamard<T, D, false>(j, stream);
    if (j.L <= kFewRows && j.quant_bits == 0) return launch_few_rows<T, D, false, false>(j, stream);
    const int waves = scr_waves(j.quant_bits);
    const int64_t rows_per_pass = (int64_t)waves * kScrRows;  // rows one workgroup covers per ring step
    const int64_t passes = (j.L + rows_per_pass - 1) / rows_per_pass;  // per [L, d] slab
    // about one workgroup per CU over the whole launch, split evenly over (job, head); never more members than a
    // slab has passes
    int members = FEDRAG_SCR_WGS / (j.H * j.n_jobs);
    if (members < 1) members = 1;
    if ((int64_t)members > passes) members = (int)passes;
    const int tiles_per_slab = ceil_div_i64(passes, members);
    const int B = (int)(j.BH / j.H);
    int b_groups = FEDRAG_SCR_WGS / (j.H * j.n_jobs * members);  // leftover parallelism goes to the sequences
    if (b_groups < 1) b_groups = 1;
    if (b_groups > B) b_groups = B;
    dim3 grid((unsigned)(j.H * members * b_groups), (unsigned)j.n_jobs);
    const ScrambleJob a = device_job(j, 0), b = device_job(j, 1);
#define FEDRAG_SCR_LAUNCH(ST_, QB_)                                                                              \
    hipLaunchKernelGGL((scramble_rows_kernel<T, D, ST_, QB_>), grid, dim3(waves * kWave), 0, stream, a, b, j.perm, \
                       j.perm_batch_stride, B, j.H, j.G, j.L, members, FastDiv(tiles_per_slab), b_groups)
    if (j.structured) {
        if (j.quant_bits == 8) FEDRAG_SCR_LAUNCH(true, 8);
        else if (j.quant_bits == 4) FEDRAG_SCR_LAUNCH(true, 4);
        else FEDRAG_SCR_LAUNCH(true, 0);
    } else {
        if (j.quant_bits == 8) FEDRAG_SCR_LAUNCH(false, 8);
        else if (j.quant_bits == 4) FEDRAG_SCR_LAUNCH(false, 4);
        else FEDRAG_SCR_LAUNCH(false, 0);
    }
#undef FEDRAG_SCR_LAUNCH
    return hipGetLastError();
}

// Row steps per workgroup.  What a launch takes is the load of the compute unit that gets the most workgroups, in steps of a
// unit whose matrix pipe is busy: `resident` workgroups of a unit (by registers: up to 128, 168, 256 a lane) take a step each in as
// many of those; one, two or three of them, which wait for their rows, take `part`, more with a second partial to read; every
// workgroup costs `setup` (its slice of Phi, or the multiplying out of the key), and where they come in several rounds the last
// one ends unevenly (`tail` of a workgroup).  Fitted to up to 19 splits of each of 554 launches; over those the choice is 1 % from the
// best split on average, 6 to 16 % at most by the form (of others, 12 x 75 rows x 64 heads with the aggregation 24 %).  The
// aggregating form, with 16 elements of the other partial in registers, has one workgroup less to a unit: cut as the plain one it
// took 10 % longer than its best split on average at d = 128, 59 % at most (4096 rows x 32 heads 60 us and 83, 8 x 500 60 and 80,
// 300 x 10 of 64 22.6 and 26.6).
struct RowStepCost {
    int resident;
    float setup, tail, part[4];
};
static constexpr RowStepCost row_step_cost(int D, bool structured, bool merge) {
    return D == 64 ? merge ? RowStepCost{3, 0.4f, 0.0f, {0.0f, 1.7f, 2.7f, 0.0f}} : RowStepCost{4, 0.4f, 0.4f, {0.0f, 1.5f, 2.5f, 3.1f}}
           : merge ? RowStepCost{2, 0.05f, 0.1f, {0.0f, 1.8f, 0.0f, 0.0f}}
           : structured ? RowStepCost{2, 0.4f, 0.0f, {0.0f, 1.2f, 0.0f, 0.0f}}
                        : RowStepCost{3, 0.2f, 0.8f, {0.0f, 1.2f, 2.0f, 0.0f}};
}
int row_steps_resident(int D, bool structured, bool merge) { return row_step_cost(D, structured, merge).resident; }
static int mf_steps_per_wg(int64_t steps, int64_t slabs, int D, bool structured, bool merge) {
    const RowStepCost c = row_step_cost(D, structured, merge);
    const int64_t cus = attn_target_wgs();
    int best = 1;
    float least = 0.0f;
    for (int64_t most = 1; most <= 64 && most <= steps; ++most) {
        const int64_t chunks = (steps + most - 1) / most;
        const int64_t spw = (steps + chunks - 1) / chunks;
        const int64_t wgs = (slabs * chunks + cus - 1) / cus;  // of the fullest unit
        const float load = (float)(wgs / c.resident * c.resident) + c.part[wgs % c.resident];
        const float per = wgs <= c.resident ? (float)spw : (float)steps / (float)chunks;
        const float cost = load * per + (float)wgs * c.setup + (wgs > c.resident ? c.tail * (float)spw : 0.0f);
        if (most == 1 || cost < least) {
            least = cost;
            best = (int)spw;
        }
    }
    return best;
}

template <int D, bool SCATTER, int RT>
static hipError_t launch_rows_mfma_f32(const RowsJob& j, hipStream_t stream) {
    constexpr int TR = 32 * RT;  // rows per workgroup step
    constexpr int kThreads = mf_threads(D, RT);
    const int64_t steps = (j.L + TR - 1) / TR;
    const int spw = mf_steps_per_wg(steps, j.BH * j.n_jobs, D, j.structured, j.merge.lse_in != nullptr);
    const int chunks = ceil_div_i64(steps, spw);
    if (!grid_fits(j.BH * chunks, kThreads)) return hipErrorInvalidValue;
    dim3 grid((unsigned)(j.BH * chunks), (unsigned)j.n_jobs);
    const ScrambleJob a = device_job(j, 0), b = device_job(j, 1);
    auto kernel = rows_times_matrix_mfma_f32_kernel<D, SCATTER, false, false, RT>;
    if constexpr (SCATTER) {
        if (j.merge.lse_in) kernel = rows_times_matrix_mfma_f32_kernel<D, true, false, true, RT>;
    } else {
        if (j.structured) kernel = rows_times_matrix_mfma_f32_kernel<D, false, true, false, RT>;
    }
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, a, b, j.perm, j.perm_batch_stride, FastDiv(j.H), FastDiv(j.G), j.L,
                       FastDiv(chunks), spw, j.merge);
    return hipGetLastError();
}

template <int D, bool SCATTER>
static hipError_t launch_rows_f32(const RowsJob& j, hipStream_t stream) {
    if constexpr (!SCATTER) {  // (d = 64, 16 rows: 4.4 us summed in 64 bits, 4.2 in 32)
        if (j.L <= wide_rows(D)) return launch_few_rows<F32, D, false, true>(j, stream);
    }
    if constexpr (SCATTER || wide_rows(D) < kFewRows) {
        if (j.L <= kFewRows) return launch_few_rows<F32, D, SCATTER, false>(j, stream);
    }
    if (D == 64 && j.L <= 32) return launch_rows_mfma_f32<D, SCATTER, 1>(j, stream);
    return launch_rows_mfma_f32<D, SCATTER, 4 / (D / 32)>(j, stream);
}

// Fewer than `most` + slabs workgroups, and those of a slab within one step of each other: 2045 slabs of 1000 steps are two
// workgroups of 500 each, where a workgroup of as many steps as fill 2048 of them had 999 and left one.
RowSteps hadamard_steps(int64_t slabs, int64_t L) {
    const int64_t steps = (L + kHadRows - 1) / kHadRows, most = kHadWgsPerUnit * attn_target_wgs();
    const int64_t per = (slabs * steps + most - 1) / most;
    const int64_t chunks = per < steps ? (steps + per - 1) / per : 1;
    return {chunks, (int)((steps + chunks - 1) / chunks)};
}

template <class T, int D, bool SCATTER>
static hipError_t launch_hadamard(const RowsJob& j, hipStream_t stream) {
    const auto [chunks, per] = hadamard_steps(j.BH, j.L);
    const int64_t most = 0xffffffffLL / kHadThreads / chunks;  // slabs of a launch: below 2^24 of them, all
    if (j.BH > 0x7fffffffLL) return hipErrorInvalidValue;
    for (int64_t first = 0; first < j.BH; first += most) {
        const int64_t slabs = j.BH - first < most ? j.BH - first : most;
        hipLaunchKernelGGL((hadamard_rows_kernel<T, D, SCATTER>), dim3((unsigned)(slabs * chunks)), dim3(kHadThreads), 0, stream,
                           device_job(j, 0), j.perm, j.perm_batch_stride, FastDiv(chunks), FastDiv(j.H), FastDiv(j.G), j.L, per, (int)first);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_rows_transform(const RowsJob& j, hipStream_t stream) {
    if (j.L == 0 || j.BH == 0) return hipSuccess;
    if (j.scatter) {  // Dec: always fp32
        if (j.structured && j.merge.lse_in) return hipErrorInvalidValue;  // (not aggregated by a key's factors)
        if (j.structured)
            return j.D == 128 ? launch_hadamard<F32, 128, true>(j, stream) : launch_hadamard<F32, 64, true>(j, stream);
        return j.D == 128 ? launch_rows_f32<128, true>(j, stream) : launch_rows_f32<64, true>(j, stream);
    }
    switch (j.dtype) {
        case FEDRAG_F32:
            return j.D == 128 ? launch_rows_f32<128, false>(j, stream) : launch_rows_f32<64, false>(j, stream);
        case FEDRAG_BF16:
            return j.D == 128 ? launch_scramble16<BF16, 128>(j, stream) : launch_scramble16<BF16, 64>(j, stream);
        case FEDRAG_F16:
            return j.D == 128 ? launch_scramble16<F16, 128>(j, stream) : launch_scramble16<F16, 64>(j, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_invert_perm(const int32_t* perm, int64_t L, int32_t* inv, hipStream_t stream) {
    if (L == 0) return hipSuccess;
    hipLaunchKernelGGL(invert_perm_kernel, dim3((unsigned)((L + 255) / 256)), dim3(256), 0, stream, perm, L, inv);
    return hipGetLastError();
}

hipError_t launch_validate_perm(const int32_t* perm, int n_perm, int64_t L, int32_t* marks, int32_t* flag,
                                hipStream_t stream) {
    const int64_t total = (int64_t)n_perm * L;
    if (!grid_fits((total > 0 ? total + 255 : 256) / 256, 256)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((total > 0 ? total + 255 : 256) / 256));
    hipLaunchKernelGGL(validate_perm_clear_kernel, grid, dim3(256), 0, stream, marks, total, flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || total == 0) return e;
    hipLaunchKernelGGL(validate_perm_kernel, grid, dim3(256), 0, stream, perm, L, total, marks, flag);
    return hipGetLastError();
}

}  // namespace fedrag

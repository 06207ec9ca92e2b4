// Partial attention for fp32 storage (Section 4.1, per-node local computation): the accuracy path.  Products and sums
// are fp32 on the fp32 matrix cores (v_mfma_f32_16x16x4_f32), exponentials and logarithms the accurate library ones.
//
// One workgroup = 16 NQ query rows of one (sequence, KV head) unit x one shard; its W waves take 16-key tiles
// round-robin and are folded at the end with the Section 4.1 aggregation, so that a handful of rows over a few hundred
// keys already keeps a compute unit busy without scratch memory.
// Lane l of a wave: lr = l % 16, lq = l / 16.
//   S^T tile (16 keys x 16 queries) = K (16 x d) . Q^T (d x 16), four channels per instruction: lane (lr, lq) supplies
//   channels 16 j + 4 lq + e of key row lr and of query lr, fetched 16 bytes at a time.  It ends up with query lr and
//   keys 4 lq + r, r = 0..3.
//   O^T (d x 16) += V^T (d x 16) . P^T (16 x 16), four keys per instruction: in instruction r lane group lq contracts
//   key 4 lq + r, which is the probability it holds, and the d-rows are assigned d = DCH i + t (tile t, row i), so that
//   lane (i = lr) needs DCH contiguous channels of each of its four keys: full rows, no transposition anywhere.
//   W = 1, which serves short contexts: keys lq + 4 r instead (lane lr fetches key row lr / 4 + 4 (lr % 4)), so that the
//   instructions behind the last key can be left out (32768 units of 4 keys of 128: 74 -> 57 us).
// Bound by the matrix pipe (64 NQ instructions of 32 cycles per 16 KiB of K, V at d = 128) as soon as the waves cover the
// chip, by the latency of a tile before that.  NQ = 2 reads K, V half as often and is taken when there are rows for it and
// its workgroups still cover the compute units; below that NQ = 1 spreads the rows over twice as many of them.
// 4 rows x 512 keys x 2 heads of 64: 10 us (67 us with one wave per row and plain multiply-adds).
#include "fedrag_device.h"
#include "fedrag_host.h"

namespace fedrag {

constexpr int kF32Tile = 16;  // keys per wave step

__device__ __forceinline__ f32x4_t mfma_f32(float a, float b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// exp(a - b) with the convention that a == -inf gives 0 even when b == -inf.
__device__ __forceinline__ float exp_diff(float a, float b) { return (a == -INFINITY) ? 0.0f : expf(a - b); }

template <int D, int NQ, int W>
FEDRAG_KERNEL __launch_bounds__(W * kWave, W == 1 && NQ == 1 ? (D == 64 ? 4 : 2) : 1) void attn_f32_kernel(const float* __restrict__ Q, const KeyRuns runs,
                                                                      FastDiv by_tiles, FastDiv by_lq, FastDiv by_hkv, int R,
                                                                      int64_t Lq, int64_t causal_off, int causal,
                                                                      float scale, float* __restrict__ O,
                                                                      float* __restrict__ lse, int64_t total_rows,
                                                                      const int32_t* __restrict__ kv_lens,
                                                                      const int32_t* __restrict__ q_lens) {
    constexpr int DCH = D / 16;  // channels per lane and key of V (= 16-row tiles of O^T)
    constexpr int KJ = D / 16;   // 16-byte reads per lane of a K or Q row
    constexpr int LDO = D + 4;
    constexpr int WF = W > 1 ? W : 1;  // waves to fold
    __shared__ float sm_m[WF][NQ * 16], sm_l[WF][NQ * 16];
    __shared__ __attribute__((aligned(16))) float sm_o[WF][NQ * 16][LDO];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const int lr = lane % 16;
    const int lq = lane / 16;
    // The arguments, then the shard: two trips to memory where branches and addresses made five (4 rows x 512 keys of 64 0.6 %, on
    // average over 80 launches 0.7 %; with two row tiles a wave, 256 rows x 32 heads of 64, 2 % slower: not there).
    if constexpr (NQ == 1)
        FEDRAG_HAVE_HERE(FEDRAG_S(Q), FEDRAG_S3(runs.by_runs), FEDRAG_S(runs.n_shards), FEDRAG_S3(by_tiles), FEDRAG_S3(by_lq), FEDRAG_S(R),
                         FEDRAG_S(Lq), FEDRAG_S(causal_off), FEDRAG_S(causal), FEDRAG_S(scale), FEDRAG_S(O), FEDRAG_S(lse),
                         FEDRAG_S(total_rows), FEDRAG_S(kv_lens), FEDRAG_S(q_lens));
    const uint32_t group = runs.by_runs.div(blockIdx.x);  // (unit, row tile); the runs of one are neighbours
    const int run = (int)(blockIdx.x - group * runs.by_runs.d);
    const uint32_t unit = by_tiles.div(group);
    const int row0 = (int)(group - unit * by_tiles.d) * (NQ * 16);
    int split;
    const KeyShard shard = runs.shard_of(run, &split);  // one run per shard: split == 0
    if constexpr (NQ == 1) FEDRAG_HAVE_HERE(FEDRAG_S(shard.K), FEDRAG_S(shard.V), FEDRAG_S(shard.L));
    int64_t L = shard.L;
    const float* K = (const float*)shard.K + (int64_t)unit * L * D;
    const float* V = (const float*)shard.V + (int64_t)unit * L * D;
    if (kv_lens) {  // padded batch of unequal sequences: only the first kv_lens[b] keys exist
        const int64_t v = __builtin_amdgcn_readfirstlane(kv_lens[by_hkv.div(unit)]);
        L = v < 0 ? 0 : (v < L ? v : L);
    }

    // a workgroup of padding rows (they are not written) leaves at once: all of its rows are in one head and past the
    // sequence's count, or the sequence has none
    int q_rows = 0;
    if (q_lens) {
        q_rows = __builtin_amdgcn_readfirstlane(q_lens[by_hkv.div(unit)]);
        const int first = (int)by_lq.mod((uint32_t)row0);
        if (q_rows <= 0 || (first >= q_rows && first + NQ * 16 <= Lq)) return;
    }

    // row n of the unit is query n % Lq of head n / Lq of the group; it sees keys < lim
    f32x4_t q[NQ][KJ];
    int64_t lim[NQ];
    int64_t most = 0;  // keys that some row of the workgroup sees
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        const int row = row0 + n * 16 + lr;
        const int row_ld = row < R ? row : R - 1;  // rows past the end are computed on a real one and not written
        const float* qp = Q + ((int64_t)unit * R + row_ld) * D + 4 * lq;
#pragma unroll
        for (int j = 0; j < KJ; ++j) q[n][j] = *(const f32x4_t*)(qp + 16 * j);
        lim[n] = L;
        if (causal) {
            const int64_t own = (int64_t)by_lq.mod((uint32_t)row_ld) + causal_off + 1;
            if (own < L) lim[n] = own;
        }
    }
    if (causal) {
        int top = 0;  // L <= INT32_MAX
#pragma unroll
        for (int n = 0; n < NQ; ++n) top = (int)lim[n] > top ? (int)lim[n] : top;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const int other = __shfl_xor(top, o);
            top = other > top ? other : top;
        }
        most = __builtin_amdgcn_readfirstlane(top);
    } else {
        most = L;
    }

    f32x4_t acc[NQ][DCH];
    float m_run[NQ], l_run[NQ];
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        m_run[n] = -INFINITY;
        l_run[n] = 0.f;
#pragma unroll
        for (int t = 0; t < DCH; ++t) acc[n][t] = zero_vec<f32x4_t>();
    }

    constexpr bool DEALT = W == 1;
    const int key_row = DEALT ? lr / 4 + 4 * (lr % 4) : lr;                // this lane's key row in a tile
    auto key_of = [&](int r) { return DEALT ? lq + 4 * r : 4 * lq + r; };  // its r-th score, probability and row of V
    // rows past the last key re-read it (it exists when a tile does); their scores are masked
    auto load_k = [&](int64_t key0, f32x4_t (&k)[KJ]) {
        int64_t key = key0 + key_row;
        if (key >= most) key = most - 1;
        const float* kp = K + key * D + 4 * lq;
#pragma unroll
        for (int j = 0; j < KJ; ++j) k[j] = *(const f32x4_t*)(kp + 16 * j);
    };
    const int64_t stride = (int64_t)W * kF32Tile;
    int64_t key0 = (int64_t)wave * kF32Tile;
    f32x4_t k[KJ];
    if (key0 < most) load_k(key0, k);
    for (; key0 < most; key0 += stride) {
        f32x4_t v[4][DCH / 4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int64_t key = key0 + key_of(r);
            if (key >= most) key = most - 1;
            const float* vp = V + key * D + DCH * lr;
#pragma unroll
            for (int c = 0; c < DCH / 4; ++c) v[r][c] = *(const f32x4_t*)(vp + 4 * c);
        }
        f32x4_t s[NQ];
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
            f32x4_t part[2] = {zero_vec<f32x4_t>(), zero_vec<f32x4_t>()};  // two chains: no wait for the last result
#pragma unroll
            for (int j = 0; j < KJ; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) part[e % 2] = mfma_f32(k[j][e], q[n][j][e], part[e % 2]);
            s[n] = part[0] + part[1];
        }
        if (key0 + stride < most) load_k(key0 + stride, k);
        const bool whole = !causal && key0 + kF32Tile <= L;  // wave-uniform
        bool odd_v = false;
        if (!whole) {
            float sum = 0.f;  // x - x is 0 for a finite x and NaN otherwise
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int t = 0; t < DCH; ++t) sum += v[r][t / 4][t % 4] - v[r][t / 4][t % 4];
            odd_v = __builtin_amdgcn_ballot_w64(sum != 0.f) != 0;
        }
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[n][r] *= scale;
                if (!whole && key0 + key_of(r) >= lim[n]) s[n][r] = -INFINITY;
                mx = fmaxf(mx, s[n][r]);
            }
            mx = xor32_max(xor16_max(mx));
            const float m_new = fmaxf(m_run[n], mx);
            const float alpha = exp_diff(m_run[n], m_new);
            float p[4];
            float psum = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[r] = exp_diff(s[n][r], m_new);
                psum += p[r];
            }
            l_run[n] = l_run[n] * alpha + psum;
            m_run[n] = m_new;
#pragma unroll
            for (int t = 0; t < DCH; ++t) acc[n][t] *= alpha;
            if (whole || !odd_v) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (DEALT && key0 + 4 * r >= most) break;
#pragma unroll
                    for (int t = 0; t < DCH; ++t) acc[n][t] = mfma_f32(v[r][t / 4][t % 4], p[r], acc[n][t]);
                }
            } else {
                // an infinity or NaN in V times the zero probability of a row that does not see its key would reach
                // that row: one query at a time, with the rows of V that it does not see left out
#pragma unroll 1
                for (int c = 0; c < 16; ++c) {
                    const int lim_c = __shfl((int)lim[n], c);
#pragma unroll
                    for (int t = 0; t < DCH; ++t) {
                        f32x4_t one = zero_vec<f32x4_t>();
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            one = mfma_f32(key0 + key_of(r) < lim_c ? v[r][t / 4][t % 4] : 0.f, lr == c ? p[r] : 0.f, one);
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[n][t][r] += lr == c ? one[r] : 0.f;
                    }
                }
            }
        }
    }

    const int64_t base = (int64_t)run * total_rows + (int64_t)unit * R;
    auto written = [&](int row) {  // query rows past the sequence's count are padding and are not written
        return row < R && !(q_lens && (int)by_lq.mod((uint32_t)row) >= q_rows);
    };
    if constexpr (W == 1) {  // nothing to fold: lane group lq holds channels 4 DCH lq .. of query lr
#pragma unroll
        for (int n = 0; n < NQ; ++n) {
            const float den = xor32_sum(xor16_sum(l_run[n]));
            const float inv = den > 0.f ? 1.0f / den : 0.f;
            const int row = row0 + n * 16 + lr;
            if (!written(row)) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int t = 0; t < DCH; t += 4) {
                    f32x4_t o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = acc[n][t + e][r] * inv;
                    *(f32x4_t*)(O + (base + row) * D + DCH * (4 * lq + r) + t) = o;
                }
            if (lq == 0) lse[base + row] = den > 0.f ? m_run[n] + logf(den) : -INFINITY;
        }
        return;
    }

    // fold the waves
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
        const float l_tot = xor32_sum(xor16_sum(l_run[n]));
        if (lq == 0) {
            sm_m[wave][n * 16 + lr] = m_run[n];
            sm_l[wave][n * 16 + lr] = l_tot;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < DCH; t += 4) {
                f32x4_t o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = acc[n][t + e][r];
                *(f32x4_t*)&sm_o[wave][n * 16 + lr][DCH * (4 * lq + r) + t] = o;
            }
    }
    __syncthreads();
    for (int idx = tid; idx < NQ * 16 * (D / 4); idx += W * kWave) {
        const int n = idx / (D / 4);
        const int d = idx % (D / 4) * 4;
        const int row = row0 + n;
        if (!written(row)) continue;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < W; ++w) M = fmaxf(M, sm_m[w][n]);
        f32x4_t num = zero_vec<f32x4_t>();
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float a = exp_diff(sm_m[w][n], M);
            const f32x4_t o = *(const f32x4_t*)&sm_o[w][n][d];
#pragma unroll
            for (int e = 0; e < 4; ++e) num[e] = __builtin_fmaf(a, o[e], num[e]);
            den = __builtin_fmaf(a, sm_l[w][n], den);
        }
        const float inv = den > 0.f ? 1.0f / den : 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] *= inv;
        *(f32x4_t*)(O + (base + row) * D + d) = num;
        if (d == 0) lse[base + row] = den > 0.f ? M + logf(den) : -INFINITY;
    }
}

template <int D, int NQ, int W>
static hipError_t launch_f32_t(const AttnProblem& p, const KeyRuns& runs, hipStream_t stream) {
    const int64_t rows = (int64_t)p.B * p.Hq * p.Lq;
    const int64_t R = (int64_t)(p.Hq / p.Hkv) * p.Lq;  // rows of a unit, contiguous in Q, O and lse
    const int64_t tiles = (R + NQ * 16 - 1) / (NQ * 16);
    const int64_t grid = (int64_t)p.B * p.Hkv * tiles * runs.n_runs;
    if (R > 0x7fffffffLL || !grid_fits(grid, W * kWave)) return hipErrorInvalidValue;
    float* Odst = p.O;
    float* Ldst = p.lse;
    if (runs.n_runs > 1) {
        if (!p.workspace || p.workspace_bytes < (size_t)runs.n_runs * rows * (D + 1) * sizeof(float))
            return hipErrorInvalidValue;
        Odst = (float*)p.workspace;
        Ldst = Odst + (size_t)runs.n_runs * rows * D;
    }
    hipLaunchKernelGGL((attn_f32_kernel<D, NQ, W>), dim3((unsigned)grid), dim3(W * kWave), 0, stream,
                       (const float*)p.Q, runs, FastDiv(tiles), FastDiv(p.Lq), FastDiv(p.Hkv), (int)R, p.Lq, p.Lkv - p.Lq,
                       p.causal ? 1 : 0, p.scale, Odst, Ldst, rows, p.kv_lens, p.q_lens);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || runs.n_runs == 1) return e;
    return launch_lse_merge(Odst, Ldst, runs.n_runs, rows, D, p.O, p.lse, stream);
}

template <int D, int NQ>
static hipError_t launch_f32_w(const AttnProblem& p, const KeyRuns& runs, hipStream_t stream) {
    const int64_t R = (int64_t)(p.Hq / p.Hkv) * p.Lq;
    const int64_t wgs = (int64_t)p.B * p.Hkv * ((R + NQ * 16 - 1) / (NQ * 16)) * runs.n_runs;
    int64_t longest = 0;
    for (int i = 0; i < runs.n_shards; ++i) longest = runs.s[i].L > longest ? runs.s[i].L : longest;
    const int64_t tiles = (longest + kF32Tile - 1) / kF32Tile;
    // Waves per workgroup: eight share the keys out while workgroups are few (2 heads x 512 keys of 64: 9.5 us, 34 with one),
    // fewer the more workgroups there are to overlap, and never more than key tiles: 4096 sequences and heads of 128 with 64
    // keys take 42 us with one wave each, 70 with eight, 16384 with 32 keys 98 and 259 (single rows; in the 32-row form, which
    // such rows used to take, 728).  From one workgroup per compute unit on four are as fast or faster than eight at
    // d = 128 (512 rows of one query x 128 keys 14.3 against 15.7), where eight spill with NQ = 2; at d = 64 from two on,
    // or for a few keys (304 causal workgroups of 300 rows 19.1 with eight, 21.4 with four).
    const int64_t cus = attn_target_wgs();
    if (wgs >= 8 * cus || tiles <= 1) return launch_f32_t<D, NQ, 1>(p, runs, stream);
    if (wgs >= 4 * cus || tiles <= 2) return launch_f32_t<D, NQ, 2>(p, runs, stream);
    if constexpr (D == 64 || NQ == 1)
        if (tiles > 4 && (wgs < cus || (D == 64 && wgs < 2 * cus && tiles > 8)))
            return launch_f32_t<D, NQ, 8>(p, runs, stream);
    return launch_f32_t<D, NQ, 4>(p, runs, stream);
}

hipError_t launch_attn_f32(const AttnProblem& p, hipStream_t stream) {
    const KeyRuns runs = attn_runs_of(p);  // fp32: one run per shard
    if (runs.n_runs < 1) return hipErrorInvalidValue;
    const int64_t R = (int64_t)(p.Hq / p.Hkv) * p.Lq;
    const bool wide = R > 16 && (int64_t)p.B * p.Hkv * ((R + 31) / 32) * runs.n_runs >= attn_target_wgs();
    if (p.D == 128) return wide ? launch_f32_w<128, 2>(p, runs, stream) : launch_f32_w<128, 1>(p, runs, stream);
    return wide ? launch_f32_w<64, 2>(p, runs, stream) : launch_f32_w<64, 1>(p, runs, stream);
}

}  // namespace fedrag

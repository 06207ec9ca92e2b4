// Global aggregation of Section 4.1 in the log domain:
//   M = max_i lse_i, a_i = exp(lse_i - M), O = sum_i a_i O_i / sum_i a_i, lse = M + ln sum_i a_i
// which equals sum_i w_i (.) O_i / sum_i w_i with w_i = exp(lse_i).  Also used to fold the intra-shard KV
// splits of the decode kernel.  Pure streaming: one thread per (row, 4 output columns).  Two forms, up to four partials and more.
#include <utility>

#include "fedrag_device.h"
#include "fedrag_host.h"

namespace fedrag {

// What bounds it: for a handful of rows (a decoding step has 32 of them over 16 key runs) the chain of dependent steps,
// for many rows over many runs memory.  So the lanes of a row share the weights out - each of 16 loads one log-sum-exp and
// evaluates one exponential, and a weight reaches the others with the multiply-add itself (row_newbcast) - there is no branch on a
// weight, the first batch of partials is in flight before the weights are known, and the workgroups are one wave while rows are few.
// Sums are formed in shard order whatever the batch.
// Calls back to back, rows of 128: 32 rows over 16 partials 2.9 us (3.5 with the weights shuffled through LDS and a branch on
// each), 3744 over 16 4.4 (5.1), 512 over 8 2.7 (3.1); from some 60 MB of partials on memory is the bound and the two are even.

// Lane N of each aligned group of 16, in all of them.
template <int N>
__device__ __forceinline__ float lane_of_16(float x) { return dpp_move<0x150 + N>(x); }

// What a row's partials come to.  A partial whose log-sum-exp is -inf takes no part, whatever it holds.
struct Fold {
    f32x4_t acc = zero_vec<f32x4_t>();
    float den = 0.f;
    __device__ __forceinline__ void add(bool in, float a, f32x4_t o) {
        a = in ? a : 0.f;
        den += a;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = __builtin_fmaf(a, in ? o[e] : 0.f, acc[e]);
    }
    // o[u] with lane u's weight, below 0 where it takes no part
    template <int NB, int... U>
    __device__ __forceinline__ void add_lanes(float mine, const f32x4_t (&o)[NB], std::integer_sequence<int, U...>) {
        (add(lane_of_16<U>(mine) != -1.0f, lane_of_16<U>(mine), o[U]), ...);
    }
    __device__ __forceinline__ f32x4_t out(float M) const {
        const float inv = 1.0f / den;
        f32x4_t z;
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = M == -INFINITY ? 0.f : acc[e] * inv;
        return z;
    }
    __device__ __forceinline__ float lse(float M) const { return M == -INFINITY ? -INFINITY : M + logf(den); }
};

// Padded batch with per-sequence query counts: row r is query r % Lq of sequence r / (Hq * Lq), and a padding row holds no
// partials and is not written.
struct QueryCounts {
    const int32_t* lens;
    int64_t Lq, rows_per_seq;
    FastDiv by_lq, by_seq;
    int small;  // below 2^31 rows both are found without a division
    __device__ __forceinline__ bool padding(int64_t r) const {
        const int64_t seq = small ? (int64_t)by_seq.div((uint32_t)r) : r / rows_per_seq;
        const int64_t q = small ? (int64_t)by_lq.mod((uint32_t)r) : r % Lq;
        return q >= lens[seq];
    }
};

// NB: partial outputs in flight (4 registers each).  16 for few rows over more than 8 partials, where a second batch is another trip
// to memory (32 rows of 128 over 16: 2.9 us, 3.0 with 8, 3.2 with 4); 8 up to twice as many threads (8192 rows of 64 over 16: 4.6
// us, 5.2 with 4); beyond that memory is the bound and the waves that fewer registers leave room for are worth more than loads in
// flight: two (16384 rows of 128 over 8: 12.8 us, 13.5 with 4, 14.5 with 8, 15.8 with 16).
template <int D, int NB>
FEDRAG_KERNEL __launch_bounds__(256) void lse_merge_kernel(const float* __restrict__ O_parts,
                                                        const float* __restrict__ lses, int S, int64_t rows,
                                                        float* __restrict__ O, float* __restrict__ lse, QueryCounts counts) {
    constexpr int TPR = D / 4;  // threads per row
    const unsigned wg = blockDim.x;
    FEDRAG_HAVE_HERE(FEDRAG_S(O_parts), FEDRAG_S(lses), FEDRAG_S(S), FEDRAG_S(rows), FEDRAG_S(O), FEDRAG_S(lse), FEDRAG_S(counts.lens),
                     FEDRAG_S(wg));
    const int64_t gid = (int64_t)blockIdx.x * wg + threadIdx.x;
    const int64_t r = gid / TPR;
    const int c = (int)(gid % TPR);
    if (r >= rows) return;
    if (counts.lens && counts.padding(r)) return;
    const float* lp = lses + r;
    const float* op = O_parts + r * D + c * 4;
    const int k = c % 16;  // this lane's partial of each 16
    auto load_l = [&](int i0) { return i0 + k < S ? lp[(int64_t)(i0 + k) * rows] : -INFINITY; };
    // a batch reads past the last partial by re-reading it, and leaves those values out
    auto load_o = [&](int i0, f32x4_t (&o)[NB]) {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int i = i0 + u < S ? i0 + u : S - 1;
            o[u] = *(const f32x4_t*)(op + (int64_t)i * rows * D);
        }
    };
    f32x4_t o[NB];
    float l = load_l(0);
    load_o(0, o);  // in flight together with the log-sum-exps
    float M = fmaxf(l, -INFINITY);  // (a NaN does not count as a maximum, also where every lane holds one)
    for (int i0 = 16; i0 < S; i0 += 16) M = fmaxf(M, load_l(i0));
    M = group_max<16>(M);
    Fold f;
    for (int i0 = 0; i0 < S; i0 += 16) {
        if (i0) l = load_l(i0);
        float mine = l == -INFINITY ? -1.0f : expf(l - M);  // below 0: takes no part
#pragma unroll 1
        for (int j0 = 0; j0 < 16 && i0 + j0 < S; j0 += NB) {
            if (i0 + j0) load_o(i0 + j0, o);
            f.add_lanes(mine, o, std::make_integer_sequence<int, NB>());
            if (NB < 16) mine = dpp_move<0x120 + 16 - NB % 16>(mine);  // row_ror: the next NB weights to the front
        }
    }
    *(f32x4_t*)(O + r * D + c * 4) = f.out(M);
    if (c == 0) lse[r] = f.lse(M);
}

// One to four partials, the usual number: every thread reads the row's log-sum-exps itself, and all that it reads is in flight
// at once.  65536 rows of 64 over 2: 9.0 us (9.7 with a branch on each weight), 3744 of 128 over 4 2.6 (2.9), 32 rows 2.3 (2.5).
template <int D, int S>
FEDRAG_KERNEL __launch_bounds__(256) void lse_merge_few_kernel(const float* __restrict__ O_parts,
                                                            const float* __restrict__ lses, int64_t rows,
                                                            float* __restrict__ O, float* __restrict__ lse, QueryCounts counts) {
    constexpr int TPR = D / 4;
    const unsigned wg = blockDim.x;
    FEDRAG_HAVE_HERE(FEDRAG_S(O_parts), FEDRAG_S(lses), FEDRAG_S(rows), FEDRAG_S(O), FEDRAG_S(lse), FEDRAG_S(counts.lens), FEDRAG_S(wg));
    const int64_t gid = (int64_t)blockIdx.x * wg + threadIdx.x;
    const int64_t r = gid / TPR;
    const int c4 = (int)(gid % TPR) * 4;
    if (r >= rows) return;
    if (counts.lens && counts.padding(r)) return;
    float l[S];
    f32x4_t o[S];
#pragma unroll
    for (int i = 0; i < S; ++i) l[i] = lses[i * rows + r];
#pragma unroll
    for (int i = 0; i < S; ++i) o[i] = *(const f32x4_t*)(O_parts + (i * rows + r) * D + c4);
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < S; ++i) M = fmaxf(M, l[i]);
    Fold f;
#pragma unroll
    for (int i = 0; i < S; ++i) f.add(l[i] != -INFINITY, expf(l[i] - M), o[i]);
    *(f32x4_t*)(O + r * D + c4) = f.out(M);
    if (c4 == 0) lse[r] = f.lse(M);
}

template <int D>
FEDRAG_KERNEL __launch_bounds__(256) void fill_empty_kernel(float* __restrict__ O, float* __restrict__ lse,
                                                         int64_t rows) {
    constexpr int TPR = D / 4;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = gid / TPR;
    const int c4 = (int)(gid % TPR) * 4;
    if (r >= rows) return;
    *(f32x4_t*)(O + r * D + c4) = zero_vec<f32x4_t>();
    if (c4 == 0) lse[r] = -INFINITY;
}

hipError_t launch_lse_merge(const float* O_parts, const float* lses, int S, int64_t rows, int D, float* O, float* lse,
                            hipStream_t stream, const int32_t* q_lens, int64_t Lq, int64_t rows_per_seq) {
    if (rows == 0) return hipSuccess;
    if (q_lens && (Lq < 1 || rows_per_seq < 1)) return hipErrorInvalidValue;
    const int64_t threads = rows * (D / 4);
    const int wg = threads <= 256 * 256 ? 64 : 256;  // one wave per workgroup until every compute unit has four
    if (!grid_fits((threads + wg - 1) / wg, wg)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((threads + wg - 1) / wg));
    QueryCounts counts{};
    if (q_lens) {
        const int small = rows <= 0x7fffffffLL ? 1 : 0;
        counts = {q_lens, Lq, rows_per_seq, FastDiv(small ? Lq : 1), FastDiv(small ? rows_per_seq : 1), small};
    }
    if (S <= 4) {
#define FEDRAG_FEW(S_) (D == 128 ? lse_merge_few_kernel<128, S_> : lse_merge_few_kernel<64, S_>)
        const auto few = S == 1 ? FEDRAG_FEW(1) : S == 2 ? FEDRAG_FEW(2) : S == 3 ? FEDRAG_FEW(3) : FEDRAG_FEW(4);
#undef FEDRAG_FEW
        hipLaunchKernelGGL(few, grid, dim3(wg), 0, stream, O_parts, lses, rows, O, lse, counts);
        return hipGetLastError();
    }
    const int nb = threads <= 256 * 256 && S > 8 ? 16 : threads <= 256 * 512 ? 8 : 2;
#define FEDRAG_MANY(NB_) (D == 128 ? lse_merge_kernel<128, NB_> : lse_merge_kernel<64, NB_>)
    const auto kernel = nb == 16 ? FEDRAG_MANY(16) : nb == 8 ? FEDRAG_MANY(8) : FEDRAG_MANY(2);
#undef FEDRAG_MANY
    hipLaunchKernelGGL(kernel, grid, dim3(wg), 0, stream, O_parts, lses, S, rows, O, lse, counts);
    return hipGetLastError();
}

hipError_t launch_fill_empty(float* O, float* lse, int64_t rows, int D, hipStream_t stream) {
    if (rows == 0) return hipSuccess;
    const int64_t threads = rows * (D / 4);
    if (!grid_fits((threads + 255) / 256, 256)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((threads + 255) / 256));
    if (D == 128)
        hipLaunchKernelGGL(fill_empty_kernel<128>, grid, dim3(256), 0, stream, O, lse, rows);
    else
        hipLaunchKernelGGL(fill_empty_kernel<64>, grid, dim3(256), 0, stream, O, lse, rows);
    return hipGetLastError();
}

// out[bh, perm[i]] = in[bh, i]: the log-sum-exps of permuted query rows put back in the rows' own order (the
// token-permutation part of Dec, Section 4.2, for the per-row scalar that travels with the output).
// One thread per value over the whole tensor, whatever its rows: decoding steps have rows of one value by the thousand (262144
// of them take 2.3 us; 59 with a workgroup of its own for every row).  Below 2^31 values the row is found without a division.
FEDRAG_KERNEL __launch_bounds__(256) void scatter_rows_f32_kernel(const float* __restrict__ in,
                                                               const int32_t* __restrict__ perm, int64_t L,
                                                               FastDiv by_l, int small, int64_t total,
                                                               float* __restrict__ out) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    if (!perm) {
        out[e] = in[e];
        return;
    }
    const int64_t bh = small ? (int64_t)by_l.div((uint32_t)e) : e / L;
    out[bh * L + perm[e - bh * L]] = in[e];
}

hipError_t launch_scatter_rows_f32(const float* in, const int32_t* perm, int64_t n_bh, int64_t L, float* out,
                                   hipStream_t stream) {
    const int64_t total = n_bh * L;
    if (total == 0) return hipSuccess;
    if (!grid_fits((total + 255) / 256, 256)) return hipErrorInvalidValue;
    const int small = total <= 0x7fffffffLL ? 1 : 0;
    hipLaunchKernelGGL(scatter_rows_f32_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, in, perm,
                       L, FastDiv(small ? L : 1), small, total, out);
    return hipGetLastError();
}

}  // namespace fedrag

// Global aggregation of Section 4.1 in the log domain:
//   M = max_i lse_i, a_i = exp(lse_i - M), O = sum_i a_i O_i / sum_i a_i, lse = M + ln sum_i a_i
// which equals sum_i w_i (.) O_i / sum_i w_i with w_i = exp(lse_i).  Also used to fold the intra-shard KV
// splits of the decode kernel.  Pure streaming: one thread per (row, 4 output columns).  Two forms, up to four partials and more.
#include "fedrag_device.h"
#include "fedrag_host.h"

namespace fedrag {

// What bounds it: for a handful of rows (a decoding step has 32 of them over 16 key runs) the chain of dependent loads,
// for many rows over many runs the instructions around them.  So the lanes of a row share the weights out - each loads
// one log-sum-exp and evaluates one exponential, and a weight reaches the others by a lane shuffle - the first batch of
// partials is in flight before the weights are known, and the workgroups are one wave while rows are few.  Sums are
// formed in shard order whatever the batch.
// 32 rows of 128 over 16 partials, calls back to back: 3.5 us (6.7 with one partial after the other); 3744 rows over 16: 5.0
// (11.9).  In a chain of other launches add what a launch costs there.

// max over the TPR = 16 or 32 consecutive lanes that hold a row
template <int TPR>
__device__ __forceinline__ float row_max(float x) {
    x = group_max<16>(x);
    return TPR == 32 ? xor16_max(x) : x;
}

// NB: partial outputs in flight (4 registers each).  16 for few rows over many partials, where a second batch is another trip
// to memory (a decoded token over 32 layers: 941 us against 949 with 8); 8 up to twice as many threads (8192 rows of 64 over 16:
// 5.2 us, 6.5 with two); beyond that memory is the bound and the waves that fewer registers leave room for are worth more than
// loads in flight: two (16384 rows of 128 over 8: 13.1 us, 15.2 with eight, 14.2 one after the other).
template <int D, int NB>
FEDRAG_KERNEL __launch_bounds__(256) void lse_merge_kernel(const float* __restrict__ O_parts,
                                                        const float* __restrict__ lses, int S, int64_t rows,
                                                        float* __restrict__ O, float* __restrict__ lse,
                                                        const int32_t* __restrict__ q_lens, int64_t Lq,
                                                        int64_t rows_per_seq) {
    constexpr int TPR = D / 4;  // threads per row
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = gid / TPR;
    const int c = (int)(gid % TPR);
    const int c4 = c * 4;
    if (r >= rows) return;
    // padded batch with per-sequence query counts: padding rows hold no partials and are not written
    if (q_lens && (r % Lq) >= q_lens[r / rows_per_seq]) return;
    const float* lp = lses + r;
    const float* op = O_parts + r * D + c4;
    // a batch reads past the last partial by re-reading it, and leaves those values out
    auto load_o = [&](int i0, f32x4_t (&o)[NB]) {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int i = i0 + u < S ? i0 + u : S - 1;
            o[u] = *(const f32x4_t*)(op + (int64_t)i * rows * D);
        }
    };
    auto load_l = [&](int i0) { return i0 + c < S ? lp[(int64_t)(i0 + c) * rows] : -INFINITY; };  // this lane's partial
    f32x4_t o[NB];
    load_o(0, o);  // in flight together with the log-sum-exps
    float l = load_l(0);
    float M = fmaxf(l, -INFINITY);  // (a NaN does not count as a maximum, also where every lane holds one)
    for (int i0 = TPR; i0 < S; i0 += TPR) M = fmaxf(M, load_l(i0));
    M = row_max<TPR>(M);
    f32x4_t acc = zero_vec<f32x4_t>();
    float den = 0.f;
    if (M != -INFINITY) {
        for (int i0 = 0; i0 < S; i0 += TPR) {
            if (i0) l = load_l(i0);
            const float mine = l == -INFINITY ? -1.0f : expf(l - M);  // below 0: weight zero, its O takes no part
#pragma unroll 1
            for (int j0 = 0; j0 < TPR && i0 + j0 < S; j0 += NB) {
                if (i0 + j0) load_o(i0 + j0, o);
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    const float a = __shfl(mine, j0 + u, TPR);
                    if (a == -1.0f) continue;
                    den += a;
                    acc[0] = __builtin_fmaf(a, o[u][0], acc[0]);
                    acc[1] = __builtin_fmaf(a, o[u][1], acc[1]);
                    acc[2] = __builtin_fmaf(a, o[u][2], acc[2]);
                    acc[3] = __builtin_fmaf(a, o[u][3], acc[3]);
                }
            }
        }
        const float inv = 1.0f / den;
        acc[0] *= inv; acc[1] *= inv; acc[2] *= inv; acc[3] *= inv;
    }
    *(f32x4_t*)(O + r * D + c4) = acc;
    if (c == 0) lse[r] = (M == -INFINITY) ? -INFINITY : M + logf(den);
}

// One to four partials, the usual number: every thread reads the row's log-sum-exps itself, and all that it reads is in flight
// at once.  65536 rows of 128 over 2: 16.6 us (18.7 one after the other, 18.2 in the form above, whose batch reads the last
// partial again); 32 rows: 2.3 (2.5, 2.9).
template <int D, int S>
FEDRAG_KERNEL __launch_bounds__(256) void lse_merge_few_kernel(const float* __restrict__ O_parts,
                                                            const float* __restrict__ lses, int64_t rows,
                                                            float* __restrict__ O, float* __restrict__ lse,
                                                            const int32_t* __restrict__ q_lens, int64_t Lq,
                                                            int64_t rows_per_seq) {
    constexpr int TPR = D / 4;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = gid / TPR;
    const int c4 = (int)(gid % TPR) * 4;
    if (r >= rows) return;
    if (q_lens && (r % Lq) >= q_lens[r / rows_per_seq]) return;
    float l[S];
    f32x4_t o[S];
#pragma unroll
    for (int i = 0; i < S; ++i) l[i] = lses[i * rows + r];
#pragma unroll
    for (int i = 0; i < S; ++i) o[i] = *(const f32x4_t*)(O_parts + (i * rows + r) * D + c4);
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < S; ++i) M = fmaxf(M, l[i]);
    f32x4_t acc = zero_vec<f32x4_t>();
    float den = 0.f;
    if (M != -INFINITY) {
#pragma unroll
        for (int i = 0; i < S; ++i) {
            if (l[i] == -INFINITY) continue;  // weight zero: its O takes no part
            const float a = expf(l[i] - M);
            den += a;
            acc[0] = __builtin_fmaf(a, o[i][0], acc[0]);
            acc[1] = __builtin_fmaf(a, o[i][1], acc[1]);
            acc[2] = __builtin_fmaf(a, o[i][2], acc[2]);
            acc[3] = __builtin_fmaf(a, o[i][3], acc[3]);
        }
        const float inv = 1.0f / den;
        acc[0] *= inv; acc[1] *= inv; acc[2] *= inv; acc[3] *= inv;
    }
    *(f32x4_t*)(O + r * D + c4) = acc;
    if (c4 == 0) lse[r] = (M == -INFINITY) ? -INFINITY : M + logf(den);
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
    if (S <= 4) {
#define FEDRAG_FEW(S_) (D == 128 ? lse_merge_few_kernel<128, S_> : lse_merge_few_kernel<64, S_>)
        const auto few = S == 1 ? FEDRAG_FEW(1) : S == 2 ? FEDRAG_FEW(2) : S == 3 ? FEDRAG_FEW(3) : FEDRAG_FEW(4);
#undef FEDRAG_FEW
        hipLaunchKernelGGL(few, grid, dim3(wg), 0, stream, O_parts, lses, rows, O, lse, q_lens, Lq, rows_per_seq);
        return hipGetLastError();
    }
    const int nb = threads <= 256 * 256 && S > 8 ? 16 : threads <= 256 * 512 ? 8 : 2;
#define FEDRAG_MANY(NB_) (D == 128 ? lse_merge_kernel<128, NB_> : lse_merge_kernel<64, NB_>)
    const auto kernel = nb == 16 ? FEDRAG_MANY(16) : nb == 8 ? FEDRAG_MANY(8) : FEDRAG_MANY(2);
#undef FEDRAG_MANY
    hipLaunchKernelGGL(kernel, grid, dim3(wg), 0, stream, O_parts, lses, S, rows, O, lse, q_lens, Lq, rows_per_seq);
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
    hipLaunchKernelGGL(scatter_rows_f32_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, in, perm,
                       L, FastDiv(L), total <= 0x7fffffffLL ? 1 : 0, total, out);
    return hipGetLastError();
}

}  // namespace fedrag

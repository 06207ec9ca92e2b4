// Host-side internal interface between the C-ABI entry points (fedrag_api.hip) and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/fedrag.h"

namespace fedrag {

// A launch grid's x dimension of n workgroups: the launchers refuse (hipErrorInvalidValue) what would not fit instead of
// truncating.  A dispatch counts its threads in 32 bits, and the runtime starts fewer of them without an error beyond that.
constexpr bool grid_fits(int64_t n, int64_t threads) { return n >= 1 && n <= 0xffffffffLL / threads; }
static_assert(grid_fits((1 << 24) - 1, 256) && !grid_fits(1 << 24, 256) && !grid_fits(0, 64), "32 bits of threads");

// Second partial for the scatter form (Dec followed by the Section 4.1 aggregation of two partials): row i of X has
// log-sum-exp lse_in[bh, i]; (O_other, lse_other) is the other partial, already in destination row order.
struct RowsMerge {
    const float* lse_in;     // [BH, L]; NULL = plain transform
    const float* O_other;    // [BH, L, D]
    const float* lse_other;  // [BH, L]
    float* lse_out;          // [BH, L]
};

// Rows-times-matrix job: up to two tensors (K and V) transformed in one launch.
struct RowsJob {
    int n_jobs;               // 1 or 2
    const void* X[2];
    const void* Phi[2];       // dense form: [Hkv, D, D]
    bool structured;          // true: the matrix is given as S1 P1 H P2 S2 by the four arrays below, [Hkv, D] each
    const float* s_in[2];
    const int32_t* p_in[2];
    const int32_t* p_out[2];
    const float* s_out[2];
    int quant_bits;           // 0, or 8 / 4: 16-bit gather form only - Y[i] receives the transport codes of the rows
    float* params[2];         //   and params[i] their (scale, lo), [BH * L, 2]
    void* Y[2];
    const int32_t* perm;      // NULL = identity
    int64_t perm_batch_stride;  // 0 (one permutation for all sequences) or L
    int64_t BH;               // batch * heads
    int H;                    // heads per sequence
    int G;                    // heads per scrambling matrix
    int64_t L;                // rows per (batch, head)
    int D;                    // 64 or 128
    int dtype;                // fedrag_dtype of X / Phi / Y (ignored when scatter: fp32)
    bool scatter;             // false: Y[j] = X[perm[j]].Phi ; true: Y[perm[i]] = X[i].Phi (fp32)
    RowsMerge merge;          // scatter, one job: aggregate every transformed row with a second partial (lse_in != NULL)
};
hipError_t launch_rows_transform(const RowsJob& job, hipStream_t stream);
// Workgroups of the fp32 row products a compute unit holds, as their split over workgroups counts them.
int row_steps_resident(int D, bool structured, bool merge);
// Workgroups per slab of the product with a key's factors, and row steps of each.
struct RowSteps {
    int64_t chunks;
    int per;
};
RowSteps hadamard_steps(int64_t slabs, int64_t L);
hipError_t launch_invert_perm(const int32_t* perm, int64_t L, int32_t* inv, hipStream_t stream);
// flag[0] = 0 if every row of perm [n_perm, L] is a permutation of 0..L-1, else bit 0 (index out of range) and / or
// bit 1 (index repeated); marks [n_perm, L] is scratch.
hipError_t launch_validate_perm(const int32_t* perm, int n_perm, int64_t L, int32_t* marks, int32_t* flag,
                                hipStream_t stream);

// Partial attention problem: one KV shard (K, V, Lkv), or - n_shards > 1 - the shards a Compute Node holds for
// the same queries, (Ks[i], Vs[i], Ls[i]), whose partials are aggregated inside the call.
constexpr int kMaxShards = 16;
struct AttnProblem {
    int B, Hq, Hkv, D, dtype;
    int64_t Lq, Lkv;
    const void *Q, *K, *V;
    float scale;
    int quant_bits;          // 0, or 8 / 4: K, V hold the transport codec's codes and K_params, V_params their
    const float* K_params;   //   per-row (scale, lo), [B,Hkv,Lkv,2] (decode shapes, 16-bit dtype, D = 128 only)
    const float* V_params;
    int n_shards;            // 0 or 1: K, V, Lkv above; else Ks, Vs, Ls below (no codes, no lengths, no mask)
    const void* Ks[kMaxShards];
    const void* Vs[kMaxShards];
    int64_t Ls[kMaxShards];
    const int32_t* kv_lens;  // NULL, or [B] device array: sequence b has only its first kv_lens[b] keys (<= Lkv)
    const int32_t* q_lens;   // NULL, or [B] device array: only the first q_lens[b] query rows of sequence b are computed
                             //   and written (prefill and fp32 kernels; the decode kernel computes all its <= 16 rows)
    bool causal;  // the Lq queries are the last Lq of the Lkv tokens and see nothing after themselves
    float* O;     // [B,Hq,Lq,D]
    float* lse;   // [B,Hq,Lq]
    void* workspace;
    size_t workspace_bytes;
};
// Division of an index below 2^31 by a number the host knows: n / d = (n * m) >> s, exact because m = ceil(2^s / d) with
// s = 31 + ceil(log2 d) leaves an error n * (m d - 2^s) < 2^31 * 2^ceil(log2 d) = 2^s.  Three scalar instructions in a
// kernel's first lines instead of some twenty-five with a reciprocal estimate in them.
struct FastDiv {
    uint32_t m, s, d;
    FastDiv() = default;
    explicit FastDiv(int64_t div) : d((uint32_t)div) {
        s = 31 + (div > 1 ? 64 - (uint32_t)__builtin_clzll((uint64_t)div - 1) : 0);  // + ceil(log2(div))
        m = (uint32_t)((((uint64_t)1 << s) + (uint64_t)div - 1) / (uint64_t)div);
    }
    __host__ __device__ uint32_t div(uint32_t n) const { return (uint32_t)(((uint64_t)n * m) >> s); }
    __host__ __device__ uint32_t mod(uint32_t n) const { return n - div(n) * d; }
};

// 32-bit outputs (with several runs: partials) of a prefill launch from this size on are stored past the L2s, 4 MiB on each of the
// 8 XCDs.  All workgroups store at about the same time, at their end, and lines left dirty there are
// written back before the next launch may start: 4 x 777 tokens x 16 heads of 128 with a mask (24 MiB) 31.0 us and 28.1, 8 x 300 x
// 32 of 64 (19 MiB) 17.2 and 15.2, 2048 x 32 of 128 (32 MiB) 61.2 and 58.8, 117 x 32 x (4001 + 3277) of 64 (17 MiB of partials)
// 22.5 and 20.6.  Below, what reads them next finds them in L2: 117 x 32 x 300 of 64 (1 MiB) 9.0 and 9.3, 128 x 16 x 1024 (2 MiB)
// 10.1 and 10.3; from 4 to 8 MiB even.
// Partials are read again at once, by the fold: beyond the 32 MiB that all L2s hold, from where they are on their way out before the
// launch ends either way, being sent past them costs up to 6 % (1277 x 16 x (307 + 330) of 128, 40 MiB, 33.9 us and 36.0; 2048 x 16 x
// 600 on codes, 32 MiB, 33.7 and 35.5; over 106 launches 0.8 % on average); below it gains up to 10 % (266 x 32 x (638 + 638), 25 MiB,
// 29.5 and 27.5).  Two partials of rows of 128 are so many rows that it is over sooner (800 x 32 x (500 + 400), 25 MiB, 34.0 and
// 34.9; 1500 x 16 x 1500 on codes, 23 MiB, 46.0 and 46.9), rows of 64 go on a little longer (1300 x 32 x 4 x 200, 41 MiB, 35.2 and 33.9;
// from 42 MiB on even, then 1 % slower).
constexpr int64_t kPastL2Bytes = 8 << 20;
constexpr int64_t kPastL2Partials = 32 << 20;
constexpr int64_t kPastL2TwoPartials = 20 << 20;
constexpr int64_t kPastL2Partials64 = 42 << 20;

// How a launch cuts the keys into runs, one workgroup per (unit of queries, run): what both attention kernels
// receive by value.  Shard i contributes runs first[i] .. first[i+1]-1 of s[i].per keys each (the last one shorter);
// first[i] = INT_MAX past the last shard, so a kernel finds its shard with compares only.  With more than one run
// the kernels write one normalised partial per run into the workspace, [n_runs][rows][D] then [n_runs][rows], and
// the Section 4.1 aggregation folds them.
struct KeyShard {
    const void* K;
    const void* V;
    int64_t L;
    int64_t per;
};
struct KeyRuns {
    int n_runs;
    int n_shards;
    FastDiv by_runs;  // n_runs (1 when there is none)
    int first[kMaxShards + 1];
    KeyShard s[kMaxShards];
    // The shard that run `run` (0 <= run < n_runs) belongs to; *split = index of the run inside it.  All of first[] is
    // read at once and counted (one compare after the other, each waiting for its own scalar load, kept a short
    // kernel from starting for 1.5 us); a single shard needs none of it.
    __device__ __forceinline__ KeyShard shard_of(int run, int* split) const {
        *split = run;
        if (n_shards == 1) return s[0];
        int i = 0, begin = 0;
#pragma unroll
        for (int j = 1; j < kMaxShards; ++j) {
            const bool past = run >= first[j];
            i += past ? 1 : 0;
            begin = past ? first[j] : begin;
        }
        *split = run - begin;
        return s[i];
    }
};
// Plans the runs for n shards of lengths Ls (n >= 1); pointers are left unset.  codes4: the streaming kernel will
// read 4-bit transport codes (d = 128 decode shapes), where it wants kDecCodesOcc workgroups per compute unit.
KeyRuns attn_plan_runs(int B, int Hq, int Hkv, int dtype, int64_t Lq, int n, const int64_t* Ls, bool codes4 = false);
// Workgroups that make one round over the chip: the compute units of the device that is current in the calling thread.
int attn_target_wgs();
bool attn_uses_decode_kernel(int Hq, int Hkv, int64_t Lq);  // G * Lq <= 16: the HBM-bound streaming kernel
// bytes of workspace the plan needs (0 when there is a single run)
size_t attn_workspace_bytes(int B, int Hq, int Hkv, int D, int dtype, int64_t Lq, int n, const int64_t* Ls);
inline size_t attn_workspace_bytes(int B, int Hq, int Hkv, int D, int dtype, int64_t Lq, int64_t Lkv) {
    return attn_workspace_bytes(B, Hq, Hkv, D, dtype, Lq, 1, &Lkv);
}
// The plan of problem p with its pointers filled in.  *part: keys of a run that the streaming kernel sums by themselves, where its
// runs were made longer than the plan's; else 0.
KeyRuns attn_runs_of(const AttnProblem& p, int64_t* part = nullptr);
// Cuts the shards of r (s[].L, n_shards) into runs of about `per` keys, a multiple of `quantum` and rebalanced inside a shard.
void attn_cut_runs(KeyRuns& r, int64_t per, int64_t quantum);
hipError_t launch_partial_attn(const AttnProblem& p, hipStream_t stream);
// Device address, on the current device, of the library's static scratch array of FEDRAG_STATIC_SCRATCH_BYTES bytes.
hipError_t attn_static_scratch(void** ptr_out);

// decode kernel geometry (shared by the split planner and the kernel)
constexpr int kDecWaves = 4;  // twice that for runs of two steps of 128 columns, half for runs of half a step
constexpr int kDecThreads = kDecWaves * 64;
constexpr int kDecTile = 32;                      // keys per wave step
constexpr int kDecStride = kDecWaves * kDecTile;  // keys per workgroup step
#ifndef FEDRAG_DECQ_OCC
#define FEDRAG_DECQ_OCC 2
#endif
constexpr int kDecCodesOcc = FEDRAG_DECQ_OCC;     // workgroups per compute unit when the kernel reads 4-bit codes
// prefill kernel geometry (shared by the split planner and the kernel)
constexpr int kPreQ = 32;                     // query rows per wave (one 32-wide MFMA column tile)
constexpr int kPrePlanRows = 8 * kPreQ;       // query rows the planner counts per workgroup (the larger of the two forms)
constexpr int kPreK = 64;                     // keys per LDS tile
constexpr int kPreMinTilesPerSplit = 4;       // a KV split is at least this many tiles
constexpr int64_t kPrePair = 2 * kPreK;       // a tile for each of two key groups
// The form a prefill launch takes (attn_prefill.hip), a host decision from sizes alone.
struct PrefillForm {
    enum Kind { kPlain, kWalk, kTwoGroups } kind;  // a run a workgroup; all shards in turn; a run's keys halved between two groups
    bool four;      // plain, walk: four waves of 32 query rows per workgroup instead of eight
    int Hq;         // heads and query rows per head as the kernel sees them
    int64_t Lq;
    KeyRuns runs;   // n_runs < 1: refused; more than one: partials
};
PrefillForm prefill_form(const AttnProblem& p);
bool prefill_stores_past_l2(const AttnProblem& p, const PrefillForm& f);  // see kPastL2Bytes
int64_t prefill_least_run(const KeyRuns& shards, int64_t from, int64_t most);
hipError_t launch_attn_f32(const AttnProblem& p, hipStream_t stream);      // fp32 storage, any L_q
hipError_t launch_decode_attn(const AttnProblem& p, hipStream_t stream);   // 16-bit storage, G * L_q <= 16
hipError_t launch_prefill_attn(const AttnProblem& p, hipStream_t stream);  // 16-bit storage, any L_q

// Aggregation of S partials: O_parts [S, rows, D], lses [S, rows] -> O [rows, D], lse [rows].
// q_lens (device, [B]) with Lq and rows_per_seq = Hq * Lq: row r is query r % Lq of sequence r / rows_per_seq, and rows
// at or past q_lens[sequence] are skipped (neither read nor written).
hipError_t launch_lse_merge(const float* O_parts, const float* lses, int S, int64_t rows, int D, float* O, float* lse,
                            hipStream_t stream, const int32_t* q_lens = nullptr, int64_t Lq = 1,
                            int64_t rows_per_seq = 1);
// O = 0, lse = -inf for `rows` rows (a shard with no keys).
hipError_t launch_fill_empty(float* O, float* lse, int64_t rows, int D, hipStream_t stream);
// out[bh, perm[i]] = in[bh, i] for n_bh rows of L values each (perm NULL = copy).
hipError_t launch_scatter_rows_f32(const float* in, const int32_t* perm, int64_t n_bh, int64_t L, float* out,
                                   hipStream_t stream);

// Transport codec job: quantize (X -> codes, params) or dequantize (codes, params -> X); X has n_rows rows of D values.
struct CodecJob {
    bool quantize;
    int64_t n_rows;
    int D;       // 64 or 128
    int dtype;   // fedrag_dtype of X
    int bits;    // 8 or 4
    void* X;
    uint8_t* codes;   // [n_rows, D * bits / 8]
    float* params;    // [n_rows, 2] = (scale, lo)
};
hipError_t launch_codec(const CodecJob& job, hipStream_t stream);

}  // namespace fedrag

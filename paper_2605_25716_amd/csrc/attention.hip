// The Compute Node's work on one KV shard (Section 4.1, per-node local computation):
//   O_i = softmax(Q' K_i'^T * scale) V_i'   and   lse_i = ln sum_t exp(Q' K_i'^T * scale)   (= ln w_i)
// evaluated with a running maximum so that outlier logits cannot overflow.  Three kernels:
//   attn_f32_kernel     (attn_f32.hip)     fp32 storage on the fp32 matrix cores (accuracy path)
//   decode_attn_kernel  (attn_decode.hip)  16-bit storage, <= 16 query rows per KV head: HBM-bound streaming
//   prefill_attn_kernel (attn_prefill.hip) 16-bit storage, many query rows: MFMA-bound tiled kernel
// This file holds the plan of the key runs and the dispatch between the three.
#include "fedrag_device.h"
#include "fedrag_host.h"

#include <atomic>
#include <climits>
#include <cstdint>

namespace fedrag {

// ------------------------------------------------------------------------------------------------ dispatch
// Decode workgroups to aim for over the whole launch: one per CU (the kernel is sized for one resident
// workgroup per CU; a single round of equal-sized workgroups measured fastest).  256 CUs on MI355X; the
// attribute query is host-only and falls back to that number when no device is present.
int attn_target_wgs() {
    // the count belongs to the device that is current in the calling thread; it is cached per device ordinal in
    // atomics, so concurrent first calls only repeat the query
    constexpr int kMaxDev = 64;
    static std::atomic<int> cached[kMaxDev];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDev) {
        (void)hipGetLastError();
        return 256;
    }
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            return 256;
        }
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}
// Shortest run of the decode kernel, in 128-key steps of a workgroup.  A run costs the launch a partial to fold and its
// workspace, so 512 keys, although runs of 256 are faster (a decoded token over 32 layers and two Context Owners of 4096 keys
// 901 us against 940): every decode shape is promised to need at most about 4.3 MB, and the host test of the entry points
// holds the size query to the number of runs it has always answered.  A context of no more than 512 keys is one run and no
// fold (300 keys: 25.7 us a layer against 27.8 in two runs).  In between a context would be two to four runs, which leaves the
// chip idle: 400 + 700 keys take 23.1 us a layer in 256-key runs against 24.9 - as long as those are one round of workgroups:
// 9 sequences x 8 KV heads x 1024 keys take 15.0 us in 144 workgroups of 512 keys and 17.9 in 288 of 256 (8-bit codes; 16-bit
// 16.2 and 17.5 for 12 sequences).  On 4-bit codes, two workgroups to a unit, a second round begun costs less than longer runs
// (20 x 8 x 800 keys 13.2 us in 640 workgroups, 14.2 in 320; the launch makes 480 of them, 13.0).
constexpr int kDecMinSteps = 4;
constexpr int kDecMinStepsShort = 2;
constexpr int64_t kDecShortContext = 2048;  // keys of all shards of a unit up to which the shorter run is taken
static bool use_decode_kernel(int Hq, int Hkv, int64_t Lq) { return (int64_t)(Hq / Hkv) * Lq <= 16; }

// Decode kernel: about one workgroup per compute unit over the whole launch; a run is a whole number of 128-key
// workgroup steps, at least kDecMinSteps (kDecMinStepsShort) of them, and stays below 2^31 bytes (32-bit buffer offsets).
// Prefill kernel: one workgroup per (sequence, query head, 256 query rows) walks a run, about 2 us per 64-key tile.
// When those workgroups cover less than half of the compute units, the keys are cut into runs of at least
// kPreMinTilesPerSplit tiles (so that a workgroup's fixed cost stays small beside its tiles) for one round of
// workgroups over the chip; otherwise every shard is one run.  The launch may cut them anew into fewer (two key groups to a workgroup).
KeyRuns attn_plan_runs(int B, int Hq, int Hkv, int dtype, int64_t Lq, int n, const int64_t* Ls, bool codes4) {
    KeyRuns r;
    for (int i = 0; i < kMaxShards; ++i) {
        r.s[i] = KeyShard{nullptr, nullptr, 0, 1};
        r.first[i] = INT_MAX;
    }
    r.first[kMaxShards] = INT_MAX;
    r.n_runs = 0;
    r.n_shards = n;
    r.by_runs = FastDiv(1);
    if (n < 1 || n > kMaxShards) return r;
    int64_t total = 0;
    for (int i = 0; i < n; ++i) total += Ls[i] > 0 ? Ls[i] : 0;
    const bool decode = use_decode_kernel(Hq, Hkv, Lq);
    const int64_t cus = (int64_t)attn_target_wgs() * ((codes4 && decode) ? kDecCodesOcc : 1);
    int64_t per = INT64_MAX;  // keys per run before rebalancing inside a shard
    int64_t quantum = 1;
    if (dtype != FEDRAG_F32 && total > 0 && Lq > 0) {
        if (decode) {
            const int64_t units = (int64_t)B * Hkv;
            const int64_t want = units > 0 ? (cus + units - 1) / units : 1;
            quantum = kDecStride;
            per = (total + want - 1) / want;
            per = ((per + quantum - 1) / quantum) * quantum;
            int64_t least = kDecMinSteps * quantum;
            if (total <= kDecShortContext && total > least) {
                const int64_t shorter = per > kDecMinStepsShort * quantum ? per : kDecMinStepsShort * quantum;
                int64_t runs = 0;
                for (int i = 0; i < n; ++i) runs += Ls[i] > 0 ? (Ls[i] + shorter - 1) / shorter : 0;
                if (codes4 || units * runs <= cus) least = shorter;
            }
            if (per < least) per = least;
            if (per > (int64_t)1 << 22) per = (int64_t)1 << 22;
        } else {
            // the query heads of a KV head form one run of G * Lq rows (see launch_prefill_t)
            const int64_t wgs = (int64_t)B * Hkv * (((int64_t)(Hq / Hkv) * Lq + kPrePlanRows - 1) / kPrePlanRows);
            quantum = kPreK;
            if (wgs > 0 && wgs * 2 <= cus) {
                const int64_t want = cus / wgs;
                const int64_t tiles = (total + kPreK - 1) / kPreK;
                int64_t per_t = (tiles + want - 1) / want;
                if (per_t < kPreMinTilesPerSplit) per_t = kPreMinTilesPerSplit;
                per = per_t * kPreK;
            }
        }
    }
    for (int i = 0; i < n; ++i) r.s[i].L = Ls[i] > 0 ? Ls[i] : 0;
    attn_cut_runs(r, per, quantum);
    return r;
}

void attn_cut_runs(KeyRuns& r, int64_t per, int64_t quantum) {
    const int n = r.n_shards;
    int at = 0;
    for (int i = 0; i < n; ++i) {
        const int64_t L = r.s[i].L;
        r.first[i] = at;
        if (L == 0) continue;  // no runs: first[i] == first[i + 1]
        const int64_t runs = per == INT64_MAX ? 1 : (L + per - 1) / per;
        int64_t mine = (L + runs - 1) / runs;  // rebalanced inside the shard
        mine = ((mine + quantum - 1) / quantum) * quantum;
        r.s[i].per = mine;
        at += (int)((L + mine - 1) / mine);
    }
    for (int i = n; i <= kMaxShards; ++i) r.first[i] = i == n ? at : INT_MAX;
    r.n_runs = at;
    r.by_runs = FastDiv(at > 0 ? at : 1);
}

// One round of workgroups where the streaming kernel would have one and a bit.  The plan above rounds the runs of a unit up, as the
// workspace is sized, and a few workgroups over a round take as long as the round did; their number is rounded down here.  Never
// more runs than the plan has.  Where the shards alone are more than a round the rounds even out (20 x (4001 + 3277 + 300) keys:
// 135 us, 139 with a run a shard), and a shard much longer than the others would be a run too long (9 of them: 55.6 us, 57.0).
// 16-bit values, the plan's runs and one round, 8192 keys x 8 heads of 128: 3 sequences (264 workgroups and 240) 27.7 and 22.2 us,
// 9 (288, 216) 67.6 and 52.8, 17 (272, 136) 122 and 103, 31 (496, 248) 164 and 160; of 64, 9 and 17 sequences 35.0 and 28.6, 64.1
// and 53.1; 5 x (4001 + 3277 + 300) 39.7 and 31.4.  What is left idle costs little: a compute unit takes more of the memory's rate
// when others rest.
// Codes are bound by the instructions that rebuild them, so there what counts is the load of the compute unit that has the most
// workgroups, in keys, each with its start and end (`start`), and one round has to be ahead by that: of 8-bit codes by 5 % (3 and 9
// x 8192 27.6 and 21.9 us, 56.8 and 44.3, 30 x 600 22.3 and 15.7, 20 x 8192 even; 20 x 16384 188 and 194: as planned).  Of 4-bit codes,
// two workgroups to a unit, by 15 %, and three quarters full (20 x 800 13.2 and 13.0, 60 x 600 19.8 and 15.1, 9 x 8192 31.9 and 29.6; 22 x
// 1100, 352 workgroups, 16.3 and 17.6: as planned), because where two runs a sequence, three on some units, would be one run, two on
// some units, it is a third more: 33 x 3000 42.5 and 50.4, 33 x 8192 101 and 127, 40 x 16384 199 and 254.
// Returns the keys of a part, as attn_runs_of does.
static int64_t decode_one_round(KeyRuns& r, int64_t units, int quant_bits) {
    const int64_t cus = attn_target_wgs(), round = cus * (quant_bits == 4 ? kDecCodesOcc : 1);
    auto longest = [](const KeyRuns& k) {
        int64_t most = 0;
        for (int i = 0; i < k.n_shards; ++i) {
            const int64_t run = k.s[i].L < k.s[i].per ? k.s[i].L : k.s[i].per;
            most = run > most ? run : most;
        }
        return most;
    };
    int64_t shards = 0, per = kDecStride;
    for (int i = 0; i < r.n_shards; ++i) {
        shards += r.s[i].L > 0 ? 1 : 0;
        if (r.s[i].L > 0 && r.s[i].per > per) per = r.s[i].per;
    }
    if (units < 1 || units * r.n_runs <= round || units * shards > round) return 0;
    static_assert(kPrePair == kDecStride, "runs of whole steps");
    const int64_t least = prefill_least_run(r, per, round / units);
    if (least > (int64_t)1 << 22) return 0;  // (a run is addressed in 32 bits)
    KeyRuns one = r;
    attn_cut_runs(one, least, kDecStride);
    auto cost = [&](const KeyRuns& k, int64_t start) { return (units * k.n_runs + cus - 1) / cus * (longest(k) + start); };
    if (quant_bits == 0 && cost(r, 0) < cost(one, 0)) return 0;
    if (quant_bits == 8 && cost(r, 500) * 20 < cost(one, 500) * 21) return 0;
    if (quant_bits == 4 && (cost(r, 400) * 20 < cost(one, 400) * 23 || units * one.n_runs * 4 < round * 3)) return 0;
    // Summed in parts no longer than the plan's runs, with a maximum of their own: in one go a run twice as long left up to 17 % more
    // error (fp16, 17 x 2 rows x 20000 keys 6.1e-7 and 7.1e-7; bf16 1 to 3 %), as fp32 sums are longer and half as many keys have the
    // probability 1 exactly.
    const int64_t parts = (longest(one) + longest(r) - 1) / longest(r);
    r = one;
    return parts > 1 ? (longest(one) + parts - 1) / parts : 0;
}

KeyRuns attn_runs_of(const AttnProblem& p, int64_t* part) {
    int64_t keys = 0;
    if (!part) part = &keys;
    *part = 0;
    const bool streaming = use_decode_kernel(p.Hq, p.Hkv, p.Lq) && p.dtype != FEDRAG_F32 && !p.causal && (p.quant_bits == 0 || p.D == 128);
    const int64_t units = (int64_t)p.B * p.Hkv;
    if (p.n_shards <= 1) {
        const bool codes4 = p.quant_bits == 4 && p.D == 128;
        KeyRuns r = attn_plan_runs(p.B, p.Hq, p.Hkv, p.dtype, p.Lq, 1, &p.Lkv, codes4);
        if (streaming) *part = decode_one_round(r, units, p.quant_bits);
        r.s[0].K = p.K;
        r.s[0].V = p.V;
        return r;
    }
    KeyRuns r = attn_plan_runs(p.B, p.Hq, p.Hkv, p.dtype, p.Lq, p.n_shards, p.Ls);
    if (streaming) *part = decode_one_round(r, units, 0);
    for (int i = 0; i < p.n_shards && i < kMaxShards; ++i) {
        r.s[i].K = p.Ks[i];
        r.s[i].V = p.Vs[i];
    }
    return r;
}

bool attn_uses_decode_kernel(int Hq, int Hkv, int64_t Lq) { return use_decode_kernel(Hq, Hkv, Lq); }

size_t attn_workspace_bytes(int B, int Hq, int Hkv, int D, int dtype, int64_t Lq, int n, const int64_t* Ls) {
    // one size serves a call on 16-bit values and the same call on 4-bit transport codes (more, shorter runs)
    int runs = attn_plan_runs(B, Hq, Hkv, dtype, Lq, n, Ls, false).n_runs;
    if (n == 1 && D == 128 && dtype != FEDRAG_F32) {
        const int on_codes = attn_plan_runs(B, Hq, Hkv, dtype, Lq, n, Ls, true).n_runs;
        if (on_codes > runs) runs = on_codes;
    }
    if (runs <= 1) return 0;
    const size_t rows = (size_t)B * Hq * (size_t)Lq;
    return (size_t)runs * rows * (size_t)(D + 1) * sizeof(float);
}

// Scratch for callers that cannot allocate: the key-run partials of a launch land in this file-scope device array
// instead of a caller's workspace.  Every GPU the library runs on holds its own copy (at its own address) until the
// process ends.  The name below is only the host's handle for the symbol: the device address is looked up once per
// device, with that device current, and only that pointer is ever handed to a kernel.
namespace {
__attribute__((used)) static __device__ __align__(256) unsigned char scratch[FEDRAG_STATIC_SCRATCH_BYTES];
}

hipError_t attn_static_scratch(void** ptr_out) {
    constexpr int kMaxDev = 64;
    static std::atomic<void*> ptrs[kMaxDev];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDev) return hipErrorInvalidDevice;
    void* p = ptrs[dev].load(std::memory_order_acquire);
    if (!p) {  // first call on this device (concurrent first calls look the same address up twice)
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptrs[dev].store(p, std::memory_order_release);
    }
    *ptr_out = p;
    return hipSuccess;
}

hipError_t launch_partial_attn(const AttnProblem& p_in, hipStream_t stream) {
    AttnProblem p = p_in;
    if (p.Lq == 1) p.causal = false;  // a single query at the last position sees every key
    const int64_t rows = (int64_t)p.B * p.Hq * p.Lq;
    if (rows == 0) return hipSuccess;
    if (p.n_shards > 1) {
        if (p.n_shards > kMaxShards || p.quant_bits != 0 || p.causal || p.kv_lens || p.q_lens) return hipErrorInvalidValue;
        int64_t total = 0;
        for (int i = 0; i < p.n_shards; ++i) total += p.Ls[i];
        if (total == 0) return launch_fill_empty(p.O, p.lse, rows, p.D, stream);
        const bool decode = use_decode_kernel(p.Hq, p.Hkv, p.Lq);
        if (p.dtype == FEDRAG_F32) return launch_attn_f32(p, stream);
        if (p.dtype != FEDRAG_BF16 && p.dtype != FEDRAG_F16) return hipErrorInvalidValue;
        // Prefill shapes: one launch, with a partial per run (never less than one per shard), or, where the query tiles cover the
        // chip, with workgroups that visit all shards and need none
        if (!decode) return launch_prefill_attn(p, stream);
        bool one_launch_per_shard = (int64_t)p.B * p.Hkv >= attn_target_wgs();
        if (one_launch_per_shard) {
            // The chip is already covered by one shard's workgroups (as many (sequence, KV head) units as compute units)
            // and every shard is one run: a launch per shard keeps the workgroups of a launch on one shard's K', V'
            // (8 shards of 8 GiB: 9.55 against 10.05 ms); the partials and their aggregation are the same
            const KeyRuns plan = attn_runs_of(p);
            for (int i = 0; i < p.n_shards; ++i)
                if (plan.first[i + 1] - plan.first[i] > 1) one_launch_per_shard = false;
        }
        if (one_launch_per_shard) {
            // one launch per non-empty shard into the workspace ([n][rows][D] then [n][rows]), then the aggregation.  A shard
            // alone is planned as one run too (units >= compute units), so its launch needs no workspace of its own.
            int idx[kMaxShards], n = 0;
            for (int i = 0; i < p.n_shards; ++i)
                if (p.Ls[i] > 0) idx[n++] = i;
            if (n > 1 && (!p.workspace || p.workspace_bytes < (size_t)n * rows * (p.D + 1) * sizeof(float)))
                return hipErrorInvalidValue;
            float* Ow = n > 1 ? (float*)p.workspace : p.O;
            float* Lw = n > 1 ? Ow + (size_t)n * rows * p.D : p.lse;
            for (int j = 0; j < n; ++j) {
                AttnProblem one = p;
                one.n_shards = 1;
                one.K = p.Ks[idx[j]];
                one.V = p.Vs[idx[j]];
                one.Lkv = p.Ls[idx[j]];
                one.workspace = nullptr;
                one.workspace_bytes = 0;
                one.O = Ow + (size_t)j * rows * p.D;
                one.lse = Lw + (size_t)j * rows;
                const hipError_t e = launch_partial_attn(one, stream);
                if (e != hipSuccess) return e;
            }
            return n > 1 ? launch_lse_merge(Ow, Lw, n, rows, p.D, p.O, p.lse, stream) : hipSuccess;
        }
        return launch_decode_attn(p, stream);
    }
    if (p.Lkv == 0) return launch_fill_empty(p.O, p.lse, rows, p.D, stream);
    if (p.quant_bits != 0) {  // K', V' as transport codes: 16-bit storage, no mask
        if (p.dtype == FEDRAG_F32 || p.causal) return hipErrorInvalidValue;
        // the streaming kernel's code path is laid out for d = 128; everything else takes the tiled kernel
        return (use_decode_kernel(p.Hq, p.Hkv, p.Lq) && p.D == 128) ? launch_decode_attn(p, stream)
                                                                    : launch_prefill_attn(p, stream);
    }
    if (p.dtype == FEDRAG_F32) return launch_attn_f32(p, stream);
    if (p.dtype != FEDRAG_BF16 && p.dtype != FEDRAG_F16) return hipErrorInvalidValue;
    return (!p.causal && use_decode_kernel(p.Hq, p.Hkv, p.Lq)) ? launch_decode_attn(p, stream)
                                                               : launch_prefill_attn(p, stream);
}

}  // namespace fedrag

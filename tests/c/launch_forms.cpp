// The host's choice of a prefill launch's form, looked at without a device (no call here enqueues anything).  Commands on stdin,
// one answer a line:
//   form B Hq Hkv d dtype Lq n L... / codes B Hq Hkv d dtype Lq 1 L (4 bits)   ->  kind four n_runs past_l2   (kind: 0 plain, 1 shards in turn, 2 two key groups)
//   decode B Hq Hkv d dtype Lq n L... / decode4, decode8 (codes)  ->  n_runs, keys that the runs cover, longest run, runs the workspace
//       holds, longest run of the plan, keys of a part (0: runs are summed in one go), runs of the plan
//   factors slabs L  ->  workgroups per slab of a product with a key's factors, row steps of each
//   runs from most n L...             ->  keys a run by halving, by trying every length in turn
//   time B Hq Hkv d dtype Lq n L...   ->  microseconds a choice takes, the least of many
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "fedrag_host.h"

using namespace fedrag;

static bool read_problem(AttnProblem& p, std::vector<int64_t>& L) {
    std::memset(&p, 0, sizeof p);
    long lq;
    int n;
    if (std::scanf("%d %d %d %d %d %ld %d", &p.B, &p.Hq, &p.Hkv, &p.D, &p.dtype, &lq, &n) != 7 || n < 1 || n > kMaxShards) return false;
    p.Lq = lq;
    p.scale = 1.0f;
    p.n_shards = n;
    L.resize(n);
    for (int i = 0; i < n; ++i) {
        long x;
        if (std::scanf("%ld", &x) != 1) return false;
        p.Ls[i] = L[i] = x;
    }
    p.Lkv = L[0];
    return true;
}

static int64_t one_after_the_other(KeyRuns cut, int64_t from, int64_t most) {
    int64_t longest = 0, per = from;
    for (int i = 0; i < cut.n_shards; ++i) longest = std::max(longest, cut.s[i].L);
    attn_cut_runs(cut, per, kPrePair);
    while (cut.n_runs > most && per < longest) attn_cut_runs(cut, per += kPrePair, kPrePair);
    return per;
}

int main() {
    char what[16];
    while (std::scanf("%15s", what) == 1) {
        AttnProblem p;
        std::vector<int64_t> L;
        if (!std::strcmp(what, "form") || !std::strcmp(what, "codes")) {
            if (!read_problem(p, L)) return 2;
            if (what[0] == 'c') p.quant_bits = 4;
            const PrefillForm f = prefill_form(p);
            std::printf("%d %d %d %d\n", (int)f.kind, f.four ? 1 : 0, f.runs.n_runs, prefill_stores_past_l2(p, f) ? 1 : 0);
        } else if (!std::strncmp(what, "decode", 6)) {
            if (!read_problem(p, L)) return 2;
            p.quant_bits = std::atoi(what + 6);
            int64_t part;
            const KeyRuns r = attn_runs_of(p, &part);
            long covered = 0, longest = 0;
            for (int run = 0; run < r.n_runs; ++run) {  // as the kernel finds its keys
                int i = 0;
                while (i + 1 < r.n_shards && run >= r.first[i + 1]) ++i;
                const int64_t begin = (run - r.first[i]) * r.s[i].per, keys = std::min(r.s[i].per, r.s[i].L - begin);
                covered += keys;
                longest = std::max<long>(longest, keys);
            }
            const size_t bytes = attn_workspace_bytes(p.B, p.Hq, p.Hkv, p.D, p.dtype, p.Lq, p.n_shards, p.Ls);
            const KeyRuns plan = attn_plan_runs(p.B, p.Hq, p.Hkv, p.dtype, p.Lq, p.n_shards > 1 ? p.n_shards : 1, p.n_shards > 1 ? p.Ls : &p.Lkv, p.quant_bits == 4);
            long planned = 0;
            for (int i = 0; i < plan.n_shards; ++i) planned = std::max<long>(planned, std::min(plan.s[i].per, plan.s[i].L));
            std::printf("%d %ld %ld %ld %ld %ld %d\n", r.n_runs, covered, longest, (long)(bytes / ((size_t)p.B * p.Hq * p.Lq * (p.D + 1) * 4)), planned, (long)part, plan.n_runs);
        } else if (!std::strcmp(what, "factors")) {
            long slabs, rows;
            if (std::scanf("%ld %ld", &slabs, &rows) != 2) return 2;
            const RowSteps r = hadamard_steps(slabs, rows);
            std::printf("%ld %d\n", (long)r.chunks, r.per);
        } else if (!std::strcmp(what, "runs")) {
            long from, most;
            int n;
            if (std::scanf("%ld %ld %d", &from, &most, &n) != 3 || n < 1 || n > kMaxShards) return 2;
            KeyRuns r;
            r.n_shards = n;
            for (int i = 0; i < n; ++i) {
                long x;
                if (std::scanf("%ld", &x) != 1) return 2;
                r.s[i] = KeyShard{nullptr, nullptr, x, 1};
            }
            std::printf("%ld %ld\n", (long)prefill_least_run(r, from, most), (long)one_after_the_other(r, from, most));
        } else if (!std::strcmp(what, "time")) {
            if (!read_problem(p, L)) return 2;
            double least = 1e30;
            int sum = 0;
            for (int i = 0; i < 200; ++i) {
                const auto t0 = std::chrono::steady_clock::now();
                sum += prefill_form(p).runs.n_runs;
                least = std::min(least, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count());
            }
            std::printf("%.3f %d\n", least, sum);
        } else {
            return 2;
        }
    }
    return 0;
}

"""The work whose speed counts: what users of this library have it do, through its public entry points.

Kinds of cases (key "kind"):
  protocol  one decoder layer's remote attention as a whole, call by call: Enc of the context's shards and of the
            queries, attention on every shard, aggregation, Dec.  With "graph" the calls are recorded once into a HIP
            graph and a pass replays it, as a serving loop does; without, every pass calls eagerly.
  request   one step of a request over all decoder layers at the paper's request sizes (Section 7.1): per layer
            scramble_q, attention over the Context Owners' shards, the Inquirer's own causal attention, Dec and
            aggregation, recorded into one HIP graph (Section 5.3; Lq = 1 is a decoded token, otherwise a segment).
  attn      a Compute Node's attention over the shards it holds (prefill and decode shapes).
  local     the Inquirer's own causal attention over its plaintext segment (Section 5.3).
  rerank    attention over a padded batch of query-document pairs (Section 5.2), on 16-bit K', V' or transport codes.
  enc       a Context Owner's Enc of one KV shard, plain or through the transport codec (Section 7.5).
  codes     decoding queries against a shard that arrived as transport codes.

Inputs: activations N(0,1) with 1 % of the (head, channel) axis scaled by 20 (fixed per tensor), Haar-random
orthogonal Phi per KV head, uniform random permutations.  Calls that start from scrambled operands get the same
activations multiplied by Phi and narrowed to the storage type.
"""
import math

import torch

from paper_2605_25716_amd import binding as fb

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
LLAMA8B = dict(Hq=32, Hkv=8, d=128)


def listed():
    return [
        # the smallest whole call chain in fp32 storage: a single user's parity or debug run, bound by latency and
        # launches
        dict(name="tiny_f32", kind="protocol", B=1, Hq=2, Hkv=2, d=64, Lq=4, S=1, L=512, dtype="f32", graph=False),
        # one decoded token of a request, all 32 layers, two Context Owners with 4096 tokens each, 192 local tokens:
        # what is paid per generated token
        dict(name="request_token", kind="request", layers=32, Lq=1, ctx="4096,4096", local=192, dtype="bf16",
             structured=False, **LLAMA8B),
        # the same request's prefill of a query segment of odd length over contexts of odd lengths, structured keys
        dict(name="request_segment", kind="request", layers=32, Lq=117, ctx="4001,3277", local=117, dtype="bf16",
             structured=True, **LLAMA8B),
        # batched decode step with the context's Enc in it: the workload the headline figure is quoted on
        dict(name="llama8b_decode", kind="protocol", B=16, S=4, L=8192, Lq=1, dtype="bf16", graph=True, **LLAMA8B),
        # long-context decode of a large batch over resident shards (16 GiB of K', V')
        dict(name="long_decode", kind="attn", B=64, Lq=1, S=2, L=32768, dtype="bf16", **LLAMA8B),
        # a RAG prompt's 2048 query tokens against 16384 retrieved tokens
        dict(name="rag_prefill", kind="attn", B=1, Lq=2048, S=1, L=16384, dtype="bf16", **LLAMA8B),
        # a 4096-token prefill chunk of a 70B-shaped model over 8 shards: the largest call
        dict(name="mixed70b_prefill", kind="attn", B=1, Hq=64, Hkv=8, d=128, Lq=4096, S=8, L=8192, dtype="bf16"),
        # the Inquirer's own segment, every token seeing itself and its predecessors
        dict(name="local_2048", kind="local", B=1, Lq=2048, L=2048, dtype="bf16", **LLAMA8B),
        # collaborative re-ranking of 10 candidate documents, bf16 as it arrives from Enc
        dict(name="rerank_bf16", kind="rerank", H=16, d=64, dtype="bf16", bits=0,
             lens="1024,896,777,640,512,512,400,333,256,130"),
        # the same on the 4-bit transport codes the paper recommends for this phase
        dict(name="rerank_codes4", kind="rerank", H=16, d=64, dtype="bf16", bits=4,
             lens="1024,896,777,640,512,512,400,333,256,130"),
        # Enc of a shard that leaves through the 8-bit codec: fp16 storage, structured keys, an odd shard length
        dict(name="enc_codes8_f16", kind="enc", B=16, H=8, d=128, L=8111, dtype="f16", bits=8, structured=True),
        # a decode step's attention on a shard that arrived as 4-bit codes
        dict(name="decode_codes4", kind="codes", B=16, L=8192, Lq=1, dtype="bf16", bits=4, **LLAMA8B),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["protocol", "protocol", "request", "attn", "attn", "local", "rerank", "enc", "codes"])
    dt16 = rng.choice(["bf16", "bf16", "f16"])
    if kind == "protocol":
        dtype = rng.choice(["f32", "bf16", "f16"])
        d, Hkv, G = rng.choice([64, 128]), rng.choice([2, 4, 8]), rng.choice([1, 2, 4])
        c = dict(kind=kind, B=_log_int(rng, 1, 16), Hq=Hkv * G, Hkv=Hkv, d=d, Lq=rng.choice([1, 1, _log_int(rng, 2, 64)]),
                 S=rng.choice([1, 2, 4]), L=_log_int(rng, 256, 8192), dtype=dtype, graph=rng.random() < 0.5)
        while dtype == "f32" and c["B"] * c["Hq"] * c["Lq"] * c["S"] * c["L"] > 1.6e7:
            if c["Lq"] > 4:
                c["Lq"] //= 2
            else:
                c["L"] = c["L"] * 2 // 3
        return c
    if kind == "request":
        Lq = rng.choice([1, _log_int(rng, 8, 512)])
        ctx = [_log_int(rng, 256, 6144) for _ in range(rng.choice([1, 2, 3]))]
        return dict(kind=kind, layers=rng.choice([8, 16, 32]), Lq=Lq, ctx=",".join(map(str, ctx)),
                    local=Lq + rng.choice([0, _log_int(rng, 16, 1024)]), dtype=dt16, structured=rng.random() < 0.5,
                    Hq=rng.choice([16, 32, 64]), Hkv=8, d=rng.choice([64, 128, 128]))
    if kind == "attn":
        shape = dict(Hq=rng.choice([16, 32, 64]), Hkv=8, d=rng.choice([64, 128, 128]))
        if rng.random() < 0.4:
            c = dict(kind=kind, B=_log_int(rng, 1, 64), Lq=rng.choice([1, 1, 2]), S=rng.choice([1, 2, 4, 8]),
                     L=_log_int(rng, 1000, 32768), dtype=dt16, **shape)
            while work(c)["bytes"] > 1.6e10:
                c["B"] //= 2
        else:
            c = dict(kind=kind, B=rng.choice([1, 1, 2]), Lq=_log_int(rng, 128, 4096), S=rng.choice([1, 1, 2, 4, 8]),
                     L=_log_int(rng, 512, 16384), dtype=dt16, **shape)
            while work(c)["flops"] > 6e12:
                c["L"] = c["L"] * 2 // 3
        return c
    if kind == "local":
        Lq = _log_int(rng, 64, 4096)
        return dict(kind=kind, B=rng.choice([1, 1, 2]), Lq=Lq, L=Lq + rng.choice([0, 0, _log_int(rng, 64, 2048)]),
                    dtype=dt16, Hq=rng.choice([16, 32]), Hkv=8, d=rng.choice([64, 128]))
    if kind == "rerank":
        top = _log_int(rng, 128, 1536)
        lens = sorted((rng.randint(max(1, top // 8), top) for _ in range(_log_int(rng, 2, 20))), reverse=True)
        return dict(kind=kind, H=rng.choice([12, 16]), d=64, dtype=dt16, bits=rng.choice([0, 0, 8, 4]),
                    lens=",".join(map(str, lens)))
    if kind == "enc":
        return dict(kind=kind, B=_log_int(rng, 1, 16), H=rng.choice([4, 8]), d=rng.choice([64, 128, 128]),
                    L=_log_int(rng, 500, 16384), dtype=dt16, bits=rng.choice([0, 0, 8, 4]), structured=rng.random() < 0.5)
    return dict(kind=kind, B=_log_int(rng, 1, 16), L=_log_int(rng, 1000, 16384), Lq=rng.choice([1, 1, 2]), dtype=dt16,
                bits=rng.choice([8, 4]), Hq=rng.choice([16, 32, 64]), Hkv=8, d=128)


# ----------------------------------------------------------------------------------------------- inputs
class _Inputs:
    """Seeded generators of activations, keys and permutations (plain torch)."""

    def __init__(self, case, seed):
        self.dt = DTYPES[case["dtype"]]
        self.dev = "cuda"
        self.gen = torch.Generator(device=self.dev)
        self.gen.manual_seed(seed * 7919 + 17)
        self.cpu = torch.Generator()
        self.cpu.manual_seed(seed * 104729 + 5)

    def act32(self, B, H, L, d):
        x = torch.randn((B, H, L, d), generator=self.gen, dtype=torch.float32, device=self.dev)
        s = torch.ones(H * d)
        s[torch.randperm(H * d, generator=self.cpu)[: max(1, round(0.01 * H * d))]] = 20.0
        return x.mul_(s.view(1, H, 1, d).to(self.dev))

    def act(self, B, H, L, d):
        if B * H * L * d <= 1 << 28:
            return self.act32(B, H, L, d).to(self.dt)
        out = torch.empty((B, H, L, d), dtype=self.dt, device=self.dev)
        s = torch.ones(H * d)
        s[torch.randperm(H * d, generator=self.cpu)[: max(1, round(0.01 * H * d))]] = 20.0
        s = s.view(1, H, 1, d).to(self.dev)
        for b in range(B):
            out[b:b + 1] = torch.randn((1, H, L, d), generator=self.gen, dtype=torch.float32, device=self.dev).mul_(s)
        return out

    def haar(self, H, d):
        q, r = torch.linalg.qr(torch.randn((H, d, d), generator=self.cpu, dtype=torch.float64))
        return q * torch.sign(torch.diagonal(r, dim1=-2, dim2=-1)).unsqueeze(-2)

    def scrambled(self, B, H, G, L, d, phi=None):
        """Activations of H heads as they look after Enc: times one matrix per group of G heads (default orthogonal)."""
        phi = (self.haar(H // G, d) if phi is None else phi).float().repeat_interleave(G, 0).to(self.dev)
        out = torch.empty((B, H, L, d), dtype=self.dt, device=self.dev)
        for b in range(B):
            out[b] = torch.bmm(self.act32(1, H, L, d)[0], phi)
        return out

    def perm(self, L):
        return torch.randperm(L, generator=self.cpu).to(torch.int32).to(self.dev)

    def dense_keys(self, Hkv, d):
        """Phi_Q, Phi_K, Phi_V in the storage type, Phi_V^{-1} in fp32; the derived ones from the stored ones."""
        phi_q = self.haar(Hkv, d).to(self.dt)
        phi_v = self.haar(Hkv, d).to(self.dt)
        phi_k = torch.linalg.inv(phi_q.double()).transpose(1, 2).to(self.dt)
        phi_vi = torch.linalg.inv(phi_v.double()).float()
        return tuple(t.contiguous().to(self.dev) for t in (phi_q, phi_k, phi_v, phi_vi))

    def structured_keys(self, Hkv, d):
        """The same four as (scale_in, perm_in, perm_out, scale_out) of S1 P1 H P2 S2, magnitudes in [1/8, 8]."""
        def diag(hi=3.0):
            e = (torch.rand((Hkv, d), generator=self.cpu, dtype=torch.float64) * 2 - 1) * hi
            sgn = torch.randint(0, 2, (Hkv, d), generator=self.cpu) * 2 - 1
            return torch.exp2(e.round()) * sgn  # powers of two: exact in every storage type, exact reciprocals

        def perms():
            return torch.stack([torch.randperm(d, generator=self.cpu) for _ in range(Hkv)])

        def put(a, g1, g2, b):
            return tuple(t.contiguous().to(self.dev) for t in (a.float(), g1.to(torch.int32), g2.to(torch.int32), b.float()))
        a, g1, g2, b = diag(), perms(), perms(), diag()
        key_q, key_k = put(a, g1, g2, b), put(1 / a, g1, g2, 1 / b)
        a, g1, g2, b = diag(), perms(), perms(), diag()
        return key_q, key_k, put(a, g1, g2, b), put(1 / b, g2.argsort(1), g1.argsort(1), 1 / a)


def _quantize(x, bits):
    """The transport codec in plain torch: codes and (scale, lo) per row."""
    levels = float(2 ** bits - 1)
    codes, params = [], []
    for b in range(x.shape[0]):
        f = x[b].float()
        lo, hi = f.amin(-1, keepdim=True), f.amax(-1, keepdim=True)
        rng = hi - lo
        q = torch.clamp(torch.floor((f - lo) * (levels / rng) + 0.5), 0, levels).to(torch.uint8)
        codes.append(q if bits == 8 else q[..., 0::2] | (q[..., 1::2] << 4))
        params.append(torch.cat([rng / levels, lo], -1))
    return torch.stack(codes), torch.stack(params)


def _dequantize64(codes, params, bits, dt):
    """Values the codes stand for: one narrowing to the storage type, then 64 bits."""
    q = codes if bits == 8 else torch.stack([codes & 15, codes >> 4], -1).flatten(-2)
    return (q.double() * params[..., :1].double() + params[..., 1:].double()).float().to(dt).double()


def _inputs(c, seed):
    """Every input of the case, on the GPU, without this repository's code."""
    g, k = _Inputs(c, seed), c["kind"]
    if k == "protocol":
        B, Hq, Hkv, d, Lq, S, L = (c[n] for n in ("B", "Hq", "Hkv", "d", "Lq", "S", "L"))
        return dict(keys=g.dense_keys(Hkv, d), Q=g.act(B, Hq, Lq, d), K=[g.act(B, Hkv, L, d) for _ in range(S)],
                    V=[g.act(B, Hkv, L, d) for _ in range(S)], perm_q=g.perm(Lq) if Lq > 1 else None,
                    perm_kv=[g.perm(L) for _ in range(S)])
    if k == "request":
        Hq, Hkv, d, Lq, n = (c[m] for m in ("Hq", "Hkv", "d", "Lq", "layers"))
        ctx = [int(x) for x in c["ctx"].split(",")]
        keys = (g.structured_keys if c["structured"] else g.dense_keys)(Hkv, d)
        stack = lambda f, L: [x for x in f(n, L).split(1)]  # noqa: E731
        mk, mv = (_matrix64(keys[m], d) for m in (1, 2))  # the order of the context's rows drops out
        Kr = [stack(lambda m, L: g.scrambled(m, Hkv, 1, L, d, mk), L) for L in ctx]
        Vr = [stack(lambda m, L: g.scrambled(m, Hkv, 1, L, d, mv), L) for L in ctx]
        return dict(keys=keys, Q=stack(lambda m, L: g.act(m, Hq, L, d), Lq), K=Kr, V=Vr,
                    Kl=stack(lambda m, L: g.act(m, Hkv, L, d), c["local"]),
                    Vl=stack(lambda m, L: g.act(m, Hkv, L, d), c["local"]), perm_q=g.perm(Lq) if Lq > 1 else None)
    if k == "attn":
        B, Hq, Hkv, d = c["B"], c["Hq"], c["Hkv"], c["d"]
        # Q' and K' share one orthogonal matrix in earnest; its effect on the logits cancels, so each may have its own
        return dict(Q=g.scrambled(B, Hq, Hq // Hkv, c["Lq"], d),
                    K=[g.scrambled(B, Hkv, 1, c["L"], d) for _ in range(c["S"])],
                    V=[g.scrambled(B, Hkv, 1, c["L"], d) for _ in range(c["S"])])
    if k == "local":
        B, Hq, Hkv, d = c["B"], c["Hq"], c["Hkv"], c["d"]
        return dict(Q=g.act(B, Hq, c["Lq"], d), K=g.act(B, Hkv, c["L"], d), V=g.act(B, Hkv, c["L"], d))
    if k == "rerank":
        lens = [int(x) for x in c["lens"].split(",")]
        t = [g.scrambled(len(lens), c["H"], 1, max(lens), c["d"]) for _ in range(3)]
        s = dict(Q=t[0], lens=torch.tensor(lens, dtype=torch.int32, device="cuda"))
        if c["bits"] == 0:
            return dict(s, K=t[1], V=t[2])
        return dict(s, K=_quantize(t[1], c["bits"]), V=_quantize(t[2], c["bits"]))
    if k == "enc":
        keys = (g.structured_keys if c["structured"] else g.dense_keys)(c["H"], c["d"])
        return dict(keys=keys, K=g.act(c["B"], c["H"], c["L"], c["d"]), V=g.act(c["B"], c["H"], c["L"], c["d"]),
                    perm=g.perm(c["L"]))
    B, Hq, Hkv, d = c["B"], c["Hq"], c["Hkv"], c["d"]
    return dict(Q=g.scrambled(B, Hq, Hq // Hkv, c["Lq"], d),
                K=_quantize(g.scrambled(B, Hkv, 1, c["L"], d), c["bits"]),
                V=_quantize(g.scrambled(B, Hkv, 1, c["L"], d), c["bits"]))


# ----------------------------------------------------------------------------------------------- passes
def _record(fn):
    """fn's calls as a HIP graph (they only enqueue kernels; all their memory is given to them)."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        fn()  # once eagerly: code objects are loaded outside the capture
        with torch.cuda.graph(graph, stream=side):
            fn()
    torch.cuda.current_stream().wait_stream(side)
    return graph.replay


def _bytes(n):
    return torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda")


def prepare(case, seed):
    c, i = case, _inputs(case, seed)
    k, dt = c["kind"], DTYPES[c["dtype"]]
    if k == "protocol":
        phi_q, phi_k, phi_v, phi_vi = i["keys"]
        if not c["graph"]:
            def call():
                Qs = fb.fedrag_scramble_q(i["Q"], phi_q, i["perm_q"])
                Os, ls = _f32(c["S"], c["B"], c["Hq"], c["Lq"], c["d"]), _f32(c["S"], c["B"], c["Hq"], c["Lq"])
                for s in range(c["S"]):
                    Ks, Vs = fb.fedrag_scramble_kv(i["K"][s], i["V"][s], phi_k, phi_v, i["perm_kv"][s], n_q_heads=c["Hq"])
                    fb.fedrag_partial_attn(Qs, Ks, Vs, None, O_part=Os[s], lse=ls[s])
                O, lse = fb.fedrag_lse_merge(Os, ls, n_kv_heads=c["Hkv"])
                return fb.fedrag_unscramble(O, phi_vi, i["perm_q"]), lse
            return dict(call=call, keep=i)
        B, Hq, Hkv, d, Lq, S, L = (c[n] for n in ("B", "Hq", "Hkv", "d", "Lq", "S", "L"))
        Qs, Ks, Vs = torch.empty_like(i["Q"]), torch.empty_like(i["K"][0]), torch.empty_like(i["V"][0])
        Os, ls, Om, lm, out = _f32(S, B, Hq, Lq, d), _f32(S, B, Hq, Lq), _f32(B, Hq, Lq, d), _f32(B, Hq, Lq), _f32(B, Hq, Lq, d)
        ws = _bytes(fb.fedrag_partial_attn_workspace_bytes(B, Hq, Hkv, d, dt, Lq, L))

        def step():
            fb.fedrag_scramble_q(i["Q"], phi_q, i["perm_q"], Q_out=Qs)
            for s in range(S):
                fb.fedrag_scramble_kv(i["K"][s], i["V"][s], phi_k, phi_v, i["perm_kv"][s], n_q_heads=Hq, K_out=Ks, V_out=Vs)
                fb.fedrag_partial_attn(Qs, Ks, Vs, None, O_part=Os[s], lse=ls[s], workspace=ws)
            fb.fedrag_lse_merge(Os, ls, n_kv_heads=Hkv, O_out=Om, lse_out=lm)
            fb.fedrag_unscramble(Om, phi_vi, i["perm_q"], O_out=out)
        replay = _record(step)

        def call():
            replay()
            return out, lm
        return dict(call=call, keep=(i, Qs, Ks, Vs, Os, ls, Om, ws))
    if k == "request":
        Hq, Hkv, d, Lq, n = (c[m] for m in ("Hq", "Hkv", "d", "Lq", "layers"))
        ctx = [int(x) for x in c["ctx"].split(",")]
        Qs, Om, lm, Ol, ll = torch.empty_like(i["Q"][0]), _f32(1, Hq, Lq, d), _f32(1, Hq, Lq), _f32(1, Hq, Lq, d), _f32(1, Hq, Lq)
        out, lse = _f32(n, 1, Hq, Lq, d), _f32(n, 1, Hq, Lq)
        ws = _bytes(fb.fedrag_partial_attn_shards_workspace_bytes(1, Hq, Hkv, d, dt, Lq, ctx))
        wl = _bytes(fb.fedrag_partial_attn_workspace_bytes(1, Hq, Hkv, d, dt, Lq, c["local"]))
        key_q, key_vi = i["keys"][0], i["keys"][3]
        pq, O_plain, l_plain = i["perm_q"], _f32(2, 1, Hq, Lq, d), _f32(2, 1, Hq, Lq)

        def layers():
            for m in range(n):
                (fb.fedrag_scramble_q_structured if c["structured"] else fb.fedrag_scramble_q)(i["Q"][m], key_q, pq, Q_out=Qs)
                fb.fedrag_partial_attn_shards(Qs, [t[m] for t in i["K"]], [t[m] for t in i["V"]], None, O=Om, lse=lm, workspace=ws)
                if c["structured"]:  # Dec by the key's factors, then the aggregation of the two partials
                    fb.fedrag_unscramble_structured(Om, key_vi, pq, O_out=O_plain[0])
                    fb.fedrag_unpermute_lse(lm, pq, lse_out=l_plain[0])
                    fb.fedrag_local_attn(i["Q"][m], i["Kl"][m], i["Vl"][m], None, O_part=O_plain[1], lse=l_plain[1], workspace=wl)
                    fb.fedrag_lse_merge(O_plain, l_plain, n_kv_heads=Hkv, O_out=out[m], lse_out=lse[m])
                else:
                    fb.fedrag_local_attn(i["Q"][m], i["Kl"][m], i["Vl"][m], None, O_part=Ol, lse=ll, workspace=wl)
                    fb.fedrag_unscramble_merge(Om, lm, key_vi, pq, Ol, ll, O_out=out[m], lse_out=lse[m], n_kv_heads=Hkv)
        replay = _record(layers)

        def call():
            replay()
            return out, lse
        return dict(call=call, keep=(i, Qs, Om, lm, Ol, ll, ws, wl, O_plain, l_plain))
    if k == "attn":
        O, lse = _f32(c["B"], c["Hq"], c["Lq"], c["d"]), _f32(c["B"], c["Hq"], c["Lq"])
        if c["S"] == 1:
            ws = _bytes(fb.fedrag_partial_attn_workspace_bytes(c["B"], c["Hq"], c["Hkv"], c["d"], dt, c["Lq"], c["L"]))
            return dict(call=lambda: fb.fedrag_partial_attn(i["Q"], i["K"][0], i["V"][0], None, O_part=O, lse=lse, workspace=ws))
        ws = _bytes(fb.fedrag_partial_attn_shards_workspace_bytes(c["B"], c["Hq"], c["Hkv"], c["d"], dt, c["Lq"], [c["L"]] * c["S"]))
        return dict(call=lambda: fb.fedrag_partial_attn_shards(i["Q"], i["K"], i["V"], None, O=O, lse=lse, workspace=ws))
    if k == "local":
        O, lse = _f32(c["B"], c["Hq"], c["Lq"], c["d"]), _f32(c["B"], c["Hq"], c["Lq"])
        ws = _bytes(fb.fedrag_partial_attn_workspace_bytes(c["B"], c["Hq"], c["Hkv"], c["d"], dt, c["Lq"], c["L"]))
        return dict(call=lambda: fb.fedrag_local_attn(i["Q"], i["K"], i["V"], None, O_part=O, lse=lse, workspace=ws))
    if k == "rerank":
        B, _, L, _ = i["Q"].shape
        O, lse = torch.zeros(i["Q"].shape, device="cuda"), torch.zeros(i["Q"].shape[:3], device="cuda")
        ws = _bytes(fb.fedrag_partial_attn_workspace_bytes(B, c["H"], c["H"], c["d"], dt, L, L))
        if c["bits"] == 0:
            return dict(call=lambda: fb.fedrag_partial_attn_varlen(i["Q"], i["K"], i["V"], i["lens"], None, O_part=O, lse=lse,
                                                                   workspace=ws, q_lens=i["lens"]))
        return dict(call=lambda: fb.fedrag_partial_attn_varlen_quantized(i["Q"], *i["K"], *i["V"], c["bits"], i["lens"], None,
                                                                         O_part=O, lse=lse, workspace=ws, q_lens=i["lens"]))
    if k == "enc":
        _, key_k, key_v, _ = i["keys"]
        B, H, L, d = i["K"].shape
        if c["bits"] == 0:
            out = torch.empty_like(i["K"]), torch.empty_like(i["V"])
            f = fb.fedrag_scramble_kv_structured if c["structured"] else fb.fedrag_scramble_kv
            return dict(call=lambda: f(i["K"], i["V"], key_k, key_v, i["perm"], K_out=out[0], V_out=out[1]))
        codes = lambda: torch.empty((B, H, L, d * c["bits"] // 8), dtype=torch.uint8, device="cuda")  # noqa: E731
        out = codes(), _f32(B, H, L, 2), codes(), _f32(B, H, L, 2)
        return dict(call=lambda: fb.fedrag_scramble_kv_quantized(i["K"], i["V"], key_k, key_v, i["perm"], c["bits"],
                                                                 structured=c["structured"], out=out))
    O, lse = _f32(c["B"], c["Hq"], c["Lq"], c["d"]), _f32(c["B"], c["Hq"], c["Lq"])
    ws = _bytes(fb.fedrag_partial_attn_workspace_bytes(c["B"], c["Hq"], c["Hkv"], c["d"], dt, c["Lq"], c["L"]))
    return dict(call=lambda: fb.fedrag_partial_attn_quantized(i["Q"], *i["K"], *i["V"], c["bits"], None, O_part=O, lse=lse,
                                                              workspace=ws))


def run(state):
    return state["call"]()


# ----------------------------------------------------------------------------------------------- what a pass needs
def work(case):
    """Inputs read once, outputs written once; two flops per multiply-add of every product of the path."""
    c, k = case, case["kind"]
    e = 4 if c["dtype"] == "f32" else 2
    if k == "protocol":
        rq, rk, d = c["B"] * c["Hq"] * c["Lq"], c["B"] * c["Hkv"] * c["S"] * c["L"], c["d"]
        # Enc's outputs are written and attended: the calls are separate
        by = rq * d * (2 * e + 4) + rk * d * 2 * e * 3 + 4 * rq + c["Hkv"] * d * d * (3 * e + 4) + 4 * c["S"] * c["L"]
        return dict(bytes=by, flops=4 * rq * c["S"] * c["L"] * d + 2 * d * d * (2 * rq + 2 * rk))
    if k == "request":
        rq, d = c["Hq"] * c["Lq"], c["d"]
        keys = sum(int(x) for x in c["ctx"].split(","))
        seen = sum(range(c["local"] - c["Lq"] + 1, c["local"] + 1))
        by = rq * (e * d + 4 * d + 4) + (keys + c["local"]) * c["Hkv"] * d * 2 * e
        return dict(bytes=c["layers"] * by, flops=c["layers"] * (4 * d * (rq * keys + c["Hq"] * seen) + 4 * d * d * rq))
    if k in ("attn", "codes"):
        rq, rk, d = c["B"] * c["Hq"] * c["Lq"], c["B"] * c["Hkv"] * c.get("S", 1) * c["L"], c["d"]
        row = 2 * d if k == "attn" else d * c["bits"] // 8 + 8
        return dict(bytes=rq * (e * d + 4 * d + 4) + 2 * rk * row, flops=4 * rq * c.get("S", 1) * c["L"] * d)
    if k == "local":
        rq, rk, d = c["B"] * c["Hq"] * c["Lq"], c["B"] * c["Hkv"] * c["L"], c["d"]
        seen = sum(range(c["L"] - c["Lq"] + 1, c["L"] + 1))
        return dict(bytes=rq * (e * d + 4 * d + 4) + 2 * rk * d * e, flops=4 * d * c["B"] * c["Hq"] * seen)
    if k == "rerank":
        lens, d = [int(x) for x in c["lens"].split(",")], c["d"]
        row = 2 * d if c["bits"] == 0 else d * c["bits"] // 8 + 8
        return dict(bytes=c["H"] * sum(lens) * (e * d + 4 * d + 4 + 2 * row), flops=4 * d * c["H"] * sum(n * n for n in lens))
    rows, d = c["B"] * c["H"] * c["L"] * 2, c["d"]
    return dict(bytes=rows * (d * e + (d * e if c["bits"] == 0 else d * c["bits"] // 8 + 8)) + 4 * c["L"], flops=2 * d * d * rows)


def tolerance(case):
    c, k = case, case["kind"]
    if c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 2e-4}  # fp32 sums in another order, over a chain of four products
    if k == "enc":
        # one rounding to the storage type, a few per cent of the fp32 sums on the other side of a rounding boundary;
        # codes one step apart where a value lies on one
        return {"rel": 2e-3 if c["dtype"] == "bf16" else 3e-4, "max": 0.02, "differ": 0.01}
    if k in ("protocol", "request"):
        # K', V', Q' rounded to 16 bits move the logits of peaked rows (6e-3 .. 4e-2 against 64 bits)
        return {"rel": 2e-2, "max": 0.5}
    if k == "local" or (k in ("attn", "codes") and c["Hq"] // c["Hkv"] * c["Lq"] <= 16):
        return {"rel": 2e-5, "max": 2e-3}  # probabilities carry 16 significant bits or more (1e-6 against 64 bits)
    return {"rel": 2e-3, "max": 0.1}       # probabilities enter the second product in 16 bits (4e-4 against 64 bits)


# ----------------------------------------------------------------------------------------------- in 64 bits
def _attend64(Q, K, V, scale, first_seen=None):
    """(O, lse) of [H, Lq, d] queries on [Hkv, L, d] keys in 64 bits; first_seen: query i sees keys < first_seen + i."""
    Hq, Lq, d = Q.shape
    Hkv, L, _ = K.shape
    O, lse = torch.empty((Hq, Lq, d), dtype=torch.float64, device=Q.device), torch.empty((Hq, Lq), dtype=torch.float64, device=Q.device)
    G = Hq // Hkv
    step = max(1, (1 << 27) // max(1, L))
    for h in range(Hkv):
        q, kt, v = Q[h * G:(h + 1) * G].reshape(G * Lq, d).double(), K[h].double().t().contiguous(), V[h].double()
        for r in range(0, G * Lq, step):
            s = (q[r:r + step] @ kt) * scale
            if first_seen is not None:
                seen = first_seen + torch.arange(r, min(r + step, G * Lq), device=Q.device) % Lq
                s.masked_fill_(torch.arange(L, device=Q.device)[None, :] >= seen[:, None], -math.inf)
            l = torch.logsumexp(s, -1)
            lse.view(Hkv, G * Lq)[h, r:r + step] = l
            O.view(Hkv, G * Lq, d)[h, r:r + step] = torch.exp(s - l[:, None]) @ v
    return O, lse


def _matrix64(key, d):
    """A key as [Hkv, d, d] matrices in 64 bits: dense as given, structured multiplied out."""
    if isinstance(key, torch.Tensor):
        return key.double()
    a, g1, g2, b = key
    idx = torch.arange(d, device=a.device)
    par = torch.zeros((d, d), dtype=torch.long, device=a.device)
    x = idx[:, None] & idx[None, :]
    for s in range(8):
        par += (x >> s) & 1
    had = (1 - 2 * (par & 1)).double() / math.sqrt(d)
    out = []
    for h in range(a.shape[0]):
        eye = torch.eye(d, dtype=torch.float64, device=a.device)
        m = ((eye * a[h].double())[:, g1[h].long()]) @ had
        out.append(m[:, g2[h].long()] * b[h].double())
    return torch.stack(out)


def exact(case, seed):
    c, i, k = case, _inputs(case, seed), case["kind"]
    scale = float(c["d"]) ** -0.5
    if k == "protocol":
        phi_q, phi_k, phi_v, phi_vi = (t.double() for t in i["keys"])
        G, outs, lses = c["Hq"] // c["Hkv"], [], []
        for b in range(c["B"]):
            Q = torch.matmul(i["Q"][b].double(), phi_q.repeat_interleave(G, 0))
            if i["perm_q"] is not None:
                Q = Q[:, i["perm_q"].long()].contiguous()
            K = torch.cat([torch.matmul(t[b].double(), phi_k) for t in i["K"]], 1)  # row order drops out
            V = torch.cat([torch.matmul(t[b].double(), phi_v) for t in i["V"]], 1)
            O, lse = _attend64(Q, K, V, scale)
            O = torch.matmul(O, phi_vi.repeat_interleave(G, 0))
            if i["perm_q"] is not None:
                back = torch.empty_like(O)
                back[:, i["perm_q"].long()] = O
                O = back
            outs.append(O)
            lses.append(lse)
        return torch.stack(outs), torch.stack(lses)
    if k == "request":
        G = c["Hq"] // c["Hkv"]
        mq, mvi = (_matrix64(i["keys"][n], c["d"]).repeat_interleave(G, 0) for n in (0, 3))
        outs, lses = [], []
        for m in range(c["layers"]):
            Q = i["Q"][m][0]
            Qr = torch.matmul(Q.double(), mq)  # the permutation of the query rows is undone by Dec
            O, l = _attend64(Qr, torch.cat([t[m][0] for t in i["K"]], 1), torch.cat([t[m][0] for t in i["V"]], 1), scale)
            O = torch.matmul(O, mvi)
            Ol, ll = _attend64(Q, i["Kl"][m][0], i["Vl"][m][0], scale, c["local"] - c["Lq"] + 1)
            lse = torch.logaddexp(l, ll)
            outs.append((O * torch.exp(l - lse)[..., None] + Ol * torch.exp(ll - lse)[..., None])[None])
            lses.append(lse[None])
        return torch.stack(outs), torch.stack(lses)
    if k == "attn":
        both = [_attend64(i["Q"][b], torch.cat([t[b] for t in i["K"]], 1), torch.cat([t[b] for t in i["V"]], 1), scale)
                for b in range(c["B"])]
        return torch.stack([o for o, _ in both]), torch.stack([l for _, l in both])
    if k == "local":
        both = [_attend64(i["Q"][b], i["K"][b], i["V"][b], scale, c["L"] - c["Lq"] + 1) for b in range(c["B"])]
        return torch.stack([o for o, _ in both]), torch.stack([l for _, l in both])
    if k in ("rerank", "codes"):
        K, V = ((_dequantize64(*i[n], c["bits"], DTYPES[c["dtype"]]) if c["bits"] else i[n]) for n in ("K", "V"))
        if k == "codes":
            both = [_attend64(i["Q"][b], K[b], V[b], scale) for b in range(c["B"])]
            return torch.stack([o for o, _ in both]), torch.stack([l for _, l in both])
        O = torch.zeros(i["Q"].shape, dtype=torch.float64, device="cuda")  # padding rows are not written
        lse = torch.zeros(i["Q"].shape[:3], dtype=torch.float64, device="cuda")
        for b, n in enumerate(i["lens"].tolist()):
            O[b, :, :n], lse[b, :, :n] = _attend64(i["Q"][b, :, :n], K[b, :, :n], V[b, :, :n], scale)
        return O, lse
    outs = []
    for x, key in ((i["K"], i["keys"][1]), (i["V"], i["keys"][2])):
        m = _matrix64(key, c["d"])
        y = torch.stack([torch.matmul(x[b][:, i["perm"].long()].double(), m) for b in range(c["B"])])
        if c["bits"] == 0:
            outs.append(y)
            continue
        y = y.to(DTYPES[c["dtype"]]).double()  # rows are narrowed to the storage type, then quantised
        lo, hi = y.amin(-1, keepdim=True), y.amax(-1, keepdim=True)
        outs += [None, torch.cat([(hi - lo) / (2 ** c["bits"] - 1), lo], -1)]
    return tuple(outs)

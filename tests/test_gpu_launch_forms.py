"""The launch forms of the attention and aggregation kernels at the sizes where they change over or end raggedly:
tiles of query rows and of keys, key runs, shards of one run each, partials per batch.  Against the oracle, with the
bounds of parity.py; what a form must not touch is poisoned."""
import numpy as np
import pytest
import torch

import parity as PT
from paper_2605_25716_amd import binding as fb
from paper_2605_25716_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


def rnd(B, H, L, d, dt, tid, seed=5):
    return W.activations(B, H, L, d, seed=seed, tensor_id=tid, outliers=False, dtype=W.torch_dtype(dt))


# query tiles cover the chip (8 units of 4132 rows): every shard is one run, with a partial of its own
@pytest.mark.parametrize("d,dt,Ls", [(64, "bf16", [64, 1, 65]), (128, "bf16", [63, 0, 128, 40, 129]), (128, "f16", [1]),
                                     (64, "f16", [192, 191, 0])])
def test_shards_of_one_run_each(oracle, d, dt, Ls):
    Q = rnd(1, 32, 1033, d, dt, W.TID_Q)
    Ks = [rnd(1, 8, L, d, dt, W.TID_K + 16 * (i + 1)) for i, L in enumerate(Ls)]
    Vs = [rnd(1, 8, L, d, dt, W.TID_V + 16 * (i + 1)) for i, L in enumerate(Ls)]
    print(f"shards {d} {dt} {Ls}", flush=True)
    O, lse = fb.fedrag_partial_attn_shards(Q.to(DEV), [k.to(DEV) for k in Ks], [v.to(DEV) for v in Vs])
    torch.cuda.synchronize()
    Or, lr = oracle.partial_attn(Q, torch.cat(Ks, dim=2), torch.cat(Vs, dim=2))
    PT.check_attn(O, lse, Or, lr, Q.dtype, f"{d} {dt} {Ls}")


@pytest.mark.parametrize("d,dt,Ls", [(128, "bf16", [192, 63, 300]), (64, "f16", [128, 0, 65, 512])])
def test_weights_between_shards_are_fp32(d, dt, Ls):
    """The weight of a shard's partial is an fp32 number whatever the storage type: the call equals the shards one by one and
    the aggregation of their partials, bit for bit."""
    Q = rnd(1, 32, 1033, d, dt, W.TID_Q).to(DEV)
    Ks = [rnd(1, 8, L, d, dt, W.TID_K + 16 * (i + 1)).to(DEV) for i, L in enumerate(Ls)]
    Vs = [rnd(1, 8, L, d, dt, W.TID_V + 16 * (i + 1)).to(DEV) for i, L in enumerate(Ls)]
    O, lse = fb.fedrag_partial_attn_shards(Q, Ks, Vs)
    parts = [fb.fedrag_partial_attn(Q, k, v) for k, v in zip(Ks, Vs)]
    Om, lm = fb.fedrag_lse_merge(torch.stack([p[0] for p in parts]), torch.stack([p[1] for p in parts]), n_kv_heads=8)
    torch.cuda.synchronize()
    assert torch.equal(O, Om) and torch.equal(lse, lm)


# query tiles of a whole round and more: a workgroup visits the shards one after the other (which form a call takes is held on
# the host, by test_boundary_cpu.py)
IN_TURN = [(1, 32, 128, "bf16", 2048, [70, 64, 0, 1, 200]), (1, 32, 64, "f16", 2048, [128, 65, 500]),
           (2, 32, 128, "f16", 1500, [64, 192]), (1, 64, 64, "bf16", 4096, [1, 1, 63, 129]),
           (1, 32, 128, "bf16", 2048, [1000, 70, 0, 640]), (1, 32, 64, "f16", 2048, [2000, 1500])]  # in eight waves
IN_TURN_ANY_SIZE = [70, 64, 130, 1, 200]
IN_TURN_FAR_BELOW = [70, 64, 130]


@pytest.mark.parametrize("B,Hq,d,dt,Lq,Ls", IN_TURN)
@pytest.mark.parametrize("spread", [0.0, 40.0])
def test_shards_visited_in_turn(B, Hq, d, dt, Lq, Ls, spread):
    """A shard's probabilities are rounded as in a launch of its own and the weight between shards is an fp32 number: the call
    agrees with the shards one by one and the aggregation of their partials to fp32 sums.  Per shard these differ by a factor
    (2^-21: two exponentials of 2^-22) and a rescale per tile (2^-24 each, 56 of them at most) of outputs of at most max |v| <= 6.
    Also with shards whose scores are far apart, so far that a shard weighs nothing, in rising and in falling order."""
    Q = rnd(B, Hq, Lq, d, dt, W.TID_Q).to(DEV)
    Ks = [rnd(B, 8, L, d, dt, W.TID_K + 16 * (i + 1)) for i, L in enumerate(Ls)]
    Vs = [rnd(B, 8, L, d, dt, W.TID_V + 16 * (i + 1)).to(DEV) for i, L in enumerate(Ls)]
    Q[..., 0] = torch.where(torch.arange(Lq, device=DEV) % 2 == 0, 16.0, -16.0).to(Q.dtype)
    for i, k in enumerate(Ks):
        k[..., 0] = spread * i  # scores of +-16 * 40 * i / sqrt(d): hundreds apart
    Ks = [k.to(DEV) for k in Ks]
    print(f"shards in turn {B} {Hq} {d} {dt} {Lq} {Ls} {spread}", flush=True)
    O, lse = fb.fedrag_partial_attn_shards(Q, Ks, Vs)
    parts = [fb.fedrag_partial_attn(Q, k, v) for k, v in zip(Ks, Vs)]
    Om, lm = fb.fedrag_lse_merge(torch.stack([p[0] for p in parts]), torch.stack([p[1] for p in parts]), n_kv_heads=8)
    torch.cuda.synchronize()
    # lse itself is held to 2^-23 of its size by either form, and the weights with it
    tol = 2.0 ** -21 + 56 * 2.0 ** -24 + 2.0 ** -22 * float(lm.abs().max())
    assert float((lse - lm).abs().max()) <= tol
    assert float((O - Om).abs().max()) <= 6.0 * tol


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("size", [1.0, 2.0 ** 40, 2.0 ** 80, 2.0 ** 100, 2.0 ** 118])
def test_shards_visited_in_turn_take_values_of_any_size(d, size):
    """bf16 values far beyond any activation's: where the call with a partial per shard is finite, so is the visiting form, and
    agrees with it as above, whatever the order of the shards' scores.  (Above 2^112 the weight of a shard that lies below another
    rests in the 16 bits of its probabilities, 2^-9 of a weight of at most 2^-1.)"""
    Ls = IN_TURN_ANY_SIZE
    Q = rnd(1, 32, 2048, d, "bf16", W.TID_Q).to(DEV)
    Q[..., 0] = torch.where(torch.arange(2048, device=DEV) % 2 == 0, 16.0, -16.0).to(Q.dtype)
    Q[..., 1] = torch.where(torch.arange(2048, device=DEV) % 4 < 2, 16.0, 0.0).to(Q.dtype)
    Ks = [rnd(1, 8, L, d, "bf16", W.TID_K + 16 * (i + 1)) for i, L in enumerate(Ls)]
    Vs = [(rnd(1, 8, L, d, "f32", W.TID_V + 16 * (i + 1)) * size).to(torch.bfloat16).to(DEV) for i, L in enumerate(Ls)]
    for i, k in enumerate(Ks):
        k[..., 0] = 20.0 * i         # rising, falling
        k[..., 1] = 60.0 * (i % 2)   # and up and down for every other pair of rows
    Ks = [k.to(DEV) for k in Ks]
    print(f"values of any size {d} {size}", flush=True)
    O, lse = fb.fedrag_partial_attn_shards(Q, Ks, Vs)
    parts = [fb.fedrag_partial_attn(Q, k, v) for k, v in zip(Ks, Vs)]
    Om, lm = fb.fedrag_lse_merge(torch.stack([p[0] for p in parts]), torch.stack([p[1] for p in parts]), n_kv_heads=8)
    torch.cuda.synchronize()
    assert torch.isfinite(Om).all() and torch.isfinite(O).all()
    tol = 2.0 ** -21 + 2.0 ** -19 + 2.0 ** -22 * float(lm.abs().max())
    assert float((lse - lm).abs().max()) <= tol
    assert float((O / size - Om / size).abs().max()) <= 6.0 * (tol if size < 2.0 ** 112 else 2.0 ** -9)


@pytest.mark.parametrize("d", [128, 64])
def test_a_shard_far_below_leaves_the_log_sum_exp_exact(d):
    """A first shard with a log-sum-exp of order one and others far below it: their weight is nothing, and what the visit does to
    the running maximum must not be seen either.  Maximum and logarithm of the sum are below 2^5 in base 2, so either form rounds
    their sum by 2^-20 and what it makes of it by 2^-22 a step."""
    Ls = IN_TURN_FAR_BELOW
    Q = (rnd(1, 32, 2048, d, "f32", W.TID_Q) * 0.25).to(torch.bfloat16).to(DEV)
    Q[..., 0] = 16.0
    Ks = [rnd(1, 8, L, d, "bf16", W.TID_K + 16 * (i + 1)) for i, L in enumerate(Ls)]
    Vs = [rnd(1, 8, L, d, "bf16", W.TID_V + 16 * (i + 1)).to(DEV) for i, L in enumerate(Ls)]
    for i, k in enumerate(Ks):
        k[..., 0] = -60.0 * (i > 0)
    Ks = [k.to(DEV) for k in Ks]
    print(f"shards far below {d}", flush=True)
    O, lse = fb.fedrag_partial_attn_shards(Q, Ks, Vs)
    parts = [fb.fedrag_partial_attn(Q, k, v) for k, v in zip(Ks, Vs)]
    Om, lm = fb.fedrag_lse_merge(torch.stack([p[0] for p in parts]), torch.stack([p[1] for p in parts]), n_kv_heads=8)
    torch.cuda.synchronize()
    assert float(lm.abs().max()) < 16.0
    assert float((lse - lm).abs().max()) <= 3 * 2.0 ** -20


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("height", [64.0, 1024.0, 8192.0, 16384.0, 2.0 ** 20])
def test_a_shard_far_below_leaves_the_weights_of_the_others(d, height):
    """Two shards of the same keys and, between them, one far below: each of the two has half the weight, also where scores are so
    large (height squared, 10^5 to 10^11 after scaling) that fp32 cannot hold a step of the maximum down and back."""
    L = 70
    Q = torch.zeros((1, 32, 2048, d), dtype=torch.bfloat16, device=DEV)
    Q[..., 0] = height
    K = torch.zeros((1, 8, L, d), dtype=torch.bfloat16, device=DEV)
    K[..., 0] = height
    Ks = [K, K * (1 - 2.0 ** -7), K] if height > 100.0 else [K, K * 0.5, K]
    Vs = [rnd(1, 8, L, d, "bf16", W.TID_V + 16 * (i + 1)).to(DEV) for i in range(3)]
    print(f"between two equal shards {d} {height}", flush=True)
    O, lse = fb.fedrag_partial_attn_shards(Q, Ks, Vs)
    parts = [fb.fedrag_partial_attn(Q, k, v) for k, v in zip(Ks, Vs)]
    torch.cuda.synchronize()
    # 3 tiles: outputs of at most 6, a rescale and a sum of 2^-24 each, 2^-22 an exponential
    assert float((O - 0.5 * (parts[0][0] + parts[2][0])).abs().max()) <= 6.0 * 2.0 ** -19
    assert float((lse - parts[0][1] - np.log(2.0)).abs().max()) <= 2.0 ** -19 + 2.0 ** -22 * float(parts[0][1].abs().max())


def test_every_shard_boundary_keeps_its_keys():
    """One key tile of one shard holds all the weight of a query row: a tile lost or read twice at a shard's end moves that
    row's log-sum-exp by ln 2 or more."""
    d, L, S, Lq = 128, 256, 3, 1024
    tile = torch.arange(L) // 64
    Q = torch.nn.functional.one_hot(torch.arange(Lq) % 4, d).to(torch.bfloat16).expand(1, 32, Lq, d).contiguous().to(DEV)
    hot = (torch.nn.functional.one_hot(tile, d) * 226.0).to(torch.bfloat16).expand(1, 8, L, d).contiguous().to(DEV)
    zero = torch.zeros_like(hot)
    expect = np.log(64 * np.exp(226.0 / np.sqrt(d)) + (S * L - 64))
    for which in range(S):
        _, lse = fb.fedrag_partial_attn_shards(Q, [hot if s == which else zero for s in range(S)], [zero] * S)
        torch.cuda.synchronize()
        assert float((lse.double() - expect).abs().max()) <= PT.TOL_16_LSE_ABS, which


# key tiles are visited first to last: odd and even counts, with and without a ragged one; 8- and 4-wave workgroups
@pytest.mark.parametrize("d,dt,Lq,tiles,tail", [(128, "bf16", 512, 5, 0), (128, "bf16", 40, 6, 1), (64, "bf16", 300, 3, 63),
                                                (64, "f16", 512, 4, 30), (128, "f16", 100, 2, 0), (64, "bf16", 512, 8, 2)])
@pytest.mark.parametrize("form", ["plain", "lengths"])
def test_keys_that_raise_the_maximum_are_exact(d, dt, Lq, tiles, tail, form):
    """One key per tile carries the weight and each has a higher score than the one before: it is the row's maximum when
    its tile is visited, so its probability is exactly 1 and what is left are fp32 rescales.  In another order the lower
    ones would be rounded to the storage type (2^-9 or 2^-12 of their weight)."""
    L = 64 * tiles + tail
    Q = torch.zeros(1, 32, Lq, d)
    Q[..., 0] = 16.0
    K = torch.zeros(1, 8, L, d)
    K[..., 0] = -300.0
    hot = [min(64 * t + (37 * t) % 64, L - 1) for t in range((L + 63) // 64)]
    K[:, :, hot, 0] = torch.arange(len(hot)) * 0.3
    K, V = K.to(W.torch_dtype(dt)), rnd(1, 8, L, d, dt, W.TID_V)
    Qd, Kd, Vd = Q.to(W.torch_dtype(dt)).to(DEV), K.to(DEV), V.to(DEV)
    if form == "plain":
        O, _ = fb.fedrag_partial_attn(Qd, Kd, Vd, 1.0 / 16.0)
    else:
        O, _ = fb.fedrag_partial_attn_varlen(Qd, Kd, Vd, torch.tensor([L], dtype=torch.int32, device=DEV), 1.0 / 16.0)
    torch.cuda.synchronize()
    p = torch.softmax(K[..., 0].double(), -1)  # [1, 8, L]
    want = (p[..., None] * V.double()).sum(2)  # [1, 8, d]
    # one fp32 exponential (2^-22) and rescale per tile of a weighted mean of |v| <= 5
    assert float((O.cpu().double() - want.repeat_interleave(4, 1)[:, :, None]).abs().max()) <= 1e-5


# 128-row tiles and 64-key tiles of the masked form; the last two launches are one past the fold of the tile order
@pytest.mark.parametrize("B,Hq,d,Lq,L,dt", [(1, 4, 128, 128, 128, "bf16"), (1, 4, 128, 129, 129, "bf16"),
                                            (1, 2, 128, 127, 191, "f16"), (1, 4, 64, 65, 130, "bf16"),
                                            (2, 4, 64, 257, 300, "f16"), (1, 4, 128, 2, 64, "bf16"),
                                            (1, 4, 128, 640, 640, "bf16"), (4, 32, 64, 515, 515, "bf16"),
                                            (4, 32, 128, 520, 583, "bf16")])
def test_masked_tiles(oracle, B, Hq, d, Lq, L, dt):
    Hkv = max(2, Hq // 4)
    Q, K, V = rnd(B, Hq, Lq, d, dt, W.TID_Q), rnd(B, Hkv, L, d, dt, W.TID_K), rnd(B, Hkv, L, d, dt, W.TID_V)
    print(f"local {B} {Hq} {d} {Lq} {L} {dt}", flush=True)
    O, lse = fb.fedrag_local_attn(Q.to(DEV), K.to(DEV), V.to(DEV))
    torch.cuda.synchronize()
    Or, lr = oracle.local_causal_attn(Q, K, V)
    PT.check_attn(O, lse, Or, lr, Q.dtype, f"local {Lq} of {L}")


# fp32: 16 query rows per workgroup, 32 where there are more and those cover the chip (last three cases); 16-key tiles over
# 8, 4, 2 or 1 waves, by the number of workgroups and of tiles
@pytest.mark.parametrize("B,Hq,Hkv,d,Lq,L", [(1, 2, 2, 64, 16, 1), (1, 2, 2, 128, 17, 15), (1, 4, 2, 128, 8, 16),
                                             (2, 4, 1, 64, 5, 127), (1, 2, 1, 128, 3, 128), (1, 2, 2, 64, 33, 129),
                                             (1, 8, 2, 128, 1, 513), (1, 2, 2, 64, 5, 20), (1, 4, 2, 128, 3, 50),
                                             (1, 2, 2, 64, 3, 65), (128, 8, 8, 64, 1, 40), (64, 8, 8, 128, 1, 90),
                                             (257, 8, 8, 64, 2, 5), (256, 8, 8, 128, 1, 4), (256, 8, 8, 128, 1, 21),
                                             (33, 8, 8, 128, 40, 60), (4, 8, 8, 64, 250, 70), (4, 8, 8, 128, 256, 33)])
def test_fp32_tiles(oracle, B, Hq, Hkv, d, Lq, L):
    Q, K, V = (rnd(B, h, n, d, "f32", t) for h, n, t in ((Hq, Lq, W.TID_Q), (Hkv, L, W.TID_K), (Hkv, L, W.TID_V)))
    print(f"f32 {B} {Hq} {Hkv} {d} {Lq} {L}", flush=True)
    O, lse = fb.fedrag_partial_attn(Q.to(DEV), K.to(DEV), V.to(DEV))
    O2, lse2 = fb.fedrag_partial_attn_shards(Q.to(DEV), [K[:, :, :L // 2].contiguous().to(DEV), K[:, :, L // 2:].contiguous().to(DEV)],
                                             [V[:, :, :L // 2].contiguous().to(DEV), V[:, :, L // 2:].contiguous().to(DEV)])
    torch.cuda.synchronize()
    Or, lr = oracle.partial_attn(Q, K, V)
    PT.check_attn(O, lse, Or, lr, torch.float32, "plain")
    PT.check_attn(O2, lse2, Or, lr, torch.float32, "two shards")
    if L >= Lq:
        O, lse = fb.fedrag_local_attn(Q.to(DEV), K.to(DEV), V.to(DEV))
        torch.cuda.synchronize()
        Or, lr = oracle.local_causal_attn(Q, K, V)
        PT.check_attn(O, lse, Or, lr, torch.float32, "masked")


@pytest.mark.parametrize("B,H,d,Lq,L", [(3, 2, 64, 70, 90), (128, 16, 128, 40, 17), (64, 8, 64, 33, 50)])
def test_fp32_padding_rows(oracle, B, H, d, Lq, L):
    """Per-sequence counts in fp32: whole tiles of padding rows, partly filled ones and sequences without rows or keys; what is
    padding is neither read nor written."""
    Q, K, V = (rnd(B, H, n, d, "f32", t) for n, t in ((Lq, W.TID_Q), (L, W.TID_K), (L, W.TID_V)))
    ql = torch.tensor([(7 * b + 1) % (Lq + 1) for b in range(B)], dtype=torch.int32)
    kl = torch.tensor([(5 * b + L) % (L + 1) for b in range(B)], dtype=torch.int32)
    O, lse = torch.full((B, H, Lq, d), -7.0, device=DEV), torch.full((B, H, Lq), -7.0, device=DEV)
    Kp, Vp = K.clone(), V.clone()
    for b in range(B):
        Kp[b, :, kl[b]:], Vp[b, :, kl[b]:] = float("nan"), float("inf")
    fb.fedrag_partial_attn_varlen(Q.to(DEV), Kp.to(DEV), Vp.to(DEV), kl.to(DEV), None, O_part=O, lse=lse, q_lens=ql.to(DEV))
    torch.cuda.synchronize()
    for b in sorted({0, 1, 2, B // 2, B - 1}):
        q, k = int(ql[b]), int(kl[b])
        assert bool((O[b, :, q:] == -7.0).all()) and bool((lse[b, :, q:] == -7.0).all())
        if q:
            Or, lr = oracle.partial_attn(Q[b:b + 1, :, :q].contiguous(), K[b:b + 1, :, :k].contiguous(), V[b:b + 1, :, :k].contiguous())
            PT.check_attn(O[b:b + 1, :, :q], lse[b:b + 1, :, :q], Or, lr, torch.float32, f"sequence {b}: {q} of {k}")


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_fp32_rows_do_not_see_a_later_token(oracle, bad):
    """A token whose K, V are not finite leaves the rows before it as they are (0 x inf must not reach them)."""
    Q, K, V = (rnd(1, h, 40, 64, "f32", t) for h, t in ((4, W.TID_Q), (2, W.TID_K), (2, W.TID_V)))
    Or, lr = oracle.local_causal_attn(Q, K, V)
    K[:, :, 21], V[:, :, 21] = bad, bad
    O, lse = fb.fedrag_local_attn(Q.to(DEV), K.to(DEV), V.to(DEV))
    torch.cuda.synchronize()
    PT.check_attn(O[:, :, :21], lse[:, :, :21], Or[:, :, :21], lr[:, :, :21], torch.float32, "rows before the token")


@pytest.mark.parametrize("S", [1, 2, 3, 4, 5, 8, 9, 16, 17, 33])
@pytest.mark.parametrize("rows,d", [(3, 128), (5, 64), (2500, 128), (8300, 64)])  # the more rows the fewer partials in flight
def test_aggregation_of_many_partials(oracle, S, rows, d):
    g = torch.Generator().manual_seed(S * 100 + rows)
    O, lse = torch.randn((S, 1, 1, rows, d), generator=g), torch.randn((S, 1, 1, rows), generator=g) * 30
    lse[S // 2, 0, 0, ::3] = float("-inf")
    lse[:, 0, 0, 1] = float("-inf")
    Or, lr = oracle.lse_merge(O, lse)
    O[lse == float("-inf")] = float("nan")  # a partial without weight takes no part, whatever it holds
    got, got_l = fb.fedrag_lse_merge(O.to(DEV), lse.to(DEV))
    torch.cuda.synchronize()
    assert PT.max_abs(got, Or) <= 1e-4 and PT.max_abs(got_l, lr) <= 1e-4


@pytest.mark.parametrize("S", [2, 16, 33])
def test_aggregation_of_partials_without_a_number(S):
    """A row whose log-sum-exps are all NaN has no weight, like one where all are -inf, whatever the number of partials."""
    O, lse = torch.ones((S, 1, 1, 3, 64)), torch.zeros((S, 1, 1, 3))
    lse[:, 0, 0, 1] = float("nan")
    got, got_l = fb.fedrag_lse_merge(O.to(DEV), lse.to(DEV))
    torch.cuda.synchronize()
    assert bool((got[0, 0, 1] == 0).all()) and float(got_l[0, 0, 1]) == float("-inf")
    assert bool((got[0, 0, ::2] == 1).all())


# one run up to 512 keys, 256-key runs up to 2048 in all where those are one round, 512-key runs otherwise
@pytest.mark.parametrize("Ls", [[31], [512], [513], [2047], [2049], [400, 700], [300, 0, 213], [9000]])
@pytest.mark.parametrize("d", [64, 128])
def test_decode_key_runs(oracle, Ls, d):
    Q = rnd(1, 8, 1, d, "bf16", W.TID_Q)
    Ks = [rnd(1, 2, L, d, "bf16", W.TID_K + 16 * (i + 1)) for i, L in enumerate(Ls)]
    Vs = [rnd(1, 2, L, d, "bf16", W.TID_V + 16 * (i + 1)) for i, L in enumerate(Ls)]
    O, lse = fb.fedrag_partial_attn_shards(Q.to(DEV), [k.to(DEV) for k in Ks], [v.to(DEV) for v in Vs])
    torch.cuda.synchronize()
    Or, lr = oracle.partial_attn(Q, torch.cat(Ks, dim=2), torch.cat(Vs, dim=2))
    PT.check_attn(O, lse, Or, lr, Q.dtype, str(Ls))


# 8 B workgroups: one tile of LDS per wave (runs of up to 128 keys; up to 1024, of 64 columns 256, with more workgroups than compute
# units, or of 128 columns from 385 on where they fill one round), also on eight waves (129 to 256 keys of 128) and on two (up to
# 64), two, and registers (whole rounds of runs from 2048 keys on); a wave's one to nine tiles, whole and ragged
@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("B,L,d", [(1, 1, 128), (2, 128, 64), (1, 129, 128), (2, 255, 128), (4, 256, 128), (1, 257, 128), (3, 353, 64), (3, 511, 128), (33, 200, 128), (33, 1000, 128),
                                   (40, 256, 64), (40, 257, 64), (1, 1, 64), (2, 32, 64), (3, 33, 64), (40, 64, 64), (300, 63, 64), (3, 65, 64), (3, 32, 128), (40, 63, 128), (300, 5, 128), (32, 385, 128), (30, 511, 128), (33, 1100, 128), (32, 2113, 128), (33, 2050, 128), (32, 2100, 64)])
def test_decode_tile_forms(oracle, B, L, d, dt):
    Q, K, V = rnd(B, 16, 1, d, dt, W.TID_Q), rnd(B, 8, L, d, dt, W.TID_K), rnd(B, 8, L, d, dt, W.TID_V)
    lens = torch.tensor([(L * (b + 1) // B) if b else 0 for b in range(B)], dtype=torch.int32)
    for kv_lens in (None, lens):
        if kv_lens is None:
            Or, lr = oracle.partial_attn(Q, K, V)
            O, lse = fb.fedrag_partial_attn(Q.to(DEV), K.to(DEV), V.to(DEV))
        else:
            Or, lr = oracle.partial_attn_varlen(Q, K, V, kv_lens)
            for b in range(B):  # what lies past a sequence's keys is not looked at
                K[b, :, int(lens[b]):], V[b, :, int(lens[b]):] = float("nan"), float("inf")
            O, lse = fb.fedrag_partial_attn_varlen(Q.to(DEV), K.to(DEV), V.to(DEV), kv_lens.to(DEV))
        torch.cuda.synchronize()
        PT.check_attn(O, lse, Or, lr, Q.dtype, f"{B} {L} {d}")


# launches cut into fewer, longer runs than planned, which are summed in parts (that they are cut is held on the host, by
# test_boundary_cpu.py): two tiles of LDS per wave, registers, codes; several shards; one part, two, and a ragged end
CUT_ANEW = [(9, 128, 0, [2001]), (9, 64, 0, [2300]), (31, 128, 0, [2100]), (5, 128, 0, [4001, 3277, 300]), (9, 64, 0, [700, 1300]),
            (17, 128, 0, [1025]), (11, 128, 8, [2048]), (17, 128, 8, [600]), (17, 128, 4, [3000]), (20, 128, 4, [1023])]


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("B,d,bits,Ls", CUT_ANEW)
def test_decode_launches_cut_anew(oracle, B, d, bits, Ls, dt):
    print(f"cut anew {B} {d} {bits} {Ls} {dt}", flush=True)
    Q = rnd(B, 16, 1, d, dt, W.TID_Q)
    Ks = [rnd(B, 8, L, d, dt, W.TID_K + 16 * (i + 1)) for i, L in enumerate(Ls)]
    Vs = [rnd(B, 8, L, d, dt, W.TID_V + 16 * (i + 1)) for i, L in enumerate(Ls)]
    Qd, Kd, Vd = Q.to(DEV), [k.to(DEV) for k in Ks], [v.to(DEV) for v in Vs]
    if bits:
        codes = fb.fedrag_quantize_rows(Kd[0], bits) + fb.fedrag_quantize_rows(Vd[0], bits)
        Ks, Vs = ([fb.fedrag_dequantize_rows(c, p, bits, Q.dtype).cpu()] for c, p in (codes[:2], codes[2:]))
        O, lse = fb.fedrag_partial_attn_quantized(Qd, *codes, bits)
    else:
        O, lse = fb.fedrag_partial_attn_shards(Qd, Kd, Vd)
    torch.cuda.synchronize()
    Or, lr = oracle.partial_attn(Q, torch.cat(Ks, dim=2), torch.cat(Vs, dim=2))
    PT.check_attn(O, lse, Or, lr, Q.dtype, f"{B} {Ls}")
    if len(Ls) > 1:
        return
    lens = torch.tensor([(Ls[0] * (b + 1) // B) if b else 0 for b in range(B)], dtype=torch.int32)
    Or, lr = oracle.partial_attn_varlen(Q, Ks[0], Vs[0], lens)
    if bits:
        O, lse = fb.fedrag_partial_attn_varlen_quantized(Qd, *codes, bits, lens.to(DEV))
    else:
        O, lse = fb.fedrag_partial_attn_varlen(Qd, Kd[0], Vd[0], lens.to(DEV))
    torch.cuda.synchronize()
    PT.check_attn(O, lse, Or, lr, Q.dtype, f"{B} {Ls} padded")


def test_longer_runs_keep_the_error_of_the_plan():
    """A batch of 16 takes two runs of 10000 keys a sequence, one of 17 a single run: it is summed in two parts, so the same
    sequences come out with the same error against 64 bits (in one go it was 1.17 times that; the two differ by some 3 % in either
    direction by where a part ends)."""
    g = torch.Generator(device=DEV).manual_seed(4)
    Q, K, V = (torch.randn((17, h, n, 128), generator=g, device=DEV).half() for h, n in ((32, 2), (8, 20000), (8, 20000)))
    S = torch.matmul(Q[:3].double().view(3, 8, 8, 128), K[:3].double().transpose(2, 3).contiguous()) / np.sqrt(128)
    ref, ref_l = torch.matmul(torch.softmax(S, -1), V[:3].double()).view(3, 32, 2, 128), torch.logsumexp(S, -1).view(3, 32, 2)
    err = []
    for B in (16, 17):
        O, lse = fb.fedrag_partial_attn(Q[:B].contiguous(), K[:B].contiguous(), V[:B].contiguous())
        err.append((float((O[:3] - ref).norm() / ref.norm()), float((lse[:3] - ref_l).norm() / ref_l.norm())))
    torch.cuda.synchronize()
    print(err, flush=True)
    assert err[1][0] <= 1.06 * err[0][0] and err[1][1] <= 1.5 * err[0][1], err


@pytest.mark.parametrize("bits", [0, 8])
@pytest.mark.parametrize("B,L", [(17, 8192), (31, 8192)])
def test_longer_runs_keep_the_range_of_the_plan(B, L, bits):
    """8192 equal scores, values of 1.5 x 2^115: 4096 of them fit fp32, a sum of all would not."""
    Q, K = torch.zeros((B, 8, 1, 128), dtype=torch.bfloat16, device=DEV), rnd(1, 8, L, 128, "bf16", W.TID_K).to(DEV).repeat(B, 1, 1, 1)
    V = torch.full((B, 8, L, 128), 1.5 * 2.0 ** 115, dtype=torch.bfloat16, device=DEV)
    if bits:
        O, lse = fb.fedrag_partial_attn_quantized(Q, *fb.fedrag_quantize_rows(K, bits), *fb.fedrag_quantize_rows(V, bits), bits)
    else:
        O, lse = fb.fedrag_partial_attn(Q, K, V)
    torch.cuda.synchronize()
    assert float((O.double() / (1.5 * 2.0 ** 115) - 1).abs().max()) <= 1e-5  # 64 additions of a tile's sum and the fold
    assert float((lse.double() - np.log(L)).abs().max()) <= 1e-5


@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_decode_on_4bit_codes_of_every_scale(dt):
    """Rows of every magnitude, tiny, ordinary and (bf16) beyond 2^100, rebuild to what fedrag_dequantize_rows gives: with one
    key per sequence the output is that row of V' itself."""
    B, d = 24, 128
    V = rnd(B, 1, 1, d, "f32", W.TID_V)
    e = torch.linspace(-14.0, 14.0, B) if dt == "f16" else torch.linspace(-120.0, 124.0, B)
    V = (V.clamp(-3, 3) * torch.exp2(e).view(B, 1, 1, 1)).to(W.torch_dtype(dt)).to(DEV)
    K = rnd(B, 1, 1, d, dt, W.TID_K).to(DEV)
    Kc, Kp = fb.fedrag_quantize_rows(K, 4)
    Vc, Vp = fb.fedrag_quantize_rows(V, 4)
    ref = fb.fedrag_dequantize_rows(Vc, Vp, 4, V.dtype).float()
    O, _ = fb.fedrag_partial_attn_quantized(rnd(B, 2, 1, d, dt, W.TID_Q).to(DEV), Kc, Kp, Vc, Vp, 4)
    torch.cuda.synchronize()
    # the probability is 1, exactly representable; fp32 division by a denominator of 1
    assert torch.equal(O, ref.expand(B, 2, 1, d))


@pytest.mark.parametrize("bits", [8, 4, 0])
def test_decode_rounds_the_exponent_once(bits):
    """Scores around 960, exact in fp32: rounding score x scale before the maximum is taken off would leave up to 2^-14 in the
    exponent, 4e-5 of a probability, the same for all keys of a score.  What is left otherwise, times a mean |v| of 0.8: the
    exponential (2^-22) and two fp16 terms of probabilities >= e^-3.75 (2^-25 absolute from subnormals)."""
    L, d = 1024, 128
    K = torch.zeros(1, 1, L, d)
    K[..., 0], K[..., 1] = 60.0, 4.0 * (torch.arange(L) * 7 % 16)  # rows of range 60: 4- (8-) bit codes are exact
    Q = torch.zeros(1, 4, 1, d)
    Q[..., 0], Q[..., 1] = 16.0, 0.0625
    V = rnd(1, 1, 16, d, "f16", W.TID_V)[:, :, torch.arange(L) * 7 % 16]  # one value per score
    Q, K, V = Q.half().to(DEV), K.half().to(DEV), V.contiguous().to(DEV)
    if bits:
        Vc, Vp = fb.fedrag_quantize_rows(V, bits)
        V = fb.fedrag_dequantize_rows(Vc, Vp, bits, V.dtype)
        O, _ = fb.fedrag_partial_attn_quantized(Q, *fb.fedrag_quantize_rows(K, bits), Vc, Vp, bits, 1.0)
    else:
        O, _ = fb.fedrag_partial_attn(Q, K, V, 1.0)
    torch.cuda.synchronize()
    p = torch.softmax(960.0 + K[0, 0, :, 1].double() / 16.0, 0)
    err = float((O[0].double() - (p[:, None] * V[0, 0].double()).sum(0)).abs().max())
    print(f"bits {bits}: {err:.2e}")
    assert err <= 1e-6


@pytest.mark.parametrize("B,H,L", [(2, 3, 1), (2, 3, 64), (2, 3, 65), (2, 3, 256), (2, 3, 300), (700, 5, 3), (4097, 3, 1)])
def test_lse_scatter(B, H, L):
    lse = torch.randn((B, H, L))
    perm = torch.randperm(L, generator=torch.Generator().manual_seed(L)).to(torch.int32)
    out = fb.fedrag_unpermute_lse(lse.to(DEV), perm.to(DEV)).cpu()
    assert torch.equal(out[:, :, perm.long()], lse)


def test_lse_scatter_of_many_rows():
    """2^26 rows and more of one value each, which a workgroup per row could not launch."""
    lse = torch.randn((1 << 21, 33, 1), device=DEV)
    out = fb.fedrag_unpermute_lse(lse, torch.zeros(1, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    assert torch.equal(out, lse)


@pytest.mark.parametrize("B,Hkv,G,Lq,L,d", [
    (1, 8, 2, 300, 300, 128), (1, 9, 2, 300, 300, 128), (3, 3, 3, 129, 200, 64), (2, 8, 4, 1024, 1024, 64),  # together
    (64, 64, 1, 64, 64, 64), (65, 64, 1, 64, 64, 64), (5, 821, 1, 40, 64, 64)])  # 8 MiB of keys an XCD, and beyond
def test_masked_batches_reach_every_tile_of_every_unit(oracle, B, Hkv, G, Lq, L, d):
    """The order in which the tiles of several units are handed out must not show: the outputs, filled with NaN before, are
    those of the sequences one by one, and the last sequence matches the oracle."""
    g = torch.Generator().manual_seed(B * Hkv + Lq)
    Q, K, V = (torch.randn(s, generator=g).to(torch.bfloat16) for s in ((B, Hkv * G, Lq, d), (B, Hkv, L, d), (B, Hkv, L, d)))
    O = torch.full((B, Hkv * G, Lq, d), float("nan"), device=DEV)
    lse = torch.full((B, Hkv * G, Lq), float("nan"), device=DEV)
    Qd, Kd, Vd = Q.to(DEV), K.to(DEV), V.to(DEV)
    fb.fedrag_local_attn(Qd, Kd, Vd, O_part=O, lse=lse)
    for b in range(B):
        Ob, lb = fb.fedrag_local_attn(Qd[b:b + 1], Kd[b:b + 1], Vd[b:b + 1])
        assert torch.equal(O[b:b + 1], Ob) and torch.equal(lse[b:b + 1], lb), b
    heads = slice(0, min(Hkv, 16) * G)
    Or, lr = oracle.local_causal_attn(Q[-1:, heads], K[-1:, :min(Hkv, 16)], V[-1:, :min(Hkv, 16)])
    PT.check_attn(O[-1:, heads], lse[-1:, heads], Or, lr, torch.bfloat16, f"masked batch {B}x{Hkv}x{G} {Lq}/{L}", report=True)


@pytest.mark.parametrize("L", [1, 2, 7, 8, 9, 16, 17, 32, 33, 65])  # at most 16 rows a head have a kernel of their own
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("structured", [False, True])
def test_few_rows(L, d, structured):
    """A handful of rows per head, every storage type, gathered and scattered, several sequences, and the few more that the tiled
    kernels begin with: fp32 sums of d products (d + 2 roundings of 2^-24 of the sum of the terms' sizes at most), narrowed once."""
    B, Hkv, G = 3, 2, 2
    H = Hkv * G
    g = torch.Generator().manual_seed(100 * L + d)
    perm = torch.randperm(L, generator=g).to(torch.int32)
    for dt in ("f32", "bf16", "f16"):
        dtype = W.torch_dtype(dt)
        x = torch.randn((B, H, L, d), generator=g).to(dtype)
        if structured:
            key = W.make_structured_keys(Hkv, d, L, 64, 1, seed=d + L, dtype=dtype).q
            a, g1, g2, b = (t.double() if t.is_floating_point() else t.long() for t in key)
            had = torch.from_numpy(W.sylvester_hadamard(d)).double()
            had /= had[0, 0] * np.sqrt(d)
            m = torch.stack([((torch.eye(d, dtype=torch.float64) * a[h])[:, g1[h]] @ had)[:, g2[h]] * b[h] for h in range(Hkv)])
            key = tuple(t.to(DEV) for t in key)
        else:
            m = torch.randn((Hkv, d, d), generator=g).to(dtype)
            key, m = m.to(DEV), m.double()
        m = m.repeat_interleave(G, 0)
        want, size = x.double() @ m, x.double().abs() @ m.abs()
        tol = size * (d + 4) * 2.0 ** -24 + want.abs() * {"f32": 0.0, "bf16": 2.0 ** -8, "f16": 2.0 ** -11}[dt] + 1e-7
        print(f"few rows {L} {d} {structured} {dt}", flush=True)
        got = (fb.fedrag_scramble_q_structured if structured else fb.fedrag_scramble_q)(x.to(DEV), key, perm.to(DEV)).cpu()
        assert ((got.double() - want[:, :, perm.long()]).abs() <= tol[:, :, perm.long()]).all(), dt
        if dt == "f32":  # Dec: the same rows scattered
            got = (fb.fedrag_unscramble_structured if structured else fb.fedrag_unscramble)(x.to(DEV), key, perm.to(DEV)).cpu()
            assert ((got.double()[:, :, perm.long()] - want).abs() <= tol).all()


# few workgroups: two groups of four waves share 128 query rows and halve their keys
TWO_GROUPS = [(1, 32, 128, "bf16", 500, [960]), (1, 32, 128, "f16", 500, [1000]),
              (1, 32, 64, "bf16", 109, [1732, 6100, 30]), (2, 16, 64, "f16", 958, [513]),
              (2, 16, 128, "f16", 30, [569, 0, 718, 7521]), (2, 16, 128, "bf16", 958, [769])]


@pytest.mark.parametrize("B,Hq,d,dt,Lq,Ls", TWO_GROUPS)
def test_keys_halved_between_two_groups(oracle, B, Hq, d, dt, Lq, Ls):
    """Runs of an odd number of tiles, ragged ones and, beside long shards, one so short that the second group has no key; with
    and without partials."""
    Q = rnd(B, Hq, Lq, d, dt, W.TID_Q)
    Ks = [rnd(B, 8, L, d, dt, W.TID_K + 16 * (i + 1)) for i, L in enumerate(Ls)]
    Vs = [rnd(B, 8, L, d, dt, W.TID_V + 16 * (i + 1)) for i, L in enumerate(Ls)]
    Or, lr = oracle.partial_attn(Q, torch.cat(Ks, dim=2), torch.cat(Vs, dim=2))
    print(f"two groups {B} {Hq} {d} {dt} {Lq} {Ls}", flush=True)
    O = torch.full(Or.shape, float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full(lr.shape, float("nan"), dtype=torch.float32, device=DEV)
    if len(Ls) > 1:
        O, lse = fb.fedrag_partial_attn_shards(Q.to(DEV), [k.to(DEV) for k in Ks], [v.to(DEV) for v in Vs], O=O, lse=lse)
    else:
        fb.fedrag_partial_attn(Q.to(DEV), Ks[0].to(DEV), Vs[0].to(DEV), O_part=O, lse=lse)
    torch.cuda.synchronize()
    PT.check_attn(O, lse, Or, lr, Q.dtype, f"{B} {Hq} {d} {dt} {Lq} {Ls}")

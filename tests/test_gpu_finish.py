"""GPU parity of fedrag_unscramble_merge: Dec of the remote result plus the aggregation with the Inquirer's own
partial (Sections 4.2 and 4.1) against the oracle's stages, and bit for bit against the three separate calls."""
import numpy as np
import pytest
import torch

import parity as PT
from paper_2605_25716_amd import binding as fb
from paper_2605_25716_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("B,Hq,Hkv,d,Lq,permute", [(2, 8, 2, 128, 1, False), (1, 4, 2, 128, 77, True),
                                                   (2, 4, 4, 64, 40, True), (1, 32, 8, 128, 128, True)])
def test_unscramble_merge(oracle, B, Hq, Hkv, d, Lq, permute):
    keys = W.make_keys(Hkv, d, Lq, 64, 1, seed=4242 + Lq, dtype=torch.float32, permute_q=permute)
    g = torch.Generator().manual_seed(99 + Lq)
    O_scr = torch.randn((B, Hq, Lq, d), generator=g)
    O_loc = torch.randn((B, Hq, Lq, d), generator=g)
    l_scr = 3.0 * torch.randn((B, Hq, Lq), generator=g)
    l_loc = 3.0 * torch.randn((B, Hq, Lq), generator=g)
    # degenerate rows: no remote keys, no local keys, neither (their outputs are never read: poison them)
    flat_s, flat_l = l_scr.view(-1), l_loc.view(-1)
    n = flat_s.numel()
    if n >= 4:
        flat_s[0] = -np.inf
        O_scr.view(-1, d)[0] = float("nan")
        flat_l[1] = -np.inf
        O_loc.view(-1, d)[1] = float("nan")
    perm = keys.perm_q
    if n >= 4 and perm is None:
        flat_s[2] = -np.inf
        flat_l[2] = -np.inf
    dv = lambda t: None if t is None else t.to(DEV)
    O, lse = fb.fedrag_unscramble_merge(dv(O_scr), dv(l_scr), dv(keys.phi_v_inv), dv(perm), dv(O_loc), dv(l_loc))
    # the three calls
    O1 = fb.fedrag_unscramble(dv(O_scr), dv(keys.phi_v_inv), dv(perm))
    l1 = fb.fedrag_unpermute_lse(dv(l_scr), dv(perm))
    O3, l3 = fb.fedrag_lse_merge(torch.stack([O1, dv(O_loc)]), torch.stack([l1, dv(l_loc)]), n_kv_heads=Hkv)
    torch.cuda.synchronize()
    assert torch.equal(torch.nan_to_num(O, nan=7.0), torch.nan_to_num(O3, nan=7.0)) and torch.equal(lse, l3)
    # the oracle's stages on the same inputs (poisoned rows replaced: the oracle multiplies before it weighs)
    Os = torch.nan_to_num(O_scr, nan=0.0)
    Ol = torch.nan_to_num(O_loc, nan=0.0)
    Ou = oracle.unscramble(Os, keys.phi_v_inv, perm)
    lu = np.empty((B, Hq, Lq))
    p = np.arange(Lq) if perm is None else perm.numpy()
    lu[:, :, p] = l_scr.double().numpy()
    Or, lr = oracle.lse_merge(np.stack([Ou, Ol.double().numpy()]), np.stack([lu, l_loc.double().numpy()]))
    assert PT.rel_normwise(O, Or) <= PT.TOL_F32_REL
    assert PT.rel_normwise(lse, lr) <= PT.TOL_F32_REL


@pytest.mark.parametrize("Lq", [2, 3, 4, 8, 15, 16, 17, 31, 32, 33, 64, 65, 129])
@pytest.mark.parametrize("d", [64, 128])
def test_unscramble_merge_at_the_edges_of_its_kernels(d, Lq):
    """At most 16 rows, at most 32 of 64 columns, one and several row tiles: the values of the three calls bit for bit, with rows
    that lack the first partial, the second and both throughout (what they hold is never read: poisoned)."""
    B, Hq, Hkv = 3, 4, 2
    keys = W.make_keys(Hkv, d, Lq, 64, 1, seed=17 + Lq, dtype=torch.float32)
    g = torch.Generator().manual_seed(100 * Lq + d)
    O_scr, O_loc = (torch.randn((B, Hq, Lq, d), generator=g) for _ in range(2))
    l_scr, l_loc = (3.0 * torch.randn((B, Hq, Lq), generator=g) for _ in range(2))
    perm = torch.randperm(Lq, generator=g).to(torch.int32)
    row = torch.arange(Lq) + torch.arange(B * Hq).view(B, Hq, 1)  # another phase in every slab
    no_loc = (row % 4 == 1) | (row % 4 == 2)
    no_scr = ((row % 4 == 0) | (row % 4 == 2))[:, :, perm.long()]
    l_loc[no_loc], O_loc[no_loc] = -np.inf, float("nan")
    l_scr[no_scr], O_scr[no_scr] = -np.inf, float("nan")
    dv = lambda t: t.to(DEV)  # noqa: E731
    print(f"unscramble_merge {d} {Lq}", flush=True)
    for p in (perm, None):
        pd = None if p is None else dv(p)
        O, lse = fb.fedrag_unscramble_merge(dv(O_scr), dv(l_scr), dv(keys.phi_v_inv), pd, dv(O_loc), dv(l_loc))
        O1 = fb.fedrag_unscramble(dv(O_scr), dv(keys.phi_v_inv), pd)
        l1 = fb.fedrag_unpermute_lse(dv(l_scr), pd)
        O3, l3 = fb.fedrag_lse_merge(torch.stack([O1, dv(O_loc)]), torch.stack([l1, dv(l_loc)]), n_kv_heads=Hkv)
        torch.cuda.synchronize()
        assert torch.isfinite(O3).all()
        assert torch.equal(O.view(torch.int32), O3.view(torch.int32)) and torch.equal(lse, l3)


@pytest.mark.parametrize("rows", [1, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dt", ["bf16", "f16", "f32"])
def test_few_rows_of_few_and_of_many_slabs(oracle, dt, d, rows):
    """Columns split over two or four workgroups, or not, by the rows and by the slabs (up to 128 and more): sums in the same
    order, so the values of a sequence bit for bit in a batch of 33, and those of the oracle."""
    B, Hq, Hkv = 33, 4, 2
    dtype = W.torch_dtype(dt)
    keys = W.make_keys(Hkv, d, rows, 64, 1, seed=rows + d, dtype=dtype)
    X = W.activations(B, Hq, rows, d, seed=5, tensor_id=W.TID_Q, outliers=False, dtype=dtype)
    O, other = X.float() * 0.5, X.float().flip(0).contiguous()
    la, lb = O[..., 0].contiguous(), other[..., 1].contiguous()
    perm = torch.randperm(rows, generator=torch.Generator().manual_seed(rows)).to(torch.int32)
    print(f"few rows {dt} {d} {rows}", flush=True)
    dv = lambda t: t.to(DEV)  # noqa: E731

    def calls(b):
        s = slice(0, b)
        out = [fb.fedrag_scramble_q(dv(X[s]), dv(keys.phi_q), dv(perm)), fb.fedrag_unscramble(dv(O[s]), dv(keys.phi_v_inv), dv(perm))]
        return out + list(fb.fedrag_unscramble_merge(dv(O[s]), dv(la[s]), dv(keys.phi_v_inv), dv(perm), dv(other[s]), dv(lb[s])))

    one, many = calls(1), calls(B)
    torch.cuda.synchronize()
    for a, b in zip(one, many):
        assert torch.equal(a, b[:1])
    PT.check_scramble(many[0], oracle.scramble(X, keys.phi_q, perm), X, keys.phi_q, perm, Hq // Hkv, dtype, "Q'")
    dec = oracle.unscramble(O, keys.phi_v_inv, perm)
    assert PT.rel_normwise(many[1], dec) <= PT.TOL_F32_REL
    moved = torch.empty_like(la)
    moved[:, :, perm.long()] = la
    Or, lr = oracle.lse_merge(np.stack([dec, other.double().numpy()]), np.stack([moved.double().numpy(), lb.double().numpy()]))
    assert PT.rel_normwise(many[2], Or) <= PT.TOL_F32_REL and PT.rel_normwise(many[3], lr) <= PT.TOL_F32_REL

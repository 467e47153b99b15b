"""The router's weight gradients of renormalised gates, dense product and
segment sums (the choice falls at 8 slots per 64 experts and at sizes of x),
against plain float64, at the edges of their tiles; an infinite token touches only the rows of
the experts it is routed to."""
import numpy as np
import pytest
import torch

import paper_2601_14327_amd as laep
from _gpu import TOL_F32, case, host, rownorm_err

pytestmark = pytest.mark.gpu


def _inputs(T, E, k, d, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((T, d), generator=g, device="cuda").to(dtype)
    wr = (0.05 * torch.randn((E, d), generator=g, device="cuda")).to(dtype)
    idx, gate = laep.moe_route(x, wr, k)[:2]
    _, off, _, src = laep.moe_expert_counts(idx, E, want_row_src=True)
    dg = torch.randn((T, k), generator=g, device="cuda")
    return x, wr, idx, gate, off, src, dg


def _dw(x, wr, idx, gate, off, src, dg):
    _, dw, db, dl = laep.moe_route_bwd(dg, idx, gate, x, wr, offsets=off, row_src=src, data=False,
                                       want_dbias=True, want_dlogits=True)
    torch.cuda.synchronize()
    return dw, db, dl


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T,E,k,d", [
    (1, 8, 2, 64),          # one token
    (65, 64, 8, 136),       # one token past a split's two steps, d % 128 = 8
    (300, 65, 5, 128),      # dense by 16 k, one expert past a tile
    (300, 128, 8, 264),     # dense, two expert tiles
    (300, 130, 8, 264),     # segments
    (257, 65, 1, 128),      # segments
    (40, 200, 100, 64),     # more than 64 slots, dense
])
def test_weights(T, E, k, d, dtype):
    case(f"router renorm weights T={T} E={E} k={k} d={d} {dtype}")
    x, wr, idx, gate, off, src, dg = a = _inputs(T, E, k, d, dtype, 3 * T + E)
    dw, db, dl = _dw(*a)
    g, q = gate.double(), dg.double()
    dls = g * (q - (g * q).sum(1, keepdim=True))
    full = torch.zeros((T, E), dtype=torch.float64, device="cuda").scatter_(1, idx.long(), dls)
    # fp32 sums of at most 300 terms
    cond = (full.abs().t() @ x.double().abs()).clamp_min(1e-30)
    assert ((dw.double() - full.t() @ x.double()).abs() <= TOL_F32 * cond).all()
    assert rownorm_err(host(dl), host(full)) <= TOL_F32
    assert ((db.double() - full.sum(0)).abs() <= TOL_F32 * full.abs().sum(0) + 1e-30).all()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("T,E,k,d", [
    (24000, 64, 2, 1024),   # segments for x of 49 MB and more
    (5900, 64, 1, 1024),    # bf16 12.1 MB: segments, 11.9 MB: dense
    (5800, 64, 1, 1024),
])
def test_weights_past_the_size_of_x(T, E, k, d, dtype):
    """Against float64 on the call's own logit gradients."""
    case(f"router renorm weights by size T={T} E={E} k={k} d={d} {dtype}")
    a = _inputs(T, E, k, d, dtype, T)
    if k == 1:   # (its gradient is 0: other gates than the softmax's)
        a[3].copy_(torch.rand((T, k), device="cuda") + 0.05)
    dw, db, dl = _dw(*a)
    full, x = dl.double(), a[0].double()
    # fp32 sums of 128 rows (segments) or up to 768 tokens (splits, most of them 0),
    # then of their partial sums: about 160 roundings of 6e-8
    cond = (full.abs().t() @ x.abs()).clamp_min(1e-30)
    assert ((dw.double() - full.t() @ x).abs() <= TOL_F32 * cond).all()
    assert ((db.double() - full.sum(0)).abs() <= TOL_F32 * full.abs().sum(0) + 1e-30).all()


@pytest.mark.parametrize("T,k", [(1, 1), (300, 1), (65, 2), (1000, 3), (33, 8), (257, 13),
                                 (70, 64), (40, 65)])
def test_slots_alone(T, k):
    """Without the dense rows (several tokens share a wave, up to 64 slots) the
    slots' gradients, seen through dx, keep their bits; unrouted slots among them."""
    E, d = 128, 64
    case(f"router renorm slots T={T} k={k}")
    x, wr, idx, gate, _, _, dg = _inputs(T, E, k, d, torch.float32, 7 * T + k)
    if k > 2:
        idx[T // 2, k - 2:], gate[T // 2, k - 2:] = -1, 0.0
        dg[T // 2, k - 1] = float("nan")   # not read
    _, off, _, src = laep.moe_expert_counts(idx, E, want_row_src=True)
    kw = dict(offsets=off, row_src=src, weights=False)
    a = laep.moe_route_bwd(dg, idx, gate, x, wr, **kw)[0]
    b, _, _, dl = laep.moe_route_bwd(dg, idx, gate, x, wr, want_dlogits=True, **kw)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert rownorm_err(host(a), host(dl.double() @ wr.double())) <= TOL_F32


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("E,k", [(64, 4), (130, 4),
                                 (64, 1), (130, 1)])   # one slot: dl is 0, and 0 * inf NaN
def test_infinite_token(E, k, bad):
    T, d = 200, 136
    case(f"router renorm weights, token with {bad} E={E}")
    x, wr, idx, gate, off, src, dg = _inputs(T, E, k, d, torch.bfloat16, E)
    t, c = 131, 77
    xz, xb = x.clone(), x.clone()
    xz[t, c], xb[t, c] = 0.0, bad
    ref = _dw(xz, wr, idx, gate, off, src, dg)[0]
    got = _dw(xb, wr, idx, gate, off, src, dg)[0]
    hit = torch.zeros(E, dtype=torch.bool, device="cuda")
    hit[idx[t].long()] = True
    assert not torch.isfinite(got[hit, c]).any()
    ok = torch.ones_like(ref, dtype=torch.bool)
    ok[hit, c] = False
    assert torch.equal(got[ok], ref[ok])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("E,k", [(64, 4), (130, 4)])
def test_several_infinite_tokens(E, k, dtype):
    """Two and three tokens of one expert in one split, of both signs and NaN: the
    expert's sums are what they are in token order, every bit the same each time."""
    T, d = 640, 264
    case(f"router renorm weights, several non-finite tokens E={E} {dtype}")
    x, wr, idx, gate, off, src, dg = _inputs(T, E, k, d, dtype, E + 1)
    e = int(idx[300, 0])
    toks = (idx == e).any(1).nonzero().flatten()[:3].tolist()
    assert len(toks) == 3
    cols = {5: [float("inf"), float("inf")], 130: [float("inf"), float("-inf")],
            261: [float("-inf"), float("nan"), float("inf")]}
    xz, xb = x.clone(), x.clone()
    hit = torch.zeros((E, d), dtype=torch.bool, device="cuda")
    for c, vals in cols.items():
        for t, v in zip(toks, vals):
            xz[t, c], xb[t, c] = 0.0, v
            hit[idx[t].long(), c] = True
    ref = _dw(xz, wr, idx, gate, off, src, dg)[0]
    got, _, dl = _dw(xb, wr, idx, gate, off, src, dg)
    for _ in range(4):
        again = _dw(xb, wr, idx, gate, off, src, dg)[0]
        assert torch.equal(got.view(torch.int32), again.view(torch.int32))
    assert torch.equal(got[~hit], ref[~hit])
    for m, c in hit.nonzero().tolist():
        rows = (idx == m).any(1)
        want = (dl[rows, m] * xb[rows, c].float()).sum().item()   # inf, -inf or NaN in any order
        assert str(got[m, c].item()) == str(want)

"""Calls of so many rows that a grid of one thread per element would pass HIP's
limit of 2^32 threads per dimension."""
import pytest
import torch

import paper_2601_14327_amd as laep
from _gpu import TOL_F32, case, host, rownorm_err

pytestmark = pytest.mark.gpu


def test_f32_ffn_with_capacity_for_2_to_the_23_rows():
    """16384 M elements each way: the activations' capacity, of which offsets uses
    the first and the last rows of the experts below."""
    R, E, d, f = 1 << 23, 2, 2048, 64
    n = 70
    case(f"f32 FFN R={R} d={d} f={f}, {n} rows")
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.empty((R, d), dtype=torch.float32, device="cuda")
    y = torch.empty_like(x)
    x[:n] = torch.randn((n, d), generator=g, device="cuda")
    y[:n + 1] = 7.0
    wgu = 0.05 * torch.randn((E, 2 * f, d), generator=g, device="cuda")
    wd = 0.05 * torch.randn((E, d, f), generator=g, device="cuda")
    off = torch.tensor([0, 3, n], dtype=torch.int32, device="cuda")
    laep.moe_grouped_ffn_fwd(x, wgu, wd, off, save_act=False, y_perm=y)
    torch.cuda.synchronize()
    for e, (a, b) in enumerate([(0, 3), (3, n)]):
        p = x[a:b].double() @ wgu[e].double().t()
        h = torch.nn.functional.silu(p[:, :f]) * p[:, f:]
        assert rownorm_err(host(y[a:b]), host(h @ wd[e].double().t())) <= TOL_F32
    assert (y[n] == 7.0).all()
    del x, y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("renorm", [True, False])
def test_router_weight_gradients_of_2_to_the_26_tokens(renorm):
    T, E, k, d = 1 << 26, 2, 1, 8
    case(f"router backward, weights only T={T} E={E} d={d} renorm={renorm}")
    x = torch.zeros((T, d), dtype=torch.bfloat16, device="cuda")
    idx = torch.zeros((T, k), dtype=torch.int32, device="cuda")
    gate = torch.ones((T, k), device="cuda")
    dg = torch.zeros((T, k), device="cuda")
    logits = torch.zeros((T, E), device="cuda")
    off = torch.tensor([0, T, T], dtype=torch.int32, device="cuda")
    src = torch.arange(T, dtype=torch.int32, device="cuda")
    # the last tokens carry a gradient: full softmax p = 1/2, gate 1/2
    gate[-3:] = 0.5
    dg[-3:] = 4.0
    x[-3:] = 1.0
    wr = torch.zeros((E, d), dtype=torch.bfloat16, device="cuda")
    _, dw, db, dl = laep.moe_route_bwd(dg, idx, gate, x, wr, renorm=renorm,
                                       logits=None if renorm else logits, offsets=off,
                                       row_src=src, data=False, want_dbias=True,
                                       want_dlogits=True)
    torch.cuda.synchronize()
    # s = g dg = 2; renorm: g (dg - s) = 1; full: p (q - s) = 1 and -1
    want = [1.0, 0.0] if renorm else [1.0, -1.0]
    assert dl[-3:].tolist() == [want] * 3 and not dl[:-3].any()
    assert db.tolist() == [3 * w for w in want]
    assert dw.tolist() == [[3 * w] * d for w in want]
    torch.cuda.empty_cache()

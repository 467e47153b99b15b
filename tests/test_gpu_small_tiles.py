"""The forward products for few rows per expert (32-, 64- and 128-row tiles)
at the edges of their tiles, against the oracle and, bit for bit, against the
256-row kernels on the same rows."""
import numpy as np
import pytest
import torch

import oracle.moe as om
import paper_2601_14327_amd as laep
from workloads import random_case
from _gpu import TOL_BF16, case, dev, host, rownorm_err

pytestmark = pytest.mark.gpu

BF = torch.bfloat16


def _run(form, x, wgu, wd, counts, ids, E, d):
    idx = dev(ids.reshape(-1, 1).astype(np.int32), torch.int32)
    _, offsets, dest, src = laep.moe_expert_counts(idx, E, want_row_src=True)
    if form == "rows":
        return laep.moe_grouped_ffn_fwd(laep.moe_permute(x, dest, 1), wgu, wd, offsets)
    if form == "gather":
        return laep.moe_grouped_ffn_fwd_gather(x, src, 1, wgu, wd, offsets, save_act=True)
    g = torch.full((x.shape[0], 1), 0.5, device=x.device)
    out, y, a = laep.moe_grouped_ffn_fwd_gather_combine(x, src, g, wgu, wd, offsets, keep_y=True,
                                                        save_act=True)
    assert torch.equal(out, laep.moe_combine(y, g, dest))
    return y, a


@pytest.mark.parametrize("form", ["rows", "gather", "combine"])
@pytest.mark.parametrize("bm,E,d,f", [
    (32, 48, 320, 192),    # average below 24 rows; d % 128 = 64, f % 128 = 64
    (64, 48, 320, 192),
    (128, 48, 320, 192),
    (32, 6, 64, 64),       # a one-step k-loop in both products
    (64, 200, 128, 64),
])
def test_small_tiles(bm, E, d, f, form):
    edges = [0, 1, bm - 1, bm, bm + 1, 2 * bm + 1]
    counts = (edges + [max(1, bm // 2)] * E)[:E]
    rng = np.random.default_rng(bm + E)
    ids = rng.permutation(np.repeat(np.arange(E), counts))
    heavy = 256 * 260      # one expert more, enough rows that the 256-row kernels run
    c = random_case(17 + bm, T=len(ids), d_model=d, E=E + 1, k=1, d_ff=f, dtype="bf16")
    wgu, wd = dev(c["w_gate_up"], BF), dev(c["w_down"], BF)
    x = dev(c["x"], BF)
    case(f"small tiles bm={bm} E={E} d={d} f={f} {form}")
    y, a = _run(form, x, wgu, wd, counts, ids, E, d)
    torch.cuda.synchronize()
    R = len(ids)
    order = np.argsort(ids, kind="stable")
    offsets = np.r_[0, np.cumsum(counts)]
    ry, ra = om.grouped_ffn_fwd(c["x"][order], c["w_gate_up"][:E], c["w_down"][:E], offsets,
                                dtype="bf16")
    assert rownorm_err(host(y), ry) <= TOL_BF16
    assert rownorm_err(host(a), ra) <= TOL_BF16
    # the same rows beside the heavy expert
    xb = torch.cat([x, x[:1].expand(heavy, d)]).contiguous()
    yb, ab = _run("rows", xb, wgu, wd, None, np.r_[ids, np.full(heavy, E)], E + 1, d)
    torch.cuda.synchronize()
    assert torch.equal(y, yb[:R])
    assert torch.equal(a, ab[:R])

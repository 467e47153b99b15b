"""The backward FFN products at the edges of their k-loops: reductions of one,
two, three and six k-steps, row tiles with 0 to 4 valid 32-row blocks per wave
row, slot counts whose division is exact and not, the last expert's rows ending
inside a k-step.  Against the oracle, dY given and formed on load."""
import numpy as np
import pytest
import torch

import oracle.moe as om
import paper_2601_14327_amd as laep
from workloads import random_case
from _gpu import TOL_BF16, TOL_F32, case, dev, host, rownorm_err

pytestmark = pytest.mark.gpu

BF = torch.bfloat16


@pytest.mark.parametrize("k", [1, 3, 7])
@pytest.mark.parametrize("d,f", [(64, 64), (128, 192), (384, 64)])
def test_backward_kloop_edges(d, f, k):
    counts = [0, 1, 31, 33, 63, 65, 127, 129, 193, 225, 257, 420]
    E = len(counts)
    rng = np.random.default_rng(d + f + k)
    # slots counted one by one (a token may hold an expert twice): the FFN calls
    # take the token of routed row r as row_src[r] / k
    ids = rng.permutation(np.repeat(np.arange(E), counts)).astype(np.int32)
    R = len(ids) // k * k
    T = R // k
    c = random_case(d + k, T=T, d_model=d, E=E, k=1, d_ff=f, dtype="bf16")
    x, wgu, wd = dev(c["x"], BF), dev(c["w_gate_up"], BF), dev(c["w_down"], BF)
    gate_h = rng.uniform(0.05, 1.0, (T, k)).astype(np.float32)
    dout_h = rng.standard_normal((T, d)).astype(np.float32)
    gate, dout = dev(gate_h, torch.float32), dev(dout_h, BF)
    _, offsets, dest, src = laep.moe_expert_counts(dev(ids[:R].reshape(R, 1), torch.int32), E,
                                                      want_row_src=True)
    case(f"k-loop edges T={T} k={k} d={d} f={f}")
    xp = laep.moe_permute(x, dest, k)
    ws = torch.empty(laep.workspace_bytes(laep.LAEP_CALL_FFN_FWD, R, 1, E, d, f),
                     dtype=torch.uint8, device="cuda")
    y, act = laep.moe_grouped_ffn_fwd(xp, wgu, wd, offsets, ws=ws, save_act=True)
    h = laep.ffn_fwd_h_view(ws, R, f, BF)
    dy, _ = laep.moe_combine_bwd(dout, y, gate, dest)
    given = laep.moe_grouped_ffn_bwd_gather(dy, x, src, k, act, wgu, wd, offsets, h_fwd=h,
                                            return_ws=True)
    on_load = laep.moe_grouped_ffn_bwd_gather(None, x, src, k, act, wgu, wd, offsets, dout=dout,
                                              topk_gate=gate, h_fwd=h)
    torch.cuda.synchronize()
    for name, a, b in zip(("dx_perm", "dw_gate_up", "dw_down"), given, on_load):
        assert torch.equal(a, b), name
    # against the oracle, on the GPU's own intermediate tensors
    dA, dH = (host(t) for t in laep.ffn_bwd_ws_views(given[3], R, f, BF))
    off = host(offsets).astype(int)
    rgu, rdd = om.grouped_ffn_wgrad(host(dy), host(xp), dA, host(h), off, E)
    gu, dd = host(given[1]), host(given[2])
    dyh, wgu_h, wd_h, dx = host(dy), host(wgu), host(wd), host(given[0])
    for e in range(E):
        rows = slice(off[e], off[e + 1])
        assert rownorm_err(gu[e], rgu[e]) <= TOL_F32, e
        assert rownorm_err(dd[e], rdd[e]) <= TOL_F32, e
        if off[e + 1] > off[e]:
            ref = dyh[rows].astype(np.float64) @ wd_h[e].astype(np.float64)
            assert rownorm_err(dH[rows], ref) <= TOL_BF16, e
            ref = dA[rows].astype(np.float64) @ wgu_h[e].astype(np.float64)
            assert rownorm_err(dx[rows], ref) <= TOL_BF16, e

"""Every row-tile height of the bf16 forward (32, 64, 128: csrc/gemm_small.hip;
256: csrc/gemm_bf16.hip) at the edges of its tiles: plain rows, gathered rows
(through an expert map) and the scatter to token rows, against the oracle and bit
for bit against each other and against another height on the same rows.  A last, large expert brings the
call to the height, which is asserted."""
import numpy as np
import pytest
import torch

import oracle.moe as om
import paper_2601_14327_amd as laep
from workloads import random_case
from _gpu import TOL_BF16, case, dev, host, rownorm_err

pytestmark = pytest.mark.gpu

BF = torch.bfloat16
# 0 to 4 valid 32-row blocks in each wave row of a 256-row tile, and every
# height's rows less one, exactly, one more and two tiles and one
EDGES = [0, 1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 193, 225, 255, 256, 257, 420, 513]


def _rows_for(bm, least, E, d, f, k):
    """A row count of at least `least` (a multiple of k) that takes height bm."""
    R = -(-least // k) * k
    while laep.laep_ffn_fwd_row_tile(R, E, d, f) != bm:
        R += -(-max(1, R // 50) // k) * k
        assert R < 1 << 20, f"no size takes {bm}-row tiles"
    return R


def _offsets(R):
    return dev(np.r_[0, np.cumsum(EDGES), R].astype(np.int32), torch.int32)


@pytest.mark.parametrize("k", [1, 3])
@pytest.mark.parametrize("d,f", [
    (64, 64),     # a one-step k-loop in both products
    (128, 192),   # two and three steps; f % 128 = 64
    (320, 192),   # d % 256 = d % 128 = 64
    (192, 320),
])
@pytest.mark.parametrize("bm", [32, 64, 128, 256])
def test_row_tiles(bm, d, f, k):
    E, n = len(EDGES) + 1, sum(EDGES)
    c = random_case(d + f, T=8, d_model=d, E=E, k=1, d_ff=f, dtype="bf16")
    wgu, wd = dev(c["w_gate_up"], BF), dev(c["w_down"], BF)
    R = _rows_for(bm, n + 300, E, d, f, k)
    assert laep.laep_ffn_fwd_row_tile(R, E, d, f) == bm
    T, off = R // k, _offsets(R)
    g = torch.Generator(device="cuda").manual_seed(bm + d)
    x = torch.randn((T, d), generator=g, device="cuda").to(BF)
    src = torch.randperm(R, generator=g, device="cuda").int()   # slot of each routed row
    dest = torch.empty_like(src)
    dest[src.long()] = torch.arange(R, dtype=torch.int32, device="cuda")
    case(f"forward row tiles bm={bm} d={d} f={f} k={k} R={R}")
    xp = x[(src // k).long()].contiguous()
    y, act = laep.moe_grouped_ffn_fwd(xp, wgu, wd, off, save_act=True)
    y0, none = laep.moe_grouped_ffn_fwd(xp, wgu, wd, off, save_act=False)
    # (gathered: the experts' weights in slots of another order)
    emap = torch.arange(E - 1, -1, -1, dtype=torch.int32, device="cuda")
    yg, actg = laep.moe_grouped_ffn_fwd_gather(x, src, k, wgu.flip(0), wd.flip(0), off, rows=R,
                                               expert_map=emap, save_act=True)
    pairs = [("y without act", y0, y), ("y gathered", yg, y), ("act gathered", actg, act)]
    if k == 1:
        gate = torch.rand((T, 1), device="cuda") + 0.05
        out, yc, actc = laep.moe_grouped_ffn_fwd_gather_combine(x, src, gate, wgu, wd, off,
                                                                keep_y=True, save_act=True)
        bare = laep.moe_grouped_ffn_fwd_gather_combine(x, src, gate, wgu, wd, off)[0]
        ref = laep.moe_combine(y, gate, dest)
        pairs += [("y scatter", yc, y), ("act scatter", actc, act), ("out", out, ref),
                  ("out alone", bare, ref)]
    # the same edge rows through another height
    other = 256 if bm != 256 else 64
    R2 = _rows_for(other, n + 300, E, d, f, 1)
    assert laep.laep_ffn_fwd_row_tile(R2, E, d, f) == other
    rest = torch.randn((R2 - n, d), generator=g, device="cuda").to(BF)
    y2, act2 = laep.moe_grouped_ffn_fwd(torch.cat([xp[:n], rest]), wgu, wd, _offsets(R2),
                                        save_act=True)
    torch.cuda.synchronize()
    assert none is None
    pairs += [(f"y of {other}-row tiles", y2[:n], y[:n]),
              (f"act of {other}-row tiles", act2[:n], act[:n])]
    for name, a, b in pairs:
        assert torch.equal(a, b), name
    # the oracle on the edge experts and on rows of the last one (rows are independent)
    last = np.r_[np.arange(n), n + np.arange(40), R - 1 - np.arange(40)]
    rows = np.r_[0, np.cumsum(EDGES), n + 80]
    ry, ra = om.grouped_ffn_fwd(host(xp)[last], c["w_gate_up"], c["w_down"], rows, dtype="bf16")
    assert rownorm_err(host(y)[last], ry) <= TOL_BF16
    assert rownorm_err(host(act)[last], ra) <= TOL_BF16

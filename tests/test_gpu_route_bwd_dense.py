"""The router backward of full-softmax gates at the edges of its tiles (64
tokens or experts x 128 columns, 32 k a step, token splits) against the oracle."""
import numpy as np
import pytest
import torch

import oracle.moe as om
import paper_2601_14327_amd as laep
from workloads import random_case
from _gpu import TOL_BF16, TOL_F32, case, dev, host, rownorm_err

pytestmark = pytest.mark.gpu

TD = {"bf16": torch.bfloat16, "f32": torch.float32}


@pytest.mark.parametrize("T,d,E,k,dtype,dead", [
    (1, 8, 1, 1, "f32", 0),            # one of everything
    (63, 136, 65, 3, "bf16", 2),       # a tile less one, E and d one vector over
    (65, 128, 64, 64, "f32", 0),       # every expert selected
    (129, 72, 45, 8, "bf16", 5),       # E odd: unaligned dl rows
    (2500, 264, 256, 8, "bf16", 0),    # several splits, the last one short
    (1000, 1024, 33, 2, "f32", 1),
    (3200, 72, 8, 2, "bf16", 1),       # dx by rows: 8 experts, 400 tokens each
    (3199, 72, 8, 2, "bf16", 1),       # and dense
    (3700, 136, 9, 2, "f32", 0),
    (900, 136, 2, 1, "f32", 1),        # by rows, one expert left
    (257, 64, 32, 8, "bf16", 3),       # 32, 20 (of 32) and 3 (of 4) lanes a token
    (501, 64, 20, 20, "f32", 2),
    (101, 64, 3, 1, "f32", 0),
])
def test_dense_route_bwd(T, d, E, k, dtype, dead):
    td = TD[dtype]
    c = random_case(T + 3 * E, T=T, d_model=d, E=E, k=k, d_ff=64, dtype=dtype, bias_std=0.5)
    rng = np.random.default_rng(E)
    alive = np.ones(E, bool)
    alive[rng.choice(E, dead, replace=False)] = False
    a = dev(alive.astype(np.uint8), torch.uint8) if dead else None
    x, b = dev(c["x"], td), dev(c["bias"], torch.float32)
    wr = dev(c["w_router"], td)
    wr[torch.from_numpy(~alive).to(wr.device)] = float("nan")   # a pruned row may hold anything
    case(f"dense route bwd T={T} d={d} E={E} k={k} {dtype} dead={dead}")
    idx, gate, logits = laep.moe_route(x, wr, k, bias=b, alive=a, renorm=False, want_logits=True)
    dg = dev(rng.standard_normal((T, k)).astype(np.float32), torch.float32)
    base = dev(rng.standard_normal((T, d)).astype(np.float32), td)
    kw = dict(renorm=False, logits=logits, alive=a, want_dlogits=True, want_dbias=True)
    for acc in (False, True):
        dx0 = base.clone() if acc else torch.full_like(base, float("nan"))
        dx, dw, db, dl = laep.moe_route_bwd(dg, idx, gate, x, wr, dx=dx0, accumulate_dx=acc, **kw)
        torch.cuda.synchronize()
        rl, rw, rb, rx = om.route_bwd(host(dg), host(idx), host(gate), c["x"], c["w_router"],
                                      logits=host(logits), alive=alive if dead else None,
                                      renorm=False, dtype=dtype,
                                      dx_in=host(base) if acc else np.zeros((T, d)))
        assert rownorm_err(host(dl), rl) <= TOL_F32
        assert rownorm_err(host(dw), rw) <= TOL_F32
        assert rownorm_err(host(db), rb) <= TOL_F32
        assert rownorm_err(host(dx), rx) <= (TOL_BF16 if dtype == "bf16" else TOL_F32)


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("T,d,E,k,dtype", [(200, 136, 70, 4, "bf16"), (65, 264, 33, 2, "f32")])
def test_probability_zero_keeps_nonfinite_rows_out_of_dx(T, d, E, k, dtype, bad):
    """An expert whose logit is -inf for a token has dl = 0 there: its row of W_r,
    whatever it holds, does not reach that token's dx; elsewhere it does."""
    td = TD[dtype]
    case(f"dense route bwd, non-finite W_r T={T} d={d} E={E} k={k} {dtype} {bad}")
    g = torch.Generator(device="cuda").manual_seed(T + E)
    x = torch.randn((T, d), generator=g, device="cuda").to(td)
    wr = (0.05 * torch.randn((E, d), generator=g, device="cuda")).to(td)
    logits = torch.randn((T, E), generator=g, device="cuda")
    nowhere, some, c = E // 3, E - 1, d - 7
    logits[:, nowhere] = -float("inf")
    logits[: T // 2, some] = -float("inf")
    p = torch.softmax(logits, 1)
    gate, idx = torch.topk(p, k, dim=1)
    dg = torch.randn((T, k), generator=g, device="cuda")
    base = torch.randn((T, d), generator=g, device="cuda").to(td)
    wz, wb = wr.clone(), wr.clone()
    wz[nowhere], wb[nowhere] = 0.0, bad
    wz[some, c], wb[some, c] = 0.0, bad
    for acc in (False, True):
        ref, got = (laep.moe_route_bwd(dg, idx.int().contiguous(), gate.contiguous(), x, w,
                                       renorm=False, logits=logits, dx=base.clone(),
                                       accumulate_dx=acc, weights=False)[0] for w in (wz, wb))
        torch.cuda.synchronize()
        hit = torch.zeros((T, d), dtype=torch.bool, device="cuda")
        hit[T // 2:, c] = True
        assert not torch.isfinite(got[hit]).any()
        assert torch.isfinite(ref).all() and torch.equal(got[~hit], ref[~hit])

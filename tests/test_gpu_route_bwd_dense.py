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

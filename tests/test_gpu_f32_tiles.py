"""The fp32 FFN at the edges of its 32 x 32 tiles and of its split K loop,
against the oracle."""
import numpy as np
import pytest
import torch

import oracle.moe as om
import paper_2601_14327_amd as laep
from workloads import random_case
from _gpu import TOL_F32, case, dev, host, rownorm_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts,d,f", [
    ([1], 64, 64),                               # one row, two steps per wave
    ([0, 31, 32, 33, 64, 65, 0, 1], 128, 320),   # tile edges, K a ragged number of batches
    ([5] * 256, 64, 128),                        # every expert the library takes
    ([300, 2, 0, 900], 576, 192),
])
@pytest.mark.parametrize("save", [True, False])
def test_f32_tiles(counts, d, f, save):
    E, R = len(counts), sum(counts)
    c = random_case(sum(counts) + d, T=R, d_model=d, E=E, k=1, d_ff=f, dtype="f32")
    offsets = np.r_[0, np.cumsum(counts)]
    td = torch.float32
    case(f"f32 tiles E={E} R={R} d={d} f={f}")
    y, act = laep.moe_grouped_ffn_fwd(dev(c["x"], td), dev(c["w_gate_up"], td),
                                      dev(c["w_down"], td),
                                      dev(offsets.astype(np.int32), torch.int32), save_act=save)
    torch.cuda.synchronize()
    ry, ra = om.grouped_ffn_fwd(c["x"], c["w_gate_up"], c["w_down"], offsets, dtype="f32")
    assert rownorm_err(host(y), ry) <= TOL_F32
    assert (act is None) if not save else rownorm_err(host(act), ra) <= TOL_F32

"""Pruning loads on both sides of the 32-bit path's limit (2^23 per expert),
and repacking with every subset of the tensors, plain and streamed."""
import itertools

import numpy as np
import pytest
import torch

import oracle.laep as ol
import paper_2601_14327_amd as laep
from _gpu import case, dev, host

pytestmark = pytest.mark.gpu

LIMIT = 1 << 23


@pytest.mark.parametrize("iters,L,E", [(5, 2, 200), (17, 1, 64), (4, 3, 256), (1025, 1, 1)])
@pytest.mark.parametrize("top", [LIMIT - 1, LIMIT, 1 << 40])
def test_window_loads(iters, L, E, top):
    rng = np.random.default_rng(E + iters)
    etn = rng.integers(0, 50, (iters, L, E)).astype(np.int64)      # many ties
    hit = rng.random((iters, L, E)) < 0.3
    etn[hit] = top - rng.integers(0, 2, hit.sum())
    total = int(etn.sum(axis=2).max())
    case(f"prune window ITER={iters} L={L} E={E} top={top}")
    alive, n, marker = laep.laep_expert_pruning(dev(etn, torch.int64), total, 0.9, 0.4,
                                                want_marker=True)
    torch.cuda.synchronize()
    pruned, ref = ol.expert_pruning(etn, total, 1, [0.9] * L, 0.4, return_marker=True)
    np.testing.assert_array_equal(host(marker), ref)
    for l in range(L):
        assert np.nonzero(host(alive)[l] == 0)[0].tolist() == pruned[l].tolist()
        assert int(host(n)[l]) == len(pruned[l])


@pytest.mark.parametrize("E", [1, 63, 64, 65, 256])
@pytest.mark.parametrize("top", [LIMIT - 1, LIMIT, (1 << 31) - 1])
def test_mask_loads(E, top):
    rng = np.random.default_rng(E)
    counts = rng.integers(0, 5, E).astype(np.int64)
    counts[rng.random(E) < 0.4] = top
    total = int(counts.sum()) + 1
    case(f"prune mask E={E} top={top}")
    alive, n = laep.laep_prune_mask(dev(counts.astype(np.int32), torch.int32), total, 0.8, 0.5)
    torch.cuda.synchronize()
    ref = ol.prune_mask(counts, total, 0.8, 0.5)
    np.testing.assert_array_equal(host(alive).astype(bool), np.asarray(ref[0], bool)
                                  if isinstance(ref, tuple) else np.asarray(ref, bool))
    assert int(host(n)[0]) == int((host(alive) == 0).sum())


@pytest.mark.parametrize("d,f", [(8, 8), (520, 136), (2048, 1024)])   # the last one streams
def test_repack_subsets(d, f):
    E = 24
    g = torch.Generator(device="cuda").manual_seed(d)
    alive = torch.rand(E, device="cuda", generator=g) < 0.6
    full = {"w_router": torch.randn(E, d, device="cuda", generator=g),
            "w_gate_up": torch.randn(E, 2 * f, d, device="cuda", generator=g),
            "w_down": torch.randn(E, d, f, device="cuda", generator=g),
            "bias": torch.randn(E, device="cuda", generator=g)}
    m, na = laep.laep_compact_experts(alive.to(torch.uint8))
    n = int(na[0])
    names = sorted(full)
    for r in range(1, 5):
        for some in itertools.combinations(names, r):
            case(f"repack d={d} f={f} {some}")
            out = laep.laep_repack_experts(m, n, **{k: full[k] for k in some})
            torch.cuda.synchronize()
            for k in some:
                assert torch.equal(out[k], full[k][alive]), k

"""The router backward's workspace: a workspace sized for the largest call
serves every smaller one (fewer tokens, slots, experts or columns)."""
import pytest
import torch

import paper_2601_14327_amd as laep
from paper_2601_14327_amd._lib import LAEP_CALL_ROUTE_BWD


def _bytes(T, k, E, d):
    return laep.workspace_bytes(LAEP_CALL_ROUTE_BWD, T, k, E, d)


@pytest.mark.parametrize("T,k,E,d", [(8300, 8, 64, 2048), (3000, 2, 65, 1024), (40000, 1, 16, 64),
                                     (700, 4, 256, 4096), (130, 100, 200, 136)])
def test_workspace_grows_with_every_size(T, k, E, d):
    by_T = [_bytes(t, k, E, d) for t in range(1, T + 1)]
    assert by_T == sorted(by_T)
    by_E = [_bytes(T, k, e, d) for e in range(k, 257)]
    assert by_E == sorted(by_E)
    by_d = [_bytes(T, k, E, c) for c in range(8, d + 200, 8)]
    assert by_d == sorted(by_d)
    by_k = [_bytes(T, j, E, d) for j in range(1, E + 1)]
    assert by_k == sorted(by_k)


@pytest.mark.gpu
@pytest.mark.parametrize("large,small", [((2080, 64), (2048, 64)), ((2048, 65), (2048, 64))])
def test_larger_workspace_serves_a_smaller_call(large, small):
    k, d = 8, 512
    ws = torch.empty(_bytes(large[0], k, large[1], d), dtype=torch.uint8, device="cuda")
    T, E = small
    print(f"[gpu case] router backward T={T} E={E} on the workspace of {large}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(E)
    x = torch.randn((T, d), generator=g, device="cuda").to(torch.bfloat16)
    wr = (0.05 * torch.randn((E, d), generator=g, device="cuda")).to(torch.bfloat16)
    dg = torch.randn((T, k), generator=g, device="cuda")
    for renorm in (True, False):
        idx, gate, logits = laep.moe_route(x, wr, k, renorm=renorm, want_logits=True)
        _, off, _, src = laep.moe_expert_counts(idx, E, want_row_src=True)
        kw = dict(renorm=renorm, logits=None if renorm else logits, offsets=off, row_src=src,
                  want_dbias=True)
        a = laep.moe_route_bwd(dg, idx, gate, x, wr, ws=ws, **kw)
        b = laep.moe_route_bwd(dg, idx, gate, x, wr, **kw)
        torch.cuda.synchronize()
        assert all(torch.equal(p, q) for p, q in zip(a[:3], b[:3]))

"""Identity and square of few long examples, whose M_b go through the workspace: the same bits as from one launch (which a planner option away
from its default or a workspace without room for them takes), ragged blocks and lengths, groups of one example and of several."""
import pytest
import torch

import paper_2510_00236_amd as pex

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BOTH = ("identity", "square")

CASES = [
    (4, 1024, 768, 3072),        # groups of one example
    (3, 5000, 1000, 3000),       # blocks and slabs that are not whole; groups of two examples and of one
    (5, 2049, 2048, 2056),       # one token past a slab, one chunk past a block
    (16, 4092, 1024, 1024),      # eight groups of two
    (6, 429, 968, 1856),         # shorter examples, on the eight-wave kernel: groups of two
    (20, 261, 768, 640),
]


@pytest.mark.parametrize("B,T,din,dout", CASES)
def test_same_bits_as_one_launch(B, T, din, dout, pex_option):
    g = torch.Generator(device=DEV).manual_seed(B * T)
    X, G = (torch.randn(B, T, n, device=DEV, generator=g).bfloat16() for n in (din, dout))
    need = pex.pex_stat_multi_workspace_bytes(B, T, din, dout, pex.PEX_BF16, BOTH)
    assert need >= B * din * dout * 4, "not taken"

    def run(size):
        out = {k: torch.full((din, dout), float("nan"), device=DEV) for k in BOTH}
        ws = torch.full((size + 4096,), 77, dtype=torch.uint8, device=DEV)
        pex.pex_stat_multi(X, G, BOTH, out=out, workspace=ws[:size])
        assert (ws[size:] == 77).all(), "written outside the workspace"
        return out

    now = run(need)
    pex_option("memory_fold", 0)
    size = pex.pex_stat_multi_workspace_bytes(B, T, din, dout, pex.PEX_BF16, BOTH)
    one_launch = run(size)
    pex_option("memory_fold", 1)
    if size < need:
        without_room = run(need - 256)
        assert all(torch.equal(without_room[k], one_launch[k]) for k in BOTH)
    assert all(torch.equal(now[k], one_launch[k]) for k in BOTH)
    # fp32 sums of exact products: a few roundings per 16 tokens and example, 2^-24 each, against a norm of many entries
    ref = [0.0, 0.0]
    for b in range(B):
        M = X[b].double().t().contiguous() @ G[b].double()
        ref = [ref[0] + M, ref[1] + M * M]
    for k, r in zip(BOTH, ref):
        assert float((now[k].double() - r).norm() / r.norm()) < 2e-6


def test_replayed_from_a_graph():
    B, T, din, dout = CASES[0]
    g = torch.Generator(device=DEV).manual_seed(3)
    X, G = (torch.randn(B, T, n, device=DEV, generator=g).bfloat16() for n in (din, dout))
    out = {k: torch.empty(din, dout, device=DEV) for k in BOTH}
    ws = torch.empty(pex.pex_stat_multi_workspace_bytes(B, T, din, dout, pex.PEX_BF16, BOTH), dtype=torch.uint8, device=DEV)
    pex.pex_stat_multi(X, G, BOTH, out=out, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pex.pex_stat_multi(X, G, BOTH, out=out, workspace=ws)
    for _ in range(3):
        X.copy_(torch.randn(X.shape, device=DEV, generator=g))
        pex.pex_stat_multi(X, G, BOTH, out=out, workspace=ws)
        eager = {k: S.clone() for k, S in out.items()}
        for S in out.values():
            S.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(out[k], eager[k]) for k in BOTH)

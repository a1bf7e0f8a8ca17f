"""Identity and square of few long examples, whose M_b go through the workspace: the same bits as from one launch (which the option
stored_examples at 0 and a workspace without room for them take), ragged blocks and lengths, groups of one example, of two and of more, one group of
all of them.  That the planner takes these layers is asked of it in test_multi_plan_host.py."""
import pytest
import torch

import paper_2510_00236_amd as pex

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BOTH = ("identity", "square")

# (B, T, din, dout), examples of a group, groups
CASES = [
    ((4, 1024, 768, 3072), 2, 2),
    ((3, 5000, 1000, 3000), 2, 2),        # blocks and slabs that are not whole; a last group of one example
    ((5, 2049, 2048, 2056), 1, 5),        # one token past a slab, one chunk past a block
    ((16, 4092, 1024, 1024), 2, 8),
    ((6, 429, 968, 1856), 2, 3),          # shorter examples, on the eight-wave kernel
    ((20, 261, 768, 640), 2, 10),
    # more room than the partial sums need:
    ((4, 8192, 4096, 4096), 4, 1),        # no partial sums; the second pass in one step of four examples
    ((1, 8192, 4096, 4096), 1, 1),
    ((5, 603, 4032, 768), 5, 1),          # five in one group: a step of four and one of one
    ((7, 3190, 2176, 2816), 7, 1),
    ((69, 1604, 648, 88), 3, 23),         # groups that end inside the steps of four; fewer workgroups than units
    ((97, 1095, 512, 232), 4, 25),        # a last group of one, in a step of its own
]


@pytest.mark.parametrize("shape", [c[0] for c in CASES])
def test_same_bits_as_one_launch(shape, pex_option):
    B, T, din, dout = shape
    g = torch.Generator(device=DEV).manual_seed(B * T)
    X, G = (torch.randn(B, T, n, device=DEV, generator=g).bfloat16() for n in (din, dout))

    def run(size):
        out = {k: torch.full((din, dout), float("nan"), device=DEV) for k in BOTH}
        ws = torch.full((size + 4096,), 77, dtype=torch.uint8, device=DEV)
        pex.pex_stat_multi(X, G, BOTH, out=out, workspace=ws[:size])
        assert (ws[size:] == 77).all(), "written outside the workspace"
        return out

    need = pex.pex_stat_multi_workspace_bytes(B, T, din, dout, pex.PEX_BF16, BOTH)
    now = run(need)
    pex_option("stored_examples", 0)
    size = pex.pex_stat_multi_workspace_bytes(B, T, din, dout, pex.PEX_BF16, BOTH)
    one_launch = run(size)
    assert all(torch.equal(now[k], one_launch[k]) for k in BOTH)
    pex_option("stored_examples", 1)
    # a workspace with no room for them, down to the partial sums alone
    for less in sorted({size, max(size, need - 256)}):
        without_room = run(less)
        assert all(torch.equal(without_room[k], one_launch[k]) for k in BOTH), less
    # fp32 sums of exact products: a few roundings per 16 tokens and example, 2^-24 each, against a norm of many entries
    ref = [0.0, 0.0]
    for b in range(B):
        M = X[b].double().t().contiguous() @ G[b].double()
        ref = [ref[0] + M, ref[1] + M * M]
    for k, r in zip(BOTH, ref):
        assert float((now[k].double() - r).norm() / r.norm()) < 2e-6


def test_a_workspace_at_any_address_beside_a_layer_that_needs_none(pex_option):
    B, T, din, dout = 1, 8192, 4096, 4096
    g = torch.Generator(device=DEV).manual_seed(5)
    X, G = (torch.randn(B, T, n, device=DEV, generator=g).bfloat16() for n in (din, dout))
    ws = torch.empty(pex.pex_stat_multi_workspace_bytes(B, T, din, dout, pex.PEX_BF16, BOTH) + 8, dtype=torch.uint8, device=DEV)
    odd = pex.pex_stat_multi(X, G, BOTH, workspace=ws[8:])
    pex_option("stored_examples", 0)
    without = pex.pex_stat_multi(X, G, BOTH)
    assert all(torch.equal(odd[k], without[k]) for k in BOTH)


def test_replayed_from_a_graph():
    B, T, din, dout = CASES[0][0]
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

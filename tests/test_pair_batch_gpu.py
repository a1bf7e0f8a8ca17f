"""Identity and square of several layers in one launch: layers of one, several and ragged blocks, cut into different numbers of groups,
beside layers that cannot join (odd widths, small ones, fp32), against 64-bit sums; a workspace that only holds single layers."""
import pytest
import torch

import paper_2510_00236_amd as pex

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BOTH = ("identity", "square")

CASES = [
    # B, T, widths, dtype
    (12, 94, [(128, 384), (128, 128), (128, 512), (512, 128)], torch.bfloat16),
    (21, 285, [(320, 960), (320, 320), (320, 1280), (1280, 320)], torch.bfloat16),       # different numbers of groups
    (7, 33, [(264, 136), (8, 1032), (520, 392)], torch.bfloat16),                        # ragged blocks, one token past a slab
    (40, 31, [(256, 256), (256, 255), (256, 512), (768, 256)], torch.bfloat16),          # one layer of odd width between the others
    (1, 300, [(512, 512), (512, 1024)], torch.bfloat16),                                 # one example: no groups
    (33, 64, [(256, 384)] * 8, torch.bfloat16),                                          # more layers than a launch takes
    (64, 128, [(768, 2304), (768, 768), (768, 3072), (3072, 768)], torch.bfloat16),      # no more groups than one or two
    (5, 40, [(64, 64), (128, 96)], torch.float32),
]


@pytest.mark.parametrize("B,T,widths,dtype", CASES)
def test_layers_together(B, T, widths, dtype):
    g = torch.Generator(device=DEV).manual_seed(B * T)
    layers = []
    for din, dout in widths:
        X, G = (torch.randn(B, T, n, device=DEV, generator=g).to(dtype) for n in (din, dout))
        layers.append((X, G, {k: torch.full((din, dout), float("nan"), device=DEV) for k in BOTH}))
    code = pex.PEX_BF16 if dtype == torch.bfloat16 else pex.PEX_F32
    need = pex.pex_stat_pair_batch_workspace_bytes(widths, B, T, code)
    single = max(pex.pex_stat_multi_workspace_bytes(B, T, din, dout, code, BOTH) for din, dout in widths)
    assert need >= single
    for size in {need, single}:
        ws = torch.full((size + 4096,), 77, dtype=torch.uint8, device=DEV)
        for _, _, out in layers:
            for S in out.values():
                S.fill_(float("nan"))
        res = pex.pex_stat_pair_batch(layers, workspace=ws[:size])
        assert (ws[size:] == 77).all(), "written outside the workspace"
        for (X, G, out), r in zip(layers, res):
            assert all(r[k] is out[k] for k in BOTH)
            M = torch.matmul(X.double().transpose(1, 2).contiguous(), G.double())
            # fp32 sums of exact products: a few roundings per 16 tokens and example, 2^-24 each, against a norm of many entries
            for S, ref in ((out["identity"], M.sum(0)), (out["square"], (M * M).sum(0))):
                assert float((S.double() - ref).norm() / ref.norm()) < 2e-6


def test_too_small_a_workspace():
    B, T, widths = 21, 285, [(320, 960), (320, 320)]
    layers = [(torch.zeros(B, T, a, dtype=torch.bfloat16, device=DEV), torch.zeros(B, T, b, dtype=torch.bfloat16, device=DEV), None) for a, b in widths]
    single = max(pex.pex_stat_multi_workspace_bytes(B, T, a, b, pex.PEX_BF16, BOTH) for a, b in widths)
    with pytest.raises((ValueError, pex.PexError)):
        pex.pex_stat_pair_batch(layers, workspace=torch.empty(single - 4096, dtype=torch.uint8, device=DEV))


def test_replayed_from_a_graph():
    B, T, widths = 12, 94, [(128, 384), (128, 128), (128, 512), (512, 128)]
    g = torch.Generator(device=DEV).manual_seed(3)
    layers = [(torch.randn(B, T, a, device=DEV, generator=g).bfloat16(), torch.randn(B, T, b, device=DEV, generator=g).bfloat16(),
               {k: torch.empty(a, b, device=DEV) for k in BOTH}) for a, b in widths]
    ws = torch.empty(pex.pex_stat_pair_batch_workspace_bytes(widths, B, T, pex.PEX_BF16), dtype=torch.uint8, device=DEV)
    pex.pex_stat_pair_batch(layers, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pex.pex_stat_pair_batch(layers, workspace=ws)
    for seed in range(3):
        for X, _, _ in layers:
            X.copy_(torch.randn(X.shape, device=DEV, generator=g))
        pex.pex_stat_pair_batch(layers, workspace=ws)
        eager = [{k: out[k].clone() for k in BOTH} for _, _, out in layers]
        for _, _, out in layers:
            for S in out.values():
                S.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for (_, _, out), e in zip(layers, eager):
            assert all(torch.equal(out[k], e[k]) for k in BOTH)


@pytest.mark.parametrize("B,T,d", [(22, 70, 768), (11, 99, 768), (19, 93, 448), (8, 180, 704), (7, 478, 640)])
def test_together_as_exact_as_alone(B, T, d):
    """Fewer groups of examples are longer sums: no layer may be rounded so much more often that its error against 64 bits grows (5 %: the
    planner's line at 2.5 and what two sets of roundings of half a million entries differ)."""
    g = torch.Generator(device=DEV).manual_seed(B)
    layers = [(torch.randn(B, T, a, device=DEV, generator=g).bfloat16(), torch.randn(B, T, b, device=DEV, generator=g).bfloat16(), None)
              for a, b in ((d, 3 * d), (d, d), (d, 4 * d), (4 * d, d))]
    together = pex.pex_stat_pair_batch(layers)
    for (X, G, _), out in zip(layers, together):
        M = torch.matmul(X.double().transpose(1, 2).contiguous(), G.double())
        alone = pex.pex_stat_multi(X, G, BOTH)
        for k, ref in (("identity", M.sum(0)), ("square", (M * M).sum(0))):
            err = lambda S: float((S.double() - ref).norm() / ref.norm())
            assert err(out[k]) <= 1.05 * err(alone[k]), (k, X.shape, G.shape)


@pytest.mark.parametrize("B,T,d", [(15, 897, 704), (13, 1550, 832)])
def test_together_where_a_workspace_has_no_room_for_their_examples(B, T, d, pex_option):
    """Layers that go each by itself, with the M_b of some in the workspace, go together in a workspace of the size they ask for without."""
    g = torch.Generator(device=DEV).manual_seed(T)
    widths = [(d, 3 * d), (d, d), (d, 4 * d), (4 * d, d)]
    layers = [tuple(torch.randn(B, T, n, device=DEV, generator=g).bfloat16() for n in w) for w in widths]

    def run(size):
        out = [{k: torch.full(w, float("nan"), device=DEV) for k in ("identity", "square")} for w in widths]
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        pex.pex_stat_pair_batch([(X, G, o) for (X, G), o in zip(layers, out)], workspace=ws)
        return [S for o in out for S in o.values()]

    room = pex.pex_stat_pair_batch_workspace_bytes(widths, B, T, pex.PEX_BF16)
    alone = run(room)
    pex_option("stored_examples", 0)
    size = pex.pex_stat_pair_batch_workspace_bytes(widths, B, T, pex.PEX_BF16)
    together = run(size)
    pex_option("stored_examples", 1)
    assert size < room and not all(torch.equal(a, b) for a, b in zip(alone, together))       # (other groups of examples, other roundings)
    assert all(torch.equal(a, b) for a, b in zip(run(size), together))

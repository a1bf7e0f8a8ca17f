"""Several tensors in one call against the calls of one tensor, which the oracles pin: the same bits of every state tensor and statistic;
sums in fp64 to their rounding.  Sizes at the edges of chunks, of a group of tensors and of the workspace."""
import numpy as np
import pytest
import torch

import paper_2510_00236_amd as pex

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SIZES = [
    [1, 2, 3, 4, 5, 1023, 1024, 1025],
    [4097, 300001, 7],
    [5] * 33 + [2049, 70000],             # more tensors than a launch takes
    [24_000_003],                         # chunks of more than 1024 elements, past the caches with all seven buffers
]


def _tensors(sizes, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    r = lambda n: torch.randn(n, device=DEV, generator=g)
    return [(r(n), r(n), r(n).abs(), r(n) * 3, (r(n) * 3).square() + 1, r(n).square(), r(n).square()) for n in sizes]


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("variant,track", [("microadam", True), ("microadam_msq", False), ("adam", True), ("adam", False), ("microadam_var", True)])
def test_step_equals_the_calls_of_one_tensor(sizes, variant, track):
    B = 5
    prm = pex.AdamParams(lr=1e-2, beta1=0.9, beta2=0.95, eps=1e-8, eps_root=0.0, weight_decay=0.1, grad_scale=1.0 / B, sq_scale=1.0 / B, step=3, B=B)
    mp = pex.MomentParams(beta2=0.95, grad_scale=1.0 / B, sq_scale=1.0 / B, B=B, debias=1, step=3)
    one, many = _tensors(sizes, 1), _tensors(sizes, 1)
    if variant == "adam" and not track:
        many = [t[:4] + (None,) + t[5:] for t in many]
    acc, acc2 = (torch.zeros(1, dtype=torch.float64, device=DEV) for _ in range(2))
    for k, t in enumerate(one):
        pex.pex_sum_squares(t[3], acc=acc, accumulate=k > 0)
    sums = torch.stack([pex.pex_moment_track(t[5], t[6], t[3], t[4], mp) for t in one]) if track else None
    max_norm = 0.3 * float(acc) ** 0.5 / B
    # a workspace of the least a call makes do with: a chunk per tensor
    least = ((len(sizes) + 31) // 32 + len(sizes)) * 16
    ws = torch.empty(least, dtype=torch.uint8, device=DEV) if sum(sizes) < 1 << 20 else None
    got = pex.pex_adam_step(many, variant, prm, acc2, max_norm, moments=mp if track else None, workspace=ws)
    torch.testing.assert_close(acc2, acc, rtol=1e-13, atol=0)
    for t, u in zip(one, many):
        pex.pex_adam_update_clipped(t[0], t[1], t[2], t[3], t[4], variant, prm, acc2, max_norm)
        for a, b in zip(t, u):
            assert b is None or torch.equal(a, b)
    if track:
        # an estimate is a difference: its sum to the rounding of the terms' magnitude
        for k, t in enumerate(one):
            scale = float((t[5] + t[6]).sum()) * 10
            assert (got[k] - sums[k]).abs().max().item() <= 1e-13 * scale
    else:
        assert got is None


@pytest.mark.parametrize("B,T,dtype", [(3, 50, torch.bfloat16), (7, 33, torch.float32), (20, 129, torch.bfloat16), (2, 300, torch.float32)])
def test_vectors_equal_the_calls_of_one_vector(B, T, dtype):
    g = torch.Generator(device=DEV).manual_seed(B)
    widths = [64, 8, 1, 77, 513, 4096, 768, 5] + [16] * 12      # whole chunks and not; more vectors than a launch takes
    items = []
    for k, d in enumerate(widths):
        A = torch.randn(B, T, d, device=DEV, generator=g).to(dtype)
        items.append((A, torch.randn(B, T, d, device=DEV, generator=g).to(dtype) if k % 2 else None, None))
    for want in (("identity", "square", "sign"), ("square",)):
        one = [pex.pex_vec_stat(A, C, want) for A, C, _ in items]
        all_bytes = pex.pex_vec_stat_batch_workspace_bytes(widths, B, T, pex.PEX_BF16 if dtype == torch.bfloat16 else pex.PEX_F32)
        largest = max(pex.pex_vec_stat_workspace_bytes(B, T, d, pex.PEX_BF16 if dtype == torch.bfloat16 else pex.PEX_F32) for d in widths)
        for nbytes in (all_bytes, (largest + 255) // 256 * 256):
            many = pex.pex_vec_stat_batch(items, want, workspace=torch.empty(nbytes, dtype=torch.uint8, device=DEV))
            assert all(set(u) == set(want) and torch.equal(t[k], u[k]) for t, u in zip(one, many) for k in want)


def test_captured_steps_match_eager_ones():
    prm = lambda step: pex.AdamParams(lr=1e-2, beta1=0.9, beta2=0.95, eps=1e-8, eps_root=0.0, weight_decay=0.0, grad_scale=0.25, sq_scale=0.25, step=step, B=4)
    mp = pex.MomentParams(beta2=0.95, grad_scale=0.25, sq_scale=0.25, B=4, debias=1, step=2)
    eager, captured = _tensors([1000, 40001], 3), _tensors([1000, 40001], 3)
    A = torch.randn(4, 60, 1000, device=DEV)
    state = [(t, torch.zeros(1, dtype=torch.float64, device=DEV), torch.zeros(2, 2, dtype=torch.float64, device=DEV),
              torch.empty(1 << 20, dtype=torch.uint8, device=DEV)) for t in (eager, captured)]

    def step(t, acc, sums, ws):
        pex.pex_vec_stat_batch([(A, None, {"identity": t[0][3], "square": t[0][4]}), (A, A, {"identity": t[1][3][:1000], "square": t[1][4][:1000]})],
                               ("identity", "square"), workspace=ws)
        pex.pex_adam_step(t, "microadam", prm(2), acc, 1e-3, moments=mp, sums=sums, workspace=ws)

    step(*state[0])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(*state[1])
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(*state[1])
    for _ in range(3):
        A.normal_()
        graph.replay()
        step(*state[0])
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for t, u in zip(eager, captured) for a, b in zip(t, u))
        assert torch.equal(state[0][1], state[1][1]) and torch.equal(state[0][2], state[1][2])


def test_checks():
    t = _tensors([8, 8], 0)
    prm = pex.AdamParams(lr=1e-2, beta1=0.9, beta2=0.95, eps=1e-8, step=1, B=4, grad_scale=1.0, sq_scale=1.0)
    mp = pex.MomentParams(beta2=0.95, grad_scale=1.0, sq_scale=1.0, B=4, debias=1, step=1)
    acc = torch.zeros(1, dtype=torch.float64, device=DEV)
    bad = lambda k, x: [t[0], t[1][:k] + (x,) + t[1][k + 1:]]
    with pytest.raises(TypeError, match="m must be"):
        pex.pex_adam_step(bad(1, t[1][1].double()), "microadam", prm, acc, 1.0)
    with pytest.raises(ValueError, match="S_sq must have 8"):
        pex.pex_adam_step(bad(4, t[1][4][:7]), "microadam", prm, acc, 1.0)
    with pytest.raises(ValueError, match="v must live in GPU memory"):
        pex.pex_adam_step(bad(2, t[1][2].cpu()), "microadam", prm, acc, 1.0)
    with pytest.raises(ValueError, match="7 tensors"):
        pex.pex_adam_step([x[:5] for x in t], "microadam", prm, acc, 1.0, moments=mp)
    with pytest.raises(pex.PexError):
        pex.pex_adam_step(bad(4, None), "microadam", prm, acc, 1.0)
    A = torch.zeros(2, 3, 8, device=DEV)
    with pytest.raises(ValueError, match="one batch"):
        pex.pex_vec_stat_batch([(A, None, None), (A[:1], None, None)])
    with pytest.raises(TypeError, match="share a dtype"):
        pex.pex_vec_stat_batch([(A, None, None), (A.bfloat16(), None, None)])
    with pytest.raises(ValueError):
        pex.pex_vec_stat_batch([(A, None, None)], workspace=torch.empty(16, dtype=torch.uint8, device=DEV))

"""The elementwise kernels where their launch changes shape: tensors whose buffers are accessed past the caches (against the same
call on slices small enough for the cached flavour: elementwise, so bit for bit), and sums on both sides of the size a single
workgroup handles."""
import pytest
import torch

import paper_2510_00236_amd as pex

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N = 31_500_003          # three buffers of this many floats exceed 360 MiB; no multiple of 4


def _rand(seed, n=N):
    return torch.rand(n, device=DEV, generator=torch.Generator(device=DEV).manual_seed(seed))


def _slices(n):
    cut = n // 4 // 4 * 4
    return [(k * cut, (k + 1) * cut if k < 3 else n) for k in range(4)]


@pytest.mark.parametrize("variant", ["adam", "microadam", "microadam_var", "microadam_msq"])
def test_streamed_adam(variant):
    p = pex.AdamParams(lr=1e-2, beta1=0.9, beta2=0.95, eps=1e-8, eps_root=0.0, weight_decay=1e-3, grad_scale=0.25, sq_scale=0.25, step=2, B=4)
    S_id, S_sq = _rand(1) - 0.5, _rand(2)
    a = [_rand(3), _rand(4), _rand(5)]
    b = [t.clone() for t in a]
    pex.pex_adam_update(*a, S_id, S_sq, variant, p)
    for lo, hi in _slices(N):
        pex.pex_adam_update(*(t[lo:hi] for t in b), S_id[lo:hi], S_sq[lo:hi], variant, p)
    assert all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("variant", ["microsignsgd", "signsgd", "signema"])
def test_streamed_sign(variant):
    S, a, b = _rand(1) - 0.5, [_rand(3), _rand(4) - 0.5], None
    b = [t.clone() for t in a]
    pex.pex_sign_update(*a, S, variant, 1e-2, 0.9, 1e-3, 8, True, 3)
    for lo, hi in _slices(N):
        pex.pex_sign_update(*(t[lo:hi] for t in b), S[lo:hi], variant, 1e-2, 0.9, 1e-3, 8, True, 3)
    assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_streamed_moments():
    p = pex.MomentParams(beta2=0.95, grad_scale=0.25, sq_scale=0.25, B=4, debias=1, step=2)
    S_id, S_sq = _rand(1) - 0.5, _rand(2)
    a = [_rand(3), _rand(4)]
    b = [t.clone() for t in a]
    sums = pex.pex_moment_track(*a, S_id, S_sq, p)
    parts = sum(pex.pex_moment_track(*(t[lo:hi] for t in b), S_id[lo:hi], S_sq[lo:hi], p) for lo, hi in _slices(N))
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    # fp64 sums of 28 M terms of order 1 in another order: far below 1e-12 of the sum of their sizes
    assert (sums - parts).abs().max() <= 1e-11 * N


@pytest.mark.parametrize("n", [1, 1023, 32767, 32768, 32769, 40001])
def test_sums_of_one_workgroup_and_of_many(n):
    x, y = _rand(6, n) - 0.5, _rand(7, n)
    ref = float(x.double().square().sum())
    acc = pex.pex_sum_squares(x)
    assert abs(float(acc) - ref) <= 1e-13 * ref          # fp64 sums of at most 2^16 terms
    pex.pex_sum_squares(x, acc=acc, accumulate=True)
    assert abs(float(acc) - 2 * ref) <= 2e-13 * ref
    p = pex.MomentParams(beta2=0.0, grad_scale=1.0, sq_scale=1.0, B=4, debias=0, step=1)
    a, q = torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
    sums = pex.pex_moment_track(a, q, x, y, p).cpu()
    ah, qh = a.double(), q.double()
    mu2, s2 = ((ah - qh / 4) / 0.75).sum().cpu(), ((qh - ah) / 0.75).sum().cpu()
    assert abs(sums[0] - mu2) <= 1e-12 * n and abs(sums[1] - s2) <= 1e-12 * n

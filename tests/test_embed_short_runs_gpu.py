"""Tokens whose runs are about the sixteen sorted positions of a wave, starting at every offset to the waves' borders: on few workgroups, where the
waves share a run from 17 positions on, and on a full chip, where they do from 65 on; bf16 rows at every alignment."""
import pytest
import torch

import paper_2510_00236_amd as pex

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BOTH = ("identity", "square")


def _check(ids, G, V):
    B, T, d = G.shape
    out = {k: torch.full((V, d), float("nan"), device=DEV) for k in BOTH}
    pex.pex_embed_stat(ids, G, V, BOTH, out=out)
    S_id, S_sq, scale = (torch.zeros(V, d, dtype=torch.float64, device=DEV) for _ in range(3))
    for b in range(B):
        real = ids[b] < V
        M = torch.zeros(V, d, dtype=torch.float64, device=DEV).index_add_(0, ids[b][real], G[b][real].double())
        S_id += M
        S_sq += M * M
        scale.index_add_(0, ids[b][real], G[b][real].double().abs())
    # a sum of n terms in any order is off by at most n 2^-24 of the sum of their magnitudes; a square's terms are squares of such sums
    n = torch.bincount(ids[ids < V].flatten(), minlength=V).double().unsqueeze(1)
    eps = 2.0 ** -24
    assert ((out["identity"].double() - S_id).abs() <= (n + 1) * eps * scale).all()
    assert ((out["square"].double() - S_sq).abs() <= 3 * (n + 1) * eps * scale * scale).all()


@pytest.mark.parametrize("d,dtype", [(64, torch.bfloat16), (5, torch.bfloat16), (263, torch.bfloat16), (6, torch.bfloat16), (3, torch.bfloat16), (65, torch.float32)])
@pytest.mark.parametrize("B,each", [(1, 4000), (7, 1), (5, 19)])
def test_runs_about_a_waves_positions(d, dtype, B, each):
    runs = [1, 15, 16, 17, 18, 16, 17, 17, 31, 2, 33, 32, 1, 64, 65, 3, 66, 47, 17, 17, 17, 17, 17, 48, 16, 49] * 2      # 17 by 17: every offset
    tokens = [v for v, n in enumerate(runs) for _ in range(n)]
    rows = [[] for _ in range(B)]
    for k, v in enumerate(tokens):
        rows[k // each % B].append(v)
    T, V = max(len(r) for r in rows), len(runs)
    ids = torch.tensor([r + [V] * (T - len(r)) for r in rows], device=DEV)        # V: padding, in no run
    g = torch.Generator(device=DEV).manual_seed(d)
    _check(ids, torch.randn(B, T, d, device=DEV, generator=g).to(dtype), V)


@pytest.mark.parametrize("B,T,V,d", [(24, 1000, 900, 1024), (24, 1100, 900, 1024), (30, 1000, 700, 1021), (14, 1000, 17000, 1024)])       # 500, 552 and 628 workgroups; 292 and 17 M entries
def test_on_both_sides_of_a_full_chip(B, T, V, d):
    g = torch.Generator(device=DEV).manual_seed(T)
    ids = (torch.rand(B, T, device=DEV, generator=g) ** 2 * V).long()
    _check(ids, torch.randn(B, T, d, device=DEV, generator=g).bfloat16(), V)

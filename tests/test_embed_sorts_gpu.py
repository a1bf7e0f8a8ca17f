"""The sorts of the embedding statistics on both sides of every line between them: one launch by buckets, two, the radix sorts of
vocabularies, batches and workspaces that buckets do not fit.  Against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2510_00236_amd as pex
import synth_inputs as si
from oracle import embed as oe
from parity_util import assert_real_stat, assert_sign_stat

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _radix_bytes(N, V, d):
    """What a call needs that sorts digit by digit."""
    up = lambda x: (x + 255) // 256 * 256
    tile = (-(-N // 64) + 1023) // 1024 * 1024
    return up(1024 * -(-N // tile)) + 4 * up(4 * N) + up(4 * (V + 2)) + up(-(-N // 192) * 24 * d)


def _check(ids, B, T, V, d, workspace=None):
    _, G = si.custom(B, T, 1, d, dtype="bf16", seed=B)
    names = ("identity", "square", "sign")
    out = {k: torch.full((V, d), float("nan"), device=DEV) for k in names}
    pex.pex_embed_stat(ids.to(DEV), G.to(DEV), V, names, out=out, workspace=workspace)
    present = ids[(ids >= 0) & (ids < V)].unique()
    if V > 2000:      # the oracle materialises [V, d] per example: compare the rows that occur, all others must be zero
        zero = torch.ones(V, dtype=torch.bool, device=DEV)
        zero[present.to(DEV)] = False
        assert all(int(torch.count_nonzero(out[k][zero])) == 0 for k in names)
        out = {k: v[present.to(DEV)] for k, v in out.items()}
        ids = torch.where((ids >= 0) & (ids < V), torch.searchsorted(present, ids.clamp(0, V - 1)), -1)
        V = present.numel()
    got = {k: v.cpu().numpy().astype(np.float64) for k, v in out.items()}
    ref = oe.embed_stat(ids.numpy(), si.widen(G), V)
    assert_real_stat(got["identity"], ref.S_id, "bf16", "identity", elementwise=False)
    assert_real_stat(got["square"], ref.S_sq, "bf16", "square", elementwise=B >= 3)
    assert_sign_stat(got["sign"], ref.S_sign, ref.amb, "sign")


@pytest.mark.parametrize("B,T,V,d,exponent,pad", [
    (4, 1024, 257, 4, 1.0, 0.1),         # 4096 positions, two tokens in bucket 0 and one in the others
    (17, 241, 257, 4, 1.0, 0.1),         # 4097: five tiles, the last of one position
    (3, 1500, 1, 4, 0.0, 0.3),           # a single token
    (4, 2048, 255, 4, 0.3, 0.0),         # the last bucket is empty
    (6, 900, 262144, 4, 0.0, 0.0),       # the most tokens a bucket holds
    (6, 900, 262145, 4, 0.0, 0.0),       # one more
    (64, 4096, 300, 1, 1.0, 0.0),        # 262144 positions: 256 tiles
    (57, 4600, 300, 1, 1.0, 0.0),        # 262200
])
def test_sorts(B, T, V, d, exponent, pad):
    ids = si.token_ids(B, T, V, seed=B + T, exponent=exponent, pad_fraction=pad)
    _check(ids, B, T, V, d)


@pytest.mark.parametrize("B,T,exponent,pad", [
    (8, 256, 1.0, 0.0),      # exactly 2048 positions, frequent tokens: every wave's segment holds keys, counters of the same digit in all of them
    (3, 500, 1.0, 0.2),      # 1500: segments of several batches of 64, the last ones partly and wholly empty; padding
    (5, 26, 0.5, 0.0),       # 130: three waves, the last of two positions
    (2, 32, 0.0, 0.9),       # one batch of one wave
    (3, 683, 1.0, 0.1),      # 2049: the sort of many workgroups
])
def test_radix_sorts_of_a_vocabulary_too_large_for_buckets(B, T, exponent, pad):
    V = 300000
    _check(si.token_ids(B, T, V, seed=B + T, exponent=exponent, pad_fraction=pad), B, T, V, 3)


def test_half_of_the_positions_one_token():
    """A bucket whose workgroup meets batches of one token, of a few tokens and of many."""
    B, T, V = 12, 1000, 700
    ids = si.token_ids(B, T, V, seed=5, exponent=0.0)
    keep = torch.rand(B, T, generator=torch.Generator().manual_seed(2))
    ids = torch.where(keep < 0.5, torch.tensor(3), torch.where(keep < 0.8, ids // 256 * 256 % V + 3, ids)) % V
    _check(ids, B, T, V, 5)


def test_workspace_of_the_radix_sort_is_enough():
    B, T, V, d = 9, 1000, 600, 5
    least = _radix_bytes(B * T, V, d)
    assert least < pex.pex_embed_stat_workspace_bytes(B, T, V, d)
    ids = si.token_ids(B, T, V, seed=1, exponent=1.0)
    _check(ids, B, T, V, d, torch.empty(least, dtype=torch.uint8, device=DEV))
    with pytest.raises((ValueError, pex.PexError)):
        _check(ids, B, T, V, d, torch.empty(least - 256, dtype=torch.uint8, device=DEV))

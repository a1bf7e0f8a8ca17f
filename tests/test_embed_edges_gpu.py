"""Embedding statistics at the edges: one slice of positions and several (the sorts: test_embed_sorts_gpu.py), rows of every alignment (lengths that are multiples of 4, 2 and 1, shorter than a lane's
four columns), gaps in the vocabulary of every length.  Outputs sit inside a larger buffer."""
import numpy as np
import pytest
import torch

import paper_2510_00236_amd as pex
import synth_inputs as si
from oracle import embed as oe
from parity_util import assert_real_stat, assert_sign_stat

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # B, T, V, d, dtype, ids dtype, Zipf exponent, padding
    (8, 256, 300, 12, "bf16", torch.int64, 1.0, 0.05),       # every token in a bucket of one or two
    (64, 32, 66000, 6, "bf16", torch.int32, 0.3, 0.0),       # mostly single positions, 258 tokens to a bucket
    (3, 683, 300, 9, "bf16", torch.int32, 1.0, 0.0),         # a last batch of one position
    (1, 64, 5000, 3, "f32", torch.int64, 0.0, 0.5),          # rows shorter than four columns, long gaps
    (2, 96, 17, 5, "bf16", torch.int64, 1.0, 0.0),           # one slice of 192 positions, frequent tokens only
    (2, 97, 17, 258, "bf16", torch.int32, 1.0, 0.0),         # one position more; two column blocks, the second of two columns
    (5, 333, 40, 261, "f32", torch.int64, 1.2, 0.1),
    (4, 500, 7, 103, "bf16", torch.int32, 1.0, 0.0),         # runs over several slices, odd rows
    (3, 20, 17000000, 2, "f32", torch.int64, 0.0, 0.0),      # a radix sort of four passes by one wave
    (1, 1, 9, 1, "bf16", torch.int64, 0.0, 0.0),
]


@pytest.mark.parametrize("B,T,V,d,dtype,idt,exponent,pad", CASES)
def test_edges(B, T, V, d, dtype, idt, exponent, pad):
    ids = si.token_ids(B, T, V, seed=B + T, exponent=exponent, pad_fraction=pad) if V < 1 << 20 else \
        torch.randint(0, V, (B, T), generator=torch.Generator().manual_seed(1))
    _, G = si.custom(B, T, 1, d, dtype=dtype, seed=B)
    names = ("identity", "square", "sign")
    buf = {k: torch.full((V * d + 128,), -7.0, device=DEV) for k in names}
    out = {k: b[64:64 + V * d].view(V, d).fill_(float("nan")) for k, b in buf.items()}
    pex.pex_embed_stat(ids.to(idt).to(DEV), G.to(DEV), V, names, out=out)
    got = {}
    for k, b in buf.items():
        assert (b[:64] == -7).all() and (b[64 + V * d:] == -7).all(), "written outside the output"
        got[k] = out[k]
    if V > 1 << 20:
        # the oracle materialises [V, d] per example: compare the rows that occur, all others must be zero
        rows = ids.unique().to(DEV)
        for k in names:
            assert int((got[k] != 0).any(1).sum()) <= rows.numel()
            got[k] = got[k][rows]
        ids = torch.searchsorted(ids.unique(), ids)
        V = rows.numel()
    got = {k: v.cpu().numpy().astype(np.float64) for k, v in got.items()}
    ref = oe.embed_stat(ids.numpy(), si.widen(G), V)
    assert_real_stat(got["identity"], ref.S_id, dtype, "identity", elementwise=False)
    assert_real_stat(got["square"], ref.S_sq, dtype, "square", elementwise=B >= 3)
    assert_sign_stat(got["sign"], ref.S_sign, ref.amb, "sign")

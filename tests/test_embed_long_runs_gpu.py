"""Tokens that fill many of the 192 sorted positions of a workgroup (16 of each wave): runs on both sides of the length that one wave
does by itself, starting and ending at and beside the waves' and workgroups' borders, examples with one or with hundreds of them."""
import numpy as np
import pytest
import torch

import paper_2510_00236_amd as pex
import synth_inputs as si
from oracle import embed as oe
from parity_util import assert_real_stat, assert_sign_stat

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# positions per token, in the order the tokens are sorted in; B examples share them in turn, `each` positions at a time
CASES = [
    ([64, 65, 63, 66, 64, 65], 3, 1),              # one wave or several, all in two workgroups
    ([16, 176, 192, 193, 191, 96], 6, 4),          # runs that end with a workgroup's positions, or one before or after
    ([1, 65, 126, 300, 15, 81], 4, 2),             # a run that starts at a workgroup's last position
    ([5, 400, 200, 70], 3, 225),                   # examples longer than a workgroup's positions
    ([15, 65, 65, 65, 65, 300], 25, 23),           # several long runs in a workgroup, examples that span two waves
    ([1000], 1, 1000),                             # one example, one token
    ([0, 0, 130, 0, 62], 64, 1),                   # a different example at every position
]


@pytest.mark.parametrize("runs,B,each", CASES)
@pytest.mark.parametrize("d,dtype,names", [(64, "bf16", ("identity", "square")), (261, "f32", ("square", "sign")), (6, "bf16", ("identity", "square", "sign"))])
def test_long_runs(runs, B, each, d, dtype, names):
    tokens = [v for v, n in enumerate(runs) for _ in range(n)]
    rows = [[] for _ in range(B)]
    for k, v in enumerate(tokens):
        rows[k // each % B].append(v)
    T, V = max(len(r) for r in rows), len(runs)
    ids = torch.tensor([r + [V] * (T - len(r)) for r in rows])        # V: padding, in no run
    _, G = si.custom(B, T, 1, d, dtype=dtype, seed=len(tokens))
    out = {k: torch.full((V, d), float("nan"), device=DEV) for k in names}
    pex.pex_embed_stat(ids.to(DEV), G.to(DEV), V, names, out=out)
    got = {k: v.cpu().numpy().astype(np.float64) for k, v in out.items()}
    ref = oe.embed_stat(ids.numpy(), si.widen(G), V)
    if "identity" in names:
        assert_real_stat(got["identity"], ref.S_id, dtype, "identity", elementwise=False)
    assert_real_stat(got["square"], ref.S_sq, dtype, "square", elementwise=B >= 3)
    if "sign" in names:
        assert_sign_stat(got["sign"], ref.S_sign, ref.amb, "sign")

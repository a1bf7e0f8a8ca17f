"""The second pass of the vector statistics at the edges of its block shapes: batches on both sides of the changes of shape
(4 and 16 examples) and beyond one round of example lanes, chains of ranges longer and shorter than a lane's eight loads,
widths that are no multiples of 4 or of a block."""
import numpy as np
import pytest
import torch

import paper_2510_00236_amd as pex
import synth_inputs as si
from oracle import vec as ov

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,T,d,dtype", [(4, 2300, 44, "f32"), (3, 500, 18, "bf16"), (5, 1200, 20, "f32"), (16, 330, 65, "f32"),
                                         (17, 700, 36, "bf16"), (64, 100, 16, "f32"), (130, 70, 35, "f32")])
def test_second_pass(B, T, d, dtype):
    X, G = si.custom(B, T, d, d, dtype=dtype, seed=B + T)
    ref = ov.vec_stat(si.widen(G), si.widen(X))
    out = {k: torch.full((d,), float("nan"), device=DEV) for k in ("identity", "square", "sign")}
    pex.pex_vec_stat(G.to(DEV), X.to(DEV), out=out)
    got = {k: v.cpu().double().numpy() for k, v in out.items()}
    # fp32 sums of exact products (bf16) or rounded ones (fp32) over T, then over B: as for the other vector tests
    for name, r in (("identity", ref.s_id), ("square", ref.s_sq)):
        assert np.abs(got[name] - r).max() <= 2e-5 * np.abs(r).max(), name
    assert (np.abs(got["sign"] - ref.s_sign) <= 2 * ref.amb).all()

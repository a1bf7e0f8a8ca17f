"""The second pass of the vector statistics at the edges of its block shapes: batches on both sides of the changes of shape
(4 and 16 examples) and beyond one round of example lanes, chains of ranges longer and shorter than a lane's eight loads,
widths that are no multiples of 4 or of a block, narrow and wide blocks (rows whose last chunk overlaps its neighbour, a row of
columns beyond what a launch of narrow blocks holds)."""
import numpy as np
import pytest
import torch

import paper_2510_00236_amd as pex
import synth_inputs as si
from oracle import vec as ov

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,T,d,dtype", [(4, 2300, 44, "f32"), (3, 500, 18, "bf16"), (5, 1200, 20, "f32"), (16, 330, 65, "f32"),
                                         (17, 700, 36, "bf16"), (64, 100, 16, "f32"), (130, 70, 35, "f32"), (3, 5, 1, "f32"), (70, 9, 3, "bf16"),
                                         (40, 70, 517, "f32"), (18, 40, 1006, "bf16"), (2, 4100, 515, "f32"), (16, 330, 1027, "bf16"), (3, 30, 40961, "f32")])
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


def test_more_columns_than_a_launch_of_narrow_blocks_holds():
    d = 2**26 + 1
    A = torch.randn(1, 1, d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(1)).bfloat16()
    out = {k: torch.full((d,), float("nan"), device=DEV) for k in ("identity", "square")}
    pex.pex_vec_stat(A, want=("identity", "square"), out=out)
    a = A.view(-1).float()
    assert torch.equal(out["identity"], a) and torch.equal(out["square"], a * a)      # one addend each, exact in fp32

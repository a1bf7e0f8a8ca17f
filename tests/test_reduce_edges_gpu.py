"""The sum of partial statistics at outputs of a few entries and of sizes that are no multiples of four: the last four columns
overlap their neighbours, fewer than four are added one by one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_00236_amd as pex
import synth_inputs as si
from parity_util import assert_real_stat, assert_sign_stat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,din,dout,dtype", [(40, 3, 1, 1, "f32"), (70, 2, 1, 3, "bf16"), (40, 3, 2, 2, "f32"), (50, 2, 5, 1, "f32"), (45, 4, 3, 9, "bf16"),
                                                (33, 2, 70, 66, "f32"), (34, 2, 67, 67, "f32")])
def test_small_outputs_in_many_groups(B, T, din, dout, dtype):
    code = pex.PEX_BF16 if dtype == "bf16" else pex.PEX_F32
    assert pex.pex_stat_workspace_bytes(B, T, din, dout, code, "square") >= 5 * din * dout * 4
    X, G = si.custom(B, T, din, dout, dtype=dtype, seed=B)
    st = oracle.stat(si.widen(X), si.widen(G))
    out = {k: torch.full((din, dout), float("nan"), device="cuda:0") for k in ("identity", "square", "sign")}
    for phi, S in out.items():
        pex.pex_stat(X.to("cuda:0"), G.to("cuda:0"), phi, S=S)
    got = {k: v.cpu().numpy().astype(np.float64) for k, v in out.items()}
    # (a single entry may be small beside its addends: the bar is on the sum of their sizes, which the square's root bounds)
    assert np.abs(got["identity"] - st.S_id).max() <= 2e-5 * np.sqrt(B * st.S_sq).max()
    assert_real_stat(got["square"], st.S_sq, dtype, "square", elementwise=True)
    assert_sign_stat(got["sign"], st.S_sign, st.amb, "sign")

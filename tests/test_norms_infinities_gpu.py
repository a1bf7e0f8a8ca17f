"""Per-example norms beside infinities: an entry of M_b that is infinite makes that example's norm infinite, at tile edges too (the
fp32 kernel's overlapping and narrow tiles, rows and columns of zeros beyond the layer), and leaves the others alone."""
import numpy as np
import pytest
import torch

import paper_2510_00236_amd as pex
import synth_inputs as si
from oracle import norms as on

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,T,din,dout,dtype", [(5, 26, 68, 36, "f32"), (3, 23, 127, 200, "f32"), (4, 50, 130, 66, "f32"), (5, 300, 192, 391, "bf16"),
                                                (4, 190, 257, 40, "bf16"), (8, 256, 768, 1001, "bf16"), (6, 80, 328, 200, "bf16"), (3, 20, 70, 66, "bf16"), (3, 20, 30, 75, "f32")])
@pytest.mark.parametrize("where", ["X", "G", "sum"])
def test_infinities(pex_option, B, T, din, dout, dtype, where):
    pex_option("gram_norms", 0)
    X, G = si.custom(B, T, din, dout, dtype=dtype, seed=B + T)
    ref = on.example_norms(si.widen(X), si.widen(G))
    # one column of X or of G that the last tile shares with, or has next to, its neighbour
    i, j = (din - 64 + 1 if din > 64 else din - 1), (dout - 64 + 1 if dout > 64 else dout - 1)
    if where == "X":
        X[1, 3, i] = float("inf")
    elif where == "G":
        G[1, 3, j] = float("-inf")
    else:       # finite inputs, an entry of M_1 beyond fp32: all its products of one sign
        X[1, :, i] = 1e25
        G[1, :, j] = 1e25
    X[X == 0] = 1.0     # (no zero meets the infinity)
    G[G == 0] = 1.0
    N = pex.pex_example_norms(X.to(DEV), G.to(DEV)).cpu().double().numpy()
    assert np.isposinf(N[1]), N
    others = [b for b in range(B) if b != 1]
    assert (np.abs(N - ref)[others] <= 1e-4 * ref[others]).all()

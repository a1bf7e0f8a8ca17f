"""Per-example norms with more groups of examples than any other statistic takes: one example per group, several, and batches
beyond the largest number of groups.  Against the oracle."""
import numpy as np
import pytest
import torch

import paper_2510_00236_amd as pex
import synth_inputs as si
from oracle import norms as on

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,din,dout,dtype", [(33, 40, 64, 72, "bf16"), (300, 33, 264, 40, "bf16"), (1030, 3, 64, 40, "bf16"), (50, 190, 65, 72, "bf16"),
                                                (33, 9, 64, 64, "f32"), (1300, 2, 68, 130, "f32")])
def test_many_groups(pex_option, B, T, din, dout, dtype):
    pex_option("gram_norms", 0)
    X, G = si.custom(B, T, din, dout, dtype=dtype, seed=B)
    ref = on.example_norms(si.widen(X), si.widen(G))
    N = pex.pex_example_norms(X.to("cuda:0"), G.to("cuda:0")).cpu().double().numpy()
    # sums of din*dout squares of fp32-accumulated entries, all terms >= 0
    assert (np.abs(N - ref) <= 1e-4 * ref).all() and np.abs(N - ref).max() <= 2e-5 * ref.max()
    pex_option("max_split", 3)
    N3 = pex.pex_example_norms(X.to("cuda:0"), G.to("cuda:0")).cpu().double().numpy()
    assert np.array_equal(N, N3)          # an example is computed the same way whatever its group


@pytest.mark.parametrize("B,T,din,dout,dtype", [(61, 50, 72, 40, "bf16"), (61, 50, 72, 40, "f32"), (19, 300, 65, 67, "f32"),      # kernel of small layers
                                                (8, 512, 1152, 1280, "f32"), (40, 97, 1280, 516, "f32"),                         # fp32 layers by bf16 pieces
                                                (70, 33, 264, 40, "bf16"), (50, 190, 65, 72, "bf16"), (24, 64, 512, 1024, "bf16")])
def test_the_same_bits_whatever_the_bound_on_the_groups(pex_option, B, T, din, dout, dtype):
    X, G = si.custom(B, T, din, dout, dtype=dtype, seed=B)
    Xd, Gd = X.to("cuda:0"), G.to("cuda:0")
    N = pex.pex_example_norms(Xd, Gd)
    ref = on.example_norms(si.widen(X), si.widen(G))
    assert np.abs(N.cpu().double().numpy() - ref).max() <= 2e-5 * ref.max()
    for most in (31, 7, 1):
        pex_option("max_split", most)
        assert torch.equal(pex.pex_example_norms(Xd, Gd), N), most

"""The fp32 MFMA kernel at the edges of its tiles and of its ring of groups: widths that are no multiple of a tile (the
last tile overlaps its neighbour), sequence lengths that are no multiple of a 4-token group, fewer groups than ring slots,
plain contractions longer than one chunk, tiles of one wave and of four.  Against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_00236_amd as pex
import synth_inputs as si
from oracle import norms as on
from parity_util import assert_real_stat, assert_sign_stat

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

SHAPES = [
    (2, 9, 64, 64),        # one tile, three groups per example: fewer than the ring holds, the last one a single token
    (4, 5, 65, 66),        # one feature and two beyond a tile
    (3, 23, 127, 200),     # one feature short of two tiles; a panel of 8 features in the last column tile
    (5, 26, 68, 36),       # a column panel narrower than a tile (whole 16-byte chunks)
    (1, 17, 129, 191),     # a single example, three row tiles
    (19, 4, 100, 333),     # one group per example: a fold after every group
    (3, 700, 96, 70),      # plain contraction of two chunks and a rest
]


@pytest.mark.parametrize("B,T,din,dout", SHAPES)
def test_tile_and_ring_edges(B, T, din, dout):
    X, G = si.custom(B, T, din, dout, dtype="f32", seed=B * 31 + T)
    Xd, Gd = X.to(DEV), G.to(DEV)
    Xn, Gn = si.widen(X), si.widen(G)
    f = lambda t: t.cpu().numpy().astype(np.float64)
    st = oracle.stat(Xn, Gn)
    # outputs full of NaN: an entry no tile owns would show
    new = lambda: torch.full((din, dout), float("nan"), device=DEV)
    tag = f"B{B} T{T} {din}x{dout}"
    assert_real_stat(f(pex.pex_stat(Xd, Gd, "identity", S=new())), st.S_id, "f32", f"{tag} identity", elementwise=False)
    assert_real_stat(f(pex.pex_stat(Xd, Gd, "square", S=new())), st.S_sq, "f32", f"{tag} square", elementwise=B >= 3)
    assert_sign_stat(f(pex.pex_stat(Xd, Gd, "sign", S=new())), st.S_sign, st.amb, f"{tag} sign")
    assert_real_stat(f(pex.pex_token_sq(Xd, Gd, S=new())), oracle.token_sq(Xn, Gn), "f32", f"{tag} token_sq", elementwise=True)
    # sums of squares of entries that carry a 32-bit sum's rounding: 2e-5 of the largest, as for the statistics
    ref = on.example_norms(Xn, Gn)
    N = f(pex.pex_example_norms(Xd, Gd))
    assert np.abs(N - ref).max() <= 2e-5 * ref.max(), tag
    w = torch.linspace(-1.0, 2.0, B)
    S = f(pex.pex_weighted_sum(Xd, Gd, w.to(DEV), S=new()))
    assert_real_stat(S, on.weighted_sum(Xn, Gn, w.numpy()), "f32", f"{tag} weighted", elementwise=False)


def test_integer_inputs_are_bit_exact():
    """Every product and partial sum is a small integer, so overlapping tiles and folded chunks must match bit for bit."""
    X, G = si.integer_valued(3, 700, 101, 67, dtype="f32", seed=3)
    st = oracle.stat(si.widen(X), si.widen(G))
    for phi, ref in (("identity", st.S_id), ("square", st.S_sq), ("sign", st.S_sign)):
        got = pex.pex_stat(X.to(DEV), G.to(DEV), phi).cpu().numpy().astype(np.float64)
        assert np.array_equal(got, ref) if phi != "square" else np.abs(got - ref).max() <= 1e-6 * ref.max(), phi


@pytest.mark.parametrize("B,T,din,dout", [(3, 23, 127, 200), (19, 4, 100, 333), (140, 5, 70, 64)])
@pytest.mark.parametrize("want", [("identity", "square"), ("identity", "sign"), ("square", "sign"), ("identity", "square", "sign")])
def test_statistics_sharing_a_contraction(pex_option, B, T, din, dout, want):
    """Every combination against the oracle; with the batch in one group, 140 examples are more than a byte counter holds, so
    sign runs alone there."""
    pex_option("max_split", 1 if B > 127 else 32)
    X, G = si.custom(B, T, din, dout, dtype="f32", seed=B + T)
    st = oracle.stat(si.widen(X), si.widen(G))
    out = {k: torch.full((din, dout), float("nan"), device=DEV) for k in want}
    pex.pex_stat_multi(X.to(DEV), G.to(DEV), want, out=out)
    got = {k: v.cpu().numpy().astype(np.float64) for k, v in out.items()}
    if "identity" in got:
        assert_real_stat(got["identity"], st.S_id, "f32", "identity", elementwise=False)
    if "square" in got:
        assert_real_stat(got["square"], st.S_sq, "f32", "square", elementwise=True)
    if "sign" in got:
        assert_sign_stat(got["sign"], st.S_sign, st.amb, "sign")


@pytest.mark.parametrize("din,dout", [(152, 320), (44, 250), (250, 64), (190, 190)])
def test_arrangements_of_waves(din, dout):
    """Workgroups of 3 x 1, 1 x 4, 4 x 1 and 2 x 2 or 3 x 1 waves: layers whose tile counts leave 2 x 2 blocks half empty."""
    B, T = 5, 21
    X, G = si.custom(B, T, din, dout, dtype="f32", seed=din + dout)
    Xn, Gn = si.widen(X), si.widen(G)
    f = lambda t: t.cpu().numpy().astype(np.float64)
    st = oracle.stat(Xn, Gn)
    out = {k: torch.full((din, dout), float("nan"), device=DEV) for k in ("identity", "square")}
    pex.pex_stat_multi(X.to(DEV), G.to(DEV), ("identity", "square"), out=out)
    assert_real_stat(f(out["identity"]), st.S_id, "f32", "identity", elementwise=False)
    assert_real_stat(f(out["square"]), st.S_sq, "f32", "square", elementwise=True)
    ref = on.example_norms(Xn, Gn)
    assert np.abs(f(pex.pex_example_norms(X.to(DEV), G.to(DEV))) - ref).max() <= 2e-5 * ref.max()

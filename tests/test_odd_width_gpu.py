"""bf16 layers whose rows are not whole 16-byte chunks, on padded copies: every statistic against the fp64 oracle, on every
block shape and route the planner can choose, outputs of the layer's own widths inside a larger buffer (nothing may be
written around them)."""
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
f64 = lambda t: t.cpu().numpy().astype(np.float64)

# (B, T, din, dout), long enough that the planner takes the copies: X, G or both of odd width
SHAPES = [
    (3, 180, 65, 72),
    (2, 177, 264, 129),
    (4, 190, 257, 33),      # one feature beyond a 256-row block; padded to 40 columns
    (5, 300, 193, 391),     # the last column tile holds 7 features
    (3, 200, 250, 770),     # even widths that are no multiples of 8
]


class Guarded:
    """A [rows, cols] fp32 output full of NaN between two strips of a sentinel."""

    def __init__(self, rows, cols):
        self.n = rows * cols
        self.buf = torch.full((self.n + 128,), -7.0, device=DEV)
        self.view = self.buf[64:64 + self.n].view(rows, cols)
        self.view.fill_(float("nan"))

    def value(self):
        assert (self.buf[:64] == -7).all() and (self.buf[64 + self.n:] == -7).all(), "written outside the output"
        return f64(self.view)


def _padded(B, T, din, dout):
    odd = (din % 8 != 0) * -(-din // 8) * 8 + (dout % 8 != 0) * -(-dout // 8) * 8
    assert pex.pex_stat_workspace_bytes(B, T, din, dout, pex.PEX_BF16, "square") >= 2 * B * T * odd, "not on the copies"


@pytest.mark.parametrize("options", [{}, {"wide_blocks": 2}, {"wide_blocks": 0, "memory_fold": 0}, {"memory_fold": 2}, {"max_split": 1}])
@pytest.mark.parametrize("B,T,din,dout", SHAPES)
def test_statistics(pex_option, B, T, din, dout, options):
    for k, v in options.items():
        pex_option(k, v)
    _padded(B, T, din, dout)
    X, G = si.custom(B, T, din, dout, dtype="bf16", seed=B * 17 + T)
    Xd, Gd = X.to(DEV), G.to(DEV)
    Xn, Gn = si.widen(X), si.widen(G)
    st = oracle.stat(Xn, Gn)
    tag = f"B{B} T{T} {din}x{dout} {options}"
    out = {phi: Guarded(din, dout) for phi in ("identity", "square", "sign")}
    for phi, o in out.items():
        pex.pex_stat(Xd, Gd, phi, S=o.view)
    assert_real_stat(out["identity"].value(), st.S_id, "bf16", f"{tag} identity", elementwise=False)
    assert_real_stat(out["square"].value(), st.S_sq, "bf16", f"{tag} square", elementwise=B >= 3)
    assert_sign_stat(out["sign"].value(), st.S_sign, st.amb, f"{tag} sign")
    w = torch.linspace(-1.0, 2.0, B)
    o = Guarded(din, dout)
    pex.pex_weighted_sum(Xd, Gd, w.to(DEV), S=o.view)
    assert_real_stat(o.value(), on.weighted_sum(Xn, Gn, w.numpy()), "bf16", f"{tag} weighted", elementwise=False)
    o = Guarded(din, dout)
    pex.pex_stat_power(Xd, Gd, 1.5, S=o.view)
    ref = on.power_stat(Xn, Gn, 1.5)
    # as in the power tests: the contraction's rounding amplified by the exponent, plus that of log2 / exp2
    assert (np.abs(o.value() - ref) <= 1e-4 * ref + 1e-5 * ref.max()).all(), f"{tag} power"


@pytest.mark.parametrize("want", [("identity", "square"), ("identity", "sign"), ("square", "sign"), ("identity", "square", "sign")])
@pytest.mark.parametrize("B,T,din,dout", SHAPES[:4] + [(300, 4, 129, 250), (300, 40, 129, 250)])
def test_statistics_sharing_a_contraction(pex_option, B, T, din, dout, want):
    """With 300 examples in one group sign runs alone beside identity and square: on the SIMT kernel where the sequences are
    short, on the copies the others made where they are long."""
    if B > 127:
        pex_option("max_split", 1)
        alone, copies = pex.pex_stat_workspace_bytes(B, T, din, dout, pex.PEX_BF16, "sign"), 2 * B * T * (136 + 256)
        assert (alone == 0) if T == 4 else (copies <= alone < copies + 256)
    X, G = si.custom(B, T, din, dout, dtype="bf16", seed=B + T)
    st = oracle.stat(si.widen(X), si.widen(G))
    out = {k: Guarded(din, dout) for k in want}
    pex.pex_stat_multi(X.to(DEV), G.to(DEV), want, out={k: o.view for k, o in out.items()})
    if "identity" in want:
        assert_real_stat(out["identity"].value(), st.S_id, "bf16", "identity", elementwise=False)
    if "square" in want:
        assert_real_stat(out["square"].value(), st.S_sq, "bf16", "square", elementwise=B >= 3)
    if "sign" in want:
        assert_sign_stat(out["sign"].value(), st.S_sign, st.amb, "sign")


@pytest.mark.parametrize("route", [0, 1, 2, 3])
@pytest.mark.parametrize("B,T,din,dout", SHAPES)
def test_norms(pex_option, B, T, din, dout, route):
    pex_option("gram_norms", route)
    X, G = si.custom(B, T, din, dout, dtype="bf16", seed=B * 7 + T)
    ref = on.example_norms(si.widen(X), si.widen(G))
    N = f64(pex.pex_example_norms(X.to(DEV), G.to(DEV)))
    assert (np.abs(N - ref) <= 2e-5 * ref.max()).all() and (np.abs(N - ref) <= 1e-4 * ref).all(), (N, ref)


@pytest.mark.parametrize("route", [1, 2, 3])
@pytest.mark.parametrize("B,T,din,dout", [(4, 190, 257, 40), (16, 300, 1001, 770)])
def test_norms_of_tokens_that_are_alike(pex_option, B, T, din, dout, route):
    """Inputs near one vector and cotangents without a mean over the sequence: N_b is small against the entries of the T x T Gram
    matrices, whose product would cancel; a sum of squares cannot."""
    pex_option("gram_norms", route)
    X, G = si.custom(B, T, din, dout, dtype="f32", seed=B + 1)
    X = (1 + 0.03 * X).bfloat16()
    G = (G - G.mean(1, keepdim=True)).bfloat16()
    ref = on.example_norms(si.widen(X), si.widen(G))
    N = f64(pex.pex_example_norms(X.to(DEV), G.to(DEV)))
    # sums of T products of size |X||G| ~ 1 in fp32 against entries ~ 0.03 sqrt(T): 2e-5 as for the other sums of squares
    assert (np.abs(N - ref) <= 2e-5 * ref).all(), np.abs(N - ref) / ref


def test_without_a_workspace_large_copies_stay_on_the_simt_kernel():
    """Copies of 33 MB do not fit the library's scratch: the call still succeeds, by the other kernel."""
    B, T, din, dout = 4, 4160, 1001, 64
    assert pex.pex_stat_workspace_bytes(B, T, din, dout, pex.PEX_BF16, "identity") > pex.NOALLOC_SCRATCH_BYTES
    X, G = si.custom(B, T, din, dout, dtype="bf16", seed=2)
    o = Guarded(din, dout)
    pex.pex_stat_noalloc(X.to(DEV), G.to(DEV), "identity", o.view)
    ref = X.reshape(-1, din).double().t() @ G.reshape(-1, dout).double()
    assert_real_stat(o.value(), ref.numpy(), "bf16", "identity", elementwise=False)
    # and where they fit, pex_stat's bits
    B, T, din, dout = SHAPES[0]
    X, G = (t.to(DEV) for t in si.custom(B, T, din, dout, dtype="bf16", seed=3))
    o = Guarded(din, dout)
    pex.pex_stat_noalloc(X, G, "square", o.view)
    assert torch.equal(o.view, pex.pex_stat(X, G, "square"))


@pytest.mark.parametrize("B,T,din,dout", [(16, 300, 1001, 770), (7, 1111, 519, 904)])
def test_per_token_square_from_exact_halves(pex_option, B, T, din, dout):
    """The squares travel as two bf16 each that add up to them exactly: as accurate as fp32 squares (a rounded bf16 square alone
    would be off by up to 2^-9)."""
    halves = -(-din // 8) * 8 + -(-dout // 8) * 8
    assert pex.pex_token_sq_workspace_bytes(B, T, din, dout, pex.PEX_BF16) >= 4 * B * T * halves, "not on the halves"
    X, G = si.custom(B, T, din, dout, dtype="bf16", seed=5, g_std=1e-2, g_token="lognormal")
    o = Guarded(din, dout)
    pex.pex_token_sq(X.to(DEV), G.to(DEV), S=o.view)
    ref = (X.reshape(-1, din).to(DEV).double().square().t() @ G.reshape(-1, dout).to(DEV).double().square()).cpu().numpy()
    got = o.value()
    # terms >= 0 summed in fp32 (at most ~2000 rows per group, then the groups): 1e-5 of every entry
    assert (np.abs(got - ref) <= 1e-5 * ref).all(), float((np.abs(got - ref) / ref).max())
    pex_option("token_presquare", 0)        # fp32 squares in the SIMT kernel
    o = Guarded(din, dout)
    pex.pex_token_sq(X.to(DEV), G.to(DEV), S=o.view)
    assert (np.abs(o.value() - ref) <= 1e-5 * ref).all()


def test_per_token_square_of_infinities_and_of_the_largest_squares():
    """An infinite square meets remainders of zero and of every size and stays infinite; a zero makes it NaN; squares between the
    largest bf16 and the largest fp32 value stay finite; sums beyond fp32 overflow to infinity."""
    B, T, din, dout = 16, 300, 1001, 770
    X, G = si.custom(B, T, din, dout, dtype="bf16", seed=6)
    X[1, 3, 999] = float("inf")
    G[2, 7, 0] = float("-inf")
    X[0, 0, 2] = 1.842e19          # squared 3.393e38: finite in fp32, above the largest bf16
    G[0, 0, 769] = 1.0             # a square without a remainder
    G[1, 3, 5] = 0.0               # inf * 0
    X[:, :, 7] = 1e18
    G[:, :, 9] = 1e18              # products of 1e72
    X[4, 4, 11] = float("nan")
    halves = -(-din // 8) * 8 + -(-dout // 8) * 8
    assert pex.pex_token_sq_workspace_bytes(B, T, din, dout, pex.PEX_BF16) >= 4 * B * T * halves, "not on the halves"
    o = Guarded(din, dout)
    pex.pex_token_sq(X.to(DEV), G.to(DEV), S=o.view)
    got = o.value()
    x2, g2 = (t.reshape(B * T, -1).float().square().double() for t in (X, G))       # exact in fp32, or infinite
    ref = (x2.t() @ g2).float().double().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.isinf(ref).sum() > 1000 and np.isnan(ref).sum() > 700
    ok = np.isfinite(ref)
    assert (np.abs(got - ref)[ok] <= 1e-5 * ref[ok]).all()      # as above


def test_less_workspace_than_the_copies_take():
    """A call with enough for its partial sums alone (none, on these layers of many tiles) runs without the copies, on the SIMT
    kernel; with less than that it is refused."""
    B, T, din, dout = 8, 512, 768, 6001
    X, G = si.custom(B, T, din, dout, dtype="bf16", seed=8)
    Xd, Gd = X.to(DEV), G.to(DEV)
    Xf, Gf = Xd.double(), Gd.double()
    M = torch.stack([Xf[b].t() @ Gf[b] for b in range(B)])
    ref = {"identity": M.sum(0), "square": M.square().sum(0)}
    token = Xf.flatten(0, 1).square().t() @ Gf.flatten(0, 1).square()
    none = torch.empty(0, dtype=torch.uint8, device=DEV)
    close = lambda got, want, what: assert_real_stat(f64(got), f64(want), "bf16", what, elementwise=False)
    for phi in ref:
        assert pex.pex_stat_workspace_bytes(B, T, din, dout, pex.PEX_BF16, phi) > 0
        close(pex.pex_stat(Xd, Gd, phi, workspace=none), ref[phi], phi)
    both = pex.pex_stat_multi(Xd, Gd, ("identity", "square"), workspace=none)
    for phi in ref:
        close(both[phi], ref[phi], f"{phi} of both")
    assert pex.pex_token_sq_workspace_bytes(B, T, din, dout, pex.PEX_BF16) > 0
    close(pex.pex_token_sq(Xd, Gd, workspace=none), token, "token square")
    w = torch.linspace(-1.0, 2.0, B, device=DEV)
    close(pex.pex_weighted_sum(Xd, Gd, w, workspace=none), (w.double()[:, None, None] * M).sum(0), "weighted")
    need = -(-din // 64) * -(-dout // 64) * B * 4        # norms: a partial of every 64 x 64 tile and example
    N = pex.pex_example_norms(Xd, Gd, workspace=torch.empty(need, dtype=torch.uint8, device=DEV))
    close(N, M.square().sum((1, 2)), "norms")
    with pytest.raises(ValueError, match="workspace holds"):
        pex.pex_example_norms(Xd, Gd, workspace=torch.empty(need - 4, dtype=torch.uint8, device=DEV))
    few = (8, 256, 768, 1001)       # six groups of examples: less than their partial sums
    Xd, Gd = (t.to(DEV) for t in si.custom(*few, dtype="bf16", seed=9))
    with pytest.raises(ValueError, match="workspace holds"):
        pex.pex_stat(Xd, Gd, "square", workspace=torch.empty(768 * 1001 * 4, dtype=torch.uint8, device=DEV))


@pytest.mark.parametrize("B,T,din,dout", [(4, 190, 257, 40), (300, 40, 129, 250), (2100, 8, 129, 250)])
def test_sign_of_a_nan_counts_as_zero(pex_option, B, T, din, dout):
    """Entries of M_b that are NaN (a NaN in X or G, infinities of both signs) add nothing to the count, whatever represents it."""
    _padded(B, T, din, dout)
    X, G = si.custom(B, T, din, dout, dtype="bf16", seed=B)
    X[1, 3, din - 2] = float("nan")
    G[0, 5, 0] = float("nan")
    X[2, 0, 7], X[2, 1, 7], G[2, 0, :], G[2, 1, :] = float("inf"), float("-inf"), 1.0, 1.0
    M = [X[b].double().t() @ G[b].double() for b in range(B)]
    ref = sum(torch.nan_to_num(torch.sign(m), nan=0.0) for m in M).numpy()
    # the fp32 sum of an entry next to zero may have either sign
    amb = sum((m.abs() <= 1e-5 * torch.nan_to_num(m, nan=0.0, posinf=0.0, neginf=0.0).abs().max()).double() for m in M).numpy()
    for want in (("sign",), ("identity", "sign"), ("square", "sign"), ("identity", "square", "sign")):
        got = f64(pex.pex_stat_multi(X.to(DEV), G.to(DEV), want)["sign"])
        assert (np.abs(got - ref) <= 2 * amb).all(), want

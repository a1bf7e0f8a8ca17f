"""fp32 layers split into bf16 pieces: which layers take that route (host), and their results at the edges of its blocks, slabs and
groups, and where pieces cannot hold a value, against the fp64 oracle."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
import paper_2510_00236_amd as pex
import synth_inputs as si
from oracle import norms as on
from parity_util import assert_real_stat, assert_sign_stat

DEV = "cuda:0"
HERE = os.path.dirname(os.path.abspath(__file__))
MODES = range(7)      # identity, square, sign, per-token square, norms, weighted sum, power

SHAPES = [
    (5, 333, 1030, 900),      # last blocks overlap their neighbours in both widths; a slab of 13 tokens ends each example
    (17, 64, 1153, 1283),     # whole slabs, one feature beyond 9 blocks and 3 beyond 10
    (40, 97, 1280, 516),      # one token in the last slab
    (3, 1100, 2100, 1021),    # plain contractions of more than one chunk
]
PAIR_SHAPES = [(5, 700, 1030, 900), (6, 1025, 2100, 1021)]


def test_route(tmp_path):
    package = os.path.dirname(pex.LIB_PATH)
    exe = str(tmp_path / "probe")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(os.path.dirname(HERE), "include"),
                    "-I" + os.path.join(package, "csrc"), os.path.join(HERE, "pieces_probe.cpp"), pex.LIB_PATH, "-Wl,-rpath," + package,
                    "-Wl,--allow-shlib-undefined", "-o", exe], check=True)
    ask = lambda rows: subprocess.run([exe], input="".join("%d %d %d %d %d %d\n" % r for r in rows), stdout=subprocess.PIPE, text=True, check=True).stdout.split()
    assert set(ask([(*s, m, 0) for s in SHAPES for m in MODES] + [(*s, 1, 1) for s in PAIR_SHAPES + [(5, 666, 1030, 900)]])) == {"1"}
    # a few tokens per example, a handful of blocks, widths that are no whole chunks of a block
    assert set(ask([(64, 47, 2048, 2048, 1, 0), (8, 512, 64, 64, 1, 0), (64, 1024, 126, 4096, 1, 0), (64, 64, 2048, 2048, 1, 1)])) == {"0"}


@pytest.fixture
def large(pex_option):
    """Keeps the kernel of small layers out: the planner's options are about the others."""
    pex_option("max_split", 31)


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,din,dout", SHAPES)
def test_edges(large, B, T, din, dout):
    X, G = si.custom(B, T, din, dout, dtype="f32", seed=B * 31 + T)
    Xd, Gd = X.to(DEV), G.to(DEV)
    Xn, Gn = si.widen(X), si.widen(G)
    f = lambda t: t.cpu().numpy().astype(np.float64)
    st = oracle.stat(Xn, Gn)
    new = lambda: torch.full((din, dout), float("nan"), device=DEV)      # an entry no block owns would show
    tag = f"B{B} T{T} {din}x{dout}"
    assert_real_stat(f(pex.pex_stat(Xd, Gd, "identity", S=new())), st.S_id, "f32", f"{tag} identity", elementwise=False)
    assert_real_stat(f(pex.pex_stat(Xd, Gd, "square", S=new())), st.S_sq, "f32", f"{tag} square", elementwise=True)
    assert_sign_stat(f(pex.pex_stat(Xd, Gd, "sign", S=new())), st.S_sign, st.amb, f"{tag} sign")
    assert_real_stat(f(pex.pex_token_sq(Xd, Gd, S=new())), oracle.token_sq(Xn, Gn), "f32", f"{tag} token_sq", elementwise=True)
    ref = on.example_norms(Xn, Gn)
    assert np.abs(f(pex.pex_example_norms(Xd, Gd)) - ref).max() <= 2e-5 * ref.max(), tag
    w = torch.linspace(-1.0, 2.0, B)
    assert_real_stat(f(pex.pex_weighted_sum(Xd, Gd, w.to(DEV), S=new())), on.weighted_sum(Xn, Gn, w.numpy()), "f32", f"{tag} weighted", elementwise=False)
    # (an exponent above 1: below it an entry near zero carries the root of its rounding)
    assert_real_stat(f(pex.pex_stat_power(Xd, Gd, 1.5, S=new())), on.power_stat(Xn, Gn, 1.5), "f32", f"{tag} power", elementwise=False)


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,din,dout", PAIR_SHAPES)
def test_identity_added_up_in_memory(large, B, T, din, dout):
    """Twice into the same outputs, which hold NaN before: the first example of a group stores."""
    X, G = si.custom(B, T, din, dout, dtype="f32", seed=B + T)
    st = oracle.stat(si.widen(X), si.widen(G))
    out = {k: torch.full((din, dout), float("nan"), device=DEV) for k in ("identity", "square")}
    Xd, Gd = X.to(DEV), G.to(DEV)
    for _ in range(2):
        pex.pex_stat_multi(Xd, Gd, ("identity", "square"), out=out)
        got = {k: v.cpu().numpy().astype(np.float64) for k, v in out.items()}
        assert_real_stat(got["identity"], st.S_id, "f32", "identity", elementwise=False)
        assert_real_stat(got["square"], st.S_sq, "f32", "square", elementwise=True)


def _special(kind):
    X, G = si.custom(5, 333, 1030, 900, dtype="f32", seed=3)
    X, G = X.clone(), G.clone()
    if kind == "infinity":
        X[1, 3, 7] = float("inf")
    elif kind == "nan":
        G[2, 332, 899] = float("nan")
    elif kind == "rounds up to 2^128":
        X[0, 0, 200] = 3.4028e38
        G *= 1e-3
    elif kind == "tiny feature":
        X[3, :, 17] *= 1e-36
    elif kind == "tiny":
        X *= 1e-35
    return X, G


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["infinity", "nan", "rounds up to 2^128", "tiny feature", "tiny"])
def test_values_that_pieces_do_not_hold(large, kind):
    """The entries an infinity or NaN does not reach keep their precision, the others are what sums of products in fp32 give (signs of
    a NaN count as 0); a feature far below the others is as exact as they are."""
    X, G = _special(kind)
    Xd, Gd = X.to(DEV), G.to(DEV)
    with np.errstate(all="ignore"):
        M = np.stack([X[b].double().numpy().T @ G[b].double().numpy() for b in range(X.shape[0])])
        ref = {"identity": M.sum(0), "square": (M * M).sum(0), "sign": np.sign(np.nan_to_num(M, nan=0.0)).sum(0)}
    out = {phi: pex.pex_stat(Xd, Gd, phi) for phi in ref}
    big = {k: torch.empty_like(v) for k, v in out.items() if k != "sign"}
    pex.pex_stat_multi(torch.cat([Xd, Xd], 1), torch.cat([Gd, torch.zeros_like(Gd)], 1), ("identity", "square"), out=big)
    pairs = [(phi, out[phi], ref[phi]) for phi in ref] + [(phi, big[phi], ref[phi]) for phi in big if kind not in ("infinity",)]
    for phi, S, r in pairs:
        S = S.cpu().double().numpy()
        finite = np.abs(r) < 3.4e38          # what overflows fp32 is infinite
        assert np.array_equal(np.isfinite(S), finite), (kind, phi)
        assert np.array_equal(np.isnan(S), np.isnan(r)), (kind, phi)
        if phi == "sign":
            assert np.abs(S - r).max() <= 2 and (S != r).mean() < 1e-5, kind
        elif not (kind == "tiny" and phi == "square"):      # (those squares underflow)
            rows = [slice(17, 18), slice(0, 17), slice(18, None)]
            for k in rows:
                ok = finite[k]
                err = np.abs(S[k] - r[k])[ok].max() / np.abs(r[k])[ok].max()
                assert err <= 2e-5, (kind, phi, k, err)


# ---- a width below a block's: lanes parked outside the operand, masks of stores, norms and S_id in memory

NARROW = [(16, 512, 100, 2052), (16, 512, 2052, 100), (16, 1000, 96, 4096)]


def test_route_of_narrow_widths(tmp_path):
    package = os.path.dirname(pex.LIB_PATH)
    exe = str(tmp_path / "probe")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(os.path.dirname(HERE), "include"),
                    "-I" + os.path.join(package, "csrc"), os.path.join(HERE, "pieces_probe.cpp"), pex.LIB_PATH, "-Wl,-rpath," + package,
                    "-Wl,--allow-shlib-undefined", "-o", exe], check=True)
    rows = [(*s, m, 0) for s in NARROW + [EXACT] for m in MODES] + [(*s, 1, 1) for s in NARROW]
    out = subprocess.run([exe], input="".join("%d %d %d %d %d %d\n" % r for r in rows), stdout=subprocess.PIPE, text=True, check=True).stdout
    assert set(out.split()) == {"1"}


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,din,dout", NARROW)
def test_edges_of_narrow_widths(large, B, T, din, dout):
    test_edges(large, B, T, din, dout)
    test_identity_added_up_in_memory(large, B, T, din, dout)


# ---- no less exact than fp32 products

EXACT = (8, 512, 1152, 1280)


def _operands(kind):
    B, T, din, dout = EXACT
    g = torch.Generator(device=DEV).manual_seed(3)
    X, G = torch.randn(B, T, din, device=DEV, generator=g), torch.randn(B, T, dout, device=DEV, generator=g)
    where, _, count = kind.partition(" ")
    if kind == "no negative values":
        X.clamp_(min=0)
    elif where == "first":
        X[:, int(count):] = 0
    elif where == "apart":
        keep = torch.zeros(B, T, 1, device=DEV)
        keep[:, torch.arange(int(count), device=DEV) * 32 + 7] = 1
        X *= keep
    elif kind == "constant":                # the products left out are at their largest, 2^-24, and of one sign
        X.fill_(1.00390625 - 2.0**-16)
        G.fill_(1.00390625 - 2.0**-16)
    elif kind == "tiny beside normal":      # the normal values meet zeros
        X[:, 32:] *= 2.0**-118
        G[:, :32] = 0
        G *= 2.0**70                        # results near 2^-44, whose squares are normal numbers
    elif kind == "denormal":
        X *= 1e-41
        G *= 1e30
    return X, G


@pytest.mark.gpu
@pytest.mark.parametrize("kind,factor", [
    ("dense", 0.6), ("no negative values", 0.6), ("first 1", 1.1), ("first 4", 1.0), ("first 16", 0.8), ("constant", 1.0), ("tiny beside normal", 0.6), ("denormal", 0.6),
    # two tokens of different 32's: each product is rounded once more before it is added, sqrt(4 / 3) of the error if roundings are
    # independent; the share of that falls with their number
    ("apart 2", 1.3), ("apart 4", 1.2), ("apart 16", 1.1)])
def test_no_less_exact_than_fp32_products(large, kind, factor):
    """2-norm of the error against 64-bit sums, beside that of the fp32 MFMA kernel (all three statistics together run there)."""
    X, G = _operands(kind)
    S_id = S_sq = 0.0
    for b in range(EXACT[0]):
        M = X[b].double().t() @ G[b].double()
        S_id, S_sq = S_id + M, S_sq + M * M
    err = lambda S, R: float((S.double() - R).norm() / R.norm())
    fp32 = pex.pex_stat_multi(X, G, ("identity", "square", "sign"))
    pair = pex.pex_stat_multi(torch.cat([X, torch.zeros_like(X)], 1), torch.cat([G, torch.zeros_like(G)], 1), ("identity", "square"))
    for name, got, ref in (("square", pex.pex_stat(X, G, "square"), S_sq), ("square", pair["square"], S_sq), ("identity", pair["identity"], S_id),
                           ("identity", pex.pex_weighted_sum(X, G, torch.ones(EXACT[0], device=DEV)), S_id)):
        assert err(got, ref) <= max(factor * err(fp32[name], ref), 3e-8), name      # (half a unit in the last place, whatever the sums)
    # identity by itself adds up 1024 tokens of several examples at a time, not each example's: up to twice the additions at full size
    assert err(pex.pex_stat(X, G, "identity"), S_id) <= max(2.0 ** 0.5 * max(factor, 1.0) * err(fp32["identity"], S_id), 3e-8)


# ---- tiles made again with fp32 products: the statistics that keep something per example

@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["infinity", "nan", "rounds up to 2^128", "tiny feature"])
def test_the_other_statistics_where_pieces_do_not_hold(large, kind):
    X, G = _special(kind)
    B, _, din = X.shape
    Xd, Gd, w = X.to(DEV), G.to(DEV), torch.linspace(-1.0, 2.0, B)
    with np.errstate(all="ignore"):
        Xn, Gn = X.double().numpy(), G.double().numpy()
        M = np.stack([Xn[b].T @ Gn[b] for b in range(B)])
        ref = {"weighted": (w.double().numpy()[:, None, None] * M).sum(0), "power": (np.abs(M) ** 1.5).sum(0),
               "token": sum((Xn[b] ** 2).T @ Gn[b] ** 2 for b in range(B))}
        norms = (M * M).sum((1, 2))
    got = {"weighted": pex.pex_weighted_sum(Xd, Gd, w.to(DEV)), "power": pex.pex_stat_power(Xd, Gd, 1.5), "token": pex.pex_token_sq(Xd, Gd)}
    for name, r in ref.items():
        S = got[name].cpu().double().numpy()
        finite = np.abs(r) < 3.4e38          # what overflows fp32 is infinite
        assert np.array_equal(np.isfinite(S), finite) and np.array_equal(np.isnan(S), np.isnan(r)), (kind, name)
        for rows in (slice(0, 200), slice(200, 201), slice(201, din)):
            ok = finite[rows]
            if ok.any():
                assert np.abs(S[rows][ok] - r[rows][ok]).max() <= 2e-5 * np.abs(r[rows][ok]).max(), (kind, name, rows)
    N = pex.pex_example_norms(Xd, Gd).cpu().double().numpy()
    finite = norms < 3.4e38
    assert np.array_equal(np.isfinite(N), finite) and np.array_equal(np.isnan(N), np.isnan(norms)), kind
    assert (np.abs(N[finite] - norms[finite]) <= 2e-5 * norms[finite]).all(), kind

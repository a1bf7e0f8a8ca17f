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

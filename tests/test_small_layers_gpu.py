"""The kernel of small layers: where the planner takes it (host), its results at the edges of its tiles, steps, shares of tokens and
groups of examples against the fp64 oracle, and the other kernels on the same layers (an option away from its default keeps them)."""
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

SHAPES = [
    (9, 200, 4, 4, "f32"), (9, 200, 4, 4, "bf16"),          # one quad of features
    (2, 9, 64, 64, "bf16"), (2, 9, 64, 64, "f32"),          # one whole tile
    (5, 16, 65, 67, "f32"), (5, 17, 65, 67, "f32"),         # one step and a token; the last quad of each width overlaps
    (5, 32, 61, 130, "bf16"), (5, 33, 61, 130, "bf16"),
    (3, 257, 63, 34, "bf16"), (3, 129, 63, 34, "f32"),      # tokens divided over eight waves, one of them with a single token more
    (2, 1100, 130, 7, "bf16"), (2, 1100, 130, 7, "f32"),
    (1, 9000, 20, 31, "bf16"), (1, 9000, 20, 31, "f32"),    # a plain contraction in two shares
    (19, 20, 37, 130, "bf16"), (19, 20, 37, 130, "f32"),    # examples that do not divide by eight waves
    (61, 50, 72, 40, "bf16"), (61, 50, 72, 40, "f32"),      # groups of examples, their sums exchanged
    (200, 6, 33, 70, "bf16"), (200, 6, 33, 70, "f32"),
]


def _ask(tmp_path, rows):
    package = os.path.dirname(pex.LIB_PATH)
    exe = str(tmp_path / "probe")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(os.path.dirname(HERE), "include"),
                    "-I" + os.path.join(package, "csrc"), os.path.join(HERE, "small_probe.cpp"), pex.LIB_PATH, "-Wl,-rpath," + package,
                    "-Wl,--allow-shlib-undefined", "-o", exe], check=True)
    out = subprocess.run([exe], input="".join("%d %d %d %d %d %d\n" % r for r in rows), stdout=subprocess.PIPE, text=True, check=True).stdout
    return [tuple(int(v) for v in l.split()) for l in out.splitlines()]


def test_route(tmp_path):
    code = {"f32": pex.PEX_F32, "bf16": pex.PEX_BF16}
    got = {}
    for mode in (0, 1, 2, 4, 5, 6):
        for s, (kw, nsplit) in zip(SHAPES, _ask(tmp_path, [(*s[:4], code[s[4]], mode) for s in SHAPES])):
            got.setdefault(s, set()).add((kw, nsplit > 1))
    # every shape is on the kernel with some statistic, and among them are both ways to divide the work, with and without groups
    assert all(any(kw > 0 for kw, _ in v) for v in got.values()), got
    assert {x for v in got.values() for x in v} >= {(1, False), (1, True), (8, False), (8, True)}
    # examples of three tokens, layers that fill the chip
    assert _ask(tmp_path, [(9, 3, 64, 64, 1, 1), (16, 2048, 2048, 8192, 1, 1), (16, 1024, 1024, 4096, 0, 1), (8, 256, 768, 50257, 1, 1)]) \
        .__repr__().count("(0, ") == 4


def _check(B, T, din, dout, dtype):
    X, G = si.custom(B, T, din, dout, dtype=dtype, seed=B * 31 + T)
    Xd, Gd, Xn, Gn = X.to(DEV), G.to(DEV), si.widen(X), si.widen(G)
    f = lambda t: t.cpu().numpy().astype(np.float64)
    st = oracle.stat(Xn, Gn)
    new = lambda: torch.full((din, dout), float("nan"), device=DEV)      # an entry no tile owns would show
    tag = f"B{B} T{T} {din}x{dout} {dtype}"
    assert_real_stat(f(pex.pex_stat(Xd, Gd, "identity", S=new())), st.S_id, dtype, f"{tag} identity", elementwise=False)
    assert_real_stat(f(pex.pex_stat(Xd, Gd, "square", S=new())), st.S_sq, dtype, f"{tag} square", elementwise=False)
    assert_sign_stat(f(pex.pex_stat(Xd, Gd, "sign", S=new())), st.S_sign, st.amb, f"{tag} sign")
    if dtype == "f32":
        assert_real_stat(f(pex.pex_token_sq(Xd, Gd, S=new())), oracle.token_sq(Xn, Gn), dtype, f"{tag} token_sq", elementwise=True)
    ref = on.example_norms(Xn, Gn)
    assert np.abs(f(pex.pex_example_norms(Xd, Gd)) - ref).max() <= 2e-5 * ref.max(), tag
    w = torch.linspace(-1.0, 2.0, B)
    S = f(pex.pex_weighted_sum(Xd, Gd, w.to(DEV), S=new()))
    assert_real_stat(S, on.weighted_sum(Xn, Gn, w.numpy()), dtype, f"{tag} weighted", elementwise=False)
    assert_real_stat(f(pex.pex_stat_power(Xd, Gd, 1.5, S=new())), on.power_stat(Xn, Gn, 1.5), dtype, f"{tag} power", elementwise=False)
    out = {"identity": new(), "square": new()}
    pex.pex_stat_multi(Xd, Gd, ("identity", "square"), out=out)
    assert_real_stat(f(out["identity"]), st.S_id, dtype, f"{tag} pair", elementwise=False)
    assert_real_stat(f(out["square"]), st.S_sq, dtype, f"{tag} pair", elementwise=False)


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,din,dout,dtype", SHAPES)
def test_edges(B, T, din, dout, dtype):
    _check(B, T, din, dout, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,din,dout,dtype", [
    (3, 100, 200, 136, "bf16"), (5, 77, 520, 264, "bf16"), (2, 37, 70, 33, "bf16"), (2, 37, 70, 33, "f32"), (3, 50, 129, 65, "f32"),
    (7, 33, 256, 128, "bf16"), (1, 64, 96, 160, "bf16"), (40, 24, 512, 520, "bf16"), (3, 50, 132, 68, "f32"), (5, 77, 521, 265, "bf16"),
    (2, 9, 64, 64, "f32"), (4, 5, 65, 66, "f32"), (3, 23, 127, 200, "f32"), (5, 26, 68, 36, "f32"), (19, 4, 100, 333, "f32")])
def test_the_other_kernels_on_small_layers(pex_option, B, T, din, dout, dtype):
    pex_option("max_split", 31)
    _check(B, T, din, dout, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,din,dout", [("f32", 70, 66), ("bf16", 72, 64), ("bf16", 71, 66)])
def test_infinities_and_nan_as_on_the_other_kernels(pex_option, dtype, din, dout):
    """The same entries non-finite, the same sign counts (a NaN counts as -1 on bf16 layers of whole 16-byte chunks, as 0 elsewhere),
    the same finite norms beside an infinity of another example."""
    X, G = si.custom(11, 40, din, dout, dtype=dtype, seed=4)
    X, G = X.clone(), G.clone()
    X[1, 3, din - 1] = float("inf")
    G[2, 39, dout - 1] = float("nan")
    X[4, 0, 0] = float("inf")
    G[4, 0, 0] = 0.0
    Xd, Gd = X.to(DEV), G.to(DEV)

    def results():
        return {**{phi: pex.pex_stat(Xd, Gd, phi) for phi in ("identity", "square", "sign")}, "norms": pex.pex_example_norms(Xd, Gd),
                "weighted": pex.pex_weighted_sum(Xd, Gd, torch.ones(11, device=DEV))}

    small = results()
    pex_option("max_split", 31)
    for k, v in results().items():
        assert torch.equal(torch.isnan(small[k]), torch.isnan(v)) and torch.equal(torch.isinf(small[k]), torch.isinf(v)), k
        ok = torch.isfinite(v)
        assert torch.equal(small[k][ok], v[ok]) if k == "sign" else (small[k][ok] - v[ok]).abs().max() <= 2e-5 * v[ok].abs().max(), k


def test_layers_the_caches_bound_stay_on_the_large_kernels(tmp_path):
    """Many tokens in some dozen tiles, rows that do not start at cache lines: every tile reads its features of all tokens."""
    rows = [(22, 2887, 181, 680, 1, 0), (88, 255, 158, 1313, 1, 0), (110, 535, 328, 350, 1, 0), (110, 535, 328, 350, 1, 1), (84, 775, 579, 258, 1, 0), (20, 3261, 512, 192, 1, 0)]
    assert [kw for kw, _ in _ask(tmp_path, rows)] == [0] * len(rows)


def test_several_statistics_are_planned_for_what_they_cost(tmp_path):
    """Identity and square on tiles of half the width, twice the workgroups: layers whose square alone is one round of them stay on the large
    kernels if the pair is two; what test_several_statistics_at_once runs is on the kernel, with both ways to divide the work and with groups."""
    assert [kw for kw, _ in _ask(tmp_path, [(115, 342, 192, 807, 1, 7), (193, 176, 192, 959, 1, 7), (43, 1507, 344, 192, 1, 7)])] == [0, 0, 0]
    code = {"f32": pex.PEX_F32, "bf16": pex.PEX_BF16}
    got = _ask(tmp_path, [(*s[:4], code[s[4]], 7) for s in SEVERAL])
    assert {(kw, ns > 1) for kw, ns in got} == {(1, False), (1, True), (8, False), (8, True)}, got


SEVERAL = [(9, 200, 4, 4, "f32"), (2, 9, 64, 64, "bf16"), (5, 17, 65, 67, "f32"), (5, 33, 61, 130, "bf16"), (3, 257, 63, 34, "bf16"), (3, 129, 63, 34, "f32"),
           (2, 1100, 130, 7, "bf16"), (19, 20, 37, 130, "bf16"), (61, 50, 72, 40, "bf16"), (200, 6, 33, 70, "f32"), (61, 300, 72, 40, "bf16"), (61, 300, 72, 40, "f32"),
           (31, 40, 200, 300, "bf16"), (1, 900, 70, 130, "bf16")]


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,din,dout,dtype", SEVERAL)
def test_several_statistics_at_once(B, T, din, dout, dtype):
    X, G = si.custom(B, T, din, dout, dtype=dtype, seed=B * 31 + T)
    Xd, Gd = X.to(DEV), G.to(DEV)
    st = oracle.stat(si.widen(X), si.widen(G))
    f = lambda t: t.cpu().numpy().astype(np.float64)
    for want in (("identity", "square"), ("identity", "sign"), ("square", "sign"), ("identity", "square", "sign")):
        out = {k: torch.full((din, dout), float("nan"), device=DEV) for k in want}
        pex.pex_stat_multi(Xd, Gd, want, out=out)
        tag = f"B{B} T{T} {din}x{dout} {dtype} {want}"
        if "identity" in want:
            assert_real_stat(f(out["identity"]), st.S_id, dtype, tag, elementwise=False)
        if "square" in want:
            assert_real_stat(f(out["square"]), st.S_sq, dtype, tag, elementwise=False)
        if "sign" in want:
            assert_sign_stat(f(out["sign"]), st.S_sign, st.amb, tag)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,dout,nan_sign", [("f32", 66, 0.0), ("bf16", 64, -1.0), ("bf16", 66, 0.0)])
def test_signs_of_nan_in_company(dtype, dout, nan_sign):
    X, G = si.custom(11, 40, 72, dout, dtype=dtype, seed=4)
    G = G.clone()
    G[2, 39, dout - 1] = float("nan")
    alone = pex.pex_stat(X.to(DEV), G.to(DEV), "sign")
    got = pex.pex_stat_multi(X.to(DEV), G.to(DEV), ("identity", "square", "sign"))
    rest = [b for b in range(11) if b != 2]
    others = oracle.stat(si.widen(X[rest]), si.widen(G[rest]))
    clear = others.amb[:, -1] == 0
    assert np.array_equal(got["sign"].cpu().numpy()[clear, -1], others.S_sign[clear, -1] + nan_sign)
    assert torch.equal(got["sign"][:, :-1], alone[:, :-1]) and torch.isnan(got["square"][:, -1]).all() and torch.isfinite(got["square"][:, :-1]).all()


def test_workspace_is_what_the_layer_needs_either_way(tmp_path, pex_option):
    """The query holds the partial sums of the plan and whatever the layer asks for without the kernel, not copies that it does not make
    for each of several statistics (an option that is about neither statistic keeps the kernel out)."""
    code = {"f32": pex.PEX_F32, "bf16": pex.PEX_BF16}
    shapes = SEVERAL + [(2, 1050, 1934, 128, "bf16"), (8, 700, 300, 333, "bf16")]
    plans = _ask(tmp_path, [(*s[:4], code[s[4]], 7) for s in shapes])
    wants = (("identity", "square"), ("square", "sign"), ("identity", "square", "sign"))
    query = lambda s: [pex.pex_stat_multi_workspace_bytes(*s[:4], code[s[4]], w) for w in wants]
    got = [query(s) for s in shapes]
    pex_option("gram_norms", 0)
    for s, (kw, ns), now in zip(shapes, plans, got):
        assert kw > 0, s
        for w, bytes_now, without in zip(wants, now, query(s)):
            assert bytes_now == max(without, len(w) * ns * s[2] * s[3] * 4 if ns > 1 else 0), (s, w)


@pytest.mark.gpu
def test_workspaces_of_every_size_that_was_enough(pex_option):
    """Less than the query, but enough without the kernel or without copies: the same statistics; less than that is refused."""
    for B, T, din, dout, dtype in [(61, 300, 72, 40, "bf16"), (61, 300, 72, 40, "f32"), (200, 6, 33, 70, "f32"), (24, 700, 100, 131, "bf16"), (40, 300, 200, 201, "bf16")]:
        code = pex.PEX_F32 if dtype == "f32" else pex.PEX_BF16
        X, G = si.custom(B, T, din, dout, dtype=dtype, seed=B + T)
        Xd, Gd = X.to(DEV), G.to(DEV)
        st = oracle.stat(si.widen(X), si.widen(G))
        sizes = set()
        for option in (1, 0):
            pex_option("gram_norms", option)
            sizes.add(pex.pex_stat_multi_workspace_bytes(B, T, din, dout, code, ("identity", "square")))
            sizes.add(pex.pex_stat_workspace_bytes(B, T, din, dout, code, "square"))
        pex_option("gram_norms", 1)
        done = set()
        S = {k: torch.empty(din, dout, device=DEV) for k in ("identity", "square")}
        for size in sorted(sizes | {max(sizes) * 2}):
            ws = torch.full((size + 4096,), 77, dtype=torch.uint8, device=DEV)
            for pair in (True, False):
                for t in S.values():
                    t.fill_(float("nan"))
                if pair:
                    rc = pex.lib().pex_stat_multi(Xd.data_ptr(), Gd.data_ptr(), B, T, din, dout, code, 3, S["identity"].data_ptr(), S["square"].data_ptr(), None, ws.data_ptr(), size, None)
                else:
                    rc = pex.lib().pex_stat(Xd.data_ptr(), Gd.data_ptr(), B, T, din, dout, code, pex.PEX_PHI_SQUARE, S["square"].data_ptr(), ws.data_ptr(), size, None)
                torch.cuda.synchronize()
                assert (ws[size:] == 77).all() and rc in (0, 6)
                if rc == 0:
                    done.add(pair)
                    assert_real_stat(S["square"].cpu().double().numpy(), st.S_sq, dtype, f"{size} bytes", elementwise=False)
                    if pair:
                        assert_real_stat(S["identity"].cpu().double().numpy(), st.S_id, dtype, f"{size} bytes", elementwise=False)
                else:
                    assert torch.isnan(S["square"]).all()
        assert done == {True, False}

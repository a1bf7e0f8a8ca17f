"""Planner choices (host only): those seen in the workspace a call asks for, others through a small program linked to the
library (plan_probe.cpp); plans made while another thread sets an option (plan_race.cpp)."""
import os
import subprocess

import pytest

import paper_2510_00236_amd as pex

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
MODE = {"identity": 0, "square": 1, "sign": 2, "token_sq": 3, "norms": 4, "weighted": 5, "power": 6}


def _compile(source, exe):
    package = os.path.dirname(pex.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(package, "csrc"), os.path.join(HERE, source), pex.LIB_PATH, "-Wl,-rpath," + package, "-Wl,--allow-shlib-undefined",
                    "-pthread", "-o", exe], check=True)
    return exe


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = _compile("plan_probe.cpp", str(tmp_path_factory.mktemp("plan") / "probe"))

    def ask(shapes):
        """[(B, T, din, dout, dtype code, statistic)] -> [(kernel, nsplit, per_split, blocks, threads)]"""
        text = "".join(f"{B} {T} {i} {o} {dt} {MODE[m]}\n" for B, T, i, o, dt, m in shapes)
        out = subprocess.run([exe], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout
        return [tuple(int(v) for v in l.split()) for l in out.splitlines()]

    return ask


def test_launches_stay_below_the_grid_limit(plans):
    """gridDim.x * blockDim.x of a launch is below 2^32, however many groups of examples would pay."""
    shapes = [(1021, 16, 8192, 50257, pex.PEX_F32, "norms"), (1021, 16, 16448, 16448, pex.PEX_F32, "norms"), (997, 8, 4096, 128256, pex.PEX_F32, "norms"),
              (16, 1, 131136, 131136, pex.PEX_F32, "norms"), (1021, 16, 32768, 32776, pex.PEX_BF16, "norms"), (1021, 16, 16384, 131080, pex.PEX_BF16, "norms"),
              (1021, 16, 8192, 50257, pex.PEX_F32, "square")]
    for shape, (kernel, nsplit, per_split, blocks, threads) in zip(shapes, plans(shapes)):
        assert kernel in (1, 2), shape
        assert blocks * nsplit * threads < 2**32, (shape, nsplit, blocks, threads)
        assert (nsplit - 1) * per_split < shape[0] <= nsplit * per_split, shape      # every example in a group, none empty


def test_fp32_plans_fit_the_librarys_scratch_where_the_call_without_a_workspace_takes_them():
    # three workgroups per unit of 128 x 128 blocks, 16 groups of 1 MiB: charged 16 MiB, so held to the scratch
    assert pex.pex_stat_workspace_bytes(64, 128, 512, 512, pex.PEX_F32, "square") <= pex.NOALLOC_SCRATCH_BYTES
    # charged more than the scratch: as many groups as pay
    assert pex.pex_stat_workspace_bytes(16, 512, 1536, 1536, pex.PEX_F32, "square") > pex.NOALLOC_SCRATCH_BYTES


def test_kept_plans_are_those_of_their_options(tmp_path):
    exe = _compile("plan_race.cpp", str(tmp_path / "race"))
    out = subprocess.run([exe], stdout=subprocess.PIPE, text=True, check=True, timeout=100).stdout
    assert int(out) == 0, f"{out.strip()} plans kept under an option they were not made with"


def test_squares_inside_the_contraction_where_the_option_asks_for_it(pex_option):
    """No copies of squares under value 0, of layers of odd width either."""
    odd, even = (16, 300, 1001, 770, pex.PEX_BF16), (16, 2048, 2048, 8192, pex.PEX_BF16)
    copies = [2 * 2 * 16 * 300 * (1008 + 776), 2 * 16 * 2048 * (2048 + 8192)]
    assert [pex.pex_token_sq_workspace_bytes(*s) >= c for s, c in zip((odd, even), copies)] == [True, True]
    pex_option("token_presquare", 0)
    assert [pex.pex_token_sq_workspace_bytes(*s) >= c for s, c in zip((odd, even), copies)] == [False, False]


def test_short_examples(plans):
    """What an example costs besides its tokens is part of the plan: layers of odd width whose examples are a few tokens take more
    groups or stay on the SIMT kernel, long ones leave it; fp32 examples of one token spread over many groups; the norms take no more groups than
    save a round of workgroups."""
    BF, F = pex.PEX_BF16, pex.PEX_F32
    kernels = lambda shapes: [p[0] for p in plans(shapes)]
    assert kernels([(592, 2, 2139, 64, BF, "power"), (72, 45, 43, 5632, BF, "power"), (67, 1, 9093, 4664, BF, "token_sq")]) == [0] * 3
    assert plans([(79, 3, 4984, 259, BF, "sign")])[0][:2] == (1, 6)      # (one group of 79 examples before: 241 us, 87 on the SIMT kernel)
    assert kernels([(79, 300, 4984, 259, BF, "sign"), (592, 200, 2139, 64, BF, "power"), (8, 256, 768, 50257, BF, "square"), (14, 544, 3776, 1943, BF, "token_sq")]) == [1] * 4
    assert all(p[0] == 2 and p[1] >= 8 for p in plans([(72, 1, 880, 128, F, "power"), (26, 1, 118, 384, F, "sign"), (36, 1, 694, 64, F, "power")]))
    assert plans([(131, 67, 10304, 64, BF, "norms")])[0][1] == 6 and plans([(56, 1150, 64, 312, BF, "norms")])[0][1] == 56

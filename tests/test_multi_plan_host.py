"""Plans of several statistics at once (host only): the M_b of few long examples through the workspace, and what the calls ask for where that is not
the way they go (multi_probe.cpp, linked to the library)."""
import os
import subprocess

import pytest

import paper_2510_00236_amd as pex
from test_plan_host import _compile

BF, MIB = pex.PEX_BF16, 1 << 20


@pytest.fixture(scope="module")
def multi(tmp_path_factory):
    exe = _compile("multi_probe.cpp", str(tmp_path_factory.mktemp("multi") / "probe"))

    def ask(shapes, **env):
        """[(B, T, din, dout)] -> [(examples, nsplit, per_split, query, plain, small, within, odd)] of identity and square, bf16"""
        text = "".join(f"{B} {T} {i} {o} {BF} 3\n" for B, T, i, o in shapes)
        out = subprocess.run([exe], input=text, stdout=subprocess.PIPE, text=True, check=True, env=dict(os.environ, **env)).stdout
        return [tuple(int(v) for v in l.split()) for l in out.splitlines()]

    return ask


# On the kernel of small layers, with the workspace the layer needs without it (bytes).
SMALL = [((224, 292, 128, 256), 8 * MIB), ((66, 881, 128, 320), 7208960), ((72, 898, 64, 128), 1572864), ((110, 593, 768, 64), 11010048)]


def test_small_layers_ask_for_no_room_for_their_examples(multi):
    for (shape, needs), (examples, _, _, query, plain, small, within, _) in zip(SMALL, multi([s for s, _ in SMALL])):
        assert small and not examples, shape
        assert query == plain == needs, (shape, query, plain)
        assert within <= needs, (shape, within)


def test_partial_sums_alone_are_enough(multi):
    """Whatever way a layer goes, a workspace for its partial sums alone is accepted."""
    shapes = [(B, T, i, o) for B in (2, 3, 5, 17, 72, 224) for T in (24, 292, 898, 2048) for i in (64, 128, 768, 2304) for o in (64, 256, 1408, 4096)]
    plans = multi(shapes)
    assert any(p[0] for p in plans) and any(p[5] for p in plans)
    for shape, (_, _, _, query, plain, _, within, _) in zip(shapes, plans):
        assert within <= plain <= query, (shape, query, plain, within)


def test_layers_that_need_no_workspace_take_one_at_any_address(multi):
    shapes = [(4, 8192, 4096, 4096), (1, 8192, 4096, 4096), (7, 2864, 2944, 2304)]
    for shape, (examples, nsplit, _, query, plain, _, _, odd) in zip(shapes, multi(shapes)):
        assert examples and nsplit == 1 and query == 4 * shape[0] * shape[2] * shape[3] and plain == 0, shape
        assert odd == 0, (shape, odd)


@pytest.mark.parametrize("B,T,d,needs", [(3, 1508, 1536, 56623104), (21, 2674, 1024, 201326592), (83, 526, 256, 62914560)])
def test_layers_in_one_launch_ask_for_no_room_for_their_examples(multi, B, T, d, needs):
    """A block whose four layers share a launch, although one of them by itself would have its M_b in the workspace."""
    widths = [(d, 3 * d), (d, d), (d, 4 * d), (4 * d, d)]
    alone = multi([(B, T, i, o) for i, o in widths])
    assert any(p[0] and p[3] > needs for p in alone)
    assert pex.pex_stat_pair_batch_workspace_bytes(widths, B, T, BF) == needs


def test_examples_go_through_the_workspace_where_that_is_the_faster_way(multi):
    """Layers on both sides, each measured both ways: many short examples of few columns wait for the second pass, which a rule by traffic alone
    does not see (47 us in one launch and 73 so, 34 and 47, 26 and 41, 35 and 49, 36 and 43, 29 and 37, 271 and 297)."""
    slower = [(211, 289, 528, 152), (101, 335, 312, 296), (80, 279, 928, 64), (159, 275, 128, 512), (25, 1302, 576, 384), (16, 1050, 2944, 64), (23, 969, 2688, 1536)]
    assert [p[0] for p in multi(slower)] == [0] * 7
    faster = [(4, 8192, 4096, 4096), (16, 4096, 768, 3072), (7, 3000, 3000, 1000), (8, 684, 1280, 1152), (69, 1604, 648, 88), (38, 2641, 320, 256), (75, 1139, 144, 736)]
    assert [p[0] for p in multi(faster)] == [1] * 7


def test_the_layers_of_the_gpu_tests_go_that_way(multi):
    from test_long_pairs_gpu import CASES
    shapes, per, groups = zip(*CASES)
    plans = multi(shapes)
    assert [p[:3] for p in plans] == [(1, n, k) for k, n in zip(per, groups)]
    more_room = [p[3] > p[4] for p in plans]
    assert more_room == [False] * 6 + [True] * 6


def test_the_option_that_keeps_examples_out_of_the_workspace(multi, pex_option):
    shapes = [(4, 8192, 4096, 4096), (6, 429, 968, 1856), (224, 292, 128, 256), (16, 2048, 2048, 8192)]
    on, off = multi(shapes), multi(shapes, PEX_STORED_EXAMPLES="0")
    assert [p[0] for p in on] == [1, 1, 0, 0] and [p[0] for p in off] == [0, 0, 0, 0]
    for a, b in zip(on, off):
        assert b[3] == b[4] == a[4] and a[1:3] == b[1:3] and a[5] == b[5]        # no room for them, the same groups, the same kernel
    # a block of layers goes together again, and by itself again
    block = ([(832, 3 * 832), (832, 832), (832, 4 * 832), (4 * 832, 832)], 9, 2370, BF)
    one = (*shapes[0], BF, ("identity", "square"))
    for value, together, alone in ((1, 110755840, 1 << 28), (0, 199360512, 0), (1, 110755840, 1 << 28)):
        pex_option("stored_examples", value)
        assert pex.pex_get_option("stored_examples") == value
        assert pex.pex_stat_pair_batch_workspace_bytes(*block) == together and pex.pex_stat_multi_workspace_bytes(*one) == alone
    assert pex.lib().pex_set_option(pex.PEX_OPT_STORED_EXAMPLES, 2) == 2


def test_small_layers_have_no_more_row_tiles_than_a_grid_dimension(tmp_path):
    """65535 tiles of 64 rows, whatever the limits of the plan."""
    exe = _compile("supports_probe.cpp", str(tmp_path / "supports"))
    text = "".join(f"16 {din} {dout} {dt} 1\n" for dt in (0, 1) for din, dout in ((65535 * 64, 8), (65535 * 64 + 1, 8), (8, 65535 * 64 + 1), (64, 64)))
    out = subprocess.run([exe], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.split()
    assert out == ["1", "0", "1", "1"] * 2

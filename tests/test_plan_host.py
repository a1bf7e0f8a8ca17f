"""Planner choices that can be seen in the workspace a call asks for (host only)."""
import paper_2510_00236_amd as pex


def test_layers_of_short_sequences_are_split_by_what_an_example_costs():
    """24 examples of 23 rows on 20 blocks: the folds, not the rows, are the work, and one group would leave the chip idle."""
    B, T, din, dout = 24, 23, 176, 2496
    groups = pex.pex_weighted_sum_workspace_bytes(B, T, din, dout, pex.PEX_BF16) / (din * dout * 4)
    assert 4 <= groups <= 13
    # a layer that fills the chip by itself stays whole however short its sequences
    assert pex.pex_weighted_sum_workspace_bytes(24, 23, 4096, 6144, pex.PEX_BF16) == 0


def test_fp32_plans_fit_the_librarys_scratch_where_the_call_without_a_workspace_takes_them():
    # three workgroups per unit of 128 x 128 blocks, 16 groups of 1 MiB: charged 16 MiB, so held to the scratch
    assert pex.pex_stat_workspace_bytes(64, 128, 512, 512, pex.PEX_F32, "square") <= pex.NOALLOC_SCRATCH_BYTES
    # charged more than the scratch: as many groups as pay
    assert pex.pex_stat_workspace_bytes(16, 512, 1536, 1536, pex.PEX_F32, "square") > pex.NOALLOC_SCRATCH_BYTES

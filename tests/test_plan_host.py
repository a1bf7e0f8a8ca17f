"""Planner choices that can be seen in the workspace a call asks for (host only)."""
import paper_2510_00236_amd as pex


def test_layers_of_short_sequences_are_split_by_what_an_example_costs():
    """24 examples of 23 rows on 20 blocks: the folds, not the rows, are the work, and one group would leave the chip idle."""
    B, T, din, dout = 24, 23, 176, 2496
    groups = pex.pex_weighted_sum_workspace_bytes(B, T, din, dout, pex.PEX_BF16) / (din * dout * 4)
    assert 4 <= groups <= 13
    # a layer that fills the chip by itself stays whole however short its sequences
    assert pex.pex_weighted_sum_workspace_bytes(24, 23, 4096, 6144, pex.PEX_BF16) == 0

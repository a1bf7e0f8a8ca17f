"""Planner choices that can be seen in the workspace a call asks for (host only)."""
import paper_2510_00236_amd as pex


def test_fp32_plans_fit_the_librarys_scratch_where_the_call_without_a_workspace_takes_them():
    # three workgroups per unit of 128 x 128 blocks, 16 groups of 1 MiB: charged 16 MiB, so held to the scratch
    assert pex.pex_stat_workspace_bytes(64, 128, 512, 512, pex.PEX_F32, "square") <= pex.NOALLOC_SCRATCH_BYTES
    # charged more than the scratch: as many groups as pay
    assert pex.pex_stat_workspace_bytes(16, 512, 1536, 1536, pex.PEX_F32, "square") > pex.NOALLOC_SCRATCH_BYTES

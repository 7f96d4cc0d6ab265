"""Registers of the kernels, from the compiler's figures that the build leaves next to the library: none but the one
named uses scratch memory (a spilling loop fails no numerical test), and no workgroup asks for more LDS than there is."""
import os

import pytest

# 12 bytes a lane, measured faster than the form without (see launch_gemm_any)
SPILLS = {"gemm_kernel<Plain, true, Gather, true, 128, 256>": 16}


def test_kernels_do_not_spill():
    from paper_2401_11469_amd import build
    if not os.path.exists(build.RESOURCES):
        pytest.skip("no resource table (library not built by build.py here)")
    rows = [l.rstrip("\n").split(" | ") for l in open(build.RESOURCES) if not l.startswith("#")]
    for kind, least in (("gemm_kernel<", 30), ("f32_kernel<", 25), ("split_reduce_kernel<", 2), ("fast_kernel<", 30), ("col_sums_kernel<", 10),
                        ("row_scores_kernel<", 8), ("average_rows_kernel<", 4), ("average_cols_kernel<", 4)):
        mine = [r for r in rows if r[0].startswith(kind)]
        assert len(mine) >= least, (kind, len(mine))
        for name, vgpr, agpr, scratch, occ, lds in mine:
            assert int(scratch) <= SPILLS.get(name, 0), (name, scratch)
            assert int(lds) <= 160 * 1024, (name, lds)

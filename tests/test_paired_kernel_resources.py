"""Registers of every kind of kernel, the paired, extraction and register-selection ones among them, from the compiler's figures
that the build leaves next to the library: none uses scratch memory, and no workgroup asks for more LDS than there is."""
import os

import pytest


def test_no_kernel_spills():
    from paper_2401_11469_amd import build
    if not os.path.exists(build.RESOURCES):
        pytest.skip("no resource table (library not built by build.py here)")
    rows = [l.rstrip("\n").split(" | ") for l in open(build.RESOURCES) if not l.startswith("#")]
    for kind, least in (("gemm_kernel<", 30), ("gemm_pair_kernel<", 56), ("f32_kernel<", 25), ("f32_pair_kernel<", 24), ("fast_kernel<", 30),
                        ("pair_kernel<", 32), ("split_reduce_kernel<", 4), ("col_sums_kernel<", 10), ("row_scores_kernel<", 8),
                        ("average_rows_kernel<", 4), ("average_cols_kernel<", 4), ("select_regs_kernel<", 10), ("select_multi_kernel<", 5),
                        ("compact_rows_lds_kernel<", 8)):
        mine = [r for r in rows if r[0].startswith(kind)]
        assert len(mine) >= least, (kind, len(mine))
        for name, vgpr, agpr, scratch, occ, lds in mine:
            assert int(scratch) == 0, (name, scratch)
            assert int(lds) <= 160 * 1024, (name, lds)

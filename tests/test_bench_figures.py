"""Figures in bench.py that count what the kernels do."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_reads_of_the_long_selection():
    """bench.py's physical bytes of one long selection: the launches that are handed the score vector."""
    src = open(os.path.join(ROOT, "paper_2401_11469_amd", "csrc", "zr_select.hip")).read()
    body = src[src.index("int launch_select_wide("):]
    body = body[:body.index("\n}\n")]
    launches = re.findall(r"hipLaunchKernelGGL\((.*?)\);", body, re.S)
    reads = sum("scores" in l for l in launches)
    bench = open(os.path.join(ROOT, "bench.py")).read()
    assert int(re.search(r"^SELECT_WIDE_READS = (\d+)", bench, re.M).group(1)) == reads == 5
    assert "28.0 * nl" not in bench

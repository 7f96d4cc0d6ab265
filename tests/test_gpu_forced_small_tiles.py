"""The parity cases on the 128 x 128 and 64 x 128 tiles of the aligned bf16 kernels.

Products as small as those cases go to the kernel for any alignment by the rules on the number of tiles; the switch that
test_gpu_forced_tiles.py uses for the big tiles sends them to these, with their ragged edges, sparse lists, contraction
tails and sums of Average imputation."""
import os
import subprocess
import sys

import pytest

from test_gpu_forced_tiles import CASES, ROOT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", ["128", "64x128"])
def test_parity_cases_on_forced_small_tiles(shape):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    res = subprocess.run([sys.executable, "-u", "-m", "pytest", os.path.join(ROOT, "tests", "test_gpu_parity.py"), "-x", "-q",
                          "-p", "no:cacheprovider", "-k", CASES, "--timeout", "300", "--timeout-method", "thread"],
                         cwd=ROOT, env=dict(os.environ, ZR_FORCE_TILES=shape), stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                         text=True, timeout=900)
    tail = "\n".join(res.stdout.splitlines()[-25:])
    assert res.returncode == 0, tail
    assert " passed" in tail and "failed" not in tail, tail


@pytest.mark.parametrize("shape,kernel", [("128", "fast_kernel<DmaP, DmaP, 128, 128, 2, 2>"), ("64x128", "fast_kernel<DmaP, DmaP, 64, 128, 1, 4>")])
def test_the_switch_reaches_the_tiles(shape, kernel):
    """A product of a few tiles, and the sums of Average imputation that its tiles leave."""
    code = f"""
import sys; sys.path.insert(0, {ROOT!r})
import torch
from paper_2401_11469_amd import zr
zr.debug_record_kernel_names(True)
M, K, N, nk = 200, 128, 300, 290
X, W = (torch.randn(r, K, device="cuda").bfloat16() for r in (M, 304))
keep = torch.arange(nk, dtype=torch.int32, device="cuda")
ws = torch.full((zr.workspace_bytes(M, K, 304, nk, zr.DROP_N, torch.bfloat16),), 0x7F, dtype=torch.uint8, device="cuda")
Y = zr.resized_linear_fwd(X, W, keep, zr.DROP_N, zr.AVERAGE, workspace=ws, w_layout=zr.W_NK)
assert zr.debug_last_kernel() == {kernel!r}, zr.debug_last_kernel()
need = (3 * M * 4 + 15) // 16 * 16
off = (ws.numel() - need) // 16 * 16
means = ws[off:off + 4 * M].view(torch.float32)
want = Y[:, :nk].double().mean(dim=1)
assert float((means.double() - want).abs().max()) < 1e-4, (means[:4], want[:4])
print("reached")
"""
    res = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, ZR_FORCE_TILES=shape), stdout=subprocess.PIPE,
                         stderr=subprocess.STDOUT, text=True, timeout=300)
    assert res.returncode == 0 and "reached" in res.stdout, res.stdout[-2000:]

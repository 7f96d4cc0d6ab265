"""The stand-alone Average pass where its two kernels take another form: clustered kept lists (one long gap),
few kept slices, more columns than are marked at a time, groups of four rows with a remainder, 256-column
workgroups, and more columns than one launch has threads for.  Against float64."""
import numpy as np
import pytest

from paper_2401_11469_amd import workloads as wl
from test_gpu_parity import AVERAGE, idx_gpu, subset, to_gpu, to_np
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def kept_sets(n):
    half = max(1, n // 2)
    yield np.arange(half)                                    # everything behind the last kept one
    yield np.arange(n - half, n)
    yield np.concatenate([np.arange(min(3, half)), np.arange(n - min(2, half), n)])      # one gap in the middle
    yield np.array([n // 3])
    yield subset(n, n, max(1, n // 20))
    yield subset(n + 1, n, max(1, (3 * n) // 4))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("axis,rows,cols", [(1, 3, 700), (1, 1023, 130), (1, 1025, 260), (1, 1031, 77), (1, 5, 8192), (1, 6, 20001),
                                            (0, 700, 3), (0, 1024, 40), (0, 2600, 33), (0, 40, 16390), (0, 200, 16641),
                                            (0, 150, 65600), (0, 20, 65537)])
def test_average_of_clustered_and_sparse_lists(zr, torch_mod, dtype, axis, rows, cols):  # noqa: F811
    torch = torch_mod
    n = rows if axis == 0 else cols
    g = np.random.Generator(np.random.PCG64(rows * 7 + cols))
    data = g.standard_normal((rows, cols)).astype(np.float32)
    if dtype == "bf16":
        data = wl.round_to_bf16(data)
    for S in kept_sets(n):
        S = np.unique(S).astype(np.int32)
        if len(S) == n:
            continue
        out = to_gpu(torch, data, dtype, ld=cols + 3)
        zr.impute(out, axis, idx_gpu(torch, S), AVERAGE)
        torch.cuda.synchronize()
        got = to_np(out)
        drop = np.setdiff1d(np.arange(n), S)
        kept_in, kept_got = (data[S], got[S]) if axis == 0 else (data[:, S], got[:, S])
        assert np.array_equal(kept_got, kept_in.astype(np.float64))
        mean = kept_in.astype(np.float64).mean(axis=axis, keepdims=True)
        d = got[drop] if axis == 0 else got[:, drop]
        # fp32 sums of values of about 1, then one rounding to the type
        eps = (2.0 ** -8 if dtype == "bf16" else 0.0) * np.abs(mean) + 2e-6
        assert np.all(np.abs(d - mean) <= eps), (axis, rows, cols, len(S), float(np.max(np.abs(d - mean))))
        assert torch.all(out._base[:, cols:] == 777.0), "padding overwritten"


def test_average_over_rows_of_very_many_columns(zr, torch_mod):  # noqa: F811
    """140 million columns: workgroups of 1024 threads to 32 columns are more threads than a launch can have."""
    torch = torch_mod
    cols = 140_000_003
    out = torch.randn(2, cols, dtype=torch.float32, device="cuda").to(torch.bfloat16)
    first = out[0].clone()
    zr.impute(out, 0, idx_gpu(torch, np.array([0])), AVERAGE)
    torch.cuda.synchronize()
    assert torch.equal(out[0], first) and torch.equal(out[1], first)       # the mean of one row

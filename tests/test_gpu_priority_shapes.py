"""Priority scores at the limits of their column pieces and row batches: few and many columns, few and many rows,
the incremental rule, odd widths, and more columns than one launch has threads for in narrow pieces.  Against
float64."""
import numpy as np
import pytest

from test_gpu_parity import DROP_K, DROP_N, idx_gpu, subset
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode", [DROP_N, DROP_K])
@pytest.mark.parametrize("K,N", [(5, 8192), (512, 8448), (513, 8192), (70, 28671), (1000, 28680), (33, 65544), (2100, 1032), (4100, 264),
                                 (3, 191), (9, 768), (9, 772), (17, 1537), (6, 4096), (7, 6148), (1, 12289)])
def test_scores(zr, torch_mod, dtype, mode, K, N):  # noqa: F811
    torch = torch_mod
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(K * 31 + N)
    a, b = (torch.randn(K, N, generator=gen, device="cuda").to(dt) for _ in range(2))
    n = N if mode == DROP_N else K
    want = (a.double() - b.double()).abs().mean(dim=0 if mode == DROP_N else 1)
    prev = torch.rand(n, generator=gen, device="cuda")
    S = subset(n, n, max(1, (2 * n) // 3))
    kept = torch.zeros(n, dtype=torch.bool, device="cuda")
    kept[torch.from_numpy(S).long().cuda()] = True
    ws = torch.empty(max(16, zr.priority_workspace_bytes(K, N, mode)), dtype=torch.uint8, device="cuda")
    for w in (None, ws):
        got = zr.priority_scores(a, b, mode, workspace=w)
        assert torch.all((got.double() - want).abs() <= 2e-6 * want), float(((got.double() - want).abs() / want).max())
        inc = zr.priority_scores(a, b, mode, prev_scores=prev, prev_keep_idx=idx_gpu(torch, S), workspace=w)
        assert torch.equal(inc[kept], got[kept]) and torch.equal(inc[~kept], prev[~kept])


def test_scores_of_very_many_columns(zr, torch_mod):  # noqa: F811
    """70 million fp32 columns: workgroups of 1024 threads to 16 columns are more threads than a launch can have."""
    torch = torch_mod
    n = 70_000_000
    a, b = (torch.randn(1, n, device="cuda") for _ in range(2))
    got = zr.priority_scores(a, b, DROP_N)
    torch.cuda.synchronize()
    assert torch.equal(got, (a - b).abs()[0])

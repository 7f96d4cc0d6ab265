"""Average imputation with scratch takes its means from sums that the product's own tiles leave, also where its
remainder panel, or all of a product with many kept rows, is split: the means, left in the first slot at the tail of the
scratch buffer, show it.
Against the float64 oracle, and the means against the mean of the stored results."""
import numpy as np
import pytest

from paper_2401_11469_amd import workloads as wl
from test_gpu_parity import AVERAGE, DROP_K, DROP_N, W_KN, W_NK, check_layer, idx_gpu, run_layer, subset, to_gpu, to_np
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def means_at_the_tail(torch, ws, length, n_keep):
    """The sums' place: the last ceil(n_keep / 128) * length floats, rounded up to 16 bytes, from a 16-byte boundary."""
    need = ((n_keep + 127) // 128 * length * 4 + 15) // 16 * 16
    off = (ws.numel() - need) // 16 * 16
    return ws[off:off + 4 * length].view(torch.float32)


@pytest.mark.parametrize("what,M,K,N,mode,layout,n_keep,kernel", [
    ("fwd", 8192, 1536, 2752, DROP_N, W_NK, 2064, "remainder panel"),      # a big panel, and a split one
    ("dX", 8192, 2752, 1536, DROP_K, W_KN, 2064, "remainder panel"),
    ("dW", 4096, 264, 2600, DROP_N, W_NK, 1950, "split"),                 # row scatters
    ("dW", 4096, 2600, 264, DROP_K, W_KN, 1950, "split"),
])
def test_split_products_leave_the_sums(zr, torch_mod, what, M, K, N, mode, layout, n_keep, kernel):  # noqa: F811
    torch = torch_mod
    gen = torch.Generator(device="cuda").manual_seed(M + K + N)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda").to(torch.bfloat16)
    X, dY, W = r(M, K), r(M, N), (r(N, K) if layout == W_NK else r(K, N))
    n = N if mode == DROP_N else K
    S = subset(M + n, n, n_keep)
    keep = idx_gpu(torch, S)
    ws = torch.full((zr.workspace_bytes(M, K, N, n_keep, mode, torch.bfloat16),), 0x7F, dtype=torch.uint8, device="cuda")
    if what == "fwd":
        out = zr.resized_linear_fwd(X, W, keep, mode, AVERAGE, workspace=ws, w_layout=layout)
        axis = 1
    elif what == "dX":
        out, _ = zr.resized_linear_bwd(X, W, dY, keep, mode, AVERAGE, need_dW=False, workspace=ws, w_layout=layout)
        axis = 1
    else:
        _, out = zr.resized_linear_bwd(X, W, dY, keep, mode, AVERAGE, need_dX=False, workspace=ws, w_layout=layout)
        axis = 0 if (layout == W_KN) == (mode == DROP_K) else 1
    name = zr.debug_last_kernel()
    torch.cuda.synchronize()
    assert kernel in name, name
    kept = out[:, keep.long()] if axis == 1 else out[keep.long()]
    want = kept.double().mean(dim=axis)
    got = means_at_the_tail(torch, ws, want.numel(), n_keep).double()
    rms = float(kept.double().square().mean().sqrt())
    assert torch.all((got - want).abs() <= 1e-5 * rms), float((got - want).abs().max())
    drop = torch.ones(n, dtype=torch.bool, device="cuda")
    drop[keep.long()] = False
    filled = (out[:, drop] - want[:, None].float()) if axis == 1 else (out[drop] - want[None].float())
    assert float(filled.abs().max()) <= 2.0 ** -8 * float(want.abs().max()) + 1e-5 * rms


@pytest.mark.parametrize("mode", [DROP_N, DROP_K])
@pytest.mark.parametrize("M,K,N", [(1300, 200, 520), (200, 1300, 392), (1352, 1096, 264)])
def test_average_with_scratch_where_products_split(zr, torch_mod, oracle, mode, M, K, N):  # noqa: F811
    case = wl.random_case(M + 3 * K + 5 * N, M, K, N, "bf16")
    n = N if mode == DROP_N else K
    for layout in (W_KN, W_NK):
        for n_keep in (1, n // 3, n - 1):
            S = subset(n_keep + n, n, n_keep)
            got = run_layer(zr, torch_mod, case, S, mode, "bf16", AVERAGE, w_layout=layout, use_ws=True)
            check_layer(oracle, case, S, mode, "bf16", AVERAGE, got)

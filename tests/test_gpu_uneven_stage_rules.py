"""Which bf16 kernel a product of aligned tensors takes whose contraction is not whole 64-deep stages, by tiles and depth."""
import pytest

from test_gpu_dispatch_rules import tensors
from test_gpu_parity import DROP_N, W_KN, W_NK, idx_gpu, subset
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,layout,n_keep,kernel", [
    (1280, 768 - 8, 2048, W_KN, 2048, "fast_kernel<DmaP, DmaQ, 128, 128"), (1280, 1544, 2048, W_KN, 2048, "gemm_kernel<P, Q, 64, 256>"),
    # rows of W: below three stages, and above 1152 deep, from 129 tiles on (12.2 us against 17.6, 32.4 against 46.8)
    (2880, 80, 872, W_NK, 391, "gemm_kernel<P, P, 64, 256>"), (896, 3720, 1760, W_NK, 1760, "gemm_kernel<P, P, 64, 256>"),
    (1352, 200, 1096, W_NK, 1096, "fast_kernel<DmaP, DmaP, 64, 128, 1, 4>"), (1352, 1160, 1096, W_NK, 1096, "gemm_kernel<P, P, 64, 256>")])
def test_rules_for_all_or_rows_of_w(zr, torch_mod, M, K, N, layout, n_keep, kernel):  # noqa: F811
    torch = torch_mod
    X, W, _ = tensors(torch, M, K, N, layout, M + K + N)
    keep = idx_gpu(torch, subset(M + N, N, n_keep))
    Y = zr.resized_linear_fwd(X, W, keep, DROP_N, w_layout=layout)
    assert zr.debug_last_kernel().startswith(kernel), zr.debug_last_kernel()
    k = keep.long()
    want = X.float() @ (W.t() if layout == W_NK else W).float()[:, k]
    assert float((Y[:, k].float() - want).norm() / want.norm()) < 5e-3


@pytest.mark.parametrize("M,K,N,n_keep,same,kernel", [
    # in slices from 1665 tokens on up to 128 tiles, from 1344 on up to 160 (1194 tokens, 115 tiles: 26.4 us against 30.8)
    (1169, 808, 2240, 2240, False, "gemm_kernel<Q, Q, 64, 256>"), (1350, 808, 2456, 2456, False, "fast_kernel<DmaQ, DmaQ, 128, 128, 2, 2> split"),
    (1602, 808, 2048, 2048, False, "gemm_kernel<Q, Q, 64, 256>"), (2002, 808, 2048, 2048, False, "fast_kernel<DmaQ, DmaQ, 128, 128, 2, 2> split"),
    # more rows to copy than to compute (608 tokens, 198 tiles: 28 us against 43)
    (608 + 4, 2712, 2480, 1035, True, "gemm_kernel<Q, Q, 64, 256>"), (608 + 4, 2712, 2480, 1035, False, "fast_kernel<DmaQ, DmaQ, 128, 128, 2, 2>")])
def test_rules_for_dw_of_no_whole_stages(zr, torch_mod, M, K, N, n_keep, same, kernel):  # noqa: F811
    torch = torch_mod
    X, W, dY = tensors(torch, M, K, N, W_NK, M + K + N)
    keep = idx_gpu(torch, subset(M + N, N, n_keep))
    ws = torch.empty(zr.workspace_bytes(M, K, N, n_keep, DROP_N, torch.bfloat16), dtype=torch.uint8, device="cuda")
    prev = dict(policy=zr.SAME, prev_dW=torch.full_like(W, 3.0)) if same else {}
    _, dW = zr.resized_linear_bwd(X, W, dY, keep, DROP_N, need_dX=False, workspace=ws, w_layout=W_NK, **prev)
    assert zr.debug_last_kernel().startswith(kernel), zr.debug_last_kernel()
    k = keep.long()
    want = dY.float()[:, k].t() @ X.float()
    assert float((dW[k].float() - want).norm() / want.norm()) < 5e-3
    dropped = torch.ones(N, dtype=torch.bool, device="cuda")
    dropped[k] = False
    assert torch.all(dW[dropped] == (3.0 if same else 0.0))

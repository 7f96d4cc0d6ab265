"""Contractions that are no whole number of stages on the direct-to-LDS kernels: what lies past their end is read as
zeros, whatever the memory there holds, and infinities inside stay where they belong."""
import pytest

from parity_util import check_kept_torch

pytestmark = pytest.mark.gpu
DROP_N, W_KN, W_NK = 0, 0, 1


@pytest.fixture(scope="module")
def torch_zr():
    import torch
    from paper_2401_11469_amd import zr
    zr.debug_record_kernel_names(True)
    return torch, zr


@pytest.mark.parametrize("layout", [W_KN, W_NK])
@pytest.mark.parametrize("M,K,N", [
    (1025, 200, 2056), (1087, 520, 2048), (2049, 776, 1544),        # 128 x 128 tiles, one token more than whole stages
    (4127, 1352, 4104), (4097, 4088, 2056)])                        # the ring loops
def test_past_the_end(torch_zr, layout, M, K, N):
    torch, zr = torch_zr
    gen = torch.Generator(device="cuda").manual_seed(M + K + N)

    def inside(rows, cols, nan_cols=8):
        """A tensor in a buffer of NaN, with rows behind it and columns beside it."""
        buf = torch.full((rows + 40, cols + nan_cols), float("nan"), device="cuda", dtype=torch.bfloat16)
        buf[:rows, :cols] = torch.randn(rows, cols, generator=gen, device="cuda").to(torch.bfloat16)
        return buf[:rows, :cols]
    X, dY, W = inside(M, K), inside(M, N), inside(*((N, K) if layout == W_NK else (K, N)))
    keep = torch.arange(N, dtype=torch.int32, device="cuda")
    names, outs = [], []
    outs.append(zr.resized_linear_fwd(X, W, keep, DROP_N, w_layout=layout))
    names.append(zr.debug_last_kernel())
    outs.append(zr.resized_linear_bwd(X, W, dY, keep, DROP_N, need_dW=False, w_layout=layout)[0])
    names.append(zr.debug_last_kernel())
    outs.append(zr.resized_linear_bwd(X, W, dY, keep, DROP_N, need_dX=False, w_layout=layout)[1])
    names.append(zr.debug_last_kernel())
    print(names, flush=True)
    assert all(n.startswith("fast_kernel") for n in (names if M > 4000 else names[:1])), names
    torch.backends.cuda.matmul.allow_tf32 = False
    Wk = (W.t() if layout == W_NK else W).float()
    dW = outs[2].t() if layout == W_NK else outs[2]
    check_kept_torch("Y", outs[0], X.float() @ Wk, "bf16", K, None)
    check_kept_torch("dX", outs[1], dY.float() @ Wk.t(), "bf16", N, None)
    check_kept_torch("dW", dW, X.float().t() @ dY.float(), "bf16", M, None)
    # an infinity in the last token and feature: infinite exactly where the exact sum is
    dY[M - 1, N - 1] = float("inf")
    X[M - 1, K - 1] = 1.0
    dW = zr.resized_linear_bwd(X, W, dY, keep, DROP_N, need_dX=False, w_layout=layout)[1]
    dW = dW.t() if layout == W_NK else dW
    assert torch.isfinite(dW[:, :-1]).all() and torch.isinf(dW[X[M - 1] != 0][:, -1]).all()

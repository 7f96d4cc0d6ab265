"""Which bf16 kernel a product of aligned tensors takes by the number of its tiles, and that the choice does not show in
the result: with and without the scratch buffer (an operand extracted beforehand, or gathered in flight) products that
are not split have the same bits."""
import numpy as np
import pytest

from test_gpu_parity import DROP_K, DROP_N, W_KN, W_NK, idx_gpu, subset
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def tensors(torch, M, K, N, layout, seed, ldn=0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda a, b, ld=0: torch.randn(a, max(b, ld), generator=gen, device="cuda").to(torch.bfloat16)[:, :b]
    return r(M, K), (r(N, K) if layout == W_NK else r(K, N, ldn)), r(M, N, ldn)


@pytest.mark.parametrize("M,K,N,mode,layout,n_keep,ldn", [
    (1000, 12800, 64, DROP_K, W_KN, 64, 0),            # every tile 64 wide: dW 12800 x 64 ...
    (1000, 12800, 96, DROP_N, W_NK, 64, 0),            # ... with the kept rows of a shard stored [N x K]
    (576, 12800, 96, DROP_N, W_NK, 64, 0),
    (1024, 64, 16384, DROP_K, W_KN, 48, 0),
    (520, 270, 300, DROP_N, W_KN, 225, 304),           # column scatter into rows of odd width
    (700, 264, 520, DROP_N, W_KN, 390, 0), (264, 700, 520, DROP_K, W_NK, 530, 0),
    (64, 4096, 1400, DROP_K, W_KN, 1000, 0), (64, 900, 12800, DROP_K, W_NK, 640, 0),
    (1536, 900, 2048, DROP_K, W_KN, 672, 0), (2048, 900, 2048, DROP_K, W_NK, 672, 0),
    (2000, 2600, 900, DROP_N, W_KN, 650, 0), (3000, 3000, 600, DROP_N, W_NK, 456, 0)])
def test_same_bits_with_and_without_the_buffer(zr, torch_mod, M, K, N, mode, layout, n_keep, ldn):  # noqa: F811
    torch = torch_mod
    X, W, dY = tensors(torch, M, K, N, layout, M + K + N, ldn)
    n = N if mode == DROP_N else K
    keep = idx_gpu(torch, subset(M + n, n, min(n_keep, n - 1)))
    ws = torch.empty(zr.workspace_bytes(M, K, N, keep.numel(), mode, torch.bfloat16), dtype=torch.uint8, device="cuda")
    outs, names = [], []
    for w in (None, ws):
        Y = zr.resized_linear_fwd(X, W, keep, mode, workspace=w, w_layout=layout)
        n1 = zr.debug_last_kernel()
        dX, _ = zr.resized_linear_bwd(X, W, dY, keep, mode, need_dW=False, workspace=w, w_layout=layout)
        n2 = zr.debug_last_kernel()
        _, dW = zr.resized_linear_bwd(X, W, dY, keep, mode, need_dX=False, workspace=w, w_layout=layout)
        outs.append((Y, dX, dW))
        names.append((n1, n2, zr.debug_last_kernel()))
    torch.cuda.synchronize()
    compared = 0
    for what, a, b, na, nb in zip(("Y", "dX", "dW"), *outs, *names):
        if "split" in nb or "remainder" in nb:
            continue
        compared += 1
        assert torch.equal(a, b), (what, int((a != b).sum()), na, nb)
    assert compared, names


@pytest.mark.parametrize("M,K,N,mode,layout,n_keep,kernel", [
    # all of W stored [K x N]: the direct-to-LDS tiles from 129 on (1024 deep, 160 tiles: 14 us against 18)
    (1280, 512, 2048, DROP_N, W_KN, 2048, "fast_kernel<DmaP, DmaQ"),
    (1024, 512, 2048, DROP_N, W_KN, 2048, "gemm_kernel<P, Q, 64, 256>"),
    # ... and, in stages that are not whole, up to 768 deep (4040 deep, 183 tiles: 60 us against 67)
    (1280, 520, 2048, DROP_N, W_KN, 2048, "fast_kernel<"), (1280, 776, 2048, DROP_N, W_KN, 2048, "gemm_kernel<P, Q, 64, 256>"),
    # kept columns of both operands in flight: 128 x 128 tiles from 129 on (1024 deep, 160 tiles: 41 us against 61)
    (1280, 700, 2048, DROP_K, W_NK, 512, "gemm_kernel<Pg, Pg, 128, 256>"),
    (1280, 700, 2048, DROP_K, W_KN, 512, "gemm_kernel<Pg, Q, 128, 256>"),
    (1024, 700, 2048, DROP_K, W_NK, 512, "gemm_kernel<Pg, Pg, 64, 256>"),
    # kept columns of W across the contraction: from 129 on (100 tiles, 256 deep: 13 us against 16)
    (512, 304, 5552, DROP_N, W_KN, 4160, "fast_kernel<DmaP, LdQG"),
    (512, 304, 4272, DROP_N, W_KN, 3200, "gemm_kernel<P, Qg, 64, 256>"), (6400, 200, 344, DROP_N, W_KN, 256, "gemm_kernel<P, Qg, 64, 256>"),
    (1024, 304, 1536, DROP_N, W_KN, 1152, "gemm_kernel<P, Qg, 64, 256>"),
    # rows of W, 65 to 256 tiles: 64 x 128 (384 up to 1024 deep), and 128 x 128 above
    (1352, 192, 1096, DROP_N, W_NK, 1096, "fast_kernel<DmaP, DmaP, 64, 128, 1, 4>"),
    (3088, 64, 2104, DROP_N, W_NK, 1578, "fast_kernel<DmaP, DmaP, 64, 128, 1, 4>"),
    (2440, 136, 2600, DROP_N, W_NK, 2600, "fast_kernel<LdPV, LdPV, 128, 128, 2, 2>"),
    # any alignment: 32 x 32, 64 x 64 (512 threads from 256 deep to 256 tiles), 128 x 128
    (31, 33, 32, DROP_N, W_KN, 32, "gemm_kernel<P, Q, 32, 256>"), (833, 67, 901, DROP_N, W_KN, 901, "gemm_kernel<P, Q, 64, 256>"),
    (985, 1001, 771, DROP_N, W_KN, 771, "gemm_kernel<P, Q, 64, 512>"), (2497, 65, 2433, DROP_N, W_KN, 2433, "gemm_kernel<P, Q, 128, 256>"),
    (985, 1001, 771, DROP_K, W_NK, 751, "gemm_kernel<Pg, Pg, 64, 512>"), (2500, 2433, 65, DROP_K, W_KN, 1825, "gemm_kernel<Pg, Q, 32, 256>"),
    # one column of tiles, 100 of them: 512 threads on 64 x 64
    (64, 512, 12800, DROP_N, W_KN, 12800, "gemm_kernel<P, Q, 64, 512>"),
    (64, 256, 8192, DROP_N, W_NK, 8192, "gemm_kernel<P, P, 64, 512>")])
def test_rules_on_the_number_of_tiles(zr, torch_mod, M, K, N, mode, layout, n_keep, kernel):  # noqa: F811
    torch = torch_mod
    X, W, _ = tensors(torch, M, K, N, layout, M + K + N)
    n = N if mode == DROP_N else K
    keep = subset(M + n, n, n_keep)
    Y = zr.resized_linear_fwd(X, W, idx_gpu(torch, keep), mode, w_layout=layout)
    assert zr.debug_last_kernel().startswith(kernel), zr.debug_last_kernel()
    k = torch.from_numpy(keep).long().cuda()
    Wf = (W.t() if layout == W_NK else W).float()
    want = X.float()[:, k] @ Wf[k] if mode == DROP_K else X.float() @ Wf[:, k]
    got = (Y if mode == DROP_K else Y[:, k]).float()
    assert float((got - want).norm() / want.norm()) < 5e-3

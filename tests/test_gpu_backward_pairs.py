"""dX and dW of one backward call in one launch: against fp32 products of the masked operands, with the previous tensors
as imputed values, repeatable bit by bit, and one after the other where dW takes the place of W."""
import pytest

from parity_util import check_kept_torch

pytestmark = pytest.mark.gpu
DROP_N, DROP_K, W_KN, W_NK, ZERO, AVERAGE, SAME = 0, 1, 0, 1, 0, 1, 2


@pytest.fixture(scope="module")
def torch_zr():
    import torch
    from paper_2401_11469_amd import zr
    zr.debug_record_kernel_names(True)
    torch.backends.cuda.matmul.allow_tf32 = False
    return torch, zr


def tensors(torch, M, K, N, nk, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda a, b: torch.randn(a, b, generator=gen, device="cuda").to(torch.bfloat16)
    return r(M, K), r(*((N, K) if nk else (K, N))), r(M, N)


@pytest.mark.parametrize("policy", [ZERO, SAME])
@pytest.mark.parametrize("M,K,N,mode,n_keep", [
    # the ring loops: rows of W on the contraction, all of W, rows of W; dW whole and in slices
    (2048, 3400, 3328, DROP_N, 1897), (2048, 3400, 3328, DROP_N, 3327), (4137, 1632, 1672, DROP_N, 1672), (3743, 3296, 3096, DROP_K, 2044),
    (8192, 1024, 4096, DROP_K, 768), (12416, 3112, 200, DROP_N, 200), (5808, 2936, 544, DROP_N, 413), (9388, 1752, 632, DROP_N, 278),
    # 128 x 128 and 64 x 128 tiles
    (1576, 2584, 4176, DROP_K, 1990), (591, 3616, 1304, DROP_K, 2314), (8030, 344, 576, DROP_K, 189), (5322, 352, 1712, DROP_N, 1164),
    (788, 2576, 1416, DROP_N, 708), (2880, 744, 1408, DROP_N, 1408)])
def test_pair(torch_zr, M, K, N, mode, n_keep, policy):
    torch, zr = torch_zr
    nk = mode == DROP_N                                    # kept indices are rows of the stored shard
    layout = W_NK if nk else W_KN
    X, W, dY = tensors(torch, M, K, N, nk, M + K + N + n_keep)
    n = N if nk else K
    gen = torch.Generator(device="cuda").manual_seed(n_keep)
    keep = torch.randperm(n, generator=gen, device="cuda")[:n_keep].sort().values.to(torch.int32)
    ws = torch.empty(zr.workspace_bytes(M, K, N, n_keep, mode, torch.bfloat16), dtype=torch.uint8, device="cuda")
    prev = dict(prev_dX=torch.full_like(X, 2.0), prev_dW=torch.full_like(W, 3.0)) if policy == SAME else {}
    dX, dW = zr.resized_linear_bwd(X, W, dY, keep, mode, policy=policy, workspace=ws, w_layout=layout, **prev)
    name = zr.debug_last_kernel()
    print(name, flush=True)
    assert "beside" in name, name
    again = zr.resized_linear_bwd(X, W, dY, keep, mode, policy=policy, workspace=ws, w_layout=layout, **prev)
    assert torch.equal(dX, again[0]) and torch.equal(dW, again[1])
    kept = torch.zeros(n, dtype=torch.bool, device="cuda")
    kept[keep.long()] = True
    Wk = (W.t() if nk else W).float()
    dWk = dW.t() if nk else dW
    if mode == DROP_K:
        check_kept_torch("dX", dX, dY.float() @ (Wk * kept[:, None]).t(), "bf16", N, kept[None, :])
        check_kept_torch("dW", dWk, (X.float() * kept[None, :]).t() @ dY.float(), "bf16", M, kept[:, None])
        rest = ((dX[:, ~kept], 2.0), (dWk[~kept], 3.0))
    else:
        check_kept_torch("dX", dX, (dY.float() * kept[None, :]) @ Wk.t(), "bf16", n_keep, None)
        check_kept_torch("dW", dWk, X.float().t() @ (dY.float() * kept[None, :]), "bf16", M, kept[None, :])
        rest = ((dWk[:, ~kept], 3.0),)
    for t, v in rest:
        assert torch.all(t == (v if policy == SAME else 0.0))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("policy", [ZERO, AVERAGE, SAME])
@pytest.mark.parametrize("layout", [W_KN, W_NK])
@pytest.mark.parametrize("mode", [DROP_N, DROP_K])
@pytest.mark.parametrize("M,K,N,n_keep", [
    (2, 9, 12, 5), (31, 33, 65, 32), (200, 77, 1201, 50), (985, 1001, 771, 578),         # few tiles; sums in groups
    (2497, 1201, 803, 640), (300, 2305, 1999, 1500), (256, 512, 256, 0)])                 # 64 x 64 and 128 x 128; nothing pruned
def test_pair_of_any_alignment(torch_zr, M, K, N, n_keep, mode, layout, policy, dtype):
    """Without scratch, so that every list is applied in flight: the same bits as the two products on their own (fp32:
    to its rounding, where the tiles and with them the order may differ)."""
    torch, zr = torch_zr
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    X, W, dY = (t.to(dt) for t in tensors(torch, M, K, N, layout == W_NK, M + K + N))
    n = N if mode == DROP_N else K
    n_keep = n if n_keep == 0 else min(n_keep, n - 1)
    keep = torch.randperm(n, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")[:n_keep].sort().values.to(torch.int32)
    prev = dict(prev_dX=torch.full_like(X, 2.0), prev_dW=torch.full_like(W, 3.0)) if policy == SAME else {}
    a = zr.resized_linear_bwd(X, W, dY, keep, mode, policy=policy, w_layout=layout, **prev)
    name = zr.debug_last_kernel()
    dX = zr.resized_linear_bwd(X, W, dY, keep, mode, policy=policy, w_layout=layout, need_dW=False, **prev)[0]
    dW = zr.resized_linear_bwd(X, W, dY, keep, mode, policy=policy, w_layout=layout, need_dX=False, **prev)[1]
    print(name, flush=True)
    if M in (31, 200, 985):
        assert "beside" in name, name
    for what, x, y, C in (("dX", a[0], dX, N), ("dW", a[1], dW, M)):
        if dtype == "bf16":
            assert torch.equal(x, y), what
        else:
            # two sums of C terms in different orders: C ** 0.5 roundings of 2 ** -24 each, with a factor of 8
            assert float((x - y).abs().max()) <= 8 * max(C, 16) ** 0.5 * 2.0 ** -24 * float(y.abs().max()), what


@pytest.mark.parametrize("what", ["dW over W", "dX over X"])
def test_results_in_the_place_of_operands(torch_zr, what):
    """dW may take the place of W, which only dX reads, and dX that of X once X[:,S] is extracted."""
    torch, zr = torch_zr
    M, K, N = 2048, 2816, 2048
    X, W, dY = tensors(torch, M, K, N, False, 5)
    keep = torch.arange(0, K, 2, dtype=torch.int32, device="cuda")
    ws = torch.empty(zr.workspace_bytes(M, K, N, keep.numel(), DROP_K, torch.bfloat16), dtype=torch.uint8, device="cuda")
    dX = zr.resized_linear_bwd(X, W, dY, keep, DROP_K, need_dW=False, workspace=ws)[0]
    dW = zr.resized_linear_bwd(X, W, dY, keep, DROP_K, need_dX=False, workspace=ws)[1]
    a, b = zr.resized_linear_bwd(X, W, dY, keep, DROP_K, workspace=ws, **({"dW": W} if what == "dW over W" else {"dX": X}))
    assert "beside" not in zr.debug_last_kernel()
    assert torch.equal(a, dX) and torch.equal(b, dW)

"""The fp32 products on 128 x 128 tiles: products with many tiles take them, short contractions among
them, at the edges of tiles and of the 32-deep stages; both layouts, all loaders and epilogues, rows of
any alignment.  Against the float64 oracle with the bounds of parity_util (fp32: 1e-5 of the largest
value)."""
import numpy as np
import pytest

from paper_2401_11469_amd import workloads as wl
from parity_util import check_kept_np
from test_gpu_parity import AVERAGE, DROP_K, DROP_N, SAME, ZERO, W_KN, W_NK, check_layer, idx_gpu, run_layer, subset, to_gpu, to_np
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


# the product with many tiles: forward (short K), dX (short N), dW (few tokens); 33 to 100 deep: 1 to 4 stages
@pytest.mark.parametrize("mode", [DROP_N, DROP_K])
@pytest.mark.parametrize("layout", [W_KN, W_NK])
@pytest.mark.parametrize("M,K,N,pad", [(2041, 33, 2750, 0), (2047, 64, 2732, 3), (1793, 8, 2500, 1),      # forward
                                       (2041, 2750, 31, 0), (1921, 2730, 100, 5),                          # dX
                                       (32, 2700, 2732, 0), (65, 2741, 2729, 3), (5, 2700, 2732, 0)])       # dW
def test_f32_big_tile_edges(zr, torch_mod, oracle, mode, layout, M, K, N, pad):  # noqa: F811
    case = wl.random_case(31 * M + 7 * K + N, M, K, N, "f32")
    n = N if mode == DROP_N else K
    for n_keep, policy in (((3 * n + 3) // 4, ZERO), (n - 1, SAME), ((4 * n) // 5, AVERAGE)):
        S = subset(n_keep + n, n, n_keep)
        got = run_layer(zr, torch_mod, case, S, mode, "f32", policy, pad=pad, w_layout=layout, use_ws=policy == AVERAGE)
        check_layer(oracle, case, S, mode, "f32", policy, got)


@pytest.mark.parametrize("M,N,C,transposed", [(2048, 2048, 48, True), (2047, 2050, 17, False), (4096, 2048, 8, False)])
def test_f32_products_with_many_tiles_take_the_big_ones(zr, torch_mod, oracle, M, N, C, transposed):  # noqa: F811
    """8 to 96 deep they took 64 x 64 tiles: 8192 x 4096 results of contraction 8 in 88 us instead of 56."""
    torch = torch_mod
    g = np.random.Generator(np.random.PCG64(M + N + C))
    A = g.standard_normal((M, C)).astype(np.float32)
    B = (g.standard_normal((N, C) if transposed else (C, N)) * 0.05).astype(np.float32)
    base = g.standard_normal((M, N)).astype(np.float32)
    out = to_gpu(torch, base, "f32")
    zr.migrated_accumulate(out, to_gpu(torch, A, "f32"), to_gpu(torch, B, "f32"), transposed)
    torch.cuda.synchronize()
    assert zr.debug_last_kernel() == f"f32_kernel<P, {'P' if transposed else 'Q'}, 128>", zr.debug_last_kernel()
    check_kept_np("out", to_np(out), oracle.migrated_accumulate(base, A, B, transposed), "f32", C)
    # the resized products at the same sizes
    X, W = to_gpu(torch, A, "f32"), to_gpu(torch, np.ascontiguousarray(B if not transposed else B.T), "f32")
    zr.resized_linear_fwd(X, W, idx_gpu(torch, subset(3, N, N - 1)), DROP_N)
    assert zr.debug_last_kernel() == "f32_kernel<P, Qg, 128>", zr.debug_last_kernel()

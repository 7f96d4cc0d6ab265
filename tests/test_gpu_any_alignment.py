"""The bf16 products for any alignment at the edges of their tiles and stages: 32 x 32 tiles (256-deep stages),
64 x 64 (128-deep, from 96 tiles on; 256-deep with 512 threads up to 256 tiles, contractions from 256 on) and
128 x 128 (64-deep, from 256 tiles on), contractions of one element
up to a little over two stages, rows shorter than the eight elements of a load, odd leading dimensions; both
layouts, all loaders and epilogues.  Against the float64 oracle with the bounds of parity_util."""
import numpy as np
import pytest

from paper_2401_11469_amd import workloads as wl
from parity_util import check_kept_np
from test_gpu_parity import AVERAGE, DROP_K, DROP_N, SAME, ZERO, W_KN, W_NK, check_layer, run_layer, subset, to_gpu, to_np
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [DROP_N, DROP_K])
@pytest.mark.parametrize("layout", [W_KN, W_NK])
@pytest.mark.parametrize("M,K,N", [(31, 33, 32), (33, 255, 64), (65, 257, 3), (64, 3, 130), (2, 515, 5), (9, 1, 2),    # 32 x 32
                                   (833, 67, 901), (897, 7, 830), (70, 900, 833), (832, 896, 129), (641, 771, 1003),                # 64 x 64
                                   (2497, 65, 2433), (2500, 2433, 63), (129, 2561, 2497)])                          # 128 x 128
def test_bf16_tile_edges(zr, torch_mod, oracle, mode, layout, M, K, N):  # noqa: F811
    case = wl.random_case(31 * M + 7 * K + N, M, K, N, "bf16")
    n = N if mode == DROP_N else K
    big = M * K * N > 1 << 28
    for n_keep, policy in ((n, ZERO), ((3 * n + 3) // 4, ZERO), (max(1, n // 5), SAME), (max(1, n - 1), AVERAGE))[1 if big else 0:]:
        S = subset(n_keep + n, n, n_keep)
        got = run_layer(zr, torch_mod, case, S, mode, "bf16", policy, pad=5 if policy == SAME else 1, w_layout=layout,
                        use_ws=policy == AVERAGE)
        check_layer(oracle, case, S, mode, "bf16", policy, got)


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("M,N,C", [(40, 9, 7), (70, 131, 229), (900, 833, 131), (2497, 2433, 61)])
def test_bf16_accumulate_tile_edges(zr, torch_mod, oracle, transposed, M, N, C):  # noqa: F811
    torch = torch_mod
    g = np.random.Generator(np.random.PCG64(M + N + C))
    cast = wl.round_to_bf16
    A = cast(g.standard_normal((M, C + 3)).astype(np.float32))
    Wm = cast((g.standard_normal((N, C + 3) if transposed else (C + 3, N)) * 0.05).astype(np.float32))
    base = cast(g.standard_normal((M, N)).astype(np.float32))
    Ag, Wg, out = to_gpu(torch, A, "bf16"), to_gpu(torch, Wm, "bf16"), to_gpu(torch, base, "bf16", ld=N + 3)
    sl = slice(1, 1 + C)
    zr.migrated_accumulate(out, Ag[:, sl], Wg[:, sl] if transposed else Wg[sl, :], transposed)
    torch.cuda.synchronize()
    assert torch.all(out._base[:, N:] == 777.0), "padding overwritten"
    want = oracle.migrated_accumulate(base, A[:, sl], Wm[:, sl] if transposed else Wm[sl, :], transposed)
    check_kept_np("out", to_np(out), want, "bf16", C)

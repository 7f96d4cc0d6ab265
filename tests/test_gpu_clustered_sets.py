"""Kept sets with long dropped ranges (prefix, suffix, two ends) on the tiles of the small-tile bf16 kernel and of
the fp32 kernel: a range behind a tile's last kept column or between two kept rows is filled 16 bytes a lane.
Zero and Same (also in place), odd pitches.  Against the float64 oracle with the bounds of parity_util."""
import numpy as np
import pytest

from paper_2401_11469_amd import workloads as wl
from test_gpu_parity import DROP_K, DROP_N, SAME, ZERO, W_KN, W_NK, check_layer, idx_gpu, run_layer, to_gpu, to_np
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode", [DROP_N, DROP_K])
@pytest.mark.parametrize("M,K,N", [(70, 1330, 1331), (830, 40, 1400), (900, 1403, 70), (40, 900, 1900), (1900, 24, 2900)])
def test_long_dropped_ranges(zr, torch_mod, oracle, dtype, mode, M, K, N):  # noqa: F811
    case = wl.random_case(17 * M + K + N, M, K, N, dtype)
    n = N if mode == DROP_N else K
    sets = [np.arange(n // 3), np.arange(n - n // 3, n), np.concatenate([np.arange(n // 5), np.arange(n - 3, n)]), np.array([n - 1])]
    for i, S in enumerate(sets):
        S = S.astype(np.int32)
        for layout in (W_KN, W_NK):
            for policy, pad in ((ZERO, 0), (SAME, 1 + i)):
                got = run_layer(zr, torch_mod, case, S, mode, dtype, policy, pad=pad, w_layout=layout)
                check_layer(oracle, case, S, mode, dtype, policy, got)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_long_dropped_ranges_in_place(zr, torch_mod, oracle, dtype):  # noqa: F811
    torch = torch_mod
    M, K, N = 300, 264, 2001
    case = wl.random_case(4711, M, K, N, dtype)
    S = np.arange(700, dtype=np.int32)
    X, W, dY = (to_gpu(torch, case[k], dtype, ld=c + 3) for k, c in (("X", K), ("W", N), ("dY", N)))
    Y, dW = (to_gpu(torch, case[k], dtype, ld=N + 3) for k in ("prev_Y", "prev_dW"))
    zr.resized_linear_fwd(X, W, idx_gpu(torch, S), DROP_N, SAME, Y, Y=Y)
    dX, _ = zr.resized_linear_bwd(X, W, dY, idx_gpu(torch, S), DROP_N, SAME, None, dW, dW=dW)
    torch.cuda.synchronize()
    check_layer(oracle, case, S, DROP_N, dtype, SAME, (to_np(Y), to_np(dX), to_np(dW)))

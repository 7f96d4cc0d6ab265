"""Aligned bf16 products around the limits of the rules on the number of 128 x 128 tiles: the 64 x 128
tiles (65 to 256 tiles, to 384 up to 1024 deep; 192 and 64 deep here) with ragged last tiles, and contractions that
are no multiple of 64 (1128 and 136 deep), which leave the direct-to-LDS loaders and with them those tiles; with and
without scratch, all policies.  Against the float64 oracle with the bounds of parity_util.  (Which kernel each takes:
test_gpu_dispatch_rules.py.)"""
import pytest

from paper_2401_11469_amd import workloads as wl
from test_gpu_parity import AVERAGE, DROP_K, DROP_N, SAME, ZERO, W_KN, W_NK, check_layer, run_layer, subset
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


# (M, K, N): fwd DROP_N and dX DROP_K in the row-gather layouts have 66..., 150... and 384 / 390 tiles
@pytest.mark.parametrize("mode", [DROP_N, DROP_K])
@pytest.mark.parametrize("M,K,N", [(1352, 192, 1096), (2000, 1128, 1384), (3088, 64, 2104), (2440, 136, 2600)])
def test_few_tiles(zr, torch_mod, oracle, mode, M, K, N):  # noqa: F811
    if mode == DROP_K:
        K, N = N, K
    case = wl.random_case(M + 3 * K + 5 * N, M, K, N, "bf16")
    n = N if mode == DROP_N else K
    layout = W_NK if mode == DROP_N else W_KN
    for n_keep, policy, ws in ((n, ZERO, False), ((3 * n) // 4, ZERO, True), ((7 * n) // 8, SAME, False), (n - 1, AVERAGE, True)):
        S = subset(n_keep + n, n, n_keep)
        got = run_layer(zr, torch_mod, case, S, mode, "bf16", policy, w_layout=layout, use_ws=ws)
        check_layer(oracle, case, S, mode, "bf16", policy, got)

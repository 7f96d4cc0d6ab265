"""The fp32 products at the edges of their smaller tiles and stages: 32 x 32 tiles (128-deep stages), 64 x 64
tiles (64-deep stages, taken from 192 tiles on; 128 x 128 tiles: test_gpu_f32_big_tiles.py), contractions of one element up to a little over a
stage, and rows shorter than the four elements of a load; both layouts, all loaders.  Against the
float64 oracle with the bounds of parity_util (fp32: 1e-5 of the largest value)."""
import numpy as np
import pytest

from paper_2401_11469_amd import workloads as wl
from test_gpu_parity import AVERAGE, DROP_K, DROP_N, SAME, ZERO, W_KN, W_NK, check_layer, run_layer, subset
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [DROP_N, DROP_K])
@pytest.mark.parametrize("layout", [W_KN, W_NK])
@pytest.mark.parametrize("M,K,N", [(31, 33, 32), (33, 127, 64), (65, 129, 3), (64, 3, 130), (2, 260, 5),      # 32 x 32 tiles
                                   (833, 67, 901), (897, 2, 830), (70, 900, 833), (832, 896, 65)])            # 64 x 64 tiles
def test_f32_tile_edges(zr, torch_mod, oracle, mode, layout, M, K, N):  # noqa: F811
    case = wl.random_case(31 * M + 7 * K + N, M, K, N, "f32")
    n = N if mode == DROP_N else K
    for n_keep, policy in ((n, ZERO), ((3 * n + 3) // 4, ZERO), (max(1, n // 5), SAME), (max(1, n - 1), AVERAGE)):
        S = subset(n_keep + n, n, n_keep)
        got = run_layer(zr, torch_mod, case, S, mode, "f32", policy, pad=5 if policy == SAME else 0, w_layout=layout,
                        use_ws=policy == AVERAGE)
        check_layer(oracle, case, S, mode, "f32", policy, got)

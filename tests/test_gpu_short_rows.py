"""Products with a contiguous extent below what a vector load reads (contractions of one to seven, results of one
to seven rows or columns), which go through the element loaders: 128 x 128, 64 x 64 and 32 x 32 tiles by the number
of tiles, both layouts, all policies, rows of any alignment.  Against the float64 oracle with the bounds of
parity_util."""
import numpy as np
import pytest

from paper_2401_11469_amd import workloads as wl
from parity_util import check_kept_np
from test_gpu_parity import AVERAGE, DROP_K, DROP_N, SAME, ZERO, W_KN, W_NK, check_layer, run_layer, subset, to_gpu, to_np
from test_gpu_parity import torch_mod, zr  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layout", [W_KN, W_NK])
@pytest.mark.parametrize("M,K,N", [(2041, 3, 1930), (700, 7, 901), (65, 2, 130),          # forward: K short
                                   (1793, 2100, 2), (130, 70, 5),                          # dX, and a narrow forward
                                   (3, 2049, 1800), (7, 901, 830), (1, 33, 40),            # dW: few tokens
                                   (5, 3, 2), (4, 6, 2500)])
def test_short_rows(zr, torch_mod, oracle, dtype, layout, M, K, N):  # noqa: F811
    case = wl.random_case(31 * M + 7 * K + N, M, K, N, dtype)
    for mode in (DROP_N, DROP_K):
        n = N if mode == DROP_N else K
        for n_keep, policy, pad in ((n, ZERO, 0), (max(1, (3 * n) // 4), ZERO, 1), (max(1, (2 * n) // 3), SAME, 3),
                                    (max(1, n - 1), AVERAGE, 0)):
            S = subset(n_keep + n, n, n_keep)
            got = run_layer(zr, torch_mod, case, S, mode, dtype, policy, pad=pad, w_layout=layout, use_ws=policy == AVERAGE)
            check_layer(oracle, case, S, mode, dtype, policy, got)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("M,N,C,tile", [(2041, 1930, 3, 128), (700, 901, 1, 64), (130, 70, 2, 32)])
def test_short_contractions_take_tiles_by_their_number(zr, torch_mod, oracle, dtype, transposed, M, N, C, tile):  # noqa: F811
    """A migrated share of a few columns: on 32 x 32 tiles of 256-deep stages it took ten times as long (8192 x 4096,
    3 deep: 605 us against 43)."""
    torch = torch_mod
    if dtype == "f32" and tile == 64 and M * N < 192 * 64 * 64:
        tile = 32                       # (fp32 leaves 32 x 32 tiles at 192 of 64 x 64)
    g = np.random.Generator(np.random.PCG64(M + N + C))
    cast = wl.round_to_bf16 if dtype == "bf16" else (lambda x: x)
    A = cast(g.standard_normal((M, C)).astype(np.float32))
    B = cast((g.standard_normal((N, C) if transposed else (C, N)) * 0.05).astype(np.float32))
    base = cast(g.standard_normal((M, N)).astype(np.float32))
    out = to_gpu(torch, base, dtype, ld=N + 3)
    zr.migrated_accumulate(out, to_gpu(torch, A, dtype), to_gpu(torch, B, dtype), transposed)
    torch.cuda.synchronize()
    name = zr.debug_last_kernel()
    assert f", {tile}, 256>" in name if dtype == "bf16" else name.endswith(f", {tile}>"), name
    assert torch.all(out._base[:, N:] == 777.0), "padding overwritten"
    check_kept_np("out", to_np(out), oracle.migrated_accumulate(base, A, B, transposed), dtype, C)


def test_short_contraction_of_a_very_large_result(zr, torch_mod):  # noqa: F811
    """131104 x 131104 results of one product each (34 GB): 4097^2 tiles of 32 x 32 are more threads than a launch
    can have."""
    torch = torch_mod
    n = 131104
    if torch.cuda.mem_get_info()[0] < 48 << 30:
        pytest.skip("needs 48 GB")
    a, b = (torch.randn(n, 1, dtype=torch.float32, device="cuda").to(torch.bfloat16) for _ in range(2))
    out = torch.zeros(n, n, dtype=torch.bfloat16, device="cuda")
    zr.migrated_accumulate(out, a, b, True)
    torch.cuda.synchronize()
    rows = torch.tensor([0, 1, 127, 128, 65535, 65536, n - 129, n - 1], device="cuda")
    want = (a[rows].float() * b.float().t()).to(torch.bfloat16)           # one product: exact in fp32, one rounding
    assert torch.equal(out[rows], want)

"""The forms of the launch of dX and dW together, each by its name: against fp32 products of the masked operands, with means and
previous tensors as imputed values; what takes longer in one launch, and what may not share one."""
import os
import subprocess
import sys

import pytest

from parity_util import check_kept_torch
from test_gpu_backward_pairs import AVERAGE, DROP_K, DROP_N, SAME, W_KN, W_NK, ZERO, tensors
from test_gpu_backward_pairs import torch_zr  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def check_pair(torch_zr, M, K, N, mode, n_keep, policy, layout=None, scratch=True):
    """Both products, twice; the kernel's name.  (Default: kept indices are rows of the stored shard.)"""
    torch, zr = torch_zr
    if layout is None:
        layout = W_NK if mode == DROP_N else W_KN
    nk = layout == W_NK
    X, W, dY = tensors(torch, M, K, N, nk, M + K + N + n_keep)
    n = N if mode == DROP_N else K
    gen = torch.Generator(device="cuda").manual_seed(n_keep)
    keep = torch.randperm(n, generator=gen, device="cuda")[:n_keep].sort().values.to(torch.int32)
    ws = torch.empty(zr.workspace_bytes(M, K, N, n_keep, mode, torch.bfloat16), dtype=torch.uint8, device="cuda") if scratch else None
    prev = dict(prev_dX=torch.full_like(X, 2.0), prev_dW=torch.full_like(W, 3.0)) if policy == SAME else {}
    dX, dW = zr.resized_linear_bwd(X, W, dY, keep, mode, policy=policy, workspace=ws, w_layout=layout, **prev)
    name = zr.debug_last_kernel()
    print(name, flush=True)
    again = zr.resized_linear_bwd(X, W, dY, keep, mode, policy=policy, workspace=ws, w_layout=layout, **prev)
    assert torch.equal(dX, again[0]) and torch.equal(dW, again[1])
    kept = torch.zeros(n, dtype=torch.bool, device="cuda")
    kept[keep.long()] = True
    Wk = (W.t() if nk else W).float()
    dWk = dW.t() if nk else dW
    if mode == DROP_K:
        check_kept_torch("dX", dX, dY.float() @ (Wk * kept[:, None]).t(), "bf16", N, kept[None, :])
        check_kept_torch("dW", dWk, (X.float() * kept[None, :]).t() @ dY.float(), "bf16", M, kept[:, None])
        rest = ((dX[:, ~kept], dX[:, kept], 1, 2.0), (dWk[~kept], dWk[kept], 0, 3.0))
    else:
        check_kept_torch("dX", dX, (dY.float() * kept[None, :]) @ Wk.t(), "bf16", n_keep, None)
        check_kept_torch("dW", dWk, X.float().t() @ (dY.float() * kept[None, :]), "bf16", M, kept[None, :])
        rest = ((dWk[:, ~kept], dWk[:, kept], 1, 3.0),)
    for dropped, stored, axis, v in rest:
        if policy == AVERAGE:
            # the mean of n_keep stored values in fp32 (as in acc_term), rounded once to bf16
            want = stored.double().mean(dim=axis, keepdim=True)
            bound = 2.0 ** -8 * want.abs() * (1 + 2.0 ** -10) + 8 * n_keep ** 0.5 * 2.0 ** -24 * stored.double().abs().mean(dim=axis, keepdim=True)
            assert torch.all((dropped.double() - want).abs() <= bound)
        else:
            assert torch.all(dropped == (v if policy == SAME else 0.0))
    return name


# One shape for every form of the launch: dW's tiles (in slices: split) beside dX's, by where dX finds the rows of W.
@pytest.mark.parametrize("M,K,N,mode,n_keep,form", [
    (512, 3808, 576, DROP_K, 2067, "DmaQ, DmaQ, 128, 128> beside <DmaP, DmaP, 64, 128>"),
    (2112, 808, 352, DROP_K, 478, "DmaQ, DmaQ, 128, 128> beside <DmaP, DmaP, 64, 128> split"),
    (71, 3696, 112, DROP_K, 3696, "DmaQ, DmaQ, 128, 128> beside <DmaP, DmaP, 128, 128>"),
    (3776, 160, 64, DROP_K, 103, "DmaQ, DmaQ, 128, 128> beside <DmaP, DmaP, 128, 128> split"),
    (219, 4504, 112, DROP_N, 112, "DmaQ, DmaQ, 128, 128> beside <DmaP, DmaQ, 128, 128>"),
    (4060, 72, 80, DROP_N, 80, "DmaQ, DmaQ, 128, 128> beside <DmaP, DmaQ, 128, 128> split"),
    (128, 3328, 104, DROP_N, 87, "DmaQ, DmaQ, 128, 128> beside <DmaP, DmaQM, 128, 128>"),
    (3328, 80, 112, DROP_N, 101, "DmaQ, DmaQ, 128, 128> beside <DmaP, DmaQM, 128, 128> split"),
    (1445, 3136, 1272, DROP_K, 3136, "RingQ, RingQ, 192, 256> beside <RingP, RingP, 256, 192>"),
    (4505, 1104, 760, DROP_K, 1057, "RingQ, RingQ, 192, 256> beside <RingP, RingP, 256, 192> split"),
    (3904, 2184, 1808, DROP_K, 2054, "RingQ, RingQ, 192, 256> beside <RingP, RingP, 256, 256>"),
    (6592, 1088, 504, DROP_K, 774, "RingQ, RingQ, 192, 256> beside <RingP, RingP, 256, 256> split"),
    (1294, 4096, 1944, DROP_K, 2845, "RingQ, RingQ, 256, 256> beside <RingP, RingP, 256, 192>"),
    (1748, 3472, 568, DROP_K, 2707, "RingQ, RingQ, 256, 256> beside <RingP, RingP, 256, 192> split"),
    (1984, 3600, 2720, DROP_K, 3008, "RingQ, RingQ, 256, 256> beside <RingP, RingP, 256, 256>"),
    (3648, 3048, 456, DROP_K, 2300, "RingQ, RingQ, 256, 256> beside <RingP, RingP, 256, 256> split"),
    (2165, 1960, 2216, DROP_N, 2216, "RingQ, RingQ, 192, 256> beside <RingP, RingQ, 256, 192>"),
    (7232, 528, 1024, DROP_N, 1024, "RingQ, RingQ, 192, 256> beside <RingP, RingQ, 256, 192> split"),
    (1280, 4728, 648, DROP_N, 648, "RingQ, RingQ, 192, 256> beside <RingP, RingQ, 256, 256>"),
    (3698, 2808, 168, DROP_N, 168, "RingQ, RingQ, 192, 256> beside <RingP, RingQ, 256, 256> split"),
    (3492, 1472, 3952, DROP_N, 3952, "RingQ, RingQ, 256, 256> beside <RingP, RingQ, 256, 192>"),
    (4579, 1200, 1792, DROP_N, 1792, "RingQ, RingQ, 256, 256> beside <RingP, RingQ, 256, 192> split"),
    (2624, 4272, 4592, DROP_N, 4592, "RingQ, RingQ, 256, 256> beside <RingP, RingQ, 256, 256>"),
    (4480, 3344, 400, DROP_N, 400, "RingQ, RingQ, 256, 256> beside <RingP, RingQ, 256, 256> split"),
    (1216, 3392, 1272, DROP_N, 1059, "RingQ, RingQ, 192, 256> beside <RingP, RingQM, 256, 192>"),
    (2240, 2112, 424, DROP_N, 370, "RingQ, RingQ, 192, 256> beside <RingP, RingQM, 256, 192> split"),
    (1406, 3600, 1720, DROP_N, 1194, "RingQ, RingQ, 192, 256> beside <RingP, RingQM, 256, 256>"),
    (2496, 2472, 512, DROP_N, 342, "RingQ, RingQ, 192, 256> beside <RingP, RingQM, 256, 256> split"),
    (1856, 2416, 3528, DROP_N, 2751, "RingQ, RingQ, 256, 256> beside <RingP, RingQM, 256, 192>"),
    (2374, 2160, 1392, DROP_N, 1110, "RingQ, RingQ, 256, 256> beside <RingP, RingQM, 256, 192> split"),
    (1408, 3504, 4352, DROP_N, 2397, "RingQ, RingQ, 256, 256> beside <RingP, RingQM, 256, 256>"),
    (2396, 2600, 808, DROP_N, 625, "RingQ, RingQ, 256, 256> beside <RingP, RingQM, 256, 256> split")])
def test_every_form(torch_zr, M, K, N, mode, n_keep, form):  # noqa: F811
    name = check_pair(torch_zr, M, K, N, mode, n_keep, ZERO)
    assert name == "fast_kernel<" + form, name


@pytest.mark.parametrize("M,K,N,mode,n_keep", [
    (4096, 2048, 2048, DROP_K, 1536), (2024, 1024, 1024, DROP_K, 768), (8192, 2752, 4096, DROP_K, 2064), (8192, 1280, 5120, DROP_K, 1088),
    (8192, 5120, 1280, DROP_N, 1088), (1856, 2416, 3528, DROP_N, 2751)])
def test_pair_with_average_and_scratch(torch_zr, M, K, N, mode, n_keep):  # noqa: F811
    """One launch with the stand-alone passes behind it, although the buffer has room for the sums of two launches."""
    name = check_pair(torch_zr, M, K, N, mode, n_keep, AVERAGE)
    assert "beside" in name, name


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("policy", [ZERO, AVERAGE, SAME])
@pytest.mark.parametrize("layout", [W_KN, W_NK])
@pytest.mark.parametrize("mode", [DROP_N, DROP_K])
# 64 x 64 and 128 x 128; nothing pruned; 128 x 128; aligned rows, which other kernels take on their own
@pytest.mark.parametrize("M,K,N,n_keep", [(2497, 1201, 803, 640), (300, 2305, 1999, 1500), (256, 512, 256, 0), (1031, 2051, 2053, 1500), (1024, 2048, 2048, 1536)])
def test_larger_pair_of_any_alignment(torch_zr, M, K, N, n_keep, mode, layout, policy, dtype):  # noqa: F811
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
    assert "beside" in name, name
    for what, x, y, C in (("dX", a[0], dX, N), ("dW", a[1], dW, M)):
        if dtype == "bf16":
            assert torch.equal(x, y), what
        else:
            # two sums of C terms in different orders: C ** 0.5 roundings of 2 ** -24 each, with a factor of 8
            assert float((x - y).abs().max()) <= 8 * max(C, 16) ** 0.5 * 2.0 ** -24 * float(y.abs().max()), what


# The forms of the kernels for any alignment that the sizes above do not reach: loaders of dX and of dW, tiles of dW and of dX.
@pytest.mark.parametrize("M,K,N,mode,layout,n_keep,scratch,form", [
    (1088, 4899, 193, DROP_N, W_KN, 193, False, "P, P; Q, Q> beside each other, 128 and 128"),
    (128, 3200, 784, DROP_N, W_KN, 784, True, "P, P; Q, Q> beside each other, 128 and 64"),
    (163, 2440, 80, DROP_K, W_KN, 2008, True, "P, P; Q, Q> beside each other, 32 and 64"),
    (447, 4309, 121, DROP_N, W_KN, 121, False, "P, P; Q, Q> beside each other, 64 and 128"),
    (32, 80, 4976, DROP_K, W_KN, 75, True, "P, P; Q, Q> beside each other, 64 and 32"),
    (81, 3637, 83, DROP_K, W_KN, 3637, False, "P, P; Q, Q> beside each other, 64 and 64"),
    (192, 3241, 661, DROP_K, W_KN, 3143, False, "P, P; Qg, Q> beside each other, 128 and 64"),
    (3328, 80, 96, DROP_K, W_KN, 67, False, "P, P; Qg, Q> beside each other, 32 and 64"),
    (57, 96, 3288, DROP_K, W_KN, 87, False, "P, P; Qg, Q> beside each other, 64 and 32"),
    (517, 3304, 456, DROP_N, W_KN, 327, True, "P, Pg; Q, Q> beside each other, 128 and 128"),
    (128, 4448, 880, DROP_N, W_KN, 447, True, "P, Pg; Q, Q> beside each other, 128 and 64"),
    (68, 72, 80, DROP_N, W_KN, 37, True, "P, Pg; Q, Q> beside each other, 32 and 32"),
    (192, 2200, 72, DROP_N, W_KN, 34, True, "P, Pg; Q, Q> beside each other, 32 and 64"),
    (320, 5040, 280, DROP_N, W_KN, 189, True, "P, Pg; Q, Q> beside each other, 64 and 128"),
    (64, 2960, 168, DROP_N, W_KN, 139, True, "P, Pg; Q, Q> beside each other, 64 and 32"),
    (128, 4736, 128, DROP_N, W_KN, 74, True, "P, Pg; Q, Q> beside each other, 64 and 64"),
    (70, 4159, 343, DROP_K, W_NK, 4159, True, "P, Q; Q, Q> beside each other, 128 and 64"),
    (258, 1392, 64, DROP_N, W_NK, 41, True, "P, Q; Q, Q> beside each other, 32 and 64"),
    (883, 3296, 104, DROP_N, W_NK, 69, True, "P, Q; Q, Q> beside each other, 64 and 128"),
    (41, 144, 2144, DROP_N, W_NK, 2144, False, "P, Q; Q, Q> beside each other, 64 and 32"),
    (201, 1584, 336, DROP_K, W_NK, 1584, False, "P, Q; Q, Q> beside each other, 64 and 64"),
    (534, 3080, 440, DROP_K, W_NK, 2637, True, "P, Qg; Q, Q> beside each other, 128 and 128"),
    (259, 1704, 1424, DROP_K, W_NK, 1325, True, "P, Qg; Q, Q> beside each other, 128 and 64"),
    (81, 216, 72, DROP_K, W_NK, 197, True, "P, Qg; Q, Q> beside each other, 32 and 32"),
    (1600, 232, 112, DROP_K, W_NK, 217, True, "P, Qg; Q, Q> beside each other, 32 and 64"),
    (654, 4160, 184, DROP_K, W_NK, 3490, True, "P, Qg; Q, Q> beside each other, 64 and 128"),
    (33, 1560, 472, DROP_K, W_NK, 1399, True, "P, Qg; Q, Q> beside each other, 64 and 32"),
    (87, 3176, 136, DROP_K, W_NK, 3054, True, "P, Qg; Q, Q> beside each other, 64 and 64"),
    (768, 2913, 1193, DROP_K, W_NK, 2003, True, "P, Qg; Q, Qg> beside each other, 128 and 128"),
    (320, 4328, 416, DROP_K, W_NK, 3002, False, "P, Qg; Q, Qg> beside each other, 128 and 64"),
    (229, 2680, 80, DROP_K, W_NK, 2096, False, "P, Qg; Q, Qg> beside each other, 32 and 64"),
    (36, 1264, 352, DROP_K, W_NK, 1149, False, "P, Qg; Q, Qg> beside each other, 64 and 32"),
    (896, 449, 73, DROP_N, W_KN, 44, True, "Pg, Pg; Q, Qg> beside each other, 32 and 64"),
    (35, 112, 5048, DROP_N, W_KN, 3726, False, "Pg, Pg; Q, Qg> beside each other, 64 and 32"),
    (2240, 144, 64, DROP_N, W_NK, 31, False, "Pg, Q; Qg, Q> beside each other, 32 and 64"),
    (36, 152, 3424, DROP_N, W_NK, 2397, False, "Pg, Q; Qg, Q> beside each other, 64 and 32")])
def test_every_form_of_any_alignment(torch_zr, M, K, N, mode, layout, n_keep, scratch, form):  # noqa: F811
    name = check_pair(torch_zr, M, K, N, mode, n_keep, ZERO, layout, scratch)
    assert name == "gemm_kernel<" + form, name


@pytest.mark.parametrize("M,K,N,mode,layout,n_keep,scratch,dtype,refused", [
    # a gather in flight in dW: estimated by tokens and the share of columns kept (us in two launches and one: 189, 281; 454, 470)
    (4832, 2184, 2840, DROP_K, W_NK, 1249, False, "bf16", "beside"), (16384, 2048, 2048, DROP_K, W_KN, 2000, False, "bf16", "beside"),
    # dW in slices (208, 329)
    (9600, 704, 4800, DROP_K, W_NK, 588, True, "bf16", "beside"),
    # rows that Same copies, on 128 x 128 tiles (17.9, 33; on 64 x 64 14.8)
    (192, 2288, 608, DROP_N, W_NK, 248, True, "same", "fast_kernel"),
    # fp32 on 128 x 128 tiles (100, 138; on 64 x 64 92)
    (1088, 3324, 484, DROP_N, W_KN, 465, False, "f32", "128")])
def test_forms_that_take_longer(torch_zr, M, K, N, mode, layout, n_keep, scratch, dtype, refused):  # noqa: F811
    torch, zr = torch_zr
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    X, W, dY = (t.to(dt) for t in tensors(torch, M, K, N, layout == W_NK, 1))
    n = N if mode == DROP_N else K
    keep = torch.randperm(n, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")[:n_keep].sort().values.to(torch.int32)
    ws = torch.empty(zr.workspace_bytes(M, K, N, n_keep, mode, dt), dtype=torch.uint8, device="cuda") if scratch else None
    same = dict(policy=SAME, prev_dX=torch.zeros_like(X), prev_dW=torch.zeros_like(W)) if dtype == "same" else dict(policy=ZERO)
    zr.resized_linear_bwd(X, W, dY, keep, mode, workspace=ws, w_layout=layout, **same)
    assert refused not in zr.debug_last_kernel(), zr.debug_last_kernel()


@pytest.mark.parametrize("M,K,N,mode,layout,n_keep,form", [
    # fp32 on 128 x 128 tiles: a unit to each of them, both products gathered, depths within 1.2 of each other
    (1576, 1024, 2048, DROP_N, W_NK, 1638, "f32_kernel<Qg, Q, 128> beside <Pg, Q, 128>"),
    (1840, 1008, 2300, DROP_N, W_KN, 1861, "f32_kernel<Q, Qg, 128> beside <Pg, Pg, 128>"),
    (1753, 1100, 1985, DROP_K, W_NK, 877, "f32_kernel<Q, Qg, 128> beside <P, Qg, 128>"),
    # one more tile than units, depths further apart, too few tiles of 64 x 64, one product that gathers nothing
    (1920, 1024, 2400, DROP_N, W_NK, 2200, None), (1536, 1301, 1500, DROP_N, W_KN, 1198, None), (1400, 1000, 1700, DROP_N, W_NK, 1400, None),
    (1576, 2048, 1600, DROP_K, W_KN, 1024, None)])
def test_fp32_pair_of_one_round(torch_zr, M, K, N, mode, layout, n_keep, form):  # noqa: F811
    torch, zr = torch_zr
    X, W, dY = (t.float() for t in tensors(torch, M, K, N, layout == W_NK, M + K + N))
    n = N if mode == DROP_N else K
    keep = torch.randperm(n, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda")[:n_keep].sort().values.to(torch.int32)
    a = zr.resized_linear_bwd(X, W, dY, keep, mode, w_layout=layout)
    name = zr.debug_last_kernel()
    assert (name == form) if form else ("128> beside" not in name), name
    kept = torch.zeros(n, device="cuda")
    kept[keep.long()] = 1.0
    Xd, Wd, dYd = X.double(), (W.t() if layout == W_NK else W).double(), dY.double()
    if mode == DROP_K:
        Xd, Wd = Xd * kept[None, :], Wd * kept[:, None]
    else:
        dYd = dYd * kept[None, :]
    dX, dW = dYd @ Wd.t(), Xd.t() @ dYd
    if layout == W_NK:
        dW = dW.t()
    for what, got, want, C in (("dX", a[0], dX, n_keep if mode == DROP_N else N), ("dW", a[1], dW, M)):
        # the error of C fp32 additions in any order grows as sqrt(C); 8 covers the largest of 4 million
        assert float((got.double() - want).abs().max()) <= 8 * C ** 0.5 * 2.0 ** -24 * float(want.abs().max()), what


def test_ring_switch_keeps_the_products_apart(torch_zr):  # noqa: F811
    """ZR_NO_RING is read once per process: in a child process, a call that is paired without it."""
    M, K, N, n_keep = 1984, 3600, 2720, 3008               # (see test_every_form)
    code = f"""
import torch
from paper_2401_11469_amd import zr
zr.debug_record_kernel_names(True)
r = lambda a, b: torch.zeros(a, b, dtype=torch.bfloat16, device="cuda")
ws = torch.empty(zr.workspace_bytes({M}, {K}, {N}, {n_keep}, 1, torch.bfloat16), dtype=torch.uint8, device="cuda")
zr.resized_linear_bwd(r({M}, {K}), r({K}, {N}), r({M}, {N}), torch.arange({n_keep}, dtype=torch.int32, device="cuda"), 1, workspace=ws)
torch.cuda.synchronize()
print(zr.debug_last_kernel())
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", code], cwd=root, env=dict(os.environ, ZR_NO_RING="1"), stdout=subprocess.PIPE, text=True, timeout=100)
    assert res.returncode == 0
    name = res.stdout.splitlines()[-1]
    assert "kernel<" in name and "Ring" not in name and "beside" not in name, name


@pytest.mark.parametrize("what", ["dW over W", "dX over X", "dX over dY", "dW over dY", "dW over dX", "prev_dW in dX", "dW over prev_dX"])
def test_overlaps_of_results_and_operands(torch_zr, what):  # noqa: F811
    """Where one product writes what the other reads or writes they run one after the other, dX first: dW may take the place
    of W, which only dX reads, dX that of X once X[:,S] is extracted, either that of dY once dY[:,S] is, and the previous
    tensor of the one may lie where the other is written."""
    torch, zr = torch_zr
    M, K, N = 2048, 2816, 2048
    mode = DROP_N if "dY" in what else DROP_K              # dY[:,S] is extracted in DROP_N
    layout = W_NK if mode == DROP_N else W_KN
    X, W, dY = tensors(torch, M, K, N, layout == W_NK, 5)
    keep = torch.arange(0, N if mode == DROP_N else K, 2, dtype=torch.int32, device="cuda")
    ws = torch.empty(zr.workspace_bytes(M, K, N, keep.numel(), mode, torch.bfloat16), dtype=torch.uint8, device="cuda")
    kw = dict(workspace=ws, w_layout=layout, policy=SAME if "prev" in what else ZERO)
    prev_dX, prev_dW = (torch.full_like(X, 2.0), torch.full_like(W, 3.0)) if "prev" in what else (None, None)
    dX = zr.resized_linear_bwd(X, W, dY, keep, mode, need_dW=False, prev_dX=prev_dX, **kw)[0]
    if what == "prev_dW in dX":
        prev_dW = dX.reshape(-1)[:W.numel()].view(W.shape)             # what dX has just written
    dW = zr.resized_linear_bwd(X, W, dY, keep, mode, need_dX=False, prev_dW=prev_dW, **kw)[1]
    check = ("dX", "dW")
    if what == "dW over W":
        out = dict(dW=W)
    elif what == "dX over X":
        out = dict(dX=X)
    elif what == "dX over dY":                             # (dY at the end of dX's place)
        room = torch.empty(M * K, dtype=torch.bfloat16, device="cuda")
        room[-dY.numel():].view_as(dY).copy_(dY)
        dY, out = room[-dY.numel():].view_as(dY), dict(dX=room.view(M, K))
    elif what == "dW over dY":
        room = torch.empty(max(W.numel(), dY.numel()), dtype=torch.bfloat16, device="cuda")
        room[-dY.numel():].view_as(dY).copy_(dY)
        dY, out = room[-dY.numel():].view_as(dY), dict(dW=room[:W.numel()].view(W.shape))
    elif what == "dW over dX":
        room = torch.empty(max(W.numel(), X.numel()), dtype=torch.bfloat16, device="cuda")
        out, check = dict(dX=room[:X.numel()].view(X.shape), dW=room[:W.numel()].view(W.shape)), ("dW",)
    elif what == "prev_dW in dX":
        out = dict(dX=torch.empty_like(dX))
        prev_dW = out["dX"].reshape(-1)[:W.numel()].view(W.shape)
    else:
        out = dict(dW=prev_dX.reshape(-1)[:W.numel()].view(W.shape))
    a, b = zr.resized_linear_bwd(X, W, dY, keep, mode, prev_dX=prev_dX, prev_dW=prev_dW, **out, **kw)
    assert "beside" not in zr.debug_last_kernel()
    assert "dX" not in check or torch.equal(a, dX)
    assert torch.equal(b, dW)

"""Selection at the edges of the forms a vector's length and the number of vectors choose: exact against the oracle, with
keys that share their leading bits, keys over the whole range, and ties."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_zr():
    import torch
    from paper_2401_11469_amd import zr
    return torch, zr


def scores(kind, rng, *shape):
    if kind == "close":
        s = 1.28 + 0.0141 * rng.standard_normal(shape)
    elif kind == "wide":
        s = rng.standard_normal(shape) * 10.0 ** rng.integers(-30, 30, size=shape)
    else:
        s = rng.integers(0, 3, size=shape)
    s = s.astype(np.float32)
    if kind == "wide":
        flat = s.reshape(-1)
        flat[::7], flat[1::11], flat[2::13], flat[3::17] = 0.0, -0.0, np.inf, -np.inf
        flat[4::19] = np.nan
    return s


@pytest.mark.parametrize("kind", ["close", "wide", "ties"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 1024, 1025, 4096, 4097, 12288, 12289, 32768, 32769])
def test_one_vector(torch_zr, kind, n):
    torch, zr = torch_zr
    from oracle import oracle
    rng = np.random.default_rng(n)
    s = scores(kind, rng, n)
    t = torch.from_numpy(s).cuda()
    for ratio in (0.0, 0.25, 0.9):
        if oracle.keep_count(n, ratio) < 1:
            continue
        S, P = oracle.resize_select(s, ratio)
        keep, drop = zr.resize_select(t, ratio)
        assert np.array_equal(keep.cpu().numpy(), S) and np.array_equal(drop.cpu().numpy(), P), (kind, n, ratio)
        ks, ds = zr.resize_select_multi([t, t[: max(1, n // 2)]], [ratio, 0.0])
        assert np.array_equal(ks[0].cpu().numpy(), S) and np.array_equal(ds[0].cpu().numpy(), P)
        assert ks[1].numel() == max(1, n // 2)


@pytest.mark.parametrize("kind", ["close", "wide", "ties"])
@pytest.mark.parametrize("batch,n", [(511, 300), (512, 300), (512, 1024), (513, 1025), (512, 4097), (512, 12289)])
def test_many_vectors(torch_zr, kind, batch, n):
    torch, zr = torch_zr
    from oracle import oracle
    s = scores(kind, np.random.default_rng(n), batch, n)
    keep, drop = zr.resize_select(torch.from_numpy(s).cuda(), 0.3)
    keep, drop = keep.cpu().numpy(), drop.cpu().numpy()
    for b in (0, 1, batch // 2, batch - 1):
        S, P = oracle.resize_select(s[b], 0.3)
        assert np.array_equal(keep[b], S) and np.array_equal(drop[b], P), (kind, b)

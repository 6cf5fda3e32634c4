"""The pass that fills a volume's sorted arrays (gather or range copy, data
range, statistics, level codes) and the range check of a data change, at the
edges of steps and tiles, on aligned and unaligned inputs of every storage
type, against numpy."""
import numpy as np
import pytest
import torch

from gpu_cases import dvl, random_amr, subset

pytestmark = pytest.mark.gpu

DTYPES = [torch.float32, torch.float16, torch.bfloat16]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()


def _values(n, dtype, seed):
    g = np.random.default_rng(seed)
    v = torch.from_numpy((g.standard_normal(n) * 10.0 ** g.integers(-3, 3, n)).astype(np.float32)).to(dtype)
    v[0] = -0.0
    return v


def _offset(v, k):
    """The same values in device memory k elements past an allocation's start."""
    buf = torch.zeros(v.numel() + k, dtype=v.dtype, device="cuda")
    buf[k:] = v.to("cuda")
    return buf[k:]


def _check(V, fields):
    _, perm = V.export_order()
    p = perm.cpu().numpy().view(np.uint32).astype(np.int64)
    level, got = V.export_sorted()
    D = dvl()
    bins = D.Bins(1, len(fields))
    for m, f in enumerate(fields):
        want = f[torch.from_numpy(p)]
        assert torch.equal(got[m].cpu().view(torch.int32 if f.dtype == torch.float32 else torch.int16),
                           want.view(torch.int32 if f.dtype == torch.float32 else torch.int16)), m
        lo, hi = V.field_range(m)
        x = f.float().numpy()
        assert (lo, hi) == (x.min(), x.max()), (m, lo, hi)
        V.set_tf(m, np.linspace(0.0, 1.0, 16, dtype=np.float32), -1e4, 1e4)   # a constant field's own range is no window
    V.update(bins)
    r = V.read_bins(bins)
    for m, f in enumerate(fields):
        x = f.double().numpy()
        # four-value fp32 sums (3 roundings each), exact to fp64 rounding after, one rounding of the mean
        tol = 4 * 2.0 ** -24 * np.abs(x).mean() + 2.0 ** -24 * abs(x.mean())
        assert abs(r["mean"][m, 0] - x.mean()) <= tol, (m, r["mean"][m, 0], x.mean())
        assert r["vmin"][m, 0] == x.min() and r["vmax"][m, 0] == x.max()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n,tile_steps", [(1, 8), (5, 16), (255, 32), (257, 8), (2048, 8), (4095, 16), (4097, 16),
                                          (8193, 32), (70001, 16)])
def test_build_set_field_and_zoom(n, tile_steps, dtype):
    D = dvl()
    vol = subset(random_amr(71, 24, 3, 0.5, n_fields=1), n, seed=n)
    assert vol.n == n
    f0 = [_values(n, dtype, n + 7 * m) for m in range(3)]
    dev = vol.to("cuda")
    V = D.build_order(dev.x, dev.y, dev.z, dev.level, [_offset(f, m) for m, f in enumerate(f0)], tile_steps=tile_steps)
    try:
        _check(V, f0)
        f1 = [_values(n, dtype, 1000 + n + m) for m in range(3)]
        for m in range(3):
            V.set_field(m, _offset(f1[m], m))
        _check(V, f1)
        bad = f0[0].clone()
        bad[n - 1] = float("nan")
        with pytest.raises(D.DvlError) as e:
            V.set_field(0, _offset(bad, n & 1))
        assert e.value.status == D.E_RANGE
        _check(V, f1)
        level, fields = V.export_sorted()
        a, b = n // 3, n - 1
        Z = V.zoom(a, b, tile_steps=tile_steps)
        try:
            zl, zf = Z.export_sorted()
            assert torch.equal(zl, level[a:b + 1])
            for m in range(3):
                assert torch.equal(zf[m], fields[m][a:b + 1])
            _check(Z, [f[a:b + 1].cpu() for f in fields])
            # the level codes: mixed segments counted from the levels themselves
            pad = (-(b + 1 - a)) % (256 * tile_steps)
            seg = torch.cat([zl.cpu(), torch.zeros(pad, dtype=torch.uint8)]).view(-1, 64)
            assert Z.level_segments() == (seg.shape[0], int((seg != seg[:, :1]).any(1).sum()))
        finally:
            Z.close()
    finally:
        V.close()


def test_nan_in_any_array_is_refused_at_build():
    D = dvl()
    n = 5000
    vol = subset(random_amr(72, 24, 3, 0.5, n_fields=1), n, seed=1).to("cuda")
    for dtype in DTYPES:
        for pos in (0, 4095, n - 1):
            f = [_values(n, dtype, m).to("cuda") for m in range(2)]
            f[1][pos] = float("nan")
            with pytest.raises(D.DvlError) as e:
                D.build_order(vol.x, vol.y, vol.z, vol.level, f)
            assert e.value.status == D.E_RANGE, (dtype, pos)

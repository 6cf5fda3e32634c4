"""Batches of more units of the importance pass than workgroups fit the chip:
a workgroup takes a chain of units, whose last one may belong to the next
request, be a ragged tile or a run of fewer tiles.  Every request equals its
update alone bit for bit."""
import gc

import numpy as np
import pytest
import torch

from gpu_cases import dvl, random_amr, subset, tfs

pytestmark = pytest.mark.gpu

KEYS = ("first", "last", "mean", "vmin", "vmax", "y", "f_total", "vmax_used")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()
    yield
    gc.collect()    # nothing of these cases is freed while a later test counts device memory


@pytest.mark.parametrize("entry_cache", [1, 2])
@pytest.mark.parametrize("n_requests", [36, 70])
def test_chains_of_units(n_requests, entry_cache):
    """Volumes whose tiles are shared by four waves (16 steps), runs of one
    tile (8 steps) and runs of several tiles (few runs asked for)."""
    D = dvl()
    base = random_amr(7, 40, 2, 0.3, n_fields=3)
    opts = [dict(), dict(), dict(tile_steps=8), dict(tile_steps=8, run_waves=64)]
    sizes = [45 * 4096, 44 * 4096 + 1000, 80 * 2048 + 700, 90 * 2048]
    Vs = []
    for n, o in zip(sizes, opts):
        d = subset(base, n, seed=n).to("cuda")
        Vs.append(D.build_order(d.x, d.y, d.z, d.level, d.fields, entry_cache=entry_cache, **o))
    ex = D.Executor()
    try:
        kinds = [dict(), dict(exponent=2.0), dict(), dict(scan_mode=1), dict(vmax_mode=2), dict(clamp_mode=1)]
        reqs, kws = [], []
        for i in range(n_requests):
            kw = kinds[i % len(kinds)]
            W = (1, 7, 64, 333)[i % 4]
            reqs.append(D.Request(Vs[(i * 5) // n_requests % 4], tfs(300 + i % 5, 3), D.Bins(W, 3), **kw))
            kws.append(kw)
        ex.update_batch(reqs)
        got = [r.vol.read_bins(r.bins) for r in reqs]
        for i, r in enumerate(reqs):
            for m in range(3):
                r.vol.set_tf(m, r.alpha[m])
            b = D.Bins(r.bins.n_bins, 3)
            r.vol.update(b, **kws[i])
            ref = r.vol.read_bins(b)
            for k in KEYS:
                assert np.asarray(got[i][k]).tobytes() == np.asarray(ref[k]).tobytes(), (i, k)
    finally:
        ex.close()
        for V in Vs:
            V.close()


@pytest.mark.parametrize("kw", [dict(), dict(vmax_mode=2), dict(scan_mode=1), dict(exponent=2.0)])
def test_cells_read_as_streams(kw):
    """280 MB of cells alone are read past the caches, two requests on them in
    one batch are not: the same bits either way, with few and with many bins."""
    D = dvl()
    s = 260
    g = torch.Generator(device="cuda").manual_seed(5)
    i = torch.arange(s ** 3, device="cuda")
    fields = [torch.rand(s ** 3, device="cuda", generator=g) for _ in range(4)]
    V = D.build_order((i % s).int(), ((i // s) % s).int(), (i // (s * s)).int(),
                      torch.zeros(s ** 3, dtype=torch.uint8, device="cuda"), fields, entry_cache=2)
    ex = D.Executor()
    try:
        A = tfs(77, 4)
        for W in (16, 1920):
            reqs = [D.Request(V, A, D.Bins(W, 4), **kw) for _ in range(2)]
            ex.update_batch(reqs)
            for m in range(4):
                V.set_tf(m, A[m])
            b = D.Bins(W, 4)
            V.update(b, **kw)
            alone = V.read_bins(b)
            for r in reqs:
                got = V.read_bins(r.bins)
                for k in KEYS:
                    assert np.asarray(got[k]).tobytes() == np.asarray(alone[k]).tobytes(), (W, k)
    finally:
        ex.close()
        V.close()

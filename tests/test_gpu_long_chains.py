"""Chains of more units than one stream of the importance pass takes (16): so
many units that every workgroup gets at least 17 of them, however many of up to
8 workgroups a compute unit holds (256 units).  Tiles shared by four waves and
runs of tiles, ragged last tiles, small volumes whose whole requests lie inside
one chain, from values and from entries, with and without the exact maximum.
Every request equals its update alone bit for bit."""
import gc

import numpy as np
import pytest
import torch

from gpu_cases import dvl, tfs

pytestmark = pytest.mark.gpu

KEYS = ("first", "last", "mean", "vmin", "vmax", "y", "f_total", "vmax_used")
RESIDENT = 8 * 256


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()
    yield
    gc.collect()    # nothing of these cases is freed while a later test counts device memory


def grid(n, **opt):
    i = torch.arange(n, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(n)
    level = torch.zeros(n, dtype=torch.uint8, device="cuda")
    return dvl().build_order((i % 256).int(), (i // 256 % 256).int(), (i // 65536).int(), level,
                             [torch.rand(n, device="cuda", generator=g).half() for _ in range(2)], **opt)


@pytest.mark.parametrize("entry_cache", [1, 2])
@pytest.mark.parametrize("big, opt, n_big", [
    (2046 * 4096 + 1000, dict(), 20),                   # 2047 units each, a ragged tile at the end
    (6999 * 2048 + 300, dict(tile_steps=8), 21),        # 1750 units of four one-tile runs each, ragged
])
def test_chains_past_one_stream(big, opt, n_big, entry_cache):
    D = dvl()
    # 1 to 37 tiles, shared by waves or not; ragged and whole (below the size from which requests on one volume share reads)
    small = [grid(n, entry_cache=entry_cache, **o) for n, o in ((3 * 4096 + 5, dict()), (4096, dict()), (37 * 2048 + 1, dict(tile_steps=8)),
                                                               (700, dict()), (16 * 4096, dict()))]
    V = grid(big, entry_cache=entry_cache, **opt)
    ex = D.Executor()
    try:
        units = n_big * (2047 if not opt else 1750)
        assert units > 16 * RESIDENT and 4 * big < 64e6     # requests on one volume do not share its reads
        kinds = [dict(), dict(exponent=2.0), dict(), dict(vmax_mode=2), dict(scan_mode=1), dict(clamp_mode=1)]
        if not opt:
            kinds[4] = dict()                           # another arithmetic shares no tile
        reqs, kws = [], []
        # requests are grouped by volume: some small ones before, between and after the large one's
        order = [small[0]] * 9 + [small[1]] * 5 + [V] * n_big + [small[2]] * 7 + [small[3]] * 6 + [small[4]] * 5
        for i, v in enumerate(order):
            kws.append(kinds[i % len(kinds)])
            reqs.append(D.Request(v, tfs(600 + i % 7, 2), D.Bins((40, 1, 333)[i % 3], 2), **kws[-1]))
        ex.update_batch(reqs)
        got = [r.vol.read_bins(r.bins) for r in reqs]
        print(f"[chains] {len(reqs)} requests, {big} cells, entries {entry_cache == 1}", flush=True)
        for i, r in enumerate(reqs):
            for m in range(2):
                r.vol.set_tf(m, r.alpha[m])
            b = D.Bins(r.bins.n_bins, 2)
            r.vol.update(b, **kws[i])
            ref = r.vol.read_bins(b)
            for key in KEYS:
                assert np.asarray(got[i][key]).tobytes() == np.asarray(ref[key]).tobytes(), (i, key)
    finally:
        ex.close()
        V.close()
        for v in small:
            v.close()

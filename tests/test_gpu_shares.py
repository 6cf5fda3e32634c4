"""Requests that read the values of one volume in one launch of the importance
pass (volumes from 64 MB of values on, up to 8 requests a launch): every request
equals its update alone bit for bit, whatever the layout, the scan arithmetic
and the size of its tables."""
import gc

import numpy as np
import pytest
import torch

from gpu_cases import dvl, tfs

pytestmark = pytest.mark.gpu

KEYS = ("first", "last", "mean", "vmin", "vmax", "y", "f_total", "vmax_used")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()
    yield
    gc.collect()    # nothing of these cases is freed while a later test counts device memory


def two_level(n, M, dtype, **opt):
    """n cells: seven eighths on a fine grid, the rest coarse above it."""
    s, nf = 256, n * 7 // 8
    i, j = torch.arange(nf, device="cuda"), torch.arange(n - nf, device="cuda")
    top = (nf + s * s - 1) // (s * s)
    top += top & 1
    x = torch.cat([i % s, 2 * (j % (s // 2))]).int()
    y = torch.cat([i // s % s, 2 * (j // (s // 2) % (s // 2))]).int()
    z = torch.cat([i // (s * s), 2 * (j // (s // 2) ** 2) + top]).int()
    level = torch.cat([torch.zeros_like(i), torch.ones_like(j)]).to(torch.uint8)
    g = torch.Generator(device="cuda").manual_seed(n)
    fields = [(torch.sin(0.02 * (m + 1) * x + 0.03 * y) + torch.cos(0.04 * z * (m + 2))
               + 0.1 * torch.rand(n, device="cuda", generator=g)).to(dtype) for m in range(M)]
    return dvl().build_order(x, y, z, level, fields, entry_cache=2, **opt)


@pytest.mark.parametrize("n, M, dtype, n_tf, opt", [
    (2047 * 4096 + 1000, 4, torch.float32, 256, dict()),                 # tiles shared by four waves, ragged end
    (2100 * 4096, 4, torch.float32, 64, dict()),                         # a wave per tile, whole
    (3000 * 4096 + 17, 6, torch.float16, 4, dict(run_waves=64)),         # few units: runs of 47 tiles
    (6000 * 2048 + 5, 3, torch.bfloat16, 1024, dict(tile_steps=8)),      # short tiles, tables of 12 KB
    (1200 * 8192 + 300, 4, torch.float32, 4096, dict(tile_steps=32)),    # tables that leave two workgroups a unit
    (1100 * 4096 + 4095, 9, torch.float32, 256, dict()),                 # more fields than the fixed counts
])
def test_shares_equal_single_updates(n, M, dtype, n_tf, opt):
    D = dvl()
    V = two_level(n, M, dtype, **opt)
    other = two_level(50_000, M, dtype)
    ex = D.Executor()
    kinds = [dict(), dict(exponent=2.0), dict(scan_mode=1), dict(vmax_mode=2), dict(), dict(scan_mode=2), dict(clamp_mode=1),
             dict(), dict(), dict(min_importance=0.0), dict(level_scale=3)]
    try:
        for k in (2, 5, 11):
            reqs, kws = [], []
            for i in range(k):
                W = (64, 1000, 7)[i % 3]
                kws.append(kinds[(i + k) % len(kinds)])
                reqs.append(D.Request(V, tfs(500 + i, M, n_tf), D.Bins(W, M), **kws[-1]))
            reqs.insert(1, D.Request(other, tfs(9, M, n_tf), D.Bins(33, M)))
            kws.insert(1, dict())
            ex.update_batch(reqs)
            got = [r.vol.read_bins(r.bins) for r in reqs]
            print(f"[share] n={n} M={M} {dtype} n_tf={n_tf} {opt} x{k}", flush=True)
            for i, r in enumerate(reqs):
                for m in range(M):
                    r.vol.set_tf(m, r.alpha[m])
                b = D.Bins(r.bins.n_bins, M)
                r.vol.update(b, **kws[i])
                ref = r.vol.read_bins(b)
                for key in KEYS:
                    assert np.asarray(got[i][key]).tobytes() == np.asarray(ref[key]).tobytes(), (k, i, key)
    finally:
        ex.close()
        V.close()
        other.close()


def test_captured_shares():
    """A captured batch whose requests share reads, replayed with new tables."""
    D = dvl()
    V = two_level(4_500_000, 4, torch.float32)
    reqs = [D.Request(V, tfs(i, 4), D.Bins(500, 4)) for i in range(3)]
    G = D.Graph(reqs)
    try:
        for rnd in range(4):
            A = [tfs(40 + 3 * rnd + i, 4) for i in range(3)]
            G.set_tf_all(A)
            G.launch()
            torch.cuda.synchronize()
            got = [V.read_bins(r.bins) for r in reqs]
            for i in range(3):
                for m in range(4):
                    V.set_tf(m, A[i][m])
                b = D.Bins(500, 4)
                V.update(b)
                ref = V.read_bins(b)
                for key in KEYS:
                    assert np.asarray(got[i][key]).tobytes() == np.asarray(ref[key]).tobytes(), (rnd, i, key)
    finally:
        G.close()
        V.close()


def test_cached_and_uncached_requests_of_one_volume():
    """Nine requests, the last with windows of its own: eight read the cached
    entries, the ninth the values; then the other way round on one volume more."""
    D = dvl()
    Vs = [two_level(300_000, 4, torch.float32), two_level(5_000_000, 4, torch.float32)]
    ex = D.Executor()
    try:
        for V in Vs:
            V.set_entry_cache(D.ENTRY_CACHE_ALWAYS)
        win = [tuple(np.array(w, np.float32) for w in zip(*[V.field_range(m) for m in range(4)])) for V in Vs]
        for n_a in (8, 1):
            reqs = []
            for V, (lo, hi) in zip(Vs, win):
                for i in range(9):
                    up = hi if i < n_a else lo + (hi - lo) / 2
                    reqs.append(D.Request(V, tfs(70 + i, 4), D.Bins(200 + i, 4), lo=lo, hi=up))
            ex.update_batch(reqs)
            got = [r.vol.read_bins(r.bins) for r in reqs]
            if n_a == 8:
                assert all(np.array_equal(V.entry_cache_info()[1], hi) for V, (_, hi) in zip(Vs, win))
            for V in Vs:
                V.set_entry_cache(D.ENTRY_CACHE_NEVER)
            for i, r in enumerate(reqs):
                for m in range(4):
                    r.vol.set_tf(m, r.alpha[m], float(r.lo[m]), float(r.hi[m]))
                b = D.Bins(r.bins.n_bins, 4)
                r.vol.update(b)
                ref = r.vol.read_bins(b)
                for key in KEYS:
                    assert np.asarray(got[i][key]).tobytes() == np.asarray(ref[key]).tobytes(), (n_a, i, key)
            for V in Vs:
                V.set_entry_cache(D.ENTRY_CACHE_ALWAYS)
    finally:
        ex.close()
        for V in Vs:
            V.close()

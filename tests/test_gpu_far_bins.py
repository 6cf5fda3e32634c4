"""Plots far wider than the volume has cells: a cell, and a tile, reach hundreds
to a million bins.  Against the oracle, with cells of very different widths (so
that narrow and wide ones meet in one step, one lane and one tile) and ends of
tiles and volumes in between."""
import numpy as np
import pytest
import torch

from gpu_cases import random_amr, run_case, subset, tfs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n, W", [(1, 1), (1, 65), (1, 1 << 20), (2, 66), (3, 300_000), (70, 4097), (255, 70_000), (257, 20_000),
                                  (4097, 1 << 18), (5000, 100_003), (5000, 4000)])
@pytest.mark.parametrize("kw", [dict(), dict(exponent=3.0, fmin=0.0, level_scale=3)])
def test_cells_of_many_bins(n, W, kw):
    vol = subset(random_amr(5, 8, 4, 0.45, n_fields=2), n, seed=W)
    # positions are fp32 pixels: an edge may move by a rounding of the plot's width
    run_case(vol, tfs(W, 2), W, label="far bins", edge_tol=1e-6, **kw)


@pytest.mark.parametrize("opt", [dict(tile_steps=8), dict(tile_steps=8, run_waves=64)])
def test_wide_tiles_among_narrow_ones(opt):
    """More tiles than bins, and one stretch of cells that takes most of the
    plot: its tiles reach many bins, the others share a few."""
    from gpu_cases import dvl
    D = dvl()
    n = 400 * 2048 + 77
    i = torch.arange(n, device="cuda")
    wide = ((i // 3000) == 60).float()                  # 3000 neighbours in z
    V = D.build_order((i % 128).int(), (i // 128 % 128).int(), (i // 16384).int(), torch.zeros(n, dtype=torch.uint8, device="cuda"),
                      [wide, torch.zeros(n, device="cuda") + (i == 0)], **opt)
    a = np.zeros((2, 16), np.float32)
    a[0, 15] = 1.0
    try:
        for m in range(2):
            V.set_tf(m, a[m], 0.0, 1.0)
        b = D.Bins(300, 2)
        V.update(b, min_importance=1e-5)
        r = V.read_bins(b)
        _, fields = V.export_sorted()
        f = fields[0].double().cpu().numpy()
        imp = np.where(f > 0, 1.0, 1e-5)
        imp = np.maximum(imp.astype(np.float32).astype(np.float64), np.float64(np.float32(1e-5)))
        end = np.cumsum(imp)
        u = np.concatenate([[0.0], end]) / end[-1] * 300
        assert r["first"][0] == 0 and r["last"][-1] == n - 1
        first, last = r["first"].astype(np.int64), r["last"].astype(np.int64)
        d = first[1:] - last[:-1]
        assert ((d == 0) | (d == 1)).all()
        k = np.arange(300)
        assert (u[first] <= k + 1e-6 * 300 + 1e-9).all() and (u[last + 1] >= k + 1 - 1e-6 * 300).all()
        assert (u[first + 1] >= k - 1e-6 * 300).all() and (u[last] <= k + 1 + 1e-6 * 300).all()
    finally:
        V.close()

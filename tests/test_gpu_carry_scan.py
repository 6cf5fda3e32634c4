"""The carry scan inside the classification: every workgroup of 1024 tiles scans
all run totals itself and keeps the bases of its own runs.  Against the oracle
with tiles up to, at and past a workgroup's edge, runs of one tile and runs that
straddle the edge, more runs than one round of the scan (8192), and all scan
arithmetics; bins must meet across the edges."""
import numpy as np
import pytest
import torch

import oracle
from gpu_cases import dvl, tfs
from parity import reconcile

pytestmark = pytest.mark.gpu

M = 2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()


def check(n, n_runs, cases, **opt):
    D = dvl()
    i = torch.arange(n, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(n)
    level = ((i // 5000) % 3 == 1).to(torch.uint8)      # the widths vary along the order
    V = D.build_order((2 * (i % 256)).int(), (2 * (i // 256 % 256)).int(), (2 * (i // 65536)).int(), level,
                      [torch.rand(n, device="cuda", generator=g) ** 3, torch.rand(n, device="cuda", generator=g)], tile_steps=8, **opt)
    try:
        lev, F = V.export_sorted()
        lev, F = lev.cpu().numpy(), np.stack([f.cpu().numpy() for f in F])
        lo, hi = oracle.default_windows(F)
        A = tfs(n % 1000, M)
        for W in (700, 3000):
            ob = oracle.update(lev, F, A, lo, hi, W, keep_cells=True)
            for mode in cases:
                for m in range(M):
                    V.set_tf(m, A[m])
                b = D.Bins(W, M)
                V.update(b, scan_mode=mode)
                r = V.read_bins(b)
                # plain fp32: a rounding per run, per tile of a run and per partial sum
                tol = 1e-6 if mode != D.SCAN_NAIVE_FP32 else (n_runs + n / 2048 / n_runs + 64) * 2.0 ** -24 + 1e-6
                rep = reconcile(r, ob, F, A, lo, hi, W, edge_tol=tol)
                assert abs(r["f_total"] - ob.f_total) <= max(1e-5, tol) * ob.f_total
                print(f"[scan] n={n} {opt} W={W} mode {mode}: edges moved {rep.edges_moved}", flush=True)
    finally:
        V.close()


@pytest.mark.parametrize("tiles", [1023, 1024, 1025, 2048, 2049])
def test_one_tile_runs(tiles):
    check(tiles * 2048 - 3, tiles, (0, 1, 2))


@pytest.mark.parametrize("tiles, run_waves", [(1025, 64), (2049, 100), (1024, 64), (3000, 64)])
def test_runs_across_the_edge_of_a_workgroup(tiles, run_waves):
    per = -(-tiles // run_waves)
    check(tiles * 2048 - 700, -(-tiles // per), (0, 1, 2), run_waves=run_waves)


def test_more_runs_than_a_round():
    check(8300 * 2048 + 1, 8301, (0, 1), run_waves=65536)

"""Bins of thousands of tiles: the statistics of a range that needs many rounds
of tile statistics, for every class of field counts and storage, against numpy
over the bins' own cell ranges."""
import numpy as np
import pytest
import torch

from gpu_cases import dvl, tfs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()


@pytest.mark.parametrize("W", [1, 3])
@pytest.mark.parametrize("M, dtype, tiles", [(1, torch.float32, 300), (2, torch.float32, 1030), (3, torch.bfloat16, 65), (8, torch.float32, 65),
                                             (8, torch.float32, 1025), (9, torch.float16, 33), (16, torch.float32, 260)])
def test_ranges_of_many_tiles(M, dtype, tiles, W):
    D = dvl()
    n = tiles * 2048 + 131
    i = torch.arange(n, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(M * tiles)
    fields = [(torch.randn(n, device="cuda", generator=g) * (m + 1)).to(dtype) for m in range(M)]
    V = D.build_order((i % 128).int(), (i // 128 % 128).int(), (i // 16384).int(), torch.zeros(n, dtype=torch.uint8, device="cuda"),
                      fields, tile_steps=8)
    try:
        A = tfs(M, M)
        for m in range(M):
            V.set_tf(m, A[m])
        b = D.Bins(W, M)
        V.update(b)
        r = V.read_bins(b)
        _, F = V.export_sorted()
        F = np.stack([f.float().cpu().numpy() for f in F]).astype(np.float64)
        assert r["first"][0] == 0 and r["last"][-1] == n - 1
        for k in range(W):
            c = F[:, int(r["first"][k]):int(r["last"][k]) + 1]
            assert np.array_equal(r["vmin"][:, k], c.min(axis=1).astype(np.float32))
            assert np.array_equal(r["vmax"][:, k], c.max(axis=1).astype(np.float32))
            # fp32 sums of four values inside the tile statistics, fp64 beyond them
            bound = 4 * 2.0 ** -24 * np.abs(c).mean(axis=1) + 2.0 ** -23 * np.abs(c.mean(axis=1))
            assert (np.abs(r["mean"][:, k] - c.mean(axis=1)) <= bound).all()
    finally:
        V.close()

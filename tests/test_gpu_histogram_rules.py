"""Per-bin histograms against the oracle on both sides of every rule that chooses
their kernel: cells a bin below and above 64, 256 and four times the buckets,
one and 512 buckets, and bins at any offset from a vector of four."""
import numpy as np
import pytest
import torch

import oracle
from gpu_cases import dvl, tfs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("n, W, H", [(1, 700, 3), (63_999, 1000, 1), (64_000, 1000, 1), (76_799, 300, 64), (76_800, 300, 64),
                                     (255_999, 1000, 300), (256_000, 1000, 300), (20_479, 10, 512), (20_480, 10, 512),
                                     (26_001, 50, 4096), (5, 1 << 16, 8)])
def test_histograms(n, W, H, dtype):
    D = dvl()
    i = torch.arange(n, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(n)
    vals = (torch.rand(n, device="cuda", generator=g) * 1.4 - 0.2).to(dtype)
    V = D.build_order((i % 64).int(), (i // 64 % 64).int(), (i // 4096).int(), torch.zeros(n, dtype=torch.uint8, device="cuda"),
                      [vals, torch.rand(n, device="cuda", generator=g).to(dtype)])
    try:
        A = tfs(n % 97, 2)
        for m in range(2):
            V.set_tf(m, A[m], 0.0, 1.0)
        b = D.Bins(W, 2)
        V.update(b)
        r = V.read_bins(b)
        got = V.bin_histograms(b, 0, H, 0.0, 1.0).cpu().numpy().view(np.uint32)
        _, fields = V.export_sorted()
        want = oracle.bin_histograms(fields[0].float().cpu().numpy(), r["first"], r["last"], H, 0.0, 1.0)
        assert np.array_equal(got, want), (n, W, H)
        assert np.array_equal(got.sum(axis=1), r["count"])
    finally:
        V.close()

"""The brushing mask against numpy where its chunks, launches and range tests
can go wrong: sizes around a chunk (256 and 2048 cells) and the sizes at which
the launch changes, one to 128 ranges, adjacent, nested, empty of cells, ending
at chunk edges, and masks at odd addresses."""
import numpy as np
import pytest
import torch

from gpu_cases import dvl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()


def select(V, ranges, offset):
    """dvl_select_mask into a guarded buffer, `offset` bytes off its alignment."""
    D = dvl()
    r = np.ascontiguousarray(np.array(ranges, np.uint64))
    buf = torch.full((V.n + 64,), 7, dtype=torch.uint8, device="cuda")
    at = buf.data_ptr() + 32 + offset
    assert D.lib().dvl_select_mask(V.handle, r.ctypes.data, len(r), at, None) == 0
    out = buf.cpu().numpy()
    assert (out[:32 + offset] == 7).all() and (out[32 + offset + V.n:] == 7).all()
    return out[32 + offset:32 + offset + V.n]


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 2049, 65535, 65536, 65537, 200_003, 4_000_000, 4_000_001, 4_100_000])
def test_masks(n):
    D = dvl()
    i = torch.arange(n, device="cuda")
    p = torch.randperm(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n))
    i = i[p]
    V = D.build_order((i % 256).int(), (i // 256 % 256).int(), (i // 65536).int(), torch.zeros(n, dtype=torch.uint8, device="cuda"),
                      [torch.rand(n, device="cuda")])
    try:
        keys, _ = V.export_order()
        k = keys.cpu().numpy().view(np.uint64)
        s = np.sort(k)
        rng = np.random.default_rng(n)
        at = lambda j: int(s[min(max(j, 0), n - 1)])
        cuts = [at(int(c)) for c in np.linspace(0, n - 1, 129)]
        cases = [
            [(at(0), at(n))],
            [(at(n // 3), at(n // 2))],
            [(at(0), at(2047)), (at(2048), at(4095)), (at(255), at(256))],
            [(at(n // 4), at(n // 4))],
            [(1 << 62, (1 << 62) + 5)],
            [(at(n // 5), at(n // 2)), (at(n // 4), at(n // 3)), (at(n // 5), at(n // 2))],
            [(cuts[j], max(cuts[j], cuts[j + 1] - 1)) for j in range(128)],
            [tuple(sorted(int(x) for x in rng.integers(0, int(s[-1]) + 2, 2))) for _ in range(65)],
            [(at(int(j)), at(int(j) + 3)) for j in rng.integers(0, n, 64)],
        ]
        for c, ranges in enumerate(cases):
            want = np.zeros(n, bool)
            for lo, hi in ranges:
                want |= (k >= np.uint64(lo)) & (k <= np.uint64(hi))
            got = select(V, ranges, c % 16)
            assert np.array_equal(got, want.astype(np.uint8)), (n, c, int((got != want).sum()))
    finally:
        V.close()

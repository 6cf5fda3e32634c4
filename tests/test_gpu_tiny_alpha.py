"""Tables whose variation is so small that V / max V is subnormal (minimum
importance 0): f rounds there, so the level scale must be applied after that
rounding in every kernel.  The same bits from values with stored f, from values
without, and from cached entries."""
import numpy as np
import pytest
import torch

from gpu_cases import dvl

pytestmark = pytest.mark.gpu

KEYS = ("first", "last", "mean", "vmin", "vmax", "y", "f_total", "vmax_used")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()


@pytest.mark.parametrize("exponent2", [-142, -130, -60])
def test_subnormal_importance_is_the_same_on_every_path(exponent2):
    D = dvl()
    s, n = 64, 64 ** 3                                  # 64 whole tiles of level 3
    i = torch.arange(n, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    f0 = torch.rand(n, device="cuda", generator=g) * 0.9 + 0.1
    f0[0] = 0.0                                         # entries 0 and 25 .. 255
    f1 = torch.rand(n, device="cuda", generator=g)
    V = D.build_order((8 * (i % s)).int(), (8 * (i // s % s)).int(), (8 * (i // (s * s))).int(),
                      torch.full((n,), 3, dtype=torch.uint8, device="cuda"), [f0, f1])
    a = np.zeros((2, 256), np.float32)
    a[0, 5] = 0.7                                       # max V of Eq. 6, taken by no cell
    a[1] = np.ldexp(np.arange(1, 257, dtype=np.float32), exponent2)
    W, kw = 1024, dict(min_importance=0.0, level_scale=3)
    try:
        for m in range(2):
            V.set_tf(m, a[m], 0.0, 1.0)
        out = [D.Bins(W, 2) for _ in range(3)]
        V.update(out[0], **kw)                          # values, f stored for the projection
        D.update_noalloc(V, D.params(W, **kw), out[1])  # values, nothing stored
        V.update(out[2], **kw)                          # the second use of the windows: entries
        assert V.entry_cache_info() is not None
        got = [V.read_bins(b) for b in out]
        # F_tot by the definition: r = V * (1 / max V) rounded to fp32, then 8^L
        e1 = np.minimum((f1.cpu().numpy() * np.float32(256)).astype(int), 255)
        e0 = np.minimum((f0.cpu().numpy() * np.float32(256)).astype(int), 255)
        v = np.abs(a[1][e1] - a[0][e0])
        r = v * (np.float32(1) / np.float32(0.7))
        total = np.ldexp(r.astype(np.float64), 9).sum()
        assert got[0]["vmax_used"] == np.float32(0.7)
        assert abs(got[0]["f_total"] - total) <= 1e-6 * total
        for k in KEYS:
            for o in got[1:]:
                assert np.asarray(o[k]).tobytes() == np.asarray(got[0][k]).tobytes(), k
    finally:
        V.close()

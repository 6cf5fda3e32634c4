"""Edges of the brushing mask and the bin histograms: sizes around the mask's
chunks of 2048 cells and 16-byte lines, mask pointers of every alignment, and
histograms on both sides of the rule for the copies of the counters.  Both
results are whole numbers: they equal the oracle's."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from gpu_cases import dvl, random_amr, subset, tfs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _volume(n, dtype):
    D = dvl()
    vol = subset(random_amr(77 + n, 28, 1), n, n)
    assert vol.n == n
    d = vol.to("cuda")
    V = D.build_order(d.x, d.y, d.z, d.level, [f.to(dtype) for f in d.fields])
    o = oracle.build_order(vol.x.numpy(), vol.y.numpy(), vol.z.numpy(), vol.level.numpy())
    F = np.stack([f.to(dtype).float().numpy()[o.perm] for f in vol.fields]).astype(np.float32)
    return D, V, o, F


@pytest.mark.parametrize("n,shift", [(1, 1), (15, 3), (2047, 15), (2048, 0), (2049, 8), (6157, 5)])
def test_mask_of_any_alignment(n, shift):
    D, V, o, _ = _volume(n, torch.float32)
    try:
        ks = np.sort(o.keys)
        at = lambda q: int(ks[int(q * (n - 1))])
        for ranges in ([(at(0), at(1))], [(at(0.3), at(0.7))], [(at(0.1), at(0.2)), (at(0.2), at(0.9))],
                       [(int(ks[-1]) + 1, int(ks[-1]) + 9)]):
            buf = torch.full((n + 64,), 7, dtype=torch.uint8, device="cuda")
            r = np.asarray(ranges, dtype=np.uint64).reshape(-1, 2)
            st = D.lib().dvl_select_mask(V.handle, r.ctypes.data_as(C.c_void_p), r.shape[0],
                                         C.c_void_p(buf.data_ptr() + shift), C.c_void_p(0))
            assert st == 0
            torch.cuda.synchronize()
            got = buf.cpu().numpy()
            want = np.full(n + 64, 7, np.uint8)
            want[shift:shift + n] = np.any([(o.keys >= lo) & (o.keys <= hi) for lo, hi in ranges], axis=0)
            assert np.array_equal(got, want), ranges
    finally:
        V.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,W,H", [(7, 3, 1), (1280, 1, 512), (1279, 1, 512), (5003, 1, 513), (9001, 9, 400), (9001, 9, 401),
                                   (9001, 4096, 3), (20011, 2, 4096)])
def test_histograms_around_the_rule(n, W, H, dtype):
    D, V, o, F = _volume(n, dtype)
    try:
        lo, hi = oracle.default_windows(F)
        A = tfs(3, V.m)
        for m in range(V.m):
            D.set_tf(V, m, A[m], float(lo[m]), float(hi[m]))
        b = D.Bins(W, V.m)
        V.update(b)
        g = V.read_bins(b)
        for m in range(V.m):
            wlo, whi = float(lo[m]), float(hi[m]) * 1.01 + 0.01
            got = V.bin_histograms(b, m, H, wlo, whi).cpu().numpy().view(np.uint32)
            assert np.array_equal(got, oracle.bin_histograms(F[m], g["first"], g["last"], H, wlo, whi))
    finally:
        V.close()

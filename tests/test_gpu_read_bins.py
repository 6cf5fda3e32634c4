"""dvl_read_bins through its staging buffer and past it: every subset of the
outputs the caller may leave out, against the device arrays."""
import ctypes as C

import numpy as np
import pytest
import torch

from gpu_cases import dvl, random_amr, tfs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()


@pytest.mark.parametrize("W", [1, 17, 1920, 18700, 18800, 60000])   # 3 fields: 56 bytes a bin, 1 MB at 18724 bins
def test_read_bins_subsets(W):
    D = dvl()
    dev = random_amr(91, 8, 3, 0.4, n_fields=3).to("cuda")
    V = D.build_order(dev.x, dev.y, dev.z, dev.level, dev.fields)
    try:
        A = tfs(91, 3)
        for m in range(3):
            V.set_tf(m, A[m])
        b = D.Bins(W, 3)
        V.update(b)
        torch.cuda.synchronize()
        want = {"first": b.first_cell, "last": b.last_cell, "mean": b.mean, "vmin": b.vmin, "vmax": b.vmax, "y": b.y,
                "f_total": b.f_total, "vmax_used": b.vmax_used}
        want = {k: t.cpu().numpy() for k, t in want.items()}
        want["first"], want["last"] = want["first"].view(np.uint32), want["last"].view(np.uint32)
        want["count"] = want["last"] - want["first"] + np.uint32(1)
        order = ("count", "first", "last", "mean", "vmin", "vmax", "y", "f_total", "vmax_used")
        st = b.struct()
        for skip in [()] + [(k,) for k in order] + [("first", "last"), ("count", "first", "last", "mean"), order[:7], order]:
            out = {k: None if k in skip else np.full_like(want[k], 7) for k in order}
            P = [None if out[k] is None else out[k].ctypes.data_as(C.c_void_p) for k in order]
            assert D.lib().dvl_read_bins(V.handle, C.byref(st), W, None, *P) == D.OK
            for k in order:
                if out[k] is not None:
                    assert out[k].tobytes() == want[k].tobytes(), (skip, k)
    finally:
        V.close()

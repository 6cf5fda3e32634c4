"""Bins whose edges fall on cell, step and tile boundaries, and cells of zero
width exactly on an edge: the cases where the rescan's rules for which bin
starts and ends with which cell can go wrong, against the oracle."""
import gc

import numpy as np
import pytest
import torch

from gpu_cases import random_amr, run_case, subset, tfs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    gc.collect()    # nothing of these cases is freed while a later test counts device memory


@pytest.mark.parametrize("n", [255, 256, 4096, 4097, 8192, 12288 + 3])
@pytest.mark.parametrize("W", [1, 2, 16, 64, 4096, 12000])
def test_edges_on_cell_boundaries(n, W):
    """f = 1 everywhere (P = 0): with n a multiple of W every edge is a cell
    boundary, with W a multiple of n every cell holds whole bins."""
    vol = subset(random_amr(81, 24, 2, 0.3, n_fields=2), n, seed=n)
    run_case(vol, tfs(81, 2), W, exponent=0.0, label=f"f=1 n={n}")


@pytest.mark.parametrize("n", [300, 4096, 9000, 20001])
@pytest.mark.parametrize("W", [7, 64, 1920])
@pytest.mark.parametrize("entry_cache", [1, 2])
def test_zero_width_cells_on_edges(n, W, entry_cache):
    """Two of three cells have V = 0 and no minimum importance: zero width, in
    runs that reach over step and tile boundaries; the others share one f."""
    vol = subset(random_amr(82, 32, 1, 0.0, n_fields=2), n, seed=n)
    a = torch.from_numpy((np.random.default_rng(n).random(n) < 1.0 / 3.0).astype(np.float32))
    vol.fields[0] = a
    vol.fields[1] = torch.zeros(n)
    vol.fields[1][0] = 1.0
    alpha = np.zeros((2, 256), np.float32)
    alpha[0, 128:] = 1.0
    run_case(vol, alpha, W, fmin=0.0, label=f"zero width n={n}", entry_cache=entry_cache)

"""Every field count with kernels of its own, from values, from cached entries
and with the importance stored or not, against the oracle."""
import gc

import pytest
import torch

from gpu_cases import dvl, random_amr, run_case, subset, tfs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dvl()
    yield
    gc.collect()    # nothing of these cases is freed while a later test counts device memory


@pytest.mark.parametrize("n_fields", [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("dtype,W,exponent,entry_cache", [
    (torch.float32, 1, 1.0, 1), (torch.float32, 700, 1.0, 2), (torch.float32, 33, 2.0, 1),
    (torch.float16, 5, 0.5, 2), (torch.bfloat16, 64, 1.0, 1)])
def test_field_counts(n_fields, dtype, W, exponent, entry_cache):
    """Three whole tiles and a ragged one."""
    vol = subset(random_amr(40 + n_fields, 24, 2, 0.3, n_fields=n_fields), 3 * 4096 + 259, seed=n_fields)
    vol.fields[:] = [f.clamp(max=6e4) for f in vol.fields]      # finite in 16 bits
    run_case(vol, tfs(n_fields, n_fields), W, exponent=exponent, dtype=dtype, label=f"M={n_fields}",
             entry_cache=entry_cache)

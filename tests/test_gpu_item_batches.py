"""Batches on both sides of the line where the per-item kernels take whole cases
per XCD (three quarters of the last turn used): every case against the same case
alone."""
import pytest

import test_gpu_items as items

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Bn", [6, 11, 12, 17, 18, 33])
@pytest.mark.parametrize("n", [2, 301])
def test_cases_match_alone(n, Bn):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    items.test_cases_match_alone(n, Bn)

"""Tiles of 9 to 24 rows of more than 8192 channels with frames beyond the Infinity Cache (workgroups that keep a CU to
themselves) against 64-bit results: tiles of two and three eights of rows."""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_slices as slices
from libutil import ensure_built

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ensure_built()


@pytest.mark.parametrize("T,H,W,C,Q", [(1050, 1, 16, 8200, 3), (300, 2, 11, 20488, 16)])
def test_long_rows(T, H, W, C, Q):
    slices.test_slices(T, H, W, C, Q)

"""The one-wave budgets at five to eight frames per lane, and the first size past them, against the oracle (whole
numbers, exact; inputs within 1e-9 of a tie of the fractional parts are skipped)."""
import pytest

torch = pytest.importorskip("torch")

import libutil
import test_gpu_parity as parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    libutil.ensure_built()


@pytest.mark.parametrize("T", [258, 320, 321, 449, 511, 512, 513])
def test_budgets(T):
    parity.test_stage_temporal_budget_random(T)

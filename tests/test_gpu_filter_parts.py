"""The filter-bank row kernel with one to four workgroups per frame: the split form's rows are the fused form's bit for
bit (the same operator entries against the same tokens in the same order), whatever share of a frame's chunks a
workgroup takes."""
import pytest

torch = pytest.importorskip("torch")

import libutil
from paper_2607_23265_amd import wavezip as wz

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    libutil.ensure_built()


# 4, 3, 2 and 1 workgroups per frame; frames keep from none to several chunks of 16 rows
@pytest.mark.parametrize("T", [5, 70, 100, 140])
def test_split_rows_are_the_fused_rows(T):
    H, W, C, Q = 27, 27, 40, 16
    B = T * 40
    g = torch.Generator().manual_seed(T)
    X = torch.randn(T, H, W, C, generator=g).bfloat16().to(DEV)
    q = (torch.randn(Q, C, generator=g) / C ** 0.5).bfloat16().to(DEV)
    p = wz.Problem(T=T, H=H, W=W, C=C, Q=Q, B=B, in_dtype=wz.WZ_BF16, out_dtype=wz.WZ_F32, spatial_basis=wz.WZ_DB4)
    tok, idx, budget, offset = wz.condense(p, X, q)
    a, _, _ = wz.relevance(p, X, q)
    fused, fidx = wz.spatial_dwt_condense(p, X, a, offset)
    torch.cuda.synchronize()
    n = int(offset[-1])
    assert n == B and torch.equal(idx[:n], fidx[:n])
    assert torch.equal(tok[:n], fused[:n])

"""The fp32 token-tiled pass (fp32 MFMA) at the edges of its tiles, against the fp64 oracle.

Tolerance: fp32 inputs, 1e-5 relative with a floor of a tenth of the largest value (as for every fp32-input case): the
sums run in chains of at most 16 products and C / 128 partial sums per wave, so their rounding stays near 1e-7.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import gpu_util as G
import oracle
from libutil import ensure_built
from paper_2607_23265_amd import synth
from paper_2607_23265_amd import wavezip as wz

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ensure_built()


# (T, H, W, C, Q): tiles of 16 to 64 tokens with one to four 16-row MFMA tiles (300 frames: too many for finer tiles),
# a ragged last tile, one token; channels short of a 32-channel chunk, one past it, more than the channel sums' LDS;
# queries at the edges of 16, 32 and 64 columns and beyond one pass
SHAPES = [(3, 1, 1, 8, 1), (2, 4, 4, 8, 16), (2, 5, 7, 40, 17), (300, 3, 3, 24, 16), (300, 4, 6, 24, 32),
          (300, 5, 8, 72, 33), (260, 8, 8, 24, 64), (260, 7, 7, 32, 65), (3, 13, 13, 264, 64), (2, 9, 9, 136, 130),
          (2, 7, 7, 8200, 20), (2, 3, 3, 65536, 3), (2, 6, 6, 96, 1024)]


@pytest.mark.parametrize("T,H,W,C,Q", SHAPES)
def test_fp32_pass(T, H, W, C, Q):
    rng = np.random.default_rng(T * 1000 + Q)
    X = rng.standard_normal((T, H, W, C)).astype(np.float32)
    q = (rng.standard_normal((Q, C)) / np.sqrt(C)).astype(np.float32)
    inp = synth.Inputs(wl=synth.small("tiny", T=T, H=H, W=W, C=C, Q=Q, B=1), X=X, query=q)
    out = oracle.condense(inp.X_f64(), inp.query_f64(), 1, 1, 1.5, 0.0)
    Xd, qd = wz.to_device(inp, DEV)
    a, r, d = wz.relevance(wz.problem_of(inp.wl), Xd, qd)
    torch.cuda.synchronize()
    assert G.within(a.cpu().numpy(), out["a"].ravel(), G.TOL_F32_IN, "a")
    assert G.within(r.cpu().numpy(), out["r"], G.TOL_F32_IN, "r")
    assert G.within(d.cpu().numpy(), out["delta"], G.TOL_F32_IN, "delta")


@pytest.mark.parametrize("Q,n", [(5, 3), (20, 3), (16, 8)])
def test_fp32_queries_share_a_pass(Q, n):
    """Queries of one video share fp32 passes of up to 64 columns; each gets its single call's outputs bit for bit."""
    T, H, W, C, B = 6, 5, 9, 200, 40
    g = torch.Generator().manual_seed(Q)
    X = torch.randn(T, H, W, C, generator=g).to(DEV)
    q = (torch.randn(n, Q, C, generator=g) / C ** 0.5).to(DEV)
    p = wz.Problem(T=T, H=H, W=W, C=C, Q=Q, B=B, in_dtype=wz.WZ_F32)
    many = wz.condense_queries(p, X, q)
    for i in range(n):
        one = wz.condense(p, X, q[i].contiguous())
        torch.cuda.synchronize()
        for x, y in zip(many, one):
            assert torch.equal(x[i], y)

"""The workgroup-shared pass with one column tile a wave (bf16, 33 to 64 query tokens, frames enough for CUs to take
turns) at the edges of its tiles and of its ring of chunks.

Tolerance: as for the wide queries, exact inputs and fp32 sums in chains of at most 6 MFMA steps: 1e-5 relative with a
floor of a tenth of the largest value.
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


# tiles of up to 64 tokens (three chunks in flight) and of up to 128 (two), ragged last tiles, one token; channels short
# of a chunk, at the ring and past it
SHAPES = [(300, 1, 1, 8, 33), (300, 8, 8, 72, 64), (300, 7, 7, 192, 48), (300, 5, 8, 200, 40), (260, 9, 9, 64, 33),
          (260, 9, 10, 136, 64), (300, 8, 16, 264, 49), (300, 13, 13, 40, 64)]


@pytest.mark.parametrize("T,H,W,C,Q", SHAPES)
def test_shared_tiles(T, H, W, C, Q):
    rng = np.random.default_rng(T * 1000 + Q)
    X = synth.f32_to_bf16_bits(rng.standard_normal((T, H, W, C)).astype(np.float32))
    q = synth.f32_to_bf16_bits((rng.standard_normal((Q, C)) / np.sqrt(C)).astype(np.float32))
    inp = synth.Inputs(wl=synth.small("t64_14x14_c3584", T=T, H=H, W=W, C=C, Q=Q, B=1), X=X, query=q)
    out = oracle.condense(inp.X_f64(), inp.query_f64(), 1, 1, 1.5, 0.0)
    Xd, qd = wz.to_device(inp, DEV)
    a, r, d = wz.relevance(wz.problem_of(inp.wl), Xd, qd)
    torch.cuda.synchronize()
    assert G.within(a.cpu().numpy(), out["a"].ravel(), G.TOL_F32_IN, "a")
    assert G.within(r.cpu().numpy(), out["r"], G.TOL_F32_IN, "r")
    assert G.within(d.cpu().numpy(), out["delta"], G.TOL_F32_IN, "delta")

"""The pass for bf16 queries of more than 128 tokens at the edges of its tiles, passes and stretches.

Tolerance: the inputs are exact in both, the pass sums bf16 products in fp32 (chains of four 64-channel chunks, eight
MFMA steps, added up in second accumulators), so its rounding stays near 1e-7: as for fp32 inputs, 1e-5 relative with a
floor of a tenth of the largest value.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import gpu_util as G
import oracle
import test_gpu_slices as slices
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


# (T, H, W, C, Q): stretches of one to four 16-row tiles with two and three column tiles a wave, a ragged last tile, one
# token; channels short of a 64-channel chunk, at and past the ring of four, beyond 8192; queries at the edges of a
# 16-column tile, of 256 columns and of one, two and three passes
SHAPES = [(3, 1, 1, 8, 129), (2, 4, 4, 64, 256), (300, 3, 3, 72, 257), (260, 5, 5, 264, 300), (260, 6, 8, 256, 384),
          (260, 7, 7, 320, 385), (3, 13, 13, 136, 400), (2, 9, 9, 584, 768), (2, 5, 7, 8200, 140), (9, 8, 8, 96, 1024),
          (260, 8, 8, 264, 300), (260, 7, 9, 136, 700), (260, 4, 8, 136, 200), (260, 5, 9, 136, 129),
          (128, 8, 8, 72, 300), (128, 8, 12, 72, 300), (3, 4, 4, 136, 450), (260, 5, 6, 136, 512),
          (260, 6, 8, 136, 400)]


@pytest.mark.parametrize("T,H,W,C,Q", SHAPES)
def test_wide_query(T, H, W, C, Q):
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


# passes of 32 columns over tiles of at most 32 tokens (long rows, up to 192 query tokens): one token, 16-row MFMA tiles
# whole, ragged and two; channel sums in LDS (C <= 8192) and stored by chunk; five and six passes, ragged last ones
@pytest.mark.parametrize("T,H,W,C,Q", [(3, 1, 1, 4104, 129), (2, 4, 4, 8192, 160), (434, 1, 1, 4104, 161),
                                       (3, 7, 9, 16392, 192), (2, 7, 8, 8256, 129), (128, 6, 6, 8192, 130)])
def test_passes_over_long_rows(T, H, W, C, Q):
    test_wide_query(T, H, W, C, Q)


def test_stretches_within_the_scratch():
    """Tiles whose sums would not fit the allocation-free call's scratch are taken in stretches: the call is accepted,
    with the scores and relevances of the definition."""
    T, H, W, C, Q = 256, 15, 15, 8192, 130
    g = torch.Generator(device=DEV).manual_seed(1)
    X = torch.randn(T, H, W, C, generator=g, device=DEV).bfloat16()
    q = (torch.randn(Q, C, generator=g, device=DEV) / C ** 0.5).bfloat16()
    p = wz.Problem(T=T, H=H, W=W, C=C, Q=Q, B=64, in_dtype=wz.WZ_BF16)
    assert wz.workspace_bytes(p) <= wz.lib().wz_noalloc_scratch_bytes()
    a, r, d = wz.relevance(p, X, q)
    qn = q.double() / q.double().norm(dim=1, keepdim=True)
    a64, s64 = [], []
    for t in range(T):
        x = X[t].reshape(-1, C).double()
        a64.append((x @ qn.t()).amax(1) / x.norm(dim=1))
        s64.append(x.sum(0))
    s64 = torch.stack(s64)
    pn = s64 / s64.norm(dim=1, keepdim=True)
    d64 = torch.cat([pn.new_zeros(1), 1 - (pn[1:] * pn[:-1]).sum(1)])
    torch.cuda.synchronize()
    for got, want, what in ((a, torch.cat(a64), "a"), (r, (pn @ qn.t()).amax(1), "r"), (d, d64, "delta")):
        assert G.within(got.cpu().numpy(), want.cpu().numpy(), G.TOL_F32_IN, what)


# one tile a frame; two and three, the last one shorter, its last stretch ragged; one pass and two (the channel and
# column sums of a stretch's passes add to those of the stretches before)
STRETCHES = [(256, 15, 15, 8192, 400), (128, 19, 21, 9216, 130), (128, 19, 21, 9216, 400), (140, 19, 21, 8000, 400)]


@pytest.mark.parametrize("T,H,W,C,Q", STRETCHES)
def test_stretches(T, H, W, C, Q):
    slices.test_slices(T, H, W, C, Q)  # a, r and delta against 64 bits


@pytest.mark.parametrize("T,H,W,C,Q", [(3, 5, 5, 264, 300), (9, 6, 8, 72, 700), (2, 1, 1, 8, 1024)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf")])
def test_infinity_in_a_small_frame(T, H, W, C, Q, value):
    """Frames of fewer than 49 tokens with more than 256 query tokens: an infinite value stays in its own channel's sum
    (the other channel of its pair does not become NaN), so r and delta are those of the same values in fp32."""
    g = torch.Generator().manual_seed(T * 1000 + Q)
    X = torch.randn(T, H, W, C, generator=g).bfloat16()
    q = (torch.randn(Q, C, generator=g) / C ** 0.5).bfloat16()
    X[0, 0, 0, 2] = value
    X[-1, -1, -1, 5] = value
    p = dict(T=T, H=H, W=W, C=C, Q=Q, B=1)
    a, r, d = wz.relevance(wz.Problem(in_dtype=wz.WZ_BF16, **p), X.to(DEV), q.to(DEV))
    a32, r32, d32 = wz.relevance(wz.Problem(in_dtype=wz.WZ_F32, **p), X.float().to(DEV), q.float().to(DEV))
    torch.cuda.synchronize()
    for got, want, what in ((a, a32, "a"), (r, r32, "r"), (d, d32, "delta")):
        got, want = got.cpu().numpy(), want.cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(want)), what
        assert G.within(np.nan_to_num(got), np.nan_to_num(want), G.TOL_F32_IN, what)

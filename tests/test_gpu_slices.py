"""The pass in slices of channels (bf16, more than 256 query tokens: a few frames with long rows, or many tokens with
short ones) at the edges of its tiles, slices and query passes.

Tolerance: exact inputs, fp32 sums in chains of at most 32 MFMA steps, the slices' partials added one after another: as
for fp32 inputs, 1e-5 relative with a floor of a tenth of the largest value.
"""
import pytest

torch = pytest.importorskip("torch")

import gpu_util as G
from libutil import ensure_built
from paper_2607_23265_amd import wavezip as wz

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# whole frames with several slices: four to sixteen 16-row tiles, the last ragged; a last slice short of a step, or of
# its steps; queries past a pass of 32 columns, not a multiple of 4 (the partial scores' padding), the most there are.
# One slice, several tiles a frame: rows of one step and of two.
SHAPES = [(2, 7, 7, 8200, 257), (1, 7, 8, 16384, 301), (3, 9, 9, 10008, 385), (9, 5, 10, 20488, 1024),
          (1, 16, 16, 65536, 260), (100, 60, 60, 8, 1000), (705, 13, 57, 56, 817)]


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ensure_built()


def inputs(T, H, W, C, Q):
    g = torch.Generator(device=DEV).manual_seed(T * 1000 + Q)
    X = torch.randn(T, H, W, C, generator=g, device=DEV).bfloat16()
    return X, (torch.randn(Q, C, generator=g, device=DEV) / C ** 0.5).bfloat16()


@pytest.mark.parametrize("T,H,W,C,Q", SHAPES)
def test_slices(T, H, W, C, Q):
    X, q = inputs(T, H, W, C, Q)
    a, r, d = wz.relevance(wz.Problem(T=T, H=H, W=W, C=C, Q=Q, B=1, in_dtype=wz.WZ_BF16), X, q)
    qn = q.double() / q.double().norm(dim=1, keepdim=True)
    a64, p64 = [], []
    for t in range(T):
        x = X[t].reshape(-1, C).double()
        a64.append((x @ qn.t()).amax(1) / x.norm(dim=1))
        p64.append(x.sum(0))
    p64 = torch.stack(p64)
    pn = p64 / p64.norm(dim=1, keepdim=True)
    d64 = torch.cat([pn.new_zeros(1), 1 - (pn[1:] * pn[:-1]).sum(1)])
    torch.cuda.synchronize()
    for got, want, what in ((a, torch.cat(a64), "a"), (r, (pn @ qn.t()).amax(1), "r"), (d, d64, "delta")):
        assert G.within(got.cpu().numpy(), want.cpu().numpy(), G.TOL_F32_IN, what)


@pytest.mark.parametrize("T,H,W,C,Q", [(2, 7, 7, 8200, 257), (3, 9, 9, 10008, 385)])
@pytest.mark.parametrize("levels", [1, 2])
def test_whole_pass(T, H, W, C, Q, levels):
    """The per-frame kernel's scores from the slices' partials rank the frames as the stage entry does, and every video
    of a batch has its single call's outputs, bit for bit; so has the call without a workspace."""
    V, B = 3, T * H * W // 4
    X, q = inputs(V * T, H, W, C, V * Q)
    X, q = X.view(V, T, H, W, C), q.view(V, Q, C)
    p = wz.Problem(T=T, H=H, W=W, C=C, Q=Q, B=B, in_dtype=wz.WZ_BF16, spatial_levels=levels)
    many = wz.condense_batch(p, X, q)
    for v in range(V):
        one = wz.condense(p, X[v], q[v].contiguous())
        static = wz.condense_noalloc(p, X[v], q[v].contiguous())
        a, r, d = wz.relevance(p, X[v], q[v].contiguous())
        budget, offset, _ = wz.temporal_budget(p, r, d)
        tok, idx = wz.spatial_dwt_condense(p, X[v], a, offset)
        torch.cuda.synchronize()
        assert int(offset[-1]) == B
        for i, x in enumerate((tok, idx, budget, offset)):
            assert torch.equal(x, one[i]) and torch.equal(x, many[i][v]) and torch.equal(x, static[i])

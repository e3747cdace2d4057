"""The decomposition of the relevance pass (csrc/wz_internal.h), evaluated on the host: a small program compiled against
the header prints the plan and the workspace of each shape.  No GPU needed."""
import os
import subprocess

import pytest

import libutil
import test_gpu_wide_query as wide
from paper_2607_23265_amd import wavezip as wz
from paper_2607_23265_amd.csrc import build

TOK, WG, WIDE, SLICES = range(4)
SCRATCH = 32 << 20
CUS = 256

PROBE = r"""
#include <cstdio>
#include "wz_internal.h"
int main() {
  wz_config c{};
  c.levels = 1; c.tau = 0.f; c.lambda_ = 1.5f; c.spatial_levels = 1; c.out_dtype = WZ_F32;
  int T, H, W, C, Q, dt, basis;
  long long B;
  while (scanf("%d %d %d %d %d %d %d %lld", &T, &H, &W, &C, &Q, &dt, &basis, &B) == 8) {
    c.T = T; c.H = H; c.W = W; c.C = C; c.Q = Q; c.in_dtype = dt; c.spatial_basis = basis; c.B = B;
    const wz::RelPlan p = wz::relevance_plan(c);
    printf("%d %d %d %d %d %d %d %zu %zu\n", p.kind, p.tiles, p.tile_tokens, p.mt, p.sub, p.ntw, p.grid,
           wz::workspace_layout(c, nullptr, true).bytes, wz::workspace_layout(c, nullptr, false).bytes);
  }
}
"""
FIELDS = ("kind", "tiles", "tile_tokens", "mt", "sub", "ntw", "grid", "bytes", "bytes_fused")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    libutil.ensure_built()
    d = tmp_path_factory.mktemp("plan")
    src, exe = str(d / "plan.hip"), str(d / "plan")
    with open(src, "w") as f:
        f.write(PROBE)
    libdir = os.path.dirname(wz.LIB_PATH)
    subprocess.run([build.hipcc(), "-O1", "-std=c++17", "--offload-host-only", "-I", build.INCLUDE, "-I", build.HERE,
                    src, f"-L{libdir}", f"-l:{os.path.basename(wz.LIB_PATH)}", f"-Wl,-rpath,{libdir}", "-o", exe],
                   check=True, capture_output=True, timeout=300)

    def run(T, H, W, C, Q, dtype=wz.WZ_BF16, basis=wz.WZ_HAAR, B=1):
        r = subprocess.run([exe], input=f"{T} {H} {W} {C} {Q} {dtype} {basis} {B}\n", capture_output=True, text=True,
                           check=True, timeout=60)
        return dict(zip(FIELDS, map(int, r.stdout.split())))

    return run


def test_kinds(plan):
    assert plan(64, 14, 14, 3584, 32)["kind"] == TOK
    assert plan(64, 14, 14, 3584, 300, wz.WZ_F32)["kind"] == TOK
    assert plan(256, 27, 27, 1152, 128)["kind"] == WG
    assert plan(64, 14, 14, 3584, 300)["kind"] == WIDE


# wz_relevance in us, channel stripes / shared tiles
@pytest.mark.parametrize("T,H,W,C,Q,kind", [
    (512, 14, 14, 768, 48, WG), (256, 27, 27, 1152, 48, WG), (96, 27, 27, 1152, 48, WG), (200, 14, 14, 2560, 48, WG),
    (512, 8, 8, 3584, 48, TOK), (110, 12, 12, 4096, 48, TOK), (128, 13, 13, 3584, 64, TOK),
    (74, 14, 14, 3168, 53, TOK),   # 40.4 / 49.8
    (33, 27, 24, 3264, 56, TOK),   # 44.1 / 52.4
    (135, 8, 13, 2344, 37, TOK),   # 34.8 / 39.0
    (289, 10, 2, 3672, 35, TOK),   # 36.6 / 53.0
    (68, 16, 16, 3664, 44, TOK),   # 44.8 / 56.4
    (1917, 2, 2, 2536, 49, TOK),   # 83.2 / 125.2
    (1, 9, 7, 200, 46, TOK),       # 7.8 / 9.2
])
def test_middle_query_kind(plan, T, H, W, C, Q, kind):
    """33 to 64 query tokens: the kernel that measured faster."""
    assert plan(T, H, W, C, Q)["kind"] == kind


# wz_relevance in us, passes of 32 columns / one pass; up to 4096 channels the one pass throughout
@pytest.mark.parametrize("T,H,W,C,Q,kind", [
    (1, 1, 1, 32768, 129, TOK),      # 232 / 302
    (434, 1, 1, 16384, 160, TOK),    # 255 / 310
    (1360, 1, 6, 36656, 130, TOK),   # 1758 / 2099
    (16, 15, 15, 16384, 129, TOK),   # 161 / 175
    (260, 14, 14, 8192, 130, WIDE),  # 715 / 610
    (3, 27, 27, 16384, 200, WIDE),   # 250 / 211
    (1, 1, 1, 4096, 129, WIDE), (64, 7, 7, 3584, 129, WIDE), (2, 4, 4, 16384, 256, WIDE),
])
def test_passes_or_one_pass(plan, T, H, W, C, Q, kind):
    """129 to 256 query tokens: the kernel that measured faster."""
    p = plan(T, H, W, C, Q)
    assert p["kind"] == kind and (kind == WIDE or p["tile_tokens"] <= 32)


# wz_relevance in us, channel slices / one pass; from 128 to 8192 channels the one pass throughout
@pytest.mark.parametrize("T,H,W,C,Q,kind", [
    (3, 33, 2, 64408, 816, SLICES),    # 1280 / 3117
    (1, 5, 12, 61904, 850, SLICES),    # 1242 / 2826
    (2, 26, 2, 32008, 397, SLICES),    # 318 / 718
    (8, 10, 12, 32768, 300, SLICES),   # 298 / 439
    (705, 13, 57, 56, 817, SLICES),    # 653 / 795
    (8, 14, 14, 16384, 1024, WIDE),    # 847 / 673
    (64, 7, 7, 16384, 300, WIDE),      # 459 / 236
    (1, 6, 8, 65536, 300, WIDE),       # frames of fewer than 49 tokens
    (1, 7, 7, 8192, 300, WIDE), (200, 28, 28, 128, 512, WIDE), (2, 7, 7, 8200, 256, WIDE),
    # the shapes of test_gpu_slices
    (2, 7, 7, 8200, 257, SLICES), (1, 7, 8, 16384, 301, SLICES), (3, 9, 9, 10008, 385, SLICES),
    (9, 5, 10, 20488, 1024, SLICES), (1, 16, 16, 65536, 260, SLICES), (100, 60, 60, 8, 1000, SLICES),
])
def test_slices_or_one_pass(plan, T, H, W, C, Q, kind):
    """More than 256 query tokens: the kernel that measured faster."""
    assert plan(T, H, W, C, Q)["kind"] == kind


def wide_cost(T, tiles, sub, mt):
    """Turns of a CU, times the 16-row tiles and the query reads (as long as four of them) of its stretches."""
    return -(-(-(-T // 8) * 8 * tiles) // CUS) * sub * (mt + 4)


# few frames of many tokens, frames enough for turns; sums past the scratch at the best tiles, or whatever the tiles
@pytest.mark.parametrize("T,H,W,C,Q", [(4, 64, 64, 32768, 300), (8, 64, 64, 16384, 300), (16, 15, 15, 65536, 230),
                                       (64, 14, 14, 65536, 129), (260, 14, 14, 16384, 130), (260, 14, 14, 8192, 130),
                                       (512, 14, 14, 3584, 300), (1040, 14, 14, 1024, 1024), (64, 14, 14, 3584, 300)])
def test_wide_query_tiles_cost(plan, T, H, W, C, Q):
    """Sums that pass the allocation-free call's scratch cost a call at most a quarter more than the best tiles, above
    256 query tokens at most half more."""
    p, N = plan(T, H, W, C, Q), H * W
    best = min(wide_cost(T, k, 1, -(-(-(-N // k)) // 16)) for k in range(-(-N // 64), -(-N // 16) + 1))
    assert p["kind"] == WIDE and wide_cost(T, p["tiles"], p["sub"], p["mt"]) <= (1.25 if Q <= 256 else 1.5) * best


# (a slightly dearer count that fits is taken, the finest ones being just past the scratch)
@pytest.mark.parametrize("T,H,W,C,Q,tiles", [(260, 14, 14, 8192, 130, 2), (260, 14, 14, 8192, 300, 2),
                                             (256, 15, 15, 8192, 130, 1), (256, 15, 15, 8192, 400, 1),
                                             (128, 19, 21, 9216, 400, 2), (856, 25, 32, 496, 815, 4)])
def test_wide_query_tiles_within_the_scratch(plan, T, H, W, C, Q, tiles):
    p = plan(T, H, W, C, Q)
    assert p["kind"] == WIDE and p["bytes"] <= SCRATCH
    assert p["tiles"] == tiles and p["sub"] > 1 and p["mt"] <= 4 and p["sub"] * 16 * p["mt"] >= p["tile_tokens"]


def test_wide_shapes_reach_every_form(plan):
    """The shapes of test_gpu_wide_query run every instantiation of the one-pass kernel, and stretches of one and of
    several tiles a frame with one and two passes over the query."""
    forms = [(p, s[1] * s[2] < 49 and s[4] > 256) for p, s in ((plan(*s), s) for s in wide.SHAPES) if p["kind"] == WIDE]
    assert {(p["mt"], p["ntw"], lone) for p, lone in forms} == {
        (m, n, lone) for m in (1, 2, 3, 4) for n in (2, 3) for lone in (False, True) if m < 4 or not lone}
    stretches = [(s, plan(*s)) for s in wide.STRETCHES]
    assert all(p["kind"] == WIDE and p["sub"] > 1 for _, p in stretches)
    assert {(p["tiles"] > 1, s[4] > 384) for s, p in stretches} == {(False, True), (True, False), (True, True)}


def test_wide_query_operator_rows_stay_in_the_scratch(plan):
    """A filter-bank call whose operator rows fitted the scratch beside coarser tiles' sums keeps them there."""
    p = plan(325, 35, 24, 280, 473, basis=wz.WZ_DB4, B=6042)
    assert p["kind"] == WIDE and p["bytes"] <= SCRATCH

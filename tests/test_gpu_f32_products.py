"""The fp32 matrix-core products at the edges of their tiles, reduction steps and slices, against the oracle: one row,
channel counts that end inside a tile or a step, slices that join, tiles of 64 and 128 rows for either product, odd ranks, tokens outside
the grid."""
import numpy as np
import pytest
import torch

import oracle
from _gpu_util import TOL, assert_matches
from paper_2309_15275_amd import binding

pytestmark = pytest.mark.gpu


def _inputs(N, T, cin, cout, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal((N, T, cin)).astype(np.float32), rng.standard_normal((N, T, cout)).astype(np.float32),
            (0.05 * rng.standard_normal((cout, cin))).astype(np.float32))


# (N, H, W, extra, Cin, Cout, patch, r)
CASES = [(1, 2, 2, 0, 4, 4, 2, 1), (1, 8, 8, 0, 4, 8, 8, 1), (2, 8, 8, 0, 68, 132, 8, 3), (3, 7, 7, 0, 60, 100, 8, 36),
         (1, 8, 16, 1, 132, 2060, 8, 10), (5, 16, 8, 2, 64, 36, 8, 64), (2, 9, 13, 0, 196, 516, 8, 27), (7, 11, 6, 1, 72, 260, 4, 5),
         (3, 8, 12, 0, 36, 1028, 4, 16), (4, 5, 5, 0, 20, 44, 2, 4), (33, 14, 14, 0, 76, 84, 8, 15)]


@pytest.mark.parametrize("case", CASES, ids=str)
@pytest.mark.parametrize("order", ["l1", "scattered"])
def test_low_rank_backward(case, order):
    N, H, W, extra, cin, cout, patch, r = case
    pp = patch * patch
    idx = oracle.select_bases(patch, r, "l1").tolist() if order == "l1" else [(k * 7 + 3) % pp for k in range(pp)][-r:]
    assert len(set(idx)) == r
    x, gy, w = _inputs(N, extra + H * W, cin, cout, 900 + r)
    gx0, gW0 = oracle.lbp_wht_backward_tokens(x, gy, w, (H, W), patch, idx)
    dx, dgy, dw = (torch.from_numpy(v).cuda() for v in (x, gy, w))
    gx, gW = torch.full_like(dx, float("nan")), torch.full_like(dw, float("nan"))
    binding.lbp_wht_backward_tokens(dx, dgy, dw, (H, W), patch, idx, gx=gx, gW=gW)
    assert_matches(gx, gx0, TOL["f32"], "gx")
    assert_matches(gW, gW0, TOL["f32"], "gW")
    again = binding.lbp_wht_backward_tokens(dx, dgy, dw, (H, W), patch, idx)        # the order of arrival does not matter
    assert torch.equal(again[0], gx) and torch.equal(again[1], gW)
    one = binding.lbp_wht_backward_tokens(dx, dgy, dw, (H, W), patch, idx, want_gw=False)
    assert_matches(one[0], gx0, TOL["f32"], "gx alone")
    one = binding.lbp_wht_backward_tokens(dx, dgy, dw, (H, W), patch, idx, want_gx=False)
    assert_matches(one[1], gW0, TOL["f32"], "gW alone")


# (N, H, W, extra, Cin, Cout, patch, r), rows of the tiles of gx and gW, and whether their slices join, on 256 compute units: every pair of
# heights with each product whole and cut, for 8 x 8 and for smaller patches; then 128 rows of many and of few patches
TILES = [((10, 3, 3, 1, 988, 92, 8, 2), 64, 128, 0, 0), ((34, 11, 11, 1, 320, 120, 8, 6), 64, 128, 0, 1), ((1, 5, 3, 0, 620, 1228, 8, 1), 64, 128, 1, 0),
         ((77, 9, 3, 0, 164, 304, 8, 2), 64, 128, 1, 1), ((26, 3, 3, 0, 652, 36, 8, 1), 128, 64, 0, 0), ((66, 11, 11, 1, 20, 52, 8, 3), 128, 64, 0, 1),
         ((59, 4, 4, 1, 212, 216, 8, 1), 128, 64, 1, 0), ((36, 24, 4, 0, 228, 212, 8, 3), 128, 64, 1, 1), ((10, 9, 25, 0, 1068, 72, 8, 2), 128, 128, 0, 0),
         ((66, 9, 25, 0, 312, 92, 8, 2), 128, 128, 0, 1), ((79, 4, 4, 0, 332, 220, 8, 1), 128, 128, 1, 0), ((38, 9, 9, 0, 140, 196, 8, 3), 128, 128, 1, 1),
         ((3, 5, 5, 0, 520, 72, 2, 1), 64, 128, 0, 0), ((70, 5, 5, 0, 204, 1176, 4, 2), 64, 128, 1, 1), ((4, 25, 5, 0, 288, 20, 4, 1), 128, 64, 0, 0),
         ((22, 17, 4, 0, 24, 232, 2, 2), 128, 64, 1, 1), ((1, 16, 16, 0, 1196, 192, 2, 3), 128, 128, 0, 0), ((19, 9, 5, 0, 444, 288, 2, 1), 128, 128, 1, 1),
         ((58, 3, 3, 0, 284, 16, 8, 10), 128, 64, 0, 1), ((25, 9, 9, 1, 204, 204, 8, 10), 128, 128, 1, 1), ((71, 27, 3, 0, 20, 36, 8, 27), 128, 64, 0, 1),
         ((77, 11, 11, 0, 20, 16, 8, 36), 128, 64, 0, 1), ((6, 26, 26, 1, 20, 976, 8, 36), 128, 64, 1, 1), ((34, 18, 18, 1, 28, 20, 8, 63), 128, 64, 0, 1),
         ((34, 20, 3, 0, 24, 968, 8, 63), 128, 64, 1, 1)]


def _plan(case):
    N, H, W, extra, cin, cout, patch, r = case
    return binding.describe_plan(binding.LbpShape(N, H, W, cin, cout, 0, 0), patch, oracle.select_bases(patch, r, "l1").tolist(), extra=extra)


@pytest.mark.parametrize("case, rows_x, rows_w, joined_x, joined_w", TILES, ids=str)
def test_tiles_of_64_and_128_rows(case, rows_x, rows_w, joined_x, joined_w):
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        plan = _plan(case)
        gw, gx = (next(t for t in plan.split("; ") if t.startswith(k)) for k in ("gW:", "gx:"))
        assert (f"fp32 {rows_x}x64" in gx, f"fp32 {rows_w}x64" in gw, "slices" in gx, "slices" in gw) == (True, True, bool(joined_x), bool(joined_w)), plan
    test_low_rank_backward(case, "l1")


@pytest.mark.parametrize("M,cin,cout", [(1, 4, 4), (3, 64, 132), (65, 68, 2052), (1030, 36, 60), (4100, 132, 68)])
def test_exact_backward(M, cin, cout):
    x, gy, w = _inputs(1, M, cin, cout, M)
    gx0 = gy[0].astype(np.float64) @ w
    gW0 = gy[0].astype(np.float64).T @ x[0]
    dx, dgy, dw = (torch.from_numpy(v).cuda() for v in (x.reshape(1, 1, M, cin), gy.reshape(1, 1, M, cout), w))
    gx, gW = torch.full_like(dx, float("nan")), torch.full_like(dw, float("nan"))
    binding.full_bp_backward(dx, dgy, dw, gx=gx, gW=gW)
    assert_matches(gx.reshape(M, cin), gx0, TOL["f32"], "gx")
    assert_matches(gW, gW0, TOL["f32"], "gW")


@pytest.mark.parametrize("steps", range(8))
@pytest.mark.parametrize("rest", [0, 4, 28])
@pytest.mark.parametrize("wide", [False, True])
def test_every_number_of_steps(steps, rest, wide):
    """Reductions of a few steps of 32 and what is left, of either product; whole numbers, exact."""
    K = 32 * steps + rest
    if K == 0:
        pytest.skip("no reduction")
    gen = torch.Generator(device="cuda").manual_seed(K)
    n = 260 if wide else 36
    for M, cin, cout in ((K, n, 68), (n, 68, K)):       # of gW, of gx
        x, gy, w = (torch.randint(-4, 5, s, generator=gen, device="cuda").float() for s in ((M, cin), (M, cout), (cout, cin)))
        gx, gW = binding.full_bp_backward(x.view(1, 1, M, cin), gy.view(1, 1, M, cout), w)
        assert torch.equal(gx.view(M, cin).double(), gy.double() @ w.double())
        assert torch.equal(gW.double(), gy.double().T @ x.double())

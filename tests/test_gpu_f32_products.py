"""The fp32 matrix-core products at the edges of their tiles, reduction steps and slices, against the oracle: one row,
channel counts that end inside a tile or a step, slices that join, both tile heights, odd ranks, tokens outside the grid."""
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

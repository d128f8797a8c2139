"""Input gradients on 128 x 256 tiles: the reverse projection takes their columns in two turns, alone and beside the weight gradient."""
import numpy as np
import pytest
import torch

import oracle
from _gpu_util import TOL, assert_matches, to_device
from paper_2309_15275_amd import binding, workloads
from paper_2309_15275_amd.autograd import lbp_wht_linear

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _defaults():
    binding.reset_options()
    yield
    binding.reset_options()


def _inputs(N, T, cin, cout, seed):
    rng = np.random.default_rng(seed)
    return [workloads.round_to_bf16(v.astype(np.float32)) for v in
            (rng.standard_normal((N, T, cin)), rng.standard_normal((N, T, cout)), 0.05 * rng.standard_normal((cout, cin)))]


# columns that end before, at and behind the second turn and the tile; reductions of 1 step, of a ring's length, and that end inside one
@pytest.mark.parametrize("patch, r, order", [(8, 1, "l1"), (8, 8, "l1"), (8, 17, "linf"), (8, 36, "l1"), (4, 3, "l1"), (4, 16, "l1")])
@pytest.mark.parametrize("N, H, W, extra, cin, cout", [(3, 7, 9, 0, 72, 32), (2, 9, 24, 1, 136, 104), (1, 16, 8, 2, 256, 96), (5, 15, 8, 0, 264, 200), (2, 24, 16, 1, 392, 328)])
def test_columns_in_two_turns(N, H, W, extra, cin, cout, patch, r, order):
    idx = oracle.select_bases(patch, r, order).tolist()
    x, gy, w = _inputs(N, extra + H * W, cin, cout, r)
    gx0, gW0 = oracle.lbp_wht_backward_tokens(x, gy, w, (H, W), patch, idx)
    dx, dgy, dw = (to_device(v, "bf16") for v in (x, gy, w))
    binding.set_option("LBP_FUSE_UNPROJECT", "1")
    got = {}
    for tile in ("4", "2"):          # an element's sum does not depend on the tile
        binding.set_option("LBP_GEMM_TILE", tile)
        gx, gW = torch.full_like(dx, float("nan")), torch.full(dw.shape, float("nan"), device="cuda")
        binding.lbp_wht_backward_tokens(dx, dgy, dw, (H, W), patch, idx, gx=gx, gW=gW)
        got[tile] = gx
        assert_matches(gx, gx0, TOL["bf16"], "gx")
        assert_matches(gW, gW0, TOL["bf16"], "gW")
    assert torch.equal(got["2"], got["4"])


# (N, H, W, tokens in front, cin, cout, patch, r): launches that the planner takes to such tiles, in one round, and of two launches otherwise
BESIDE = [(31, 10, 10, 0, 952, 688, 8, 55), (45, 20, 20, 2, 1488, 1216, 8, 10), (6, 46, 46, 1, 1216, 1080, 4, 4), (102, 8, 8, 0, 3864, 744, 8, 48)]


@pytest.mark.parametrize("case", range(len(BESIDE)))
def test_beside_the_weight_gradient(case):
    N, H, W, extra, cin, cout, patch, r = BESIDE[case]
    idx = binding.select_bases(patch, r)
    shape = binding.LbpShape(N, H, W, cin, cout, 1, 0)
    plan = binding.describe_plan(shape, patch, idx, extra=extra)
    assert "one grouped launch" in plan and "gx: tile 128x256" in plan, plan
    g = torch.Generator(device="cuda").manual_seed(case)
    x, gy = (torch.randn(N, extra + H * W, c, generator=g, device="cuda").bfloat16() for c in (cin, cout))
    w = (0.05 * torch.randn(cout, cin, generator=g, device="cuda")).bfloat16()
    got = {}
    for group in (None, "2", "0"):
        binding.set_option("LBP_GEMM_GROUP", group)
        binding.set_option("LBP_GEMM_TILE", "4" if group == "0" else None)
        gx, gW = torch.full_like(x, float("nan")), torch.full((cout, cin), float("nan"), device="cuda")
        binding.lbp_wht_backward_tokens(x, gy, w, (H, W), patch, idx, gx=gx, gW=gW)
        got[group] = gx, gW
    assert torch.equal(got[None][0], got["0"][0]) and torch.equal(got[None][0], got["2"][0])
    assert torch.equal(got[None][1], got["2"][1])
    # fp32 sums of the same products in other slices
    assert float((got[None][1] - got["0"][1]).norm() / got["0"][1].norm()) <= 2e-6


def test_bias_sums_at_the_end_of_such_a_launch():
    N, H, W, _, cin, cout, patch, r = BESIDE[0]
    idx = binding.select_bases(patch, r)
    assert "gx: tile 128x256" in binding.describe_plan(binding.LbpShape(N, H, W, cin, cout, 1, 1), patch, idx)
    g = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn(N, H, W, cin, generator=g, device="cuda").bfloat16().requires_grad_()
    w = (0.05 * torch.randn(cout, cin, generator=g, device="cuda")).bfloat16().requires_grad_()
    b = torch.zeros(cout, device="cuda", dtype=torch.bfloat16, requires_grad=True)
    gy = torch.randn(N, H, W, cout, generator=g, device="cuda").bfloat16()
    beside = torch.autograd.grad(lbp_wht_linear(x, w, b, patch, idx), (x, w, b), gy)
    binding.set_option("LBP_GEMM_GROUP", "0")
    apart = torch.autograd.grad(lbp_wht_linear(x, w, b, patch, idx), (x, w, b), gy)
    assert torch.equal(beside[0], apart[0]) and torch.equal(beside[2], apart[2])


# (as BESIDE): input gradients alone, in one round (last tiles of 128 columns and fewer, few bases, 4 x 4 patches, unpoolable ranks) and in many;
# test_host_plans.py asserts these plans without a GPU
LONE = [(119, 14, 14, 0, 1408, 680, 8, 12), (61, 14, 14, 1, 1864, 1024, 4, 8), (97, 9, 9, 1, 3224, 1312, 8, 7), (111, 20, 20, 0, 576, 3864, 8, 7),
        (56, 9, 9, 0, 1880, 1488, 8, 26), (69, 20, 20, 1, 1024, 984, 4, 14), (72, 24, 24, 0, 2176, 912, 8, 18)]


@pytest.mark.parametrize("apart", [False, True])
@pytest.mark.parametrize("case", range(len(LONE)))
def test_alone(case, apart):
    # as the planner sends them, alone and with grouping switched off, against 128 x 128 tiles: an element's sum does not depend on the tile
    N, H, W, extra, cin, cout, patch, r = LONE[case]
    idx = binding.select_bases(patch, r)
    binding.set_option("LBP_GEMM_GROUP", "0" if apart else None)
    plan = binding.describe_plan(binding.LbpShape(N, H, W, cin, cout, 1, 0), patch, idx, extra=extra, want_gw=apart)
    assert "separate launches" in plan and "gx: tile 128x256" in plan and "joined" not in plan, plan
    g = torch.Generator(device="cuda").manual_seed(case)
    x, gy = (torch.randn(N, extra + H * W, c, generator=g, device="cuda").bfloat16() for c in (cin, cout))
    w = (0.05 * torch.randn(cout, cin, generator=g, device="cuda")).bfloat16()
    got = []
    for tile in (None, "4"):
        binding.set_option("LBP_GEMM_TILE", tile)
        gx = torch.full_like(x, float("nan"))
        binding.lbp_wht_backward_tokens(x, gy, w, (H, W), patch, idx, gx=gx, want_gw=apart)
        got.append(gx)
    assert torch.equal(got[0], got[1])

"""Grouped launches of more workgroups than the device holds: which product goes first depends on how long its workgroups are.

The order decides when a workgroup runs, never what it computes, so both orders give the same bits; operands are small whole
numbers, so that the weight gradient (at most 184 products of at most 4, times 1/64) is exact.
"""
import pytest
import torch

from paper_2309_15275_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_switches():
    binding.reset_options()
    yield
    binding.reset_options()


# steps of the input gradient / of the weight gradient: 60 / 3 in joined slices, 5 / 4 and 4 / 4 (the two sides of the line), 2 / 10
@pytest.mark.parametrize("shape,cin,cout,r", [((2, 12, 12), 2688, 3800, 23), ((64, 8, 8), 16384, 320, 4), ((64, 8, 8), 20480, 256, 4),
                                              ((80, 8, 8), 16384, 128, 8)])
def test_either_order_gives_the_same(shape, cin, cout, r):
    N, H, W = shape
    idx = binding.select_bases(8, r)
    rows = binding.patch_count(N, H, W, 8) * r
    gen = torch.Generator(device="cuda").manual_seed(r)
    draw = lambda *s: torch.randint(-2, 3, s, generator=gen, device="cuda").bfloat16()
    x_r, gy_r, w = draw(rows, cin), draw(rows, cout), draw(cout, cin)

    def call(group):
        binding.set_option("LBP_GEMM_GROUP", group)
        gx = torch.full((N, H, W, cin), float("nan"), dtype=torch.bfloat16, device="cuda")
        gW = torch.full((cout, cin), float("nan"), device="cuda")
        return binding.lbp_wht_products(x_r, gy_r, w, shape, 8, idx, gx, gW)

    assert "one grouped launch" in binding.describe_plan(binding.LbpShape(N, H, W, cin, cout, 1, 0), 8, idx)
    gx, gW = call(None)
    gx2, gW2 = call("2")
    assert torch.equal(gx, gx2) and torch.equal(gW, gW2)
    assert torch.equal(gW.double(), gy_r.double().T @ x_r.double() / 64)

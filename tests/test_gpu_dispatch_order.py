"""Grouped launches of more workgroups than the device holds: which product goes first depends on how long its workgroups are.

The order decides when a workgroup runs, never what it computes, so both orders give the same bits; operands are small whole
numbers, so that the weight gradient (at most 640 products of at most 4, times 1/64) is exact.
"""
import re

import pytest
import torch

from paper_2309_15275_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_switches():
    binding.reset_options()
    yield
    binding.reset_options()


# steps of 64 of an input gradient's workgroup / of a weight gradient's, and which goes first: 10 / 3 (60 in 6 slices that join) input,
# 5 / 4 (the line) input, 4 / 4 weight, 2 / 10 weight
@pytest.mark.parametrize("shape,cin,cout,r", [((2, 12, 12), 2688, 3800, 23), ((64, 8, 8), 16384, 320, 4), ((64, 8, 8), 20480, 256, 4),
                                              ((80, 8, 8), 16384, 128, 8)])
def test_either_order_gives_the_same(shape, cin, cout, r):
    N, H, W = shape
    idx = binding.select_bases(8, r)
    rows = binding.patch_count(N, H, W, 8) * r
    gen = torch.Generator(device="cuda").manual_seed(r)
    draw = lambda *s: torch.randint(-2, 3, s, generator=gen, device="cuda").bfloat16()
    x_r, gy_r, w = draw(rows, cin), draw(rows, cout), draw(cout, cin)

    def call(**options):
        for name, value in options.items():
            binding.set_option("LBP_" + name, value)
        gx = torch.full((N, H, W, cin), float("nan"), dtype=torch.bfloat16, device="cuda")
        gW = torch.full((cout, cin), float("nan"), device="cuda")
        binding.lbp_wht_products(x_r, gy_r, w, shape, 8, idx, gx, gW)
        binding.reset_options()
        return gx, gW

    plan = binding.describe_plan(binding.LbpShape(N, H, W, cin, cout, 1, 0), 8, idx)
    assert "one grouped launch" in plan
    # more workgroups than the device holds, or there is no order: at least these many (a tile may hold fewer patches than fit)
    bm, cut = int(re.search(r"gx: tile (\d+)x128", plan)[1]), re.search(r"reduction in (\d) slices", plan)
    least = -(-rows // bm) * -(-cin // 128) * (int(cut[1]) if cut else 1) + -(-cout // 128) * -(-cin // 128)
    assert least > 2 * torch.cuda.get_device_properties(0).multi_processor_count
    gx, gW = call()
    assert torch.equal(gW.double(), gy_r.double().T @ x_r.double() / 64)
    # weight gradient first, whatever the rule; two launches in one piece each, the reverse projection in the product as in the grouped one
    for other in (call(GEMM_GROUP=2), call(GEMM_GROUP=0, GX_JOIN=1, FUSE_UNPROJECT=1)):
        assert torch.equal(gx, other[0]) and torch.equal(gW, other[1])

"""Exact gradients on 256 x 128 tiles (three stages of 64), which only the planner chooses: test_host_plans.py asserts that it does for these."""
import pytest
import torch

from paper_2309_15275_amd import binding

pytestmark = pytest.mark.gpu

# (rows, Cin, Cout, gradients, which of them are on such tiles): reductions of 9 to 11 steps that end inside one, at its end and behind it,
# longer ones and, with more columns, of 2 and 5; rows and columns that end inside a tile; a weight gradient in slices; an input gradient behind a weight gradient
CASES = [(33000, 88, 520, "gx", "gx"), (33001, 120, 576, "gx", "gx"), (33000, 128, 584, "gx", "gx"), (41615, 88, 640, "gx", "gx"), (41616, 88, 1136, "gx", "gx"),
         (33024, 128, 648, "gx", "gx"), (36801, 1552, 200, "gW", "gW"), (36800, 1552, 160, "gW", "gW"), (5184, 936, 3648, "both", "gx"), (5184, 936, 1544, "both", "gx"),
         (3400, 1176, 3824, "both", "gx"), (36864, 600, 320, "gx", "gx"), (27001, 808, 120, "gx", "gx")]


@pytest.mark.parametrize("rows, cin, cout, grads, tall", CASES)
def test_every_element_of_tall_tiles(rows, cin, cout, grads, tall):
    gen = torch.Generator(device="cuda").manual_seed(rows + cin)
    x, gy, w = (torch.randint(-2, 3, s, generator=gen, device="cuda").float() for s in ((rows, cin), (rows, cout), (cout, cin)))
    shape = lambda t: t.bfloat16().view(1, 1, rows, -1)
    gx, gW = binding.full_bp_backward(shape(x), shape(gy), w.bfloat16(), want_gx=grads != "gW", want_gw=grads != "gx")
    if grads != "gW":       # whole numbers below 2^24: exact in fp32 in any order
        assert torch.equal(gx.view(rows, cin), (gy.double() @ w.double()).bfloat16())
    if grads != "gx":
        assert torch.equal(gW, (gy.double().T @ x.double()).float())

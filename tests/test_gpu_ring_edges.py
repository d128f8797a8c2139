"""Reductions around the length of the ring that a product's main loop keeps in LDS.

Short ones end before the ring is full, the others in each of its stages, with and without a partial step.  Operands are small
whole numbers, so that every sum is exact in fp32 and results compare bit for bit (the input gradient after one rounding to bf16).
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


# 128 x 128 with four stages of 64 (0), 256 x 128 (2), 256 x 256 and 256 x 192 with five of 32 (3, 7), 64 x 128 (5)
@pytest.mark.parametrize("tile", [0, 2, 3, 5, 7])
@pytest.mark.parametrize("k", [8, 24, 32, 40, 64, 72, 96, 128, 136, 160, 168, 192, 224, 256, 264, 296, 320, 328, 352, 384, 448])
def test_reductions_around_the_ring(k, tile):
    gen = torch.Generator(device="cuda").manual_seed(k)
    draw = lambda *s: torch.randint(-2, 3, s, generator=gen, device="cuda").float()
    binding.set_option("LBP_GEMM_TILE", tile)
    other, cin = 272, 200
    # the input gradient's reduction is over Cout, the weight gradient's over the tokens
    gy, w, x = draw(other, k), draw(k, cin), draw(other, cin)
    gx, _ = binding.full_bp_backward(x.bfloat16().view(1, 1, other, cin), gy.bfloat16().view(1, 1, other, k), w.bfloat16(), want_gw=False)
    assert torch.equal(gx.view(other, cin), (gy.double() @ w.double()).bfloat16())
    gy, w, x = draw(k, other), draw(other, cin), draw(k, cin)
    _, gW = binding.full_bp_backward(x.bfloat16().view(1, 1, k, cin), gy.bfloat16().view(1, 1, k, other), w.bfloat16(), want_gx=False)
    assert torch.equal(gW, (gy.double().T @ x.double()).float())

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


STEPS = [8, 24, 32, 40, 64, 72, 96, 128, 136, 160, 168, 192, 224, 256, 264, 296, 320, 328, 352, 384, 448]


# One launch holds every workgroup: 128 x 128 with four stages of 64 (0), 128 x 256 with three of 32 (2), 256 x 256 and 256 x 192 with five of 32 (3, 7),
# 64 x 128 and 64 x 64 with three (5, 6).  13184 columns are more workgroups than that, and two stages: 64 x 128 (1, 5), 128 x 128 (4), 64 x 64 (6).
@pytest.mark.parametrize("tile, cin", [(0, 200), (2, 200), (3, 200), (5, 200), (6, 200), (7, 200), (1, 13184), (4, 13184), (5, 13184), (6, 13184)])
@pytest.mark.parametrize("k", STEPS)
def test_reductions_around_the_ring(k, tile, cin):
    gen = torch.Generator(device="cuda").manual_seed(k)
    draw = lambda *s: torch.randint(-2, 3, s, generator=gen, device="cuda").float()
    binding.set_option("LBP_GEMM_TILE", tile)
    other = 272
    # the input gradient's reduction is over Cout, the weight gradient's over the tokens
    gy, w, x = draw(other, k), draw(k, cin), draw(other, cin)
    gx, _ = binding.full_bp_backward(x.bfloat16().view(1, 1, other, cin), gy.bfloat16().view(1, 1, other, k), w.bfloat16(), want_gw=False)
    assert torch.equal(gx.view(other, cin), (gy.double() @ w.double()).bfloat16())
    gy, w, x = draw(k, other), draw(other, cin), draw(k, cin)
    _, gW = binding.full_bp_backward(x.bfloat16().view(1, 1, k, cin), gy.bfloat16().view(1, 1, k, other), w.bfloat16(), want_gx=False)
    assert torch.equal(gW, (gy.double().T @ x.double()).float())


# Both products in one resident launch, the input gradient on 64 x 128 tiles with four stages of 64 read a whole one ahead: both reductions are k
@pytest.mark.parametrize("k", STEPS)
def test_grouped_reductions_around_the_ring(k):
    gen = torch.Generator(device="cuda").manual_seed(k)
    N, r, cin = k // 8, 8, 264
    idx = binding.select_bases(8, r)
    plan = binding.describe_plan(binding.LbpShape(N, 8, 8, cin, k, 1, 0), 8, idx)
    assert "one grouped launch" in plan and "gx: tile 64x128" in plan
    draw = lambda *s: torch.randint(-2, 3, s, generator=gen, device="cuda").bfloat16()
    x_r, gy_r, w = draw(N * r, cin), draw(N * r, k), draw(k, cin)
    gx = torch.full((N, 8, 8, cin), float("nan"), dtype=torch.bfloat16, device="cuda")
    gW = torch.full((k, cin), float("nan"), device="cuda")
    binding.lbp_wht_products(x_r, gy_r, w, (N, 8, 8), 8, idx, gx, gW)
    assert torch.equal(gW.double(), gy_r.double().T @ x_r.double() / 64)
    assert torch.equal(gx, binding.wht_unproject((gy_r.double() @ w.double()).float(), (N, 8, 8, cin), torch.bfloat16, 8, idx))

"""fp32 products from three bf16 parts an operand: as exact as single precision gets, over the range of its exponents, and with values
that are not finite as the fp32 matrix cores have them."""
import numpy as np
import pytest
import torch

from paper_2309_15275_amd import binding

pytestmark = pytest.mark.gpu


def _products(M, cin, cout, seed, scale_x=1.0, scale_gy=1.0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x, gy, w = (torch.randn(s, generator=gen, device="cuda") for s in ((M, cin), (M, cout), (cout, cin)))
    return scale_x * x, scale_gy * gy, w


def _run(x, gy, w):
    gx, gW = binding.full_bp_backward(x.view(1, 1, *x.shape), gy.view(1, 1, *gy.shape), w)
    return gx.view_as(x), gW


# (rows, Cin, Cout): steps of 32 and the rest, 64- and 128-row tiles, slices that join
@pytest.mark.parametrize("M, cin, cout", [(31, 8, 36), (64, 68, 128), (700, 132, 260), (3000, 324, 96), (40, 260, 3000)])
@pytest.mark.parametrize("scale_x, scale_gy", [(1.0, 1.0), (1e-30, 1e15), (1e18, 1e-15)])
def test_error_of_the_sums(M, cin, cout, scale_x, scale_gy):
    """Six products of parts leave out 2^-24 of a product at most, 2^-26.8 of random ones in the mean square, and a sum of K products that is
    rounded K / 16 times, with K^(1/2) of cancelling, is off by less than 2^-24 (1 + (K / 16)^(1/2)) of its norm."""
    x, gy, w = _products(M, cin, cout, M, scale_x, scale_gy)
    gx, gW = _run(x, gy, w)
    for out, ref, K in ((gx, gy.double() @ w.double(), cout), (gW, gy.double().T @ x.double(), M)):
        err = float(torch.norm(out.double() - ref) / torch.norm(ref))
        assert err <= 2.0 ** -24 * (1 + (K / 16) ** 0.5), (err, K)


# the smallest normal numbers, denormals of 10 to 23 bits and their ordinary partners; operands and sums beyond what has parts
@pytest.mark.parametrize("M, cin, cout", [(31, 8, 36), (700, 132, 260), (3000, 324, 96)])
@pytest.mark.parametrize("scale_x, scale_gy", [(2.0 ** -112, 2.0 ** 60), (2.0 ** -120, 1.0), (2.0 ** -126, 2.0 ** 60), (2.0 ** -139, 2.0 ** 60),
                                               (2.0 ** 60, 2.0 ** -130), (2.0 ** 102, 2.0 ** -110), (2.0 ** 110, 2.0 ** -60), (2.0 ** 60, 2.0 ** 30)])
def test_error_at_the_ends_of_the_exponents(M, cin, cout, scale_x, scale_gy):
    """Tiny and huge operands keep the bits that they have.  Sums below 2^-126 are denormal and known to 2^-150 each; sums that leave
    the range of the parts are rounded every 2 products instead of 16."""
    x, gy, w = _products(M, cin, cout, M, scale_x, scale_gy)
    gx, gW = _run(x, gy, w)
    for out, a, b, K in ((gx, gy, w, cout), (gW, gy.T, x, M)):
        ref = a.double() @ b.double()
        large = max(float(a.abs().max()), float(b.abs().max())) >= 2.0 ** 104 or float(ref.abs().max()) >= 2.0 ** 78
        bound = 2.0 ** -24 * (1 + (K / (2 if large else 16)) ** 0.5) * float(torch.norm(ref)) + 2.0 ** -149 * ref.numel() ** 0.5
        assert float(torch.norm(out.double() - ref)) <= bound, (K, large)


@pytest.mark.parametrize("where", ["x", "gy", "w"])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38])
def test_values_that_are_not_finite(where, value):
    """Sums without such a value keep their bits; the others are what fp32 arithmetic gives (infinite, or NaN)."""
    x, gy, w = _products(200, 132, 196, 3)
    good = _run(x, gy, w)
    {"x": x, "gy": gy, "w": w}[where][70, 50] = value
    bad = _run(x, gy, w)
    for out, before, a, b in ((bad[0], good[0], gy, w), (bad[1], good[1], gy.T, x)):
        if where == "x" and out is bad[0] or where == "w" and out is bad[1]:
            assert torch.equal(out, before)
            continue
        ref = a.double() @ b.double()
        touched = torch.ones_like(out, dtype=torch.bool)
        if where == "gy":
            touched = torch.zeros_like(touched)
            touched[70 if out is bad[0] else 50] = True
        else:
            touched = torch.zeros_like(touched)
            touched[:, 50] = True
        assert torch.equal(torch.isnan(out), torch.isnan(ref))
        same = torch.isinf(ref) | (ref.abs() > 3.4028235e38)
        assert torch.equal(out[same], ref[same].float())
        # a tile that was computed again has been rounded differently: 2^-24 K^(1/2) of the operands' norms
        rest = ~touched
        assert float((out[rest] - before[rest]).abs().max()) <= 2.0 ** -22 * 200 ** 0.5 * float(before[rest].abs().max())


def test_largest_and_smallest_parts():
    """One product at a time: powers of two across the exponents, and mantissas that fill all three parts."""
    m = torch.tensor([1.0, 1 + 2.0 ** -23, 2 - 2.0 ** -23, 1 + 2.0 ** -8 + 2.0 ** -16, 1 - 2.0 ** -24], device="cuda")
    for e in (-100, -50, 0, 50, 100):
        gy = torch.zeros(4, 20, device="cuda")
        x = torch.zeros(4, 20, device="cuda")
        gy[0, :5], x[0, :5] = m * 2.0 ** e, m * 2.0 ** -e
        gW = _run(x, gy, torch.zeros(20, 20, device="cuda"))[1]
        ref = gy[0].double()[:, None] * x[0].double()[None]
        assert float((gW.double() - ref).abs().max()) <= 2.0 ** -23 * 4       # one rounding of the sum, and what is left out


def test_a_single_product_is_rounded_once():
    """One token: every element of gW is one product, which is rounded as fp32 arithmetic rounds it.  (What three parts leave out would show: the
    first pair of values has the largest middle and low parts there are, of the same sign, and m l' + l m' is 2^-24.04 of its product.)"""
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, gy = (torch.randn(1, n, generator=gen, device="cuda") for n in (516, 260))
    x[:, 0] = gy[:, 0] = 1 + 2.0 ** -8 - 2.0 ** -16 + 2.0 ** -17 - 2.0 ** -23
    gW = _run(x, gy, torch.ones(260, 516, device="cuda"))[1]
    assert torch.equal(gW, gy.T * x)


@pytest.mark.parametrize("M", [2, 3, 8, 31])
def test_short_sums(M):
    """At most 2^-24 of each product's size is left out, and three roundings follow: of h h', of the small parts' sum (2^-7 of it) and of the
    two together, 2^-24 each of no more than the sum of the products' sizes."""
    gen = torch.Generator(device="cuda").manual_seed(M)
    x, gy = (torch.randn(M, n, generator=gen, device="cuda") for n in (516, 260))
    x[:, 0] = gy[:, 0] = 1 + 2.0 ** -8 - 2.0 ** -16 + 2.0 ** -17 - 2.0 ** -23
    gW = _run(x, gy, torch.ones(260, 516, device="cuda"))[1]
    ref, size = gy.double().T @ x.double(), gy.double().abs().T @ x.double().abs()
    assert float(((gW.double() - ref).abs() / size).max()) <= 2.0 ** -24 * (3 + 2.0 ** -6) * (1 if M <= 16 else 2)

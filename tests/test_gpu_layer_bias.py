"""The layer's native autograd function: bias gradient from the projection's patch sums (pooled, unpooled, fp32 and
generic projections; ragged grids; tokens outside the grid), and what autograd asks of a function."""
import pytest
import torch

from _gpu_util import rel_fro, to_host
from paper_2309_15275_amd import binding
from paper_2309_15275_amd.autograd import LBPWHTLinear, _LbpWhtLinearFn, _LbpWhtLinearTokensFn, lbp_wht_linear

pytestmark = pytest.mark.gpu


def _tensors(shape, cout, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(shape, generator=g, device="cuda").to(dtype).requires_grad_()
    w = (0.1 * torch.randn(cout, shape[-1], generator=g, device="cuda")).to(dtype).requires_grad_()
    b = torch.randn(cout, generator=g, device="cuda").to(dtype).requires_grad_()
    gy = torch.randn(shape[:-1] + (cout,), generator=g, device="cuda").to(dtype)
    return x, w, b, gy


@pytest.mark.parametrize("patch,r", [(8, 8), (8, 21), (8, 64), (8, 40), (4, 3), (4, 16), (2, 2), (16, 5)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("grid", [None, (9, 13)])
def test_gradients_equal_the_python_function(patch, r, dtype, grid):
    shape = (3, 11, 16, 72) if grid is None else (5, 2 + 9 * 13, 72)
    x, w, b, gy = _tensors(shape, 136, dtype, r)
    idx = binding.select_bases(patch, r)
    y = lbp_wht_linear(x, w, b, patch, idx, grid)
    assert "LbpWhtLinearBackward" in y.grad_fn.name()
    y0 = (_LbpWhtLinearFn.apply(x, w, b, patch, idx) if grid is None else _LbpWhtLinearTokensFn.apply(x, w, b, patch, idx, grid))
    assert torch.equal(y, y0)
    got, want = torch.autograd.grad(y, (x, w, b), gy), torch.autograd.grad(y0, (x, w, b), gy)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    exact = gy.double().flatten(0, -2).sum(0)
    assert got[2].dtype == dtype and rel_fro(to_host(got[2]), exact.cpu().numpy()) <= (4e-3 if dtype == torch.bfloat16 else 1e-6)
    alone = torch.autograd.grad(lbp_wht_linear(x, w, b, patch, idx, grid), (b,), gy)[0]       # no product wanted
    assert rel_fro(to_host(alone), exact.cpu().numpy()) <= (4e-3 if dtype == torch.bfloat16 else 1e-6)


def test_many_patches_and_two_channel_blocks():
    x, w, b, gy = _tensors((300, 16, 16, 8), 24, torch.float32, 3)
    gb = torch.autograd.grad(lbp_wht_linear(x, w, b, 8, [0, 1]), b, gy, retain_graph=False)[0]
    y = lbp_wht_linear(x, w, b, 8, [0, 1])
    full = torch.autograd.grad(y, (x, w, b), gy)
    exact = gy.double().flatten(0, -2).sum(0).cpu().numpy()
    assert rel_fro(to_host(full[2]), exact) <= 1e-6 and rel_fro(to_host(gb), exact) <= 1e-6


def test_what_autograd_asks():
    layer = LBPWHTLinear(32, 48, patch=4, rank=4, device="cuda")
    x = torch.randn(2, 8, 8, 32, device="cuda")
    with torch.no_grad():
        assert not layer(x).requires_grad
    y = layer(x)                                        # x itself needs no gradient
    assert y.requires_grad and len(y.grad_fn.next_functions) == 3
    y.sum().backward()                                  # an expanded (not contiguous) output gradient
    assert x.grad is None and torch.allclose(layer.bias.grad, torch.full((48,), 128.0, device="cuda"))
    with pytest.raises(RuntimeError, match="second time"):
        y.sum().backward()
    y = layer(x)
    with torch.no_grad():
        layer.weight.mul_(2.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        y.sum().backward()
    xt = torch.randn(2, 32, 8, 8, device="cuda").permute(0, 2, 3, 1).requires_grad_()      # not contiguous
    assert torch.equal(layer(xt), layer(xt.detach().contiguous()))


@pytest.mark.parametrize("patch,r,cin,cout,dtype", [(8, 8, 72, 136, torch.bfloat16), (16, 5, 72, 136, torch.bfloat16),
                                                    (8, 1, 8, 2048, torch.float32), (2, 2, 16, 520, torch.float32)])
def test_bias_sums_lie_within_the_reported_workspace_or_what_a_caller_has(patch, r, cin, cout, dtype):
    x, w, b, gy = _tensors((5, 19, 16, cin), cout, dtype, r)
    idx = binding.select_bases(patch, r)
    shape = binding.LbpShape(5, 19, 16, cin, cout, int(dtype == torch.bfloat16), int(dtype == torch.bfloat16))
    want = torch.autograd.grad(lbp_wht_linear(x, w, b, patch, idx), (x, w, b), gy)
    rows, esz = binding.patch_count(5, 19, 16, patch) * r, x.element_size()
    least = sum(-(-n // 256) * 256 for n in (rows * cout * esz, rows * cin * esz, cout * cin * 4)) + (rows * cin * 4 if patch == 16 else 0)
    for size in (binding.workspace_bytes(shape, patch, r), least + 256):
        guard = torch.full((size + 4096,), 77, dtype=torch.uint8, device="cuda")
        binding.set_workspace(guard[:size])
        try:
            got = torch.autograd.grad(lbp_wht_linear(x, w, b, patch, idx), (x, w, b), gy)
            torch.cuda.synchronize()
        finally:
            binding.set_workspace(None)
        assert bool((guard[size:] == 77).all())
        for p, q in zip(got, want):      # sums in another order: one bf16 rounding (2^-8), a few fp32 ones (2^-24)
            assert rel_fro(to_host(p), to_host(q)) <= (4e-3 if dtype == torch.bfloat16 else 1e-6)


# rows of patch sums around what a workgroup takes at a time (128, 64 on thin layers), channels around its 16
@pytest.mark.parametrize("N, grid, extra, cin, cout, r", [(1, (8, 8), 0, 72, 8, 8), (1, (7, 5), 2, 128, 24, 4), (127, (8, 8), 0, 96, 136, 8),
                                                          (128, (8, 8), 1, 200, 40, 3), (129, (7, 7), 0, 264, 1032, 36), (33, (32, 32), 1, 136, 520, 2),
                                                          (65, (8, 8), 0, 48, 200, 8), (16, (33, 31), 1, 40, 72, 8), (64, (16, 16), 0, 768, 1536, 16)])
def test_bias_rows_are_added_up_beside_the_products(N, grid, extra, cin, cout, r):
    g = torch.Generator(device="cuda").manual_seed(N + cout)
    H, W = grid
    ints = lambda *s: torch.randint(-2, 3, s, generator=g, device="cuda").bfloat16()      # sums are exact in fp32
    x, gy = ints(N, extra + H * W, cin).requires_grad_(), ints(N, extra + H * W, cout)
    w, b = ints(cout, cin).requires_grad_(), ints(cout).requires_grad_()
    if not extra:
        x, gy = x.detach().view(N, H, W, cin).requires_grad_(), gy.view(N, H, W, cout)
    y = lbp_wht_linear(x, w, b, 8, binding.select_bases(8, r, "linf" if r == 16 else "l1"), grid if extra else None)
    got = torch.autograd.grad(y, (x, w, b), gy)[2]
    assert torch.equal(got, gy.double().flatten(0, -2).sum(0).bfloat16())


# Thousands of rows, whose sum depends on the order (2^20 and -2^20 among values of about 1: a partial sum keeps 3 binary places at
# times): where it is formed must not show, nor where the rows lie (on the projected input's place or behind everything, inside the reported
# workspace).  Patches 8 and 4, 64 and 128 rows of workgroup side by side, rows around multiples of 256.
@pytest.mark.parametrize("N, grid, extra, cin, cout, patch, r", [(2, (56, 56), 0, 48, 192, 8, 8), (3, (40, 44), 2, 136, 72, 4, 3), (64, (16, 16), 0, 96, 264, 8, 4),
                                                                 (31, (57, 55), 1, 40, 200, 4, 2), (41, (56, 56), 0, 192, 200, 8, 2), (86, (14, 14), 3, 256, 512, 4, 9)])
def test_the_sum_does_not_depend_on_who_adds_it_up(N, grid, extra, cin, cout, patch, r):
    H, W = grid
    x, w, b, gy = _tensors((N, extra + H * W, cin), cout, torch.bfloat16, cout)
    at = torch.randperm(N * (extra + H * W), generator=torch.Generator().manual_seed(r))[:60].cuda()
    flat = gy.view(-1, cout)
    flat[at[:30]], flat[at[30:]] = 2.0 ** 20, -2.0 ** 20
    idx = binding.select_bases(patch, r)

    def bias_gradient(group):
        binding.set_option("LBP_GEMM_GROUP", group)
        try:
            y = lbp_wht_linear(x, w, b, patch, idx, grid)
            return torch.autograd.grad(y, (x, w, b), gy)[2]
        finally:
            binding.set_option("LBP_GEMM_GROUP", None)

    shape = binding.LbpShape(N, H, W, cin, cout, 1, 1)
    assert "one grouped launch" in binding.describe_plan(shape, patch, idx, extra)
    want = bias_gradient(0)
    assert torch.equal(bias_gradient(None), want)
    size = binding.workspace_bytes(shape, patch, r, extra)
    guard = torch.full((size + 4096,), 77, dtype=torch.uint8, device="cuda")
    binding.set_workspace(guard[:size])
    try:
        assert torch.equal(bias_gradient(None), want)
        torch.cuda.synchronize()
    finally:
        binding.set_workspace(None)
    assert bool((guard[size:] == 77).all())


def test_without_memory_behind_the_products_the_sums_are_added_up_before_them():
    x, w, b, gy = _tensors((8, 256, 256, 512), 512, torch.bfloat16, 1)
    idx, shape = binding.select_bases(4, 1), binding.LbpShape(8, 256, 256, 512, 512, 1, 1)
    plan = binding.describe_plan(shape, 4, idx)
    assert "one grouped launch" in plan
    patches, products = binding.patch_count(8, 256, 256, 4), int(plan.split("workspace ")[1].split()[0])
    rows = patches * 512 * 4
    before, beside = max(products, patches * 512 * 2 + rows), products + rows      # bytes of either way, which the library rounds up by a quarter
    y = lbp_wht_linear(x, w, b, 4, idx)
    binding.release_workspace()
    want = torch.autograd.grad(y, (x, w, b), gy, retain_graph=True)
    got = [torch.empty_like(t) for t in want]      # (so that the second call's outputs are in torch's cache)
    del got
    binding.release_workspace()
    torch.cuda.synchronize()
    filler = None
    try:
        free = torch.cuda.mem_get_info()[0]
        leave = int(1.25 * (before + beside) / 2)
        filler = torch.empty(free - leave, dtype=torch.uint8, device="cuda")
        for _ in range(2):
            got = torch.autograd.grad(y, (x, w, b), gy, retain_graph=True)
            torch.cuda.synchronize()
            assert leave - torch.cuda.mem_get_info()[0] < 1.25 * beside
            for p, q in zip(got, want):
                assert torch.equal(p, q)
            del got, p, q
    finally:
        del filler
        torch.cuda.empty_cache()
        binding.release_workspace()

"""Launch shapes of small calls against the oracle: grouped and joined products of 4 x 4 patches, tiles that hold few
patches (low ranks), the exact backward's two products in one launch."""
import numpy as np
import pytest
import torch

import oracle
from _gpu_util import TOL, assert_matches, full_backward, rel_fro, to_device, to_host
from paper_2309_15275_amd import binding, workloads

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


# (N, H, W, extra, Cin, Cout, patch, r)
CASES = [(2, 7, 7, 1, 200, 480, 4, 6), (3, 8, 12, 0, 48, 72, 4, 16), (1, 9, 5, 0, 136, 2064, 4, 3), (6, 26, 26, 0, 264, 88, 4, 5),
         (1, 16, 16, 1, 72, 1032, 4, 1), (20, 34, 34, 0, 136, 112, 8, 2), (3, 15, 17, 1, 264, 136, 8, 1), (9, 8, 8, 0, 56, 520, 8, 3),
         (40, 12, 12, 0, 136, 520, 4, 2)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_backward(case):
    N, H, W, extra, cin, cout, patch, r = case
    idx = oracle.select_bases(patch, r, "l1").tolist()
    x, gy, w = _inputs(N, extra + H * W, cin, cout, 70 + r)
    gx0, gW0 = oracle.lbp_wht_backward_tokens(x, gy, w, (H, W), patch, idx)
    dx, dgy, dw = (to_device(v, "bf16") for v in (x, gy, w))
    assert "one grouped launch" in binding.describe_plan(binding.LbpShape(N, H, W, cin, cout, 1, 0), patch, idx, extra=extra)
    for join in (None, "1", "3"):
        binding.set_option("LBP_GX_JOIN", join)
        gx = torch.full_like(dx, float("nan"))
        gW = torch.full(dw.shape, float("nan"), device="cuda")
        binding.lbp_wht_backward_tokens(dx, dgy, dw, (H, W), patch, idx, gx=gx, gW=gW)
        assert_matches(gx, gx0, TOL["bf16"], "gx")
        assert_matches(gW, gW0, TOL["bf16"], "gW")
        alone = binding.lbp_wht_backward_tokens(dx, dgy, dw, (H, W), patch, idx, want_gw=False)[0]
        assert_matches(alone, gx0, TOL["bf16"], "gx alone")


@pytest.mark.parametrize("M,cin,cout", [(9, 56, 64), (100, 72, 2056), (1500, 136, 88), (3000, 264, 520)])
@pytest.mark.parametrize("gw_dtype", [torch.float32, torch.bfloat16])
def test_exact_backward_in_one_launch(M, cin, cout, gw_dtype):
    x, gy, w = _inputs(1, M, cin, cout, M)
    dev = {k: to_device(v, "bf16") for k, v in (("x", x.reshape(1, 1, M, cin)), ("gy", gy.reshape(1, 1, M, cout)), ("w", w))}
    gx, gW = full_backward(dev, gw_dtype)
    assert rel_fro(to_host(gx).reshape(M, cin), gy[0].astype(np.float64) @ w) <= 4e-3
    assert rel_fro(to_host(gW), gy[0].astype(np.float64).T @ x[0]) <= (4e-3 if gw_dtype == torch.bfloat16 else 1e-5)
    binding.set_option("LBP_GEMM_GROUP", "0")
    gx1, gW1 = full_backward(dev, gw_dtype)
    assert rel_fro(to_host(gx1), to_host(gx)) <= 4e-3 and rel_fro(to_host(gW1), to_host(gW)) <= 4e-3

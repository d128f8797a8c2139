"""Projection onto more than 32 bases: workgroups with one item, several, a last one with fewer, and both tensors in one launch."""
import numpy as np
import pytest
import torch

from paper_2309_15275_amd import binding

pytestmark = pytest.mark.gpu


def _signs(idx):
    h = np.array([[1.0]])
    while len(h) < 8:
        h = np.block([[h, h], [h, -h]])
    walsh = h[np.argsort((np.diff(h, axis=1) != 0).sum(axis=1), kind="stable")]
    return torch.tensor(np.stack([np.outer(walsh[k // 8], walsh[k % 8]).reshape(-1) for k in idx]), device="cuda")


# (images, H, W, Cin, Cout): items of 128 channels of a patch below, at and above one round of 1024 workgroups, 8190 (8 each at most) and 8307
# (past 8 each: workgroups as for fewer bases)
@pytest.mark.parametrize("N, H, W, cin, cout", [(1, 8, 8, 8, 128), (31, 16, 16, 136, 904), (32, 16, 16, 128, 896), (33, 16, 15, 256, 1024), (70, 21, 24, 320, 1160), (71, 21, 24, 320, 1160)])
@pytest.mark.parametrize("r", [33, 36, 64])
def test_every_item_once(N, H, W, cin, cout, r):
    gen = torch.Generator(device="cuda").manual_seed(N + r)
    x, gy = (torch.randint(-2, 3, (N, H, W, c), generator=gen, device="cuda").bfloat16() for c in (cin, cout))
    idx = list(range(63, 63 - r, -1))
    sign = _signs(idx)
    got = binding.wht_project_pair(x, gy, 8, idx)
    for t, out in ((x, got[0]), (gy, got[1])):
        ph, pw = -(-H // 8), -(-W // 8)
        p = torch.nn.functional.pad(t.double(), (0, 0, 0, pw * 8 - W, 0, ph * 8 - H)).view(N, ph, 8, pw, 8, -1)
        want = torch.matmul(sign, p.permute(0, 1, 3, 2, 4, 5).reshape(N * ph * pw, 64, -1).contiguous())
        assert torch.equal(out.view(N * ph * pw, r, -1), want.bfloat16())       # whole numbers below 256: exact

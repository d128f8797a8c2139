"""Projections of launches around whole runs of workgroups an XCD (8 runs of 64), rows of whole 128-byte lines and others, both tensors."""
import numpy as np
import pytest
import torch

from paper_2309_15275_amd import binding

pytestmark = pytest.mark.gpu


def _walsh(p):
    h = np.array([[1.0]])
    while len(h) < p:
        h = np.block([[h, h], [h, -h]])
    return h[np.argsort((np.diff(h, axis=1) != 0).sum(axis=1), kind="stable")]


def _coefficients(t, p, idx):
    N, H, W, C = t.shape
    walsh, ph, pw = _walsh(p), -(-H // p), -(-W // p)
    sign = torch.tensor(np.stack([np.outer(walsh[k // p], walsh[k % p]).reshape(-1) for k in idx]), device="cuda")
    tokens = torch.nn.functional.pad(t.double(), (0, 0, 0, pw * p - W, 0, ph * p - H)).view(N, ph, p, pw, p, C)
    return torch.matmul(sign, tokens.permute(0, 1, 3, 2, 4, 5).reshape(N * ph * pw, p * p, C).contiguous())


# (images, H, W, channels of either tensor, patch, bases, type): workgroups of the first tensor 508, 512, 516, 1032, 511 and 1100 in the register
# form, 512, 510, 768 and 1024 in the matrix-core one
@pytest.mark.parametrize("N, H, W, c0, c1, patch, r, dtype", [
    (4, 64, 64, 1016, 40, 8, 8, torch.bfloat16), (4, 64, 64, 1024, 48, 8, 4, torch.bfloat16), (4, 64, 64, 1032, 1024, 8, 9, torch.bfloat16),
    (2, 60, 60, 2352, 264, 4, 7, torch.bfloat16), (4, 57, 64, 511, 512, 8, 3, torch.float32), (11, 40, 40, 1024, 1028, 8, 10, torch.float32),
    (4, 64, 64, 136, 64, 8, 20, torch.bfloat16), (1, 120, 136, 136, 1024, 8, 24, torch.bfloat16), (4, 64, 64, 264, 384, 8, 36, torch.bfloat16),
    (4, 64, 59, 392, 128, 8, 15, torch.bfloat16)])
def test_every_workgroup_has_a_place(N, H, W, c0, c1, patch, r, dtype):
    if dtype == torch.float32:
        c0 = c0 // 4 * 4
    gen = torch.Generator(device="cuda").manual_seed(r)
    ts = [torch.randint(-2, 3, (N, H, W, c), generator=gen, device="cuda").to(dtype) for c in (c0, c1)]
    idx = binding.select_bases(patch, r, "l1")
    for t, out in zip(ts, binding.wht_project_pair(ts[0], ts[1], patch, idx)):
        want = _coefficients(t, patch, idx)
        assert torch.equal(out.view(want.shape), want.to(dtype))       # whole numbers below 256: exact


# the energy's loads: rows of whole lines and others
@pytest.mark.parametrize("C", [8, 64, 72, 128, 136, 192])
@pytest.mark.parametrize("patch", [2, 4, 8])
def test_energy_of_either_kind_of_rows(C, patch):
    gen = torch.Generator(device="cuda").manual_seed(C + patch)
    t = torch.randint(-2, 3, (3, 21, 24, C), generator=gen, device="cuda").bfloat16()
    want = _coefficients(t, patch, range(patch * patch)).square().sum(dim=(0, 2))
    assert torch.equal(torch.as_tensor(binding.wht_energy(t, patch)).double().cuda().view(-1), want)      # sums below 2^24: exact

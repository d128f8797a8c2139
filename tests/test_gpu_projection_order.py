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


def _workgroups(Q, channels, other, r, dtype, matrix_cores):
    """Of the first tensor of a launch of two."""
    if not matrix_cores:
        return -(-Q * channels // (512 if dtype == torch.bfloat16 else 256))
    items = Q * (-(-channels // 128) + -(-other // 128))
    one_round = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    share = -(-items // one_round) if r > 32 and items <= 8 * one_round else min(8, -(-items // 4096))
    return -(-Q * -(-channels // 128) // share)


# (images, H, W, channels of either tensor, patch, bases, type, workgroups of the first tensor on 256 units): one fewer than the 512 of 8 runs, those, one
# more, two times that and some; more than 32 bases; several items a workgroup; rows of whole 128-byte lines (1024 and 768 channels), narrow rows
# on hanging patches
@pytest.mark.parametrize("N, H, W, c0, c1, patch, r, dtype, workgroups", [
    (64, 8, 8, 4088, 40, 8, 8, torch.bfloat16, 511), (101, 8, 8, 2592, 48, 8, 4, torch.bfloat16, 512), (64, 8, 8, 4104, 1024, 8, 9, torch.bfloat16, 513),
    (4, 64, 64, 1024, 264, 8, 4, torch.bfloat16, 512), (171, 16, 8, 768, 48, 8, 3, torch.bfloat16, 513), (517, 8, 8, 1016, 56, 8, 2, torch.bfloat16, 1026),
    (2, 60, 60, 2352, 264, 4, 7, torch.bfloat16, 2068), (129, 16, 8, 508, 512, 8, 3, torch.float32, 512), (11, 40, 40, 1024, 1028, 8, 10, torch.float32, 1100),
    (37, 43, 45, 504, 136, 8, 10, torch.bfloat16, 1312), (37, 43, 45, 520, 72, 8, 4, torch.bfloat16, 1353), (29, 27, 26, 252, 128, 4, 5, torch.float32, 1399),
    (511, 8, 8, 72, 64, 8, 20, torch.bfloat16, 511), (4, 64, 64, 136, 64, 8, 20, torch.bfloat16, 512), (1, 216, 152, 72, 64, 8, 24, torch.bfloat16, 513),
    (4, 64, 64, 1032, 1032, 8, 24, torch.bfloat16, 1152), (4, 64, 59, 520, 128, 8, 15, torch.bfloat16, 1280), (4, 64, 64, 392, 64, 8, 36, torch.bfloat16, 512),
    (16, 64, 64, 1032, 72, 8, 40, torch.bfloat16, 3072)])
def test_every_workgroup_has_a_place(N, H, W, c0, c1, patch, r, dtype, workgroups):
    idx = binding.select_bases(patch, r, "l1")
    matrix_cores = "matrix-core" in binding.describe_plan(binding.LbpShape(N, H, W, c0, c1, int(dtype == torch.bfloat16), 0), patch, idx).split("(")[0]
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert _workgroups(N * -(-H // patch) * -(-W // patch), c0, c1, r, dtype, matrix_cores) == workgroups
    gen = torch.Generator(device="cuda").manual_seed(r)
    ts = [torch.randint(-2, 3, (N, H, W, c), generator=gen, device="cuda").to(dtype) for c in (c0, c1)]
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

"""The one-pass energy kernels against the oracle at the edges of their items: patch counts that do not fill an item,
channel counts that do not fill a chunk, ragged grids, one workgroup with several items."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_15275_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("patch,N,H,W,C", [(8, 1, 7, 7, 8), (8, 3, 9, 17, 136), (8, 5, 16, 24, 120), (8, 300, 16, 16, 520),
                                           (4, 1, 4, 4, 8), (4, 3, 5, 9, 136), (4, 70, 18, 15, 264), (2, 1, 3, 5, 8), (2, 5, 7, 6, 264)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_energy_at_item_edges(patch, N, H, W, C, dtype):
    g = torch.Generator().manual_seed(N * 1000 + C)
    t = torch.randn(N, H, W, C, generator=g).to(dtype)
    want = oracle.wht_energy_padded(t.float().numpy(), patch)
    got = binding.wht_energy(t.cuda(), patch)
    # squares of fp32 coefficients of the stored values; sums in double
    np.testing.assert_allclose(got.cpu().numpy(), want, rtol=2e-6)
    assert torch.equal(binding.wht_energy(t.cuda(), patch), got)
    twice = binding.wht_energy(t.cuda(), patch, energy=got.clone())
    np.testing.assert_allclose(twice.cpu().numpy(), 2 * want, rtol=2e-6)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("patch", [2, 4, 8])
def test_small_tensors_need_little_of_a_callers_workspace(patch, dtype):
    # never more than the coefficients themselves would take
    t = torch.randn(2, 19, 16, 24, device="cuda").to(dtype)
    want = binding.wht_energy(t, patch)
    size = -(-binding.patch_count(2, 19, 16, patch) * patch * patch * 24 * t.element_size() // 256) * 256
    buf = torch.full((size + 4096,), 77, dtype=torch.uint8, device="cuda")
    binding.set_workspace(buf[:size])
    try:
        got = binding.wht_energy(t, patch)
        torch.cuda.synchronize()
    finally:
        binding.set_workspace(None)
    assert torch.equal(got, want) and bool((buf[size:] == 77).all())


def test_fp32_sums_of_a_large_tensor_stay_short():
    # 64 items a lane, the first of each with 2^26 times the energy of the others: one fp32 sum would lose the other 63
    # (9e-7 of the result), sums of 8 lose the 7 that share its sum
    t = torch.full((128, 64, 64, 256), 0.25, device="cuda")
    t.view(128, 16, 4, 64, 256)[:, :, :2, :2] = 2.0 ** 11
    got = binding.wht_energy(t, 2).cpu()
    want = 2048 * 256 * (2.0 ** 26 + 63)
    assert abs(float(got[0]) - want) <= 7 * 2.0 ** -26 * want and not got[1:].any()


def test_fp32_lanes_with_ten_items():
    # more than 8 items a lane, the last of them not in every lane, ragged grids
    t = torch.randn(9, 63, 65, 520, device="cuda")
    p = torch.nn.functional.pad(t.double(), (0, 0, 0, 1, 0, 1)).view(9, 32, 2, 33, 2, 520)
    h = p[:, :, 0] + p[:, :, 1], p[:, :, 0] - p[:, :, 1]
    want = torch.stack([(c[:, :, :, 0] + s * c[:, :, :, 1]).square().sum() for c in h for s in (1, -1)])
    np.testing.assert_allclose(binding.wht_energy(t, 2).cpu().numpy(), want.cpu().numpy(), rtol=2e-6)


# workgroups of a launch: 1, 2, 31 to 33 (a group of arrivals and its edges), 64, 65, 1024 (bf16: one item each up to 1024)
@pytest.mark.parametrize("items", [1, 2, 31, 32, 33, 64, 65, 1000, 1024, 1025])
@pytest.mark.parametrize("patch,dtype", [(8, torch.bfloat16), (4, torch.bfloat16), (2, torch.bfloat16), (8, torch.float32), (2, torch.float32)])
def test_last_workgroups_add_up(items, patch, dtype):
    """Whole numbers: every sum is exact in any order.  Several calls in a row, eager and from a graph, leave the counters as found."""
    side = 8                                                                    # 64 tokens x 128 channels an item, 256 lanes a workgroup
    N, C = (items, 128) if dtype == torch.bfloat16 else (items, 256 * patch * patch // 64)
    g = torch.Generator().manual_seed(items)
    t = torch.randint(-1, 2, (N, side, side, C), generator=g).to(dtype).cuda()
    p = t.double().view(N, side // patch, patch, side // patch, patch, C).permute(0, 1, 3, 2, 4, 5).reshape(-1, patch, patch, C)
    had = torch.tensor(_walsh(patch), dtype=torch.float64, device="cuda")
    coef = torch.tensordot(had, torch.tensordot(had, p, dims=([1], [1])), dims=([1], [2]))       # [v, u, ...]
    want = coef.square().sum(dim=(2, 3)).T.reshape(-1)
    got = binding.wht_energy(t, patch)
    assert torch.equal(got, want)
    graph, total = torch.cuda.CUDAGraph(), torch.zeros_like(got)
    with torch.cuda.graph(graph):
        binding.wht_energy(t, patch, energy=total)
    for k in range(1, 4):
        graph.replay()
        assert torch.equal(binding.wht_energy(t, patch), want)
        assert torch.equal(total, k * want)


def _whole_numbers(N, C, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(-1, 2, (N, 16, 16, C), generator=g).to(torch.bfloat16).cuda()


def test_calls_on_two_streams_with_two_workspaces_are_independent():
    """Nothing orders the two streams: each call counts the workgroups of its own launch only.  Whole numbers, exact in any order."""
    t = [_whole_numbers(64, 768, 1), _whole_numbers(24, 1032, 2)]           # launches of 768 and 864 workgroups
    want = [binding.wht_energy(v, 8) for v in t]
    buf = [torch.empty(1 << 20, dtype=torch.uint8, device="cuda") for _ in t]
    out = [[torch.zeros(64, dtype=torch.float64, device="cuda") for _ in range(40)] for _ in t]
    streams = [torch.cuda.Stream() for _ in t]
    torch.cuda.synchronize()
    try:
        for i in range(40):
            for v, b, s, o in zip(t, buf, streams, out):
                binding.set_workspace(b)
                with torch.cuda.stream(s):
                    binding.wht_energy(v, 8, energy=o[i])
        torch.cuda.synchronize()
    finally:
        binding.set_workspace(None)
    for w, o in zip(want, out):
        assert all(torch.equal(e, w) for e in o)


@pytest.mark.parametrize("patch", [2, 4, 8])
def test_more_workspaces_than_sets_of_counters(patch):
    """The sums then meet in launches of their own, in the same order: the same bits, also from a graph.  (The last test of this file: the
    sets of a process are given out for good.)"""
    pool = torch.empty(40 << 20, dtype=torch.uint8, device="cuda")
    # 1 workgroup, a few, groups of 32 and one more, many groups, for both types
    ts = [torch.randn(n, 24, 16, c, device="cuda").to(dt) for n, c in ((1, 8), (2, 136), (11, 264), (37, 520), (40, 776))
          for dt in (torch.bfloat16, torch.float32)]
    want = [binding.wht_energy(t, patch) for t in ts]
    try:
        for k in range(40):
            binding.set_workspace(pool[k << 20:(k + 1) << 20])
            for t, w in zip(ts, want):
                assert torch.equal(binding.wht_energy(t, patch), w), (k, t.shape, t.dtype)
        graph, total = torch.cuda.CUDAGraph(), torch.zeros_like(want[-2])
        with torch.cuda.graph(graph):
            binding.wht_energy(ts[-2], patch, energy=total)
        for k in range(1, 4):
            total.zero_()
            graph.replay()
            assert torch.equal(total, want[-2])
            assert torch.equal(binding.wht_energy(ts[-2], patch), want[-2])
        torch.cuda.synchronize()
    finally:
        binding.set_workspace(None)


def _walsh(p):
    """Rows by number of sign changes."""
    h = np.array([[1.0]])
    while len(h) < p:
        h = np.block([[h, h], [h, -h]])
    return h[np.argsort((np.diff(h, axis=1) != 0).sum(axis=1), kind="stable")]

"""GPU: the list copies (a client's refresh, scattered and by segments) on both
sides of each change of form and at the edges of a block, a wave's run and the
64 entries that a segment loads ahead, against torch's index assignment."""
import pytest

import paper_1601_04033_amd as fa
from helpers import gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 255, 256, 257, 2047, 2048, 2049, 4099, 10_000_000, 10_000_001, 40_000_000, 40_000_001])
@pytest.mark.parametrize("density", [0.0, 0.01, 0.25, 1.0])
def test_list_copies(P, density):
    import torch
    dev = gpu()
    gen = torch.Generator(device=dev).manual_seed(P)
    copy = torch.randn(P, device=dev, generator=gen)
    listed = torch.nonzero(torch.rand(P, device=dev, generator=gen) < density).reshape(-1)
    m = listed.numel()
    idx = torch.cat([listed.int(), torch.zeros(3, device=dev, dtype=torch.int32)])   # entries past the count
    val = torch.randn(m + 3, device=dev, generator=gen)
    cnt = torch.full((1,), m, device=dev, dtype=torch.int64)
    edges = torch.arange(fa.bfasgd_list_index_length(P), device=dev) * 256
    seg = torch.searchsorted(listed, edges.clamp_(max=P)).int()
    want = copy.clone()
    want[listed] = val[:m]
    for index in (None, seg):
        got = copy.clone()
        fa.bfasgd_apply_fetch(got, idx, val, cnt, seg_start=index)
        assert torch.equal(got, want), (P, density, index is not None)
    if m > 1:                                    # the capacity cuts the list
        cut = m // 2
        want = copy.clone()
        want[listed[:cut]] = val[:cut]
        for index in (None, seg):
            got = copy.clone()
            fa.bfasgd_apply_fetch(got, idx[:cut].contiguous(), val[:cut].contiguous(), cnt, seg_start=index)
            assert torch.equal(got, want), (P, density, index is not None, "cut")


@pytest.mark.parametrize("P", [1_499_999, 1_500_000, 1_500_001])
def test_scattered_copies_around_one_entry_per_lane(P):
    import torch
    dev = gpu()
    gen = torch.Generator(device=dev).manual_seed(P)
    copy = torch.randn(P, device=dev, generator=gen)
    for m in (1, 63, 64, 65, 255, 256, 257, P // 3):
        listed = torch.randperm(P, device=dev, generator=gen)[:m]
        val = torch.randn(m, device=dev, generator=gen)
        got, want = copy.clone(), copy.clone()
        want[listed] = val
        fa.bfasgd_apply_fetch(got, listed.int(), val, torch.full((1,), m, device=dev, dtype=torch.int64))
        assert torch.equal(got, want), m


@pytest.mark.parametrize("P", [1_500_001, 30_000_000, 30_000_001, 150_000_000, 150_000_001])
def test_cached_push_without_an_index(P):
    """A push whose list is copied into the client's cache ahead of the pass, where the copy's form changes: the cache
    against torch's index assignment, the state against the push with the index, which merges the list in the pass."""
    import torch
    from helpers import new_gpu_state
    dev = gpu()
    gen = torch.Generator(device=dev).manual_seed(P)
    listed = torch.nonzero(torch.rand(P, device=dev, generator=gen) < 0.02).reshape(-1)
    m = listed.numel()
    val = torch.randn(m, device=dev, generator=gen)
    theta0, cache0 = torch.randn(P, device=dev, generator=gen), torch.randn(P, device=dev, generator=gen)
    cnt = torch.full((1,), m, device=dev, dtype=torch.int64)
    edges = torch.arange(fa.bfasgd_list_index_length(P), device=dev) * 256
    seg = torch.searchsorted(listed, edges.clamp_(max=P)).int()
    out = []
    for index in (None, seg):
        st, cache = new_gpu_state(theta0, dev, 4, 0.005, fa.MATH_FAST, v0=3.0), cache0.clone()
        fa.bfasgd_apply_cached(st, listed.int(), val, cnt, cache, 1, 0, seg_start=index)
        out.append([st.tensors[n].view(torch.int32) for n in ("theta", "n", "b", "v")] + [cache])
    for x, y in zip(*out):
        assert torch.equal(x, y)
    cache0[listed] = val
    assert torch.equal(out[0][-1], cache0)

"""GPU: the selection in three launches (every scatter wave sums the totals of
the groups of tiles before its own) against the same vector selected in
shards that take two launches, bit for bit: where one load per lane covers
the groups, one group past it, and a count that exceeds the capacity."""
import pytest

import paper_1601_04033_amd as fa
from helpers import gpu, new_gpu_state

pytestmark = pytest.mark.gpu
GROUP = 1024 * 1024       # parameters per group of tiles
SHARD = 45 * GROUP


@pytest.mark.parametrize("P,share", [(49 * GROUP + 5, 0.5), (64 * GROUP, 0.5), (65 * GROUP + 1, 0.5),
                                     (256 * GROUP, 0.12), (257 * GROUP + 1029, 0.12), (60 * GROUP, 0.05)])
def test_three_launches_equal_shards(P, share):
    import torch
    dev = gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(P)
    v = torch.rand(P, device=dev, generator=gen) * 95 + 5
    grad = torch.randn(P, device=dev, generator=gen)
    cap = int(P * share)

    def select(lo, hi, base, cap):
        st = new_gpu_state(grad[lo:hi], dev, 16, 0.005, fa.MATH_FAST)
        st.tensors["v"].copy_(v[lo:hi])
        st.c.index_base, st.c.T = base, 77
        idx = torch.full((cap,), -7, device=dev, dtype=torch.int32)
        val = torch.zeros(cap, device=dev)
        cnt = torch.zeros(1, device=dev, dtype=torch.int64)
        seg = torch.zeros(fa.bfasgd_list_index_length(hi - lo), device=dev, dtype=torch.int32)
        ws = torch.full((fa.bfasgd_workspace_bytes(hi - lo),), 0xA5, device=dev, dtype=torch.uint8)
        fa.bfasgd_select_compact(st, grad[lo:hi], 400.0, 1e-8, 5, 77, 3, idx, val, cnt, ws, seg_start=seg)
        return idx, val, int(cnt.item()), seg

    idx, val, m, seg = select(0, P, 0, cap)
    at = 0
    for lo in range(0, P, SHARD):
        hi = min(P, lo + SHARD)
        i, x, k, s = select(lo, hi, lo, hi - lo)
        n = max(0, min(k, cap - at))
        assert torch.equal(idx[at:at + n], i[:n] + lo)
        assert torch.equal(val[at:at + n].view(torch.int32), x[:n].view(torch.int32))
        assert torch.equal(seg[lo // 256:lo // 256 + s.numel() - 1], s[:-1] + at)
        at += k
    assert m == at == int(seg[-1])
    assert (m > cap) == (share == 0.05)
    if m < cap:
        assert bool((idx[m:] == -7).all())

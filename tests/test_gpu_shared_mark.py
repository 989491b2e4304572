"""GPU: pushes of a batch marked together (from 4M parameters on, groups of 4)
against single selections, bit for bit: batches that fill a group, spill into
a last group of one and of three, odd sizes, a tile whose global chunk indexes
cross a multiple of 2^32, and sizes beyond the two-launch form."""
import numpy as np
import pytest

import paper_1601_04033_amd as fa
from helpers import gpu, new_gpu_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,B,index_base", [
    (4_000_000, 2, 0),
    (4_000_003, 4, 0),
    (4_100_000, 5, 4 * (2**32 - 700)),      # chunk 700 of the vector is global chunk 2^32
    (5_000_001, 7, 4 * 2**33),
    (26_000_002, 3, 0),                     # blocks of 16 tiles
    (51_000_001, 3, 0),                     # mark, scan, scatter
])
def test_pushes_marked_together_equal_single_selections(P, B, index_base):
    import torch
    dev = gpu()
    st = new_gpu_state(np.zeros(P, dtype=np.float32), dev, 16, 0.005, fa.MATH_FAST)
    st.c.index_base = index_base
    gen = torch.Generator(device=dev)
    gen.manual_seed(P)
    st.tensors["v"].copy_(torch.rand(P, device=dev, generator=gen) * 95 + 5)
    grads = [torch.randn(P, device=dev, generator=gen) for _ in range(B)]
    st.c.T = 500
    T, clients = [500 + 3 * b for b in range(B)], [(5 * b) % 16 for b in range(B)]
    cap, L = P // 3, fa.bfasgd_list_index_length(P)

    def buffers(rows):
        return (torch.full((rows, cap), -7, device=dev, dtype=torch.int32), torch.zeros(rows, cap, device=dev),
                torch.zeros(rows, device=dev, dtype=torch.int64), torch.zeros(rows, L, device=dev, dtype=torch.int32))

    wsb = fa.bfasgd_workspace_bytes(P)
    idx, val, cnt, seg = buffers(B)
    # the workspace's previous contents do not matter
    ws = torch.full((B * wsb,), 0xA5, device=dev, dtype=torch.uint8)
    fa.bfasgd_select_compact_batch(st, grads, 150.0, 1e-8, 99, T, clients, idx, val, cnt, ws, seg_start=seg)
    i1, v1, c1, s1 = buffers(1)
    w1 = torch.empty(wsb, device=dev, dtype=torch.uint8)
    for b in range(B):
        i1.fill_(-7)
        v1.zero_()
        fa.bfasgd_select_compact(st, grads[b], 150.0, 1e-8, 99, T[b], clients[b], i1[0], v1[0], c1, w1, seg_start=s1[0])
        torch.cuda.synchronize()
        assert int(cnt[b]) == int(c1[0]) > 0
        for x, y in ((idx[b], i1[0]), (val[b].view(torch.int32), v1[0].view(torch.int32)), (seg[b], s1[0])):
            assert torch.equal(x, y), b

"""GPU: the sparse apply on both sides of each change of its form (3M and 16M
parameters) and at the ends of a wave's run of entries, in ascending and
shuffled lists with indices outside [0, P): listed parameters equal a dense
pass with the same gradient bit for bit, the others keep every bit."""
import numpy as np
import pytest

import paper_1601_04033_amd as fa
from helpers import gpu, new_gpu_state, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [fa.MATH_FAST, fa.MATH_IEEE])
@pytest.mark.parametrize("P", [1000, 3_000_000, 3_000_001, 16_000_000, 16_000_001])
def test_sparse_apply_forms(P, mode):
    import torch
    dev = gpu()
    gen = torch.Generator(device=dev).manual_seed(P)
    theta0 = torch.randn(P, device=dev, generator=gen)
    grad = torch.randn(P, device=dev, generator=gen)

    def server():
        st = new_gpu_state(theta0, dev, 4, 0.005, mode)
        st.v.fill_(3.0)
        st.c.T, st.c.dense_T = 20, 19
        return st

    dense = server()
    fa.fasgd_apply_updates(dense, [grad], [1], [5])
    rng = np.random.default_rng(P + mode)
    counts = [0, 1, 127, 128, 129, 383, 384, 385] + ([P] if P == 1000 else [P // 9, P // 2])
    for m, shuffled in [(m, s) for m in counts for s in (False, True)]:
        m = min(m, P)
        listed = torch.randperm(P, device=dev, generator=gen)[:m]
        if not shuffled:
            listed = listed.sort().values
        idx, val = listed.int(), grad[listed]
        # entries that name no parameter, one of them past the count
        out = torch.tensor([-1, P, 2 ** 31 - 1, 0], device=dev, dtype=torch.int32)
        at = int(rng.integers(0, m + 1))
        idx = torch.cat([idx[:at], out[:3], idx[at:], out[3:]])
        val = torch.cat([val[:at], val.new_ones(3), val[at:], val.new_ones(1)])
        st = server()
        fa.bfasgd_apply_sparse(st, idx, val, torch.full((1,), m + 3, device=dev, dtype=torch.int64), 1, 5)
        fresh = server()
        for name in ("theta", "n", "b", "v", "last_T"):
            got, was = st.tensors[name], fresh.tensors[name]
            want = was.clone()
            want[listed] = 20 if name == "last_T" else dense.tensors[name][listed]
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)), (name, m, shuffled)
        assert st.T == 21
    # the capacity cuts the list before the count does
    idx = torch.arange(P, device=dev, dtype=torch.int32)[: 500]
    st = server()
    fa.bfasgd_apply_sparse(st, idx, grad[:500].contiguous(), torch.full((1,), P, device=dev, dtype=torch.int64), 1, 5)
    assert torch.equal(st.theta[:500], dense.theta[:500]) and torch.equal(st.theta[500:], theta0[500:])


@pytest.mark.parametrize("mode", [fa.MATH_FAST, fa.MATH_IEEE])
@pytest.mark.parametrize("m", [196_607, 196_608, 196_609, 300_001])
@pytest.mark.parametrize("room", ["exact", "whole"])
def test_sparse_apply_around_a_short_list(m, mode, room):
    """Beyond 16M parameters, lists on both sides of 512 runs of 384 entries, in buffers of their own length and of P."""
    import torch
    dev = gpu()
    P = 16_000_001
    gen = torch.Generator(device=dev).manual_seed(m)
    theta0 = torch.randn(P, device=dev, generator=gen)
    grad = torch.randn(P, device=dev, generator=gen)

    def server():
        st = new_gpu_state(theta0, dev, 4, 0.005, mode)
        st.v.fill_(3.0)
        st.c.T, st.c.dense_T = 20, 19
        return st

    dense, st, fresh = server(), server(), server()
    fa.fasgd_apply_updates(dense, [grad], [1], [5])
    listed = torch.randperm(P, device=dev, generator=gen)[:m].sort().values
    idx = torch.zeros(m if room == "exact" else P, device=dev, dtype=torch.int32)
    val = torch.zeros(idx.numel(), device=dev)
    idx[:m], val[:m] = listed.int(), grad[listed]
    fa.bfasgd_apply_sparse(st, idx, val, torch.full((1,), m, device=dev, dtype=torch.int64), 1, 5)
    for name in ("theta", "n", "b", "v", "last_T"):
        want = fresh.tensors[name].clone()
        want[listed] = 20 if name == "last_T" else dense.tensors[name][listed]
        assert torch.equal(st.tensors[name].view(torch.int32), want.view(torch.int32)), name

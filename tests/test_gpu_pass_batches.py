"""GPU: the dense passes at the edges of their gradient batches (the remainder
after the last whole batch, the sizes where the batch changes) against the
same gradients applied one pass each, bit for bit; synchronous SGD against
SASGD on the divided gradients."""
import numpy as np
import pytest

import paper_1601_04033_amd as fa
from helpers import gpu, new_gpu_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [77, 500_000, 500_001, 2_000_000, 2_000_001])
@pytest.mark.parametrize("rule", ["fast", "ieee", "sasgd"])
def test_pass_equals_one_pass_per_gradient(P, rule):
    import torch
    dev = gpu()
    lam = 4
    gen = torch.Generator(device=dev)
    gen.manual_seed(P)
    theta0 = np.random.default_rng(P).standard_normal(P, dtype=np.float32)
    grads = [torch.randn(P, device=dev, generator=gen) * 1e-2 for _ in range(13)]
    apply = fa.sasgd_apply_updates if rule == "sasgd" else fa.fasgd_apply_updates
    mode = fa.MATH_IEEE if rule == "ieee" else fa.MATH_FAST
    for K in (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 13):
        one = new_gpu_state(theta0, dev, lam, 0.005, mode)
        each = new_gpu_state(theta0, dev, lam, 0.005, mode)
        for st in (one, each):
            st.c.T, st.c.dense_T = 50, 49
        clients, ts = [k % lam for k in range(K)], [50 + k - 3 * (k % 5) for k in range(K)]
        apply(one, grads[:K], clients, ts)
        for k in range(K):
            apply(each, grads[k:k + 1], clients[k:k + 1], ts[k:k + 1])
        torch.cuda.synchronize()
        assert one.T == each.T == 50 + K
        for name in ("theta", "n", "b", "v"):
            x, y = one.tensors[name], each.tensors[name]
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), (name, K)


@pytest.mark.parametrize("lam", [1, 2, 3, 5, 7])
def test_sync_step_equals_sasgd_on_divided_gradients(lam):
    import torch
    dev = gpu()
    P = 1033
    theta0 = np.random.default_rng(lam).standard_normal(P, dtype=np.float32)
    grads = [torch.randn(P, device=dev) for _ in range(lam)]
    sync = new_gpu_state(theta0, dev, lam, 0.04, fa.MATH_IEEE)
    plain = new_gpu_state(theta0, dev, lam, 0.04, fa.MATH_IEEE)
    fa.sgd_sync_apply(sync, grads, 0.04)
    # divided on the host, correctly rounded (torch divides by a scalar on the GPU by multiplying with 1 / lam)
    divided = [(g.cpu() / lam).to(dev) for g in grads]
    fa.sasgd_apply_updates(plain, divided, list(range(lam)), list(range(lam)))   # every tau 0
    torch.cuda.synchronize()
    assert torch.equal(sync.tensors["theta"].view(torch.int32), plain.tensors["theta"].view(torch.int32))


@pytest.mark.parametrize("P", [50_000, 50_001, 200_000, 200_001])
@pytest.mark.parametrize("rule", ["fast", "ieee"])
def test_short_passes_equal_one_pass_per_gradient(P, rule):
    """The sizes where the batch of a pass of few gradients changes."""
    import torch
    dev = gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(P)
    theta0 = torch.randn(P, device=dev, generator=gen)
    grads = [torch.randn(P, device=dev, generator=gen) * 1e-2 for _ in range(9)]
    mode = fa.MATH_IEEE if rule == "ieee" else fa.MATH_FAST
    for K in (1, 2, 3, 4, 5, 7, 8, 9):
        one, each = new_gpu_state(theta0, dev, 4, 0.005, mode), new_gpu_state(theta0, dev, 4, 0.005, mode)
        clients, ts = [k % 4 for k in range(K)], [k - k % 3 for k in range(K)]
        fa.fasgd_apply_updates(one, grads[:K], clients, ts)
        for k in range(K):
            fa.fasgd_apply_updates(each, grads[k:k + 1], clients[k:k + 1], ts[k:k + 1])
        torch.cuda.synchronize()
        for name in ("theta", "n", "b", "v"):
            x, y = one.tensors[name], each.tensors[name]
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), (name, K)

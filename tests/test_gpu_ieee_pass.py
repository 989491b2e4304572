"""GPU: the IEEE passes in the short sequences (one look at v before and after
the pass) against sparse applies of the whole vector, which look at every
divisor: bit for bit, on ordinary states and on states whose v, n or gradients
leave the range the short sequences hold for (zeros, negative, huge and
subnormal v, infinities, NaNs) in some lanes of some waves."""
import numpy as np
import pytest

import paper_1601_04033_amd as fa
from helpers import gpu, new_gpu_state, to_dev

pytestmark = pytest.mark.gpu


def _same(a, b, what):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    same = (a.view(np.uint32) == b.view(np.uint32)) | (np.isnan(a) & np.isnan(b))
    assert same.all(), (what, int((~same).sum()), np.flatnonzero(~same)[:5])


@pytest.mark.parametrize("odd", ["none", "v", "n", "grad"])
@pytest.mark.parametrize("K", [1, 3, 4, 5, 8, 13])
@pytest.mark.parametrize("beta,reading", [(0.9, fa.V_EQUATIONS), (0.9, fa.V_PROSE), (1.0, fa.V_EQUATIONS)])
def test_ieee_pass_equals_divisor_by_divisor(K, odd, beta, reading):
    import torch
    dev = gpu()
    P, lam = 3 * 256 + 77, 4
    rng = np.random.default_rng(100 * K + len(odd))
    theta0 = rng.standard_normal(P, dtype=np.float32)
    n0 = rng.uniform(1e-6, 1e-2, P).astype(np.float32)
    b0 = (rng.standard_normal(P) * 1e-3).astype(np.float32)
    v0 = rng.uniform(1.0, 100.0, P).astype(np.float32)
    grads = (rng.standard_normal((K + 1, P)) * 1e-2).astype(np.float32)
    at = rng.choice(P, 40, replace=False)
    bad = np.array([0.0, -3.0, 1e-41, 2e-31, 1e31, 3e38, np.inf, -np.inf, np.nan, -0.0], dtype=np.float32)
    if odd == "v":
        v0[at] = np.resize(bad, 40)
    elif odd == "n":
        n0[at] = np.resize(bad, 40)
    elif odd == "grad":
        grads[rng.integers(0, K + 1, 40), at] = np.resize(bad, 40)
    dg = [to_dev(g, dev) for g in grads]
    clients = [k % lam for k in range(K + 1)]
    idx = torch.arange(P, device=dev, dtype=torch.int32)
    cnt = torch.full((1,), P, device=dev, dtype=torch.int64)
    seg = torch.arange(0, P + 256, 256, device=dev, dtype=torch.int32).clamp_(max=P)

    def server():
        st = new_gpu_state(theta0, dev, lam, 0.005, fa.MATH_IEEE, beta=beta, v_reading=reading)
        for name, x in (("n", n0), ("b", b0), ("v", v0)):
            st.tensors[name].copy_(to_dev(x, dev))
        st.c.T, st.c.dense_T = 50, 49
        return st

    ts = [50 + k - 7 * (k % 5) for k in range(K + 1)]
    ref = server()
    for k in range(K + 1):
        fa.bfasgd_apply_sparse(ref, idx, dg[k], cnt, clients[k], ts[k])
    one = server()                       # the first K gradients in one pass, the last in another
    fa.fasgd_apply_updates(one, dg[:K], clients[:K], ts[:K])
    fa.fasgd_apply_updates(one, dg[K:], clients[K:], ts[K:])
    push = server()                      # the first as a push of every parameter, ahead of the others
    fa.fasgd_apply_with_push(push, idx, dg[0], cnt, seg, clients[0], ts[0], dg[1:], clients[1:], ts[1:])
    torch.cuda.synchronize()
    for name in ("theta", "n", "b", "v"):
        _same(one.tensors[name], ref.tensors[name], f"pass {name}")
        _same(push.tensors[name], ref.tensors[name], f"pass with a push {name}")

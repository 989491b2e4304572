"""GPU: the diagnostics entry points.  The IEEE mode's short correctly
rounded sequences (used when eps >= 2^-96 and 2^-20 <= |alpha| < 2^20)
equal the general sequences bit for bit, checked exhaustively on the device
through fasgd_check_ieee_sequences; the general sequences, which run outside
that range, still match the oracle; and the bandwidth anchor copies
exactly."""
import numpy as np
import pytest

import oracle
import paper_1601_04033_amd as fa
import workload
from helpers import RTOL_SEQ, assert_state_close, gpu, new_gpu_state, to_dev

pytestmark = pytest.mark.gpu

# (gamma, beta, eps, alpha): the workloads' settings, the hand trace's, the
# ends of the short range and a value drawn at random
SETTINGS = [(0.95, 0.9, 1e-4, 0.005), (0.95, 0.9, 1e-8, 0.04), (0.5, 0.5, 9 / 16, 0.25),
            (1.0, 0.0, 2.0 ** -96, 2.0 ** -20), (0.0, 1.0, 1.0, 2.0 ** 20 * (1 - 2.0 ** -24)),
            (0.9, 0.99, 3e-7, 0.0123), (0.95, 0.9, 1e-4, 1000.0)]


@pytest.mark.parametrize("gamma,beta,eps,alpha", SETTINGS)
def test_short_sequences_equal_general_ones(gamma, beta, eps, alpha):
    """Square root and 1/sqrt over every finite float x >= 2^-96 (an infinite
    or NaN x gives a NaN root), alpha / d over every d of the short range with
    either sign (every other of the 2^32 bit patterns is found to be outside
    it), and 2^24 whole updates per reading of v, infinities and NaNs among
    their states."""
    import torch
    dev = gpu()
    counts = torch.full((4,), -1, dtype=torch.int64, device=dev)
    print(f"ieee sequences: gamma={gamma} beta={beta} eps={eps} alpha={alpha}", flush=True)
    fa.fasgd_check_ieee_sequences(gamma, beta, eps, alpha, 0x1EEE + int(alpha * 1000), 1 << 24, counts)
    torch.cuda.synchronize()
    got = counts.cpu().tolist()
    assert got == [0, 0, 0, 0], dict(zip(("sqrt", "1/sqrt", "division", "updates"), got))


@pytest.mark.parametrize("reading", [fa.V_EQUATIONS, fa.V_PROSE])
@pytest.mark.parametrize("eps,alpha", [(2.0 ** -100, 0.01), (1e-4, 2.0 ** -21)])
def test_general_sequences_match_oracle(eps, alpha, reading):
    """Outside the short sequences' range (here eps below 2^-96, or alpha
    below 2^-20) IEEE passes take the general sequences: four K = 8 passes
    over a ragged P against 32 oracle updates."""
    import torch
    dev = gpu()
    w = workload.WORKLOADS["tiny"]
    P, K = 4099, 8
    theta0, m, s = workload.host_params(w, P, seed=9)
    clients, ts = workload.schedule(w, 4 * K)
    st = new_gpu_state(theta0, dev, w.lam, alpha, fa.MATH_IEEE, eps=eps, v_reading=reading)
    ref = oracle.init_state(theta0, alpha=alpha, eps=eps, v_reading=reading)
    for p in range(4):
        gs = [workload.host_gradient(w, m, s, p * K + k, seed=9) for k in range(K)]
        sl = slice(p * K, (p + 1) * K)
        fa.fasgd_apply_updates(st, [to_dev(g, dev) for g in gs], clients[sl], ts[sl])
        for k, g in enumerate(gs):
            oracle.fasgd_apply(ref, g, ts[p * K + k])
    torch.cuda.synchronize()
    assert np.isfinite(st.theta.cpu().numpy()).all()
    assert_state_close(st, ref, RTOL_SEQ, what=f"eps={eps} alpha={alpha}")


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1 << 20, (1 << 22) + 7])
def test_copy_anchor_copies_exactly(n):
    """The bandwidth anchor (fasgd_copy_anchor) copies every float bit for bit,
    the trailing n % 4 included, and writes nothing past n."""
    import torch
    dev = gpu()
    src = torch.randn(n, device=dev)
    dst = torch.full((n + 4,), 7.0, device=dev)
    fa.fasgd_copy_anchor(src, dst[:n])
    torch.cuda.synchronize()
    assert torch.equal(dst[:n].view(torch.int32), src.view(torch.int32))
    assert (dst[n:] == 7.0).all()


def test_ieee_division_fallback_inside_the_pass():
    """Inside the K-fused IEEE pass, lanes whose divisor v tau lies outside
    [2^-100, 2^100] take the general division while the other lanes of the
    same wave take the short one: v starts at 1e-33, 1e33 or 1 in turn and
    beta = 1 keeps it there, so every wave mixes the two.  Positive gradients
    keep theta's sums free of cancellation.  Two K = 8 passes over a ragged P
    against 16 oracle updates."""
    import torch
    dev = gpu()
    w = workload.WORKLOADS["tiny"]
    P, K = 4099, 8
    theta0, m, s = workload.host_params(w, P, seed=11)
    clients, ts = workload.schedule(w, 2 * K)
    v0 = np.where(np.arange(P) % 3 == 0, 1e-33, np.where(np.arange(P) % 3 == 1, 1e33, 1.0)).astype(np.float32)
    st = new_gpu_state(theta0, dev, w.lam, w.alpha_fasgd, fa.MATH_IEEE, beta=1.0)
    st.v.copy_(torch.from_numpy(v0))
    ref = oracle.init_state(theta0, alpha=w.alpha_fasgd, beta=1.0)
    ref.v = v0.astype(np.float64)
    for p in range(2):
        gs = [np.abs(workload.host_gradient(w, m, s, p * K + k, seed=11)) + np.float32(1e-3) for k in range(K)]
        sl = slice(p * K, (p + 1) * K)
        fa.fasgd_apply_updates(st, [to_dev(g, dev) for g in gs], clients[sl], ts[sl])
        for k, g in enumerate(gs):
            oracle.fasgd_apply(ref, g, ts[p * K + k])
    torch.cuda.synchronize()
    th = st.theta.cpu().numpy()
    assert np.isfinite(th).all() and (np.abs(th[0::3]) > 1e25).all()    # the tiny divisors took effect
    assert_state_close(st, ref, RTOL_SEQ, what="mixed divisor ranges")

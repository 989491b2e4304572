"""GPU: per-segment decisions and the segment apply where their forms change:
segment counts around the walk (8), the 64-wide compare and the group (128),
segments starting at every remainder of 4 and down to one parameter, sizes on
both sides of the streaming form, arrays that are only 4-byte aligned.
Decisions against the oracle; the apply against a sparse apply of the sent
segments' parameters, bit for bit (same update per parameter)."""
import numpy as np
import pytest

import oracle
import paper_1601_04033_amd as fa
import workload
from helpers import gpu, new_gpu_state, to_dev
from test_gpu_next import SEED, _check_decisions

pytestmark = pytest.mark.gpu


def _cuts(P, S, seed):
    rng = np.random.default_rng(seed)
    small = [1, 2, 4, 7][: max(0, min(4, S - 2))]           # segments of 1, 1, 2 and 3 parameters at the front
    rest = rng.choice(np.arange(8, P), S - 1 - len(small), replace=False)
    return np.concatenate([[0], np.sort(np.concatenate([small, rest])), [P]]).astype(np.int64)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("P,S", [(70_001, 1), (70_001, 2), (70_001, 8), (70_001, 9), (70_001, 64), (70_001, 65),
                                 (70_001, 66), (70_001, 128), (70_001, 129), (70_001, 257), (1_677_721, 7),
                                 (1_677_722, 7), (2_000_003, 100), (2_000_003, 130), (16384 * 5, 3)])
def test_segment_forms(P, S, offset):
    import torch
    dev = gpu()
    seg = _cuts(P, S, P + S)
    theta0 = np.random.default_rng(S).standard_normal(P + offset).astype(np.float32)
    v = workload.synthetic_v(P, seed=S)
    g = to_dev(np.random.default_rng(S + 1).standard_normal(P + offset).astype(np.float32), dev)[offset:]
    mode = fa.MATH_IEEE if S % 2 else fa.MATH_FAST

    def server():
        full = fa.allocate_state(P + offset, dev)
        views = [x[offset:] for x in full]
        views[0].copy_(to_dev(theta0[offset:], dev))
        st = fa.fasgd_init_state(*views, lam=4, alpha=0.005, math_mode=mode)
        st.v.copy_(to_dev(v, dev))
        st.n.fill_(1e-3)
        return st

    a, b = server(), server()
    send = torch.zeros(S, device=dev, dtype=torch.uint8)
    ws = torch.empty(fa.bfasgd_segments_workspace_bytes(P, S), device=dev, dtype=torch.uint8)
    sent = np.zeros(S, bool)
    for T in range(4):                                       # until some segments are sent and some are not
        fa.bfasgd_decide_segments(a, seg, 30.0, 1e-8, SEED, T, T % 4, send, ws)
        sent = send.cpu().numpy().astype(bool)
        want, mean = oracle.bfasgd_decide_segments(v, seg, 30.0, 1e-8, SEED, T, T % 4)
        _check_decisions(sent, want, mean, 30.0, SEED, T, T % 4)
        if sent.any() and (S == 1 or not sent.all()):
            break
    fa.bfasgd_apply_segments(a, g, seg, send, 1, 0)
    on = np.zeros(P, bool)
    for i in np.flatnonzero(sent):
        on[seg[i]:seg[i + 1]] = True
    j = np.flatnonzero(on).astype(np.int32)
    idx = to_dev(np.resize(j, max(j.size, 1)), dev)
    fa.bfasgd_apply_sparse(b, idx, g[idx.long()], torch.full((1,), j.size, device=dev, dtype=torch.int64), 1, 0)
    torch.cuda.synchronize()
    for name in ("theta", "n", "b", "v", "last_T"):
        assert torch.equal(a.tensors[name].view(torch.int32), b.tensors[name].view(torch.int32)), name
    assert a.T == b.T == 1

"""Waits between blocks of decodes off the persistent engine that end by count:
every block stops, every status says so, and the next decode is exact.  The
bound is forced from the host; blocks that wait for spawned tasks while the
longest pass runs reach it."""
import numpy as np
import pytest

import oracle
from workloads import hmm

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# one block per task (K = 200; 300 and 1000 in a large batch), teams, and the
# beams: blocks without a task wait from the start
@pytest.mark.parametrize("K,n,method,B", [(200, 3, "flash", 0), (300, 200, "flash", 0), (1000, 200, "flash", 0),
                                          (600, 2, "flash", 0), (1100, 2, "flash", 0), (4200, 1, "flash", 0),
                                          (300, 3, "beam", 32)])
def test_wait_that_ends_is_reported(K, n, method, B):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    T = 400 if n < 100 else 60
    lp, la, _ = hmm.random_dense(K, 1, K)
    lb = (2 * np.random.default_rng(K).standard_normal((T, K))).astype(np.float32)
    d_la, d_lp, d_lb = _dev(la), _dev(lp), _dev(lb)
    lens = [T - 50 * (b % 2) for b in range(n)]
    batch = fv.Batch([d_lb[:t] for t in lens])
    lib = fv.lib()
    assert lib.fv_debug_wait_turns(-1) == fv.FV_E_INVALID_ARG
    print(f"K={K} n={n} {method}: waits of 64 turns", flush=True)
    assert lib.fv_debug_wait_turns(1) == fv.FV_OK
    try:
        fv.decode_batch(d_la, batch, d_lp, method=method, P=8, B=B)
        torch.cuda.synchronize()
    finally:
        assert lib.fv_debug_wait_turns(0) == fv.FV_OK
    assert (batch.status.cpu().numpy() == fv.FV_E_DEVICE).all()
    fv.decode_batch(d_la, batch, d_lp, method=method, P=8, B=B)
    torch.cuda.synchronize()
    assert (batch.status.cpu().numpy() >= 0).all()
    for b in (0, 1 % n):
        po, so = (oracle.beam(lp, la, lb[:lens[b]], B, 8) if B else oracle.vanilla(lp, la, lb[:lens[b]]))[:2]
        np.testing.assert_array_equal(batch.paths[b, :lens[b]].cpu().numpy(), po)
        assert float(batch.scores[b]) == so

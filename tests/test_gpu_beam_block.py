"""FLASH-BS on one block per task against the oracle: beam widths on both sides
of a thread's share, state counts at the edges of a column group and of the
widest model, ties, missing edges, positive scores, subtasks that stay with
their block and that go to the queue, ends that a beam loses (the exact
re-decode), and sparse steps with more candidates than the block's table."""
import numpy as np
import pytest

import oracle
from workloads import hmm

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENS = [1, 2, 3, 7, 24, 25, 61]


def _dev(x):
    return None if x is None else torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _check(model, lp, lbs, B, P, ref):
    import paper_2510_19301_amd as fv
    batch = fv.Batch([_dev(b) for b in lbs])
    fv.decode_batch(model, batch, _dev(lp), method="beam", P=P, B=B)
    torch.cuda.synchronize()
    paths, scores, status = batch.paths.cpu().numpy(), batch.scores.cpu().numpy(), batch.status.cpu().numpy()
    for b, lb in enumerate(lbs):
        po, so, rc = ref(lb, B, P)[:3]
        assert np.float32(so).view(np.uint32) == scores[b].view(np.uint32), (b, so, scores[b])
        assert status[b] == rc, (b, status[b], rc)
        np.testing.assert_array_equal(paths[b][:lb.shape[0]], po)


@pytest.mark.parametrize("kind", ["float", "ties", "missing", "positive"])
@pytest.mark.parametrize("K", [63, 64, 65, 1024, 1025, 2048])
def test_dense(K, kind):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    r = np.random.default_rng([K, len(kind)])
    lp, la, _ = hmm.random_dense(K, 1, K, integer=kind in ("ties", "missing"),
                                 neg_inf_frac=0.9 if kind == "missing" else 0.0)
    lens = LENS if K <= 65 else LENS[:5]
    lbs = [2 * r.standard_normal((T, K)) for T in lens]
    if kind in ("ties", "missing"):
        lbs = [np.rint(b) for b in lbs]
    if kind == "positive":
        la, lbs = la + np.float32(4), [b + 3 for b in lbs]
    lbs = [np.ascontiguousarray(b, np.float32) for b in lbs]
    d_la = _dev(la)
    for B in (1, 16, 64, 128, 129, 256):
        for P in (1, 4):
            print(f"dense {kind} K={K} B={B} P={P}", flush=True)
            _check(d_la, lp, lbs, min(B, K - 1), P, lambda lb, b, p: oracle.beam(lp, la, lb, b, p))


@pytest.mark.parametrize("integer", [False, True])
@pytest.mark.parametrize("K,deg", [(40, 6), (1500, 6), (3000, 20)])
def test_sparse(K, deg, integer):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    lp, row_ptr, col, val, _ = hmm.random_csr(K, 1, K, deg_hi=deg, integer=integer, dup_frac=0.1)
    model = fv.CsrModel(_dev(np.asarray(row_ptr, np.int32)), _dev(np.asarray(col, np.int32)),
                        _dev(np.asarray(val, np.float32)))
    r = np.random.default_rng(K)
    lbs = [np.ascontiguousarray(np.rint(b) if integer else b, np.float32)
           for b in (2 * r.standard_normal((T, K)) for T in LENS)]
    for B in (1, 16, 128, 129, 256):
        for P in (1, 4):
            print(f"sparse K={K} deg={deg} integer={integer} B={B} P={P}", flush=True)
            _check(model, lp, lbs, min(B, K - 1), P, lambda lb, b, p: oracle.beam_csr(lp, row_ptr, col, val, lb, b, p))

"""Beams that lose the end state of a subtask: the exact re-decode and what it
spawns go to the persistent engine, the rest of the sequence stays with its
block.  Results against the oracle, and the time against the engine's alone."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _graph(r, K, p):
    """log A of a graph with a share p of the edges (one at least a state)."""
    w = np.where(r.random((K, K)) < p, r.random((K, K)), 0.0)
    w[np.arange(K), (np.arange(K) + 1) % K] += 0.1
    with np.errstate(divide="ignore"):
        return np.log(w / w.sum(1, keepdims=True)).astype(np.float32)


@pytest.mark.parametrize("K,p", [(64, 0.1), (300, 0.02), (1000, 0.005)])
def test_dense(K, p):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    r = np.random.default_rng(K)
    la = _graph(r, K, p)
    lbs = [(2 * r.standard_normal((T, K))).astype(np.float32) for T in (2, 17, 60, 90, 90, 41)]
    d_la, d_lbs = _dev(la), [_dev(x) for x in lbs]
    lost = 0
    for B in (1, 4, 16):
        for P in (1, 4, 9):
            print(f"K={K} B={B} P={P}", flush=True)
            batch = fv.Batch(d_lbs)
            fv.decode_batch(d_la, batch, None, method="beam", P=P, B=B)
            torch.cuda.synchronize()
            for b, lb in enumerate(lbs):
                po, so, rc, st = oracle.beam(None, la, lb, B, P)
                lost += st["fallbacks"]
                assert int(batch.status[b]) == rc
                assert float(batch.scores[b]) == so
                np.testing.assert_array_equal(batch.paths[b, :lb.shape[0]].cpu().numpy(), po)
    assert lost > 0


def test_sparse():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    K, deg = 2000, 4
    r = np.random.default_rng(K)
    row_ptr = np.arange(K + 1, dtype=np.int32) * deg
    col = np.sort((np.arange(K)[:, None] + r.integers(0, 40, (K, deg))) % K, axis=1).astype(np.int32).reshape(-1)
    val = np.log(r.random(K * deg) + 1e-3).astype(np.float32)
    model = fv.CsrModel(_dev(row_ptr), _dev(col), _dev(val))
    lbs = [(2 * r.standard_normal((T, K))).astype(np.float32) for T in (1, 30, 70)]
    lost = 0
    for B in (2, 8, 30):
        for P in (1, 5):
            print(f"sparse B={B} P={P}", flush=True)
            batch = fv.Batch([_dev(x) for x in lbs])
            fv.decode_batch(model, batch, None, method="beam", P=P, B=B)
            torch.cuda.synchronize()
            for b, lb in enumerate(lbs):
                po, so, rc, st = oracle.beam_csr(None, row_ptr, col, val, lb, B, P)
                lost += st["fallbacks"]
                assert int(batch.status[b]) == rc and float(batch.scores[b]) == so
                np.testing.assert_array_equal(batch.paths[b, :lb.shape[0]].cpu().numpy(), po)
    assert lost > 0


@pytest.mark.parametrize("K,n,B", [(512, 64, 4), (512, 64, 16), (1024, 1, 8)])
def test_time(K, n, B):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    r = np.random.default_rng(K)
    la = _dev(_graph(r, K, 0.02))
    batch = fv.Batch([_dev((2 * r.standard_normal((400, K))).astype(np.float32)) for _ in range(n)])
    ms = {}
    for engine in (True, False):
        ws = None
        out = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            ws = fv.decode_batch(la, batch, None, method="beam", P=16, B=B, ws=ws, engine=engine)
            e1.record()
            torch.cuda.synchronize()
            out.append(e0.elapsed_time(e1))
        ms[engine] = min(out[1:])
    print(f"K={K} n={n} B={B} engine {ms[True]:.2f} ms, default {ms[False]:.2f} ms", flush=True)
    assert ms[False] < ms[True], ms

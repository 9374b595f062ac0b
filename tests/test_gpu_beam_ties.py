"""Beam steps whose B-th best score has many others beside it: equal scores, and
rows of scores whose depth is unlike the last step's (the selection's bins
follow that).  Results against the oracle, and the time of equal scores against
the persistent engine's (the block's step takes a quarter of it otherwise)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _rows(kind, r, T, K):
    if kind == "equal":
        return np.zeros((T, K), np.float32)
    if kind == "two":
        return -np.float32(r.integers(0, 2, (T, K)))
    # very shallow and very deep steps in turn, and tiny differences beside one far ahead
    x = r.standard_normal((T, K)) * np.where(np.arange(T) % 2 == 0, 1e-4, 1e4)[:, None]
    x[T // 2, r.integers(0, K)] = 1e5
    return x.astype(np.float32)


# selections of at most, and more than, the members that are ranked one by one
@pytest.mark.parametrize("kind", ["equal", "two", "depth"])
@pytest.mark.parametrize("K", [128, 129, 130, 1024, 1500, 2048])
def test_dense(K, kind):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    r = np.random.default_rng([K, len(kind)])
    la = np.full((K, K), -7.0, np.float32)
    if kind == "depth":
        la = (la - 1e-3 * r.random((K, K))).astype(np.float32)
    lbs = [_rows(kind, r, T, K) for T in (1, 2, 9, 30)]
    d_la, d_lbs = _dev(la), [_dev(x) for x in lbs]
    for B in (1, 2, 64, 127, 256):
        B = min(B, K - 1)
        for P in (1, 4):
            print(f"{kind} K={K} B={B} P={P}", flush=True)
            batch = fv.Batch(d_lbs)
            fv.decode_batch(d_la, batch, None, method="beam", P=P, B=B)
            torch.cuda.synchronize()
            for b, lb in enumerate(lbs):
                po, so, rc = oracle.beam(None, la, lb, B, P)[:3]
                assert int(batch.status[b]) == rc
                assert float(batch.scores[b]) == so
                np.testing.assert_array_equal(batch.paths[b, :lb.shape[0]].cpu().numpy(), po)


@pytest.mark.parametrize("integer", [0, 1])
def test_sparse(integer):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    K, deg = 1700, 5
    r = np.random.default_rng(integer)
    row_ptr = np.arange(K + 1, dtype=np.int32) * deg
    col = np.sort(r.integers(0, K, (K, deg)), axis=1).astype(np.int32).reshape(-1)
    val = np.full(K * deg, -1.0, np.float32)
    model = fv.CsrModel(_dev(row_ptr), _dev(col), _dev(val))
    lbs = [-np.float32(r.integers(0, 1 + integer, (T, K))) for T in (1, 2, 20)]
    for B in (2, 100, 256):
        print(f"sparse {integer} B={B}", flush=True)
        batch = fv.Batch([_dev(x) for x in lbs])
        fv.decode_batch(model, batch, None, method="beam", P=3, B=B)
        torch.cuda.synchronize()
        for b, lb in enumerate(lbs):
            po, so, rc = oracle.beam_csr(None, row_ptr, col, val, lb, B, 3)[:3]
            assert int(batch.status[b]) == rc and float(batch.scores[b]) == so
            np.testing.assert_array_equal(batch.paths[b, :lb.shape[0]].cpu().numpy(), po)


def test_time_of_equal_scores():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    K, n, T = 1024, 64, 200
    la = torch.full((K, K), -7.0, device="cuda")
    batch = fv.Batch([torch.zeros((T, K), device="cuda") for _ in range(n)])
    ms = {}
    for engine in (True, False):
        ws = None
        out = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            ws = fv.decode_batch(la, batch, None, method="beam", P=16, B=64, ws=ws, engine=engine)
            e1.record()
            torch.cuda.synchronize()
            out.append(e0.elapsed_time(e1))
        ms[engine] = min(out[1:])
    assert ms[False] < ms[True], ms

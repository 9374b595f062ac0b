"""Bounded scans where the spread of the scores changes within a sequence: what
the scans expect to need follows the last steps, so the steps after such a
change need more than that.  Rows of zeros and then sharp rows on a sticky
chain, a spread that steps up and down, a left-to-right model.  Every sequence
ends in a row that selects one column, so that columns off the best path are
checked too."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TMAX = 14
N_REF = 48        # different sequences of a batch


def _model(kind, K):
    r = np.random.default_rng([K, len(kind)])
    lp = np.full(K, -np.log(K), np.float32)
    if kind == "dropout":
        la = np.full((K, K), np.log(0.1 / (K - 1)), np.float32)
        np.fill_diagonal(la, np.log(0.9))
        rows = np.zeros((TMAX, K), np.float32)
        for t in range(TMAX):
            if t % 5 >= 3:
                rows[t] = -50.0
                rows[t, (7 * t) % K] = -0.1
    elif kind == "spread":
        x = np.log(r.random((K, K))) / 0.1 + np.log(r.gamma(1.1, size=(K, K)))
        la = (x - np.logaddexp.reduce(x, 1, keepdims=True)).astype(np.float32)
        sigma = np.where(np.arange(TMAX) % 5 < 3, 0.1, 10.0)
        rows = (r.standard_normal((TMAX, K)) * sigma[:, None]).astype(np.float32)
    else:
        la = np.full((K, K), -np.inf, np.float32)
        for d in range(4):
            i = np.arange(K - d)
            la[i, i + d] = -0.5 - d
        lp = np.where(np.arange(K) % 97 == 0, lp, -np.inf).astype(np.float32)
        rows = (2 * r.standard_normal((TMAX, K))).astype(np.float32)
    return lp, la, rows


def _sequences(K, rows):
    out = []
    for k in range(N_REF):
        T = TMAX - k % 9
        lb = rows[:T].copy()
        col = (k * K) // N_REF + k % 5
        lb[-1] = -1e4
        lb[-1, min(col, K - 1)] = 0.0
        out.append(lb)
    return out


# n = 256: one block per sequence; 1, 40: teams
@pytest.mark.parametrize("n", [1, 40, 256])
@pytest.mark.parametrize("kind", ["dropout", "spread", "leftright"])
@pytest.mark.parametrize("K", [200, 512, 576, 640, 1000, 1024])
def test_spread_changes(K, kind, n):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    lp, la, rows = _model(kind, K)
    lbs = _sequences(K, rows)
    refs = [oracle.vanilla(lp, la, lb) for lb in lbs[:n]]
    dev = lambda x: torch.from_numpy(x).cuda()
    d_la, d_lp, d_lbs = dev(la), dev(lp), [dev(b) for b in lbs]
    for method, P in (("vanilla", 1), ("flash", 2), ("flash", 3)):
        print(f"{kind} K={K} {method} P={P} n={n}", flush=True)
        batch = fv.Batch([d_lbs[b % N_REF] for b in range(n)])
        fv.decode_batch(d_la, batch, d_lp, method=method, P=P)
        torch.cuda.synchronize()
        paths, scores, status = batch.paths.cpu().numpy(), batch.scores.cpu().numpy(), batch.status.cpu().numpy()
        for b in range(n):
            po, so, rc = refs[b % N_REF]
            T = po.shape[0]
            assert np.float32(so).view(np.uint32) == scores[b].view(np.uint32), (b, T, so, scores[b])
            assert status[b] == rc
            np.testing.assert_array_equal(paths[b][:T], po)


def test_edges_at_the_end_of_the_range():
    """An edge whose distance to its column's maximum is no float."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    K, n = 600, 200
    la = np.full((K, K), -np.inf, np.float32)
    la[0], la[1], la[5] = -3.39e38, -3.38e38, 2e36
    lp = np.full(K, -np.inf, np.float32)
    lp[0], lp[1] = -1e36, -2.1e36               # state 0 wins every column, state 5 is never reached
    lb = np.zeros((2, K), np.float32)
    po, so, rc = oracle.vanilla(lp, la, lb)
    assert rc == fv.FV_OK and po[0] == 0
    dev = lambda x: torch.from_numpy(x).cuda()
    batch = fv.Batch([dev(lb)] * n)
    fv.decode_batch(dev(la), batch, dev(lp), method="vanilla")
    torch.cuda.synchronize()
    assert (batch.scores.cpu().numpy() == so).all()
    assert (batch.paths.cpu().numpy() == po).all()


@pytest.mark.parametrize("T", [32770, 32775, 32782, 32783, 32784])
def test_tasks_after_one_given_up(T):
    """A long sequence that the bound does not prune (given up after some steps)
    and short ones that its team takes next: the scores' tags have 15 bits."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    K, n = 2100, 200
    r = np.random.default_rng(T)
    lbs = [(2 * r.standard_normal((t, K))).astype(np.float32) for t in (5, 12, 24)]
    la = np.zeros((K, K), np.float32)
    refs = [oracle.vanilla(None, la, lb) for lb in lbs]
    dev = lambda x: torch.from_numpy(x).cuda()
    d_lbs = [dev(b) for b in lbs]
    batch = fv.Batch([torch.zeros((T, K), device="cuda")] + [d_lbs[b % 3] for b in range(n)])
    print(f"T={T}", flush=True)
    fv.decode_batch(dev(la), batch, None, method="vanilla")
    torch.cuda.synchronize()
    paths, scores, status = batch.paths.cpu().numpy(), batch.scores.cpu().numpy(), batch.status.cpu().numpy()
    assert (status == fv.FV_OK).all()
    assert scores[0] == 0 and (paths[0][:T] == 0).all()
    for b in range(n):
        po, so, _ = refs[b % 3]
        assert scores[1 + b] == so, (b, scores[1 + b], so)
        np.testing.assert_array_equal(paths[1 + b][:po.shape[0]], po)

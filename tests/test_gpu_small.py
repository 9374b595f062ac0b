"""Small dense models (one block per sequence) against the oracle: scores below,
around and above zero, ties, zeros of both signs, missing edges, and lengths
at the edges of the backtrace's chunks (4096 / K rows)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("kind", ["negative", "ties", "sign", "positive", "missing", "flat"])
@pytest.mark.parametrize("K", [1, 2, 31, 32, 33, 63, 64, 65, 100, 128])
def test_small_matches_oracle(K, kind):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    r = np.random.default_rng([K, len(kind)])
    per = 4096 // K
    lens = [1, 2, 9] + ([per, per + 1, per + 2, 2 * per + 1] if K > 30 else [150])
    lp, la = r.standard_normal(K), r.standard_normal((K, K))
    lbs = [r.standard_normal((T, K)) for T in lens]
    if kind == "negative":
        lp, la, lbs = lp - 5, la - 5, [b - 5 for b in lbs]
    elif kind == "ties":
        lp, la, lbs = np.rint(lp) - 2, np.rint(la) - 3, [np.rint(b) - 2 for b in lbs]
    elif kind == "sign":
        la = np.where(r.random((K, K)) < 0.3, -0.0, np.rint(la))
        lp, lbs = np.rint(lp), [np.rint(b) for b in lbs]
    elif kind == "positive":
        lp, la, lbs = lp + 4, la + 4, [b + 4 for b in lbs]
    elif kind == "missing":
        la[r.random((K, K)) < 0.8] = -np.inf
        lp[r.random(K) < 0.5] = -np.inf
        lp, la, lbs = lp - 4, la - 4, [b - 4 for b in lbs]
    elif kind == "flat":
        lp, la, lbs = 0 * lp, 0 * la, [0 * b for b in lbs]
    c = lambda x: np.ascontiguousarray(x, np.float32)
    lp, la, lbs = c(lp), c(la), [c(b) for b in lbs]
    dev = lambda x: torch.from_numpy(x).cuda()
    for method, P in (("vanilla", 1), ("flash", 1), ("flash", 7)):
        print(f"{kind} K={K} {method} P={P}", flush=True)
        batch = fv.Batch([dev(b) for b in lbs])
        fv.decode_batch(dev(la), batch, dev(lp), method=method, P=P)
        torch.cuda.synchronize()
        paths, scores = batch.paths.cpu().numpy(), batch.scores.cpu().numpy()
        for b, lb in enumerate(lbs):
            po, so = (oracle.vanilla(lp, la, lb) if method == "vanilla" else oracle.flash(lp, la, lb, P))[:2]
            assert np.float32(so).view(np.uint32) == scores[b].view(np.uint32), (b, so, scores[b])
            np.testing.assert_array_equal(paths[b][:lb.shape[0]], po)

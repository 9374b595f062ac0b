"""Bounded scans (dense vanilla and FLASH above the small models) against the
oracle, at the edges of a group of columns, a block's share, the lists and the
kernels: exact paths and score bits, with ties, missing edges, scores around
and above zero, and rows on which the bound prunes nothing."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENS = [1, 2, 3, 6, 21, 70]
# state counts: past the small models, odd rows, a partial last group, the
# single blocks' largest, the teams' kernels on both sides
KS = [129, 130, 192, 255, 256, 257, 300, 512, 577, 1000, 1023, 1024, 1025, 2047, 4096, 4097]


def _inputs(kind, K, lens):
    r = np.random.default_rng([K, len(kind)])
    lp = r.standard_normal(K).astype(np.float32)
    la = (2 * r.standard_normal((K, K))).astype(np.float32)
    lbs = [(2 * r.standard_normal((T, K))).astype(np.float32) for T in lens]
    if kind == "ties":
        lp, la, lbs = np.rint(lp), np.rint(la / 2), [np.rint(b / 2) for b in lbs]
    elif kind == "missing":
        la[r.random((K, K)) < 0.9] = -np.inf
        la[:, K // 2] = -np.inf
        lp[r.random(K) < 0.5] = -np.inf
        lbs[-1][5] = -np.inf                  # an infeasible sequence
    elif kind == "sign":                      # scores on both sides of zero, zeros of both signs
        la = np.where(r.random((K, K)) < 0.2, np.float32(-0.0), np.rint(la)).astype(np.float32)
        lbs = [np.rint(b + (1.0 if t % 2 else -1.0)) for t, b in enumerate(lbs)]
    elif kind == "positive":
        la, lbs = la + 9, [b + 3 for b in lbs]
    elif kind == "flat":
        lp, la, lbs = lp * 0, la * 0 - 1, [b * 0 for b in lbs]
    return [np.ascontiguousarray(x, np.float32) for x in (lp, la)] + [[np.ascontiguousarray(b, np.float32) for b in lbs]]


@pytest.mark.parametrize("kind", ["normal", "ties", "missing", "sign", "positive", "flat"])
@pytest.mark.parametrize("K", KS)
def test_bounded_matches_oracle(K, kind):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    lens = LENS if K <= 1025 else [1, 2, 23]
    lp, la, lbs = _inputs(kind, K, lens)
    dev = lambda x: torch.from_numpy(x).cuda()
    d_la, d_lp = dev(la), dev(lp)
    for method, P in (("vanilla", 1), ("flash", 2), ("flash", 5), ("flash", 64)):
        for sub in (lbs, lbs[-1:]):           # a batch; one sequence on many blocks
            print(f"{kind} K={K} {method} P={P} n={len(sub)}", flush=True)
            batch = fv.Batch([dev(b) for b in sub])
            fv.decode_batch(d_la, batch, d_lp, method=method, P=P)
            torch.cuda.synchronize()
            paths, scores, status = batch.paths.cpu().numpy(), batch.scores.cpu().numpy(), batch.status.cpu().numpy()
            for b, lb in enumerate(sub):
                po, so, rc = (oracle.vanilla(lp, la, lb) if method == "vanilla" else oracle.flash(lp, la, lb, P))[:3]
                T = lb.shape[0]
                assert np.float32(so).view(np.uint32) == scores[b].view(np.uint32), (b, so, scores[b])
                assert (status[b] == fv.FV_OK) == bool(np.isfinite(so))
                np.testing.assert_array_equal(paths[b][:T], po)


@pytest.mark.parametrize("kind", ["normal", "ties", "missing", "sign", "positive", "flat"])
@pytest.mark.parametrize("K", [131, 256, 320, 512, 513, 1000, 1024])
def test_one_block_per_sequence(K, kind):
    """Batches of more sequences than the card has blocks for teams."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    lens = [1, 2, 3] + [5, 6, 7] * 75
    lp, la, lbs = _inputs(kind, K, lens)
    dev = lambda x: torch.from_numpy(x).cuda()
    d_la, d_lp = dev(la), dev(lp)
    d_lbs = [dev(b) for b in lbs]
    refs = [oracle.vanilla(lp, la, lb) for lb in lbs]
    for method, P in (("vanilla", 1), ("flash", 2)):
        print(f"{kind} K={K} {method} n={len(lens)}", flush=True)
        batch = fv.Batch(d_lbs)
        fv.decode_batch(d_la, batch, d_lp, method=method, P=P)
        torch.cuda.synchronize()
        paths, scores = batch.paths.cpu().numpy(), batch.scores.cpu().numpy()
        for b, lb in enumerate(lbs):
            po, so, _ = refs[b] if method == "vanilla" else oracle.flash(lp, la, lb, P)[:3]
            assert np.float32(so).view(np.uint32) == scores[b].view(np.uint32), (b, so, scores[b])
            np.testing.assert_array_equal(paths[b][:lb.shape[0]], po)

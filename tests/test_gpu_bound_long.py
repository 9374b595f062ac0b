"""The bounded scans' kernels for sequences above the short ones: the inputs of
test_gpu_bound.py and test_gpu_bound_shift.py in batches with one sequence that
is long enough to choose them."""
import numpy as np
import pytest

import oracle
from test_gpu_bound import _inputs
from test_gpu_bound_shift import N_REF, TMAX, _model, _sequences

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LONG = 70


def _dev(x):
    return torch.from_numpy(x).cuda()


def _check(lp, la, lbs, label, P=5):
    import paper_2510_19301_amd as fv
    d_la, d_lp = _dev(la), _dev(lp)
    seen = {}
    for lb in lbs:
        if id(lb) not in seen:
            seen[id(lb)] = (_dev(lb), oracle.vanilla(lp, la, lb))
    for method in ("vanilla", "flash"):
        print(f"{label} n={len(lbs)} {method}", flush=True)
        batch = fv.Batch([seen[id(lb)][0] for lb in lbs])
        fv.decode_batch(d_la, batch, d_lp, method=method, P=P)
        torch.cuda.synchronize()
        paths, scores, status = batch.paths.cpu().numpy(), batch.scores.cpu().numpy(), batch.status.cpu().numpy()
        for b, lb in enumerate(lbs):
            po, so, rc = seen[id(lb)][1]
            assert np.float32(so).view(np.uint32) == scores[b].view(np.uint32), (b, so, scores[b])
            assert status[b] == rc
            np.testing.assert_array_equal(paths[b][:lb.shape[0]], po)


@pytest.mark.parametrize("kind", ["normal", "ties", "missing", "sign", "positive", "flat"])
@pytest.mark.parametrize("K", [300, 577, 1000, 1024, 2049, 4096, 4097])
def test_kinds(K, kind):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    lp, la, lbs = _inputs(kind, K, [1, 3, 21, LONG] if K <= 1024 else [6, LONG])
    _check(lp, la, lbs, f"{kind} K={K}")
    _check(lp, la, lbs[-1:], f"{kind} K={K}")                       # one sequence on many blocks
    if K <= 1024:
        _check(lp, la, lbs[-1:] + lbs[:3] * 75, f"{kind} K={K}")    # one block per sequence


@pytest.mark.parametrize("n", [1, 40, 256])
@pytest.mark.parametrize("kind", ["dropout", "spread", "leftright"])
@pytest.mark.parametrize("K", [576, 700, 1024])
def test_spread_changes(K, kind, n):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    lp, la, rows = _model(kind, K)
    short = _sequences(K, rows)
    long = np.concatenate([np.tile(rows, (-(-LONG // TMAX), 1))[:LONG - 1], short[3][-1:]])
    _check(lp, la, [long] + [short[b % N_REF] for b in range(n - 1)], f"{kind} K={K}", P=3)

"""Scores that the bound does not prune: passes are left to the persistent
engine early, with the same results and in little more than the engine's time
(a bound of 1.35: what a pass may read before it is left, at most a twelfth of
these, and the bounded passes' own kernels)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _ms(f):
    out = []
    for _ in range(4):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        f()
        e1.record()
        torch.cuda.synchronize()
        out.append(e0.elapsed_time(e1))
    return min(out[1:])


# teams (K > 1024; lists with and without room for all states, the gated exchange
# above 4096), one block per sequence (K = 1024, n = 256)
@pytest.mark.parametrize("K,T,n,method,sigma", [(8000, 100, 1, "vanilla", 0.0), (8000, 100, 1, "flash", 0.3),
                                                (4096, 100, 16, "vanilla", 0.0), (4096, 200, 1, "flash", 0.3),
                                                (1024, 400, 256, "vanilla", 0.0), (1024, 400, 256, "flash", 0.0)])
def test_time_of_scores_without_information(K, T, n, method, sigma):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    g = torch.Generator(device="cuda").manual_seed(K)
    la = torch.full((K, K), -float(np.log(K)), device="cuda")
    if sigma:
        la += torch.randn((K, K), generator=g, device="cuda")
    batch = fv.Batch([torch.randn((T, K), generator=g, device="cuda") * sigma for _ in range(n)])
    print(f"K={K} T={T} n={n} {method} sigma={sigma}", flush=True)
    ms, out = {}, {}
    for engine in (True, False):
        ws = fv.decode_batch(la, batch, None, method=method, P=16, engine=engine)
        ms[engine] = _ms(lambda: fv.decode_batch(la, batch, None, method=method, P=16, ws=ws, engine=engine))
        out[engine] = (batch.paths.clone(), batch.scores.clone(), batch.status.clone())
    for a, b in zip(out[True], out[False]):
        assert torch.equal(a, b)
    assert ms[False] < 1.35 * ms[True], ms


@pytest.mark.parametrize("K,n", [(700, 200), (1024, 256), (1500, 40), (5001, 6)])
@pytest.mark.parametrize("method,P", [("vanilla", 1), ("flash", 5)])
def test_some_sequences_left_to_the_engine(K, n, method, P):
    """Sequences with and without information, and ones that change, in one batch."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    g = torch.Generator(device="cuda").manual_seed(K + n)
    la = torch.full((K, K), -8.0, device="cuda")
    la.fill_diagonal_(-0.5)
    seqs = []
    for b in range(n):
        T = 40 + 7 * (b % 9)
        x = 3 * torch.randn((T, K), generator=g, device="cuda")
        if b % 3 == 1:
            x[:-1] = 0
        if b % 3 == 2:
            x[T // 3:2 * T // 3] = 0
        seqs.append(x)
    batch = fv.Batch(seqs)
    print(f"K={K} n={n} {method} P={P}", flush=True)
    out = []
    for engine in (True, False):
        batch.paths.fill_(-7)
        fv.decode_batch(la, batch, None, method=method, P=P, engine=engine)
        torch.cuda.synchronize()
        out.append((batch.paths.clone(), batch.scores.clone(), batch.status.clone()))
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("method", ["vanilla", "flash"])
def test_time_of_long_lists(method):
    """A wide reach: most states are listed, and each step's third list is read by one wave."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    K, T = 3000, 100
    g = torch.Generator(device="cuda").manual_seed(K)
    la = torch.log_softmax(4 * torch.randn((K, K), generator=g, device="cuda"), 1)
    batch = fv.Batch([2 * torch.randn((T, K), generator=g, device="cuda")])
    ms, out = {}, {}
    for engine in (True, False):
        ws = fv.decode_batch(la, batch, None, method=method, P=4, engine=engine)
        ms[engine] = _ms(lambda: fv.decode_batch(la, batch, None, method=method, P=4, ws=ws, engine=engine))
        out[engine] = (batch.paths.clone(), batch.scores.clone(), batch.status.clone())
    for a, b in zip(out[True], out[False]):
        assert torch.equal(a, b)
    assert ms[False] < 1.35 * ms[True], ms

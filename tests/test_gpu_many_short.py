"""FLASH over many short sequences, whose tasks would take longer through the
bounded scans' queue than other ways take in all: results on both sides of the
rule, and the time against a call that the rule cannot change."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("K", [129, 200, 256, 300, 700])
@pytest.mark.parametrize("n,T,P", [(256, 8, 4), (300, 33, 16), (256, 20, 4), (200, 40, 4), (520, 16, 16)])
def test_results(K, n, T, P):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    r = np.random.default_rng([K, n])
    la = np.rint(3 * r.standard_normal((K, K)) - 4).astype(np.float32)
    lbs = [np.rint(2 * r.standard_normal((T - k, K))).astype(np.float32) for k in (0, 1, 5)]
    refs = [oracle.vanilla(None, la, lb) for lb in lbs]
    d_lbs = [torch.from_numpy(x).cuda() for x in lbs]
    batch = fv.Batch([d_lbs[b % 3] for b in range(n)])
    print(f"K={K} n={n} T={T} P={P}", flush=True)
    fv.decode_batch(torch.from_numpy(la).cuda(), batch, None, method="flash", P=P)
    torch.cuda.synchronize()
    paths, scores, status = batch.paths.cpu().numpy(), batch.scores.cpu().numpy(), batch.status.cpu().numpy()
    for b in range(n):
        po, so, rc = refs[b % 3]
        assert status[b] == rc and np.float32(so).view(np.uint32) == scores[b].view(np.uint32)
        np.testing.assert_array_equal(paths[b][:po.shape[0]], po)


def _ms(fv, la, batch, **kw):
    ws, out = None, []
    for _ in range(6):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        ws = fv.decode_batch(la, batch, None, ws=ws, **kw)
        e1.record()
        torch.cuda.synchronize()
        out.append(e0.elapsed_time(e1))
    return min(out[1:])


@pytest.mark.parametrize("K,T,P,most", [(256, 8, 4, 1.3), (256, 32, 16, 1.3), (130, 32, 16, 1.3), (512, 8, 4, 1.15)])
def test_time(K, T, P, most):
    """(K <= 256: the bisection without leaves, which is one block per sequence
    whatever the rule, is the longer tree; above: the engine.)"""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    g = torch.Generator(device="cuda").manual_seed(K)
    la = torch.log_softmax(4 * torch.randn((K, K), generator=g, device="cuda"), 1)
    batch = fv.Batch([2 * torch.randn((T, K), generator=g, device="cuda") for _ in range(256)])
    other = _ms(fv, la, batch, method="flash", P=P, **({"leaves": False} if K <= 256 else {"engine": True}))
    ms = _ms(fv, la, batch, method="flash", P=P)
    print(f"K={K} T={T} P={P}: {ms:.3f} ms, the other way {other:.3f}", flush=True)
    assert ms < most * other

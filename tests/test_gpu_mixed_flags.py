"""Batches that mix a dense model small enough for one block per sequence with
a larger one: the flags and hooks that mean the persistent engine hold for
every model of the batch."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KS = (100, 200, 300)
T = 400


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def _models():
    """Multiples of 0.1: many near ties, which the two starts round differently."""
    out = []
    for K in KS:
        r = np.random.default_rng([K, T, 1])
        la, lp, lb = [(np.rint(r.standard_normal(shape) / 0.1) * 0.1).astype(np.float32)
                      for shape in ((K, K), (K,), (T, K))]
        out.append((lp, la, lb))
    return out


@pytest.mark.parametrize("models", [(0, 2), (1, 2), (0, 1, 2)])
@pytest.mark.parametrize("flag", ["relative", "no_leaves"])
def test_flags_hold_for_every_model(models, flag):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    ms = [_models()[m] for m in models]
    rel = flag == "relative"
    for P in (4, 16):
        batch = fv.Batch([_dev(lb) for _, _, lb in ms], models=list(range(len(ms))))
        fv.decode_batch([_dev(la) for _, la, _ in ms], batch, [_dev(lp) for lp, _, _ in ms], method="flash", P=P,
                        relative_init=rel, leaves=rel)
        torch.cuda.synchronize()
        paths, scores = batch.paths.cpu().numpy(), batch.scores.cpu().numpy()
        differ = False
        for b, (lp, la, lb) in enumerate(ms):
            po, so, _, _ = oracle.flash(lp, la, lb, P, relative_init=rel)
            differ |= bool((oracle.vanilla(lp, la, lb)[0] != po).any())
            np.testing.assert_array_equal(paths[b, :T], po)
            assert scores[b] == so
        assert differ == rel


def test_wide_beam_beside_beams():
    """B >= K on the smallest model: FLASH, under the relative start."""
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    ms, B, P = _models(), 150, 4
    batch = fv.Batch([_dev(lb) for _, _, lb in ms], models=[0, 1, 2])
    fv.decode_batch([_dev(la) for _, la, _ in ms], batch, [_dev(lp) for lp, _, _ in ms], method="beam", P=P, B=B,
                    relative_init=True)
    torch.cuda.synchronize()
    paths = batch.paths.cpu().numpy()
    for b, (lp, la, lb) in enumerate(ms):
        f = oracle.flash(lp, la, lb, P, relative_init=True) if B >= KS[b] else oracle.beam(lp, la, lb, B, P,
                                                                                          relative_init=True)
        np.testing.assert_array_equal(paths[b, :T], f[0])


def test_step_limit_holds_for_every_model():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    ms = [_models()[m] for m in (0, 1)] + [_models()[2]]
    batch = fv.Batch([_dev(lb) for _, _, lb in ms], models=[0, 1, 2])
    args = [_dev(la) for _, la, _ in ms], batch, [_dev(lp) for lp, _, _ in ms]
    assert fv.lib().fv_debug_engine_limits(20, 0) == fv.FV_OK
    try:
        fv.decode_batch(*args, method="vanilla")
        torch.cuda.synchronize()
    finally:
        assert fv.lib().fv_debug_engine_limits(0, 0) == fv.FV_OK
    assert (batch.status.cpu().numpy() == fv.FV_E_DEVICE).all()
    fv.decode_batch(*args, method="vanilla")
    torch.cuda.synchronize()
    assert (batch.status.cpu().numpy() == fv.FV_OK).all()

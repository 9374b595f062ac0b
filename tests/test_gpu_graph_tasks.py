"""Graph capture of the decodes that take whole tasks, with passes and subtasks
that are left to the persistent engine: every replay, on inputs that changed in
place, against an eager call on the engine alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _model(K, p):
    r = np.random.default_rng(K)
    w = np.where(r.random((K, K)) < p, r.random((K, K)), 0.0)
    w[np.arange(K), (np.arange(K) + 1) % K] += 0.1
    with np.errstate(divide="ignore"):
        return torch.from_numpy(np.log(w / w.sum(1, keepdims=True)).astype(np.float32)).cuda()


# one block per sequence with and without the closer bound, teams, short and
# long sequences, giving up, beams that lose their ends, the queue's rule
@pytest.mark.parametrize("K,n,T,method,P,B,p", [
    (200, 8, 90, "flash", 8, 0, 1.0), (512, 200, 70, "vanilla", 1, 0, 1.0), (700, 200, 80, "flash", 4, 0, 1.0),
    (700, 3, 20, "vanilla", 1, 0, 1.0), (1500, 4, 70, "flash", 4, 0, 1.0), (5001, 2, 50, "vanilla", 1, 0, 1.0),
    (256, 256, 16, "flash", 4, 0, 1.0), (400, 6, 120, "beam", 4, 6, 0.03)])
def test_replays(K, n, T, method, P, B, p):
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    import paper_2510_19301_amd as fv
    la = _model(K, p)
    g = torch.Generator(device="cuda").manual_seed(K)
    lbs = [torch.zeros((T - b % 5, K), device="cuda") for b in range(n)]

    def fill(rep):
        for b, x in enumerate(lbs):
            x.normal_(generator=g).mul_(0.0 if (b + rep) % 3 == 0 else 2.0)   # some without information

    batch, ref = fv.Batch(lbs), fv.Batch(lbs)
    fill(0)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):   # warm-up on the capture stream
        ws = fv.decode_batch(la, batch, None, method=method, P=P, B=B)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fv.decode_batch(la, batch, None, method=method, P=P, B=B, ws=ws)
    ws_ref = None
    for rep in range(4):
        print(f"K={K} n={n} {method} replay {rep}", flush=True)
        fill(rep)
        batch.paths.fill_(-1)
        batch.scores.fill_(123.0)
        batch.status.fill_(99)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        ws_ref = fv.decode_batch(la, ref, None, method=method, P=P, B=B, ws=ws_ref, engine=True)
        torch.cuda.synchronize()
        assert torch.equal(batch.status, ref.status), rep
        assert torch.equal(batch.scores.view(torch.int32), ref.scores.view(torch.int32)), rep
        for b, x in enumerate(lbs):
            assert torch.equal(batch.paths[b, :x.shape[0]], ref.paths[b, :x.shape[0]]), (rep, b)

"""als_epoch under HIP graph capture: the call enqueues kernels only (no allocation once the workspace has its
size, no copy, no wait), so a caller may record an epoch once and replay it.  Every replay is checked against
the same epoch run eagerly, with eager library calls and synchronisations between the replays."""
import pytest
import torch

from gpu_util import f64, rel_fro, say, to_dev
from paper_2112_02194_amd import binding as als
from synth import make_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,kw", [("c1", {}), ("c3", {"rows": 60000, "cols": 60000})])
def test_a_captured_epoch_replays_like_eager_epochs(gpu_device, name, kw):
    say(f"graph capture of als_epoch, {name} {kw}")
    p = make_problem(name, **kw)
    ctx = als.Context(0)
    Y, Yt = to_dev(p, gpu_device)
    W, H = p.W0.clone().to(gpu_device), p.H0.clone().to(gpu_device)
    prm = als.make_params(p.alpha, p.lam)
    for _ in range(2):  # the workspace takes its size and the launch-size hints arrive
        als.als_epoch(ctx, Y, Yt, W, H, prm)
    als.als_status_sync(ctx)
    W0, H0 = W.clone(), H.clone()
    eager = []
    for _ in range(3):
        als.als_epoch(ctx, Y, Yt, W, H, prm)
        eager.append((W.clone(), H.clone(), als.als_loss(ctx, Y, W, H, prm)))
    W.copy_(W0)
    H.copy_(H0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        als.als_epoch(ctx, Y, Yt, W, H, prm)
    torch.cuda.synchronize()
    assert bool(torch.equal(W, W0)) and bool(torch.equal(H, H0))  # recording runs nothing
    for i in range(3):
        graph.replay()
        loss = als.als_loss(ctx, Y, W, H, prm)  # eager work and a synchronisation between the replays
        als.als_status_sync(ctx)
        We, He, le = eager[i]
        say(f"  replay {i}: errW {rel_fro(f64(W), f64(We)):.1e} errH {rel_fro(f64(H), f64(He)):.1e}")
        assert rel_fro(f64(W), f64(We)) <= 1e-6 and rel_fro(f64(H), f64(He)) <= 1e-6
        assert abs(loss - le) <= 1e-6 * abs(le)
    ctx.close()


@pytest.mark.parametrize("spread", [1.0, 1e-3])
def test_a_captured_fold_in_and_retrieval_replay_on_new_links(gpu_device, spread):
    """One serving step - rows folded in by their own entries, then the best items without the known ones - recorded once and
    replayed on links rewritten in place.  With spread 1e-3 the items are nearly parallel and the queries take the scan."""
    say(f"graph capture of als_solve_rows + als_topk, spread {spread}")
    rows, n, d, k, nnz = 200, 66_000, 64, 20, 3000
    gen = torch.Generator().manual_seed(3)
    H = (1.0 + spread * torch.randn((n, d), generator=gen)).to(gpu_device)

    def links():
        cuts = torch.sort(torch.randint(0, nnz + 1, (rows - 1,), generator=gen)).values
        ptr = torch.cat([torch.zeros(1, dtype=torch.int64), cuts, torch.tensor([nnz])])
        return ptr.to(gpu_device), torch.randint(0, n, (nnz,), generator=gen).to(torch.int32).to(gpu_device)
    prm = als.make_params(0.1, 1e-2)
    ctx, other = als.Context(0), als.Context(0)
    G = als.als_gramian(other, H)
    Y = als.Csr(rows, n, *links())
    X = torch.zeros((rows, d), device=gpu_device)

    def step(c, Yc, Xc):
        als.als_solve_rows(c, Yc, H, G, prm, Xc)
        return als.als_topk(c, Xc, H, k, Yc)
    step(ctx, Y, X)  # the workspace takes its size
    als.als_status_sync(ctx)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ids, scores = step(ctx, Y, X)
    for _ in range(3):
        ptr, idx = links()
        Y.indptr.copy_(ptr)
        Y.indices.copy_(idx)
        graph.replay()
        als.als_status_sync(ctx)
        Xe = torch.zeros_like(X)
        want = step(other, als.Csr(rows, n, ptr, idx), Xe)  # eager, with a context of its own
        als.als_status_sync(other)
        assert torch.equal(X, Xe) and torch.equal(ids, want[0]) and torch.equal(scores, want[1])
    ctx.close()
    other.close()

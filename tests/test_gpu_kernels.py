"""Single kernels at the sizes where their tiling can go wrong, against fp64 evaluations of the same quantity."""
import numpy as np
import pytest
import torch

from gpu_util import f64, rel_fro, say
from paper_2112_02194_amd import binding as als

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_device):
    c = als.Context(0)
    yield c
    c.close()


def _launches(ctx, call):
    """`call`, and the timed launches of every kernel slot in it."""
    als.als_set_timing(ctx, True)
    call()
    launches = als.als_get_timing(ctx)["launches"]
    als.als_set_timing(ctx, False)
    return launches


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_shared_factor_against_the_closed_form_of_one_entry_rows(ctx, gpu_device, d):
    """1, 2, 4 and 8 blocks of 16 columns.  A row with the single entry v solves to B^-1 v / (1 + v^T B^-1 v)
    (Sherman-Morrison), so every column of the shared factor's inverse shows in the result.  Tolerance: L^-1 and
    Z = V L^-T are fp32 with rounding errors amplified by sqrt(cond(B)) each, 4 sqrt(d cond) 2^-24 together, and the
    1 x 1 system is formed from operands cut to 16 bits (4 * 2^-16)."""
    say(f"shared factor d={d}")
    gen = torch.Generator().manual_seed(d)
    n, alpha, lam = 203, 0.1, 1e-3
    H = torch.randn((n, d), generator=gen, dtype=torch.float64) * torch.logspace(0, -2, d, dtype=torch.float64)
    Hf = H.float()
    G = (Hf.double().T @ Hf.double()).float()
    B = alpha * G.double().numpy() + lam * np.eye(d)
    ev = np.linalg.eigvalsh(B)
    Y = als.Csr(n, n, torch.arange(n + 1, device=gpu_device), torch.arange(n, device=gpu_device, dtype=torch.int32))
    X = torch.empty((n, d), device=gpu_device)
    als.als_solve_rows(ctx, Y, Hf.to(gpu_device), G.to(gpu_device), als.make_params(alpha, lam), X)
    als.als_status_sync(ctx)
    BiV = np.linalg.solve(B, f64(Hf).T).T
    ref = BiV / (1.0 + np.sum(f64(Hf) * BiV, axis=1, keepdims=True))
    assert rel_fro(f64(X), ref) <= 4 * np.sqrt(d * ev[-1] / ev[0]) * 2.0 ** -24 + 4 * 2.0 ** -16


@pytest.mark.parametrize("d", [16, 128])
def test_a_gramian_that_is_not_positive_definite_is_reported(ctx, gpu_device, d):
    Y = als.Csr(4, 4, torch.arange(5, device=gpu_device), torch.arange(4, device=gpu_device, dtype=torch.int32))
    V = torch.ones((4, d), device=gpu_device)
    G = torch.eye(d, device=gpu_device)
    G[d - 1, d - 1] = -1.0  # the last pivot of the last block
    als.als_solve_rows(ctx, Y, V, G, als.make_params(0.1, 1e-3), torch.empty((4, d), device=gpu_device))
    with pytest.raises(als.AlsError) as e:
        als.als_status_sync(ctx)
    assert e.value.status == als.ALS_ENOTSPD
    als.als_status_sync(ctx)  # reported once


def _topk_definition(Q, H, k, ex):
    """Scores in fp64 with numpy's matmul; ids by (-score, id) among the admissible items with a score."""
    S = Q.double().numpy() @ H.double().numpy().T
    out = []
    for q in range(S.shape[0]):
        bad = set() if ex is None else set(ex[1][ex[0][q]:ex[0][q + 1]].tolist())
        ok = np.array([i for i in range(S.shape[1]) if i not in bad and not np.isnan(S[q, i])], dtype=np.int64)
        out.append(ok[np.lexsort((ok, -S[q, ok]))][:k])
    return S, out


# edges of segments (32), units (128 and more), thread strides of the chunk scan (1024 chunks), query groups (64, 256, 384,
# 512) and both kernel shapes
@pytest.mark.parametrize("nq,n,d,dtype,k", [
    (1, 1, 16, torch.float32, 1), (3, 31, 32, torch.bfloat16, 40), (1, 129, 128, torch.float32, 10),
    (64, 4097, 64, torch.float32, 20), (65, 33000, 32, torch.float32, 20), (256, 8191, 128, torch.bfloat16, 64),
    (257, 5000, 128, torch.float32, 50), (385, 2047, 128, torch.bfloat16, 10), (513, 1025, 64, torch.bfloat16, 20),
    (300, 40001, 16, torch.float32, 10), (520, 3000, 32, torch.bfloat16, 50), (2, 300007, 16, torch.bfloat16, 50)])
def test_topk_at_the_edges_of_its_tiles(gpu_device, nq, n, d, dtype, k):
    """Ties broken by id, zero rows on both sides, long exclusion lists of the very best items; the returned scores are held
    to the error of an fp32 sum of d products, (d + 1) 2^-24 |q| |h|, and the ids to the definition where no neighbouring
    scores are closer than twice that."""
    say(f"topk nq={nq} n={n} d={d} {dtype} k={k}")
    gen = torch.Generator().manual_seed(n + d)
    H = (torch.randn(n, d, generator=gen) * torch.exp(0.5 * torch.randn(n, 1, generator=gen))).to(dtype)
    Q = torch.randn(nq, d, generator=gen).to(dtype)
    H[n // 2: n // 2 + 70] = H[n // 2]
    H[n // 3: n // 3 + 40] = 0
    Q[nq // 2] = 0
    if nq > 2:
        Q[1] = H[n // 2]
    best = (Q.double() @ H.double().T).topk(min(n, 100)).indices
    lens = torch.randint(0, min(n, 100) + 1, (nq,), generator=gen)
    ptr = torch.zeros(nq + 1, dtype=torch.int64)
    ptr[1:] = torch.cumsum(lens, 0)
    idx = torch.cat([best[q, :int(lens[q])] for q in range(nq)]).to(torch.int32)
    ctx = als.Context(0)
    for ex in (None, (ptr.numpy(), idx.numpy())):
        csr = None if ex is None else als.Csr(nq, n, ptr.to(gpu_device), idx.to(gpu_device))
        ids, sc = als.als_topk(ctx, Q.to(gpu_device), H.to(gpu_device), k, csr)
        torch.cuda.synchronize()
        ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
        S, ref = _topk_definition(Q, H, k, ex)
        tol = (d + 1) * 2.0 ** -24 * np.outer(np.linalg.norm(Q.double().numpy(), axis=1), np.linalg.norm(H.double().numpy(), axis=1))
        for q in range(nq):
            m = len(ref[q])
            assert np.all(ids[q, m:] == -1) and np.all(np.isneginf(sc[q, m:]))
            got, r = ids[q, :m], ref[q]
            assert len(set(got.tolist())) == m
            assert ex is None or not np.intersect1d(got, ex[1][ex[0][q]:ex[0][q + 1]]).size
            assert np.all(np.abs(sc[q, :m] - S[q, got]) <= tol[q, got])
            assert np.all(np.abs(S[q, got] - S[q, r]) <= 2 * (tol[q, got] + tol[q, r]))
            same = np.flatnonzero(np.diff(sc[q, :m]) == 0)
            assert np.all(got[same] < got[same + 1])  # equal scores by ascending id
    ctx.close()


def test_topk_with_values_that_cannot_be_bounded(gpu_device):
    """Infinite, NaN, huge and tiny entries: an item whose score is NaN is never returned, infinite ones rank as numbers do, and
    the rest of the ranking is what it is without them."""
    say("topk with inf, nan, 1e30, 1e-30")
    nq, n, d, k = 70, 3000, 64, 20
    gen = torch.Generator().manual_seed(11)
    H, Q = torch.randn(n, d, generator=gen), torch.randn(nq, d, generator=gen)
    H[5] = float("nan")
    H[700, 3] = float("inf")
    H[1500] = 1e30 * H[1500]
    H[2000:2200] *= 1e-30
    Q[7] *= 1e-30
    Q[8] *= 1e25
    Q[9, 0] = float("nan")
    Q[10, :] = 0
    ctx = als.Context(0)
    ids, sc = als.als_topk(ctx, Q.to(gpu_device), H.to(gpu_device), k)
    torch.cuda.synchronize()
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    S = (Q[:, None, :] * H[None, :, :]).sum(-1).numpy()  # fp32: overflows where the library's products do
    for q in range(nq):
        ok = np.flatnonzero(~np.isnan(S[q]))
        ref = ok[np.lexsort((ok, -S[q, ok]))][:k]
        assert np.all(ids[q, len(ref):] == -1)
        got = ids[q, :len(ref)]
        assert 5 not in got
        with np.errstate(invalid="ignore"):
            close = np.abs(S[q, got] - S[q, ref]) <= 1e-4 * np.abs(S[q, ref])
        assert np.all(close | (S[q, got] == S[q, ref])), (q, got, ref)
    ctx.close()


@pytest.mark.parametrize("d,dtype", [(64, torch.float32), (64, torch.bfloat16), (128, torch.float32), (128, torch.bfloat16)])
@pytest.mark.parametrize("solver", [als.SOLVER_DIRECT, als.SOLVER_CG])
def test_primal_rows_at_the_edges_of_their_batches(ctx, gpu_device, d, dtype, solver):
    """One entry, the batch of 32 and the split threshold with a neighbour on each side, segments with a short tail; labels of
    both signs and a Gramian whose base is not 16-byte aligned.  Tolerance: rounding of d-long sums amplified by the
    system's condition, 4 sqrt(d) 2^-24 cond (CG stops at 1e-6 |b|: plus 1e-6 cond; it starts
    from the row's content, whose size its rounding errors would follow: here 0); bf16 results round by 2^-8."""
    say(f"primal rows d={d} {dtype} solver={solver}")
    gen = torch.Generator().manual_seed(d)
    lens = [1, 2, 31, 32, 33, 63, 64, 65, 96, 127, 129, 511, 512, 513, 1025, 1100, 0]
    n, alpha, lam, rows = 4001, 0.1, 1e-1, len(lens)
    H = (0.3 * torch.randn((n, d), generator=gen)).to(dtype)
    ptr = torch.tensor([0] + lens).cumsum(0)
    idx = torch.cat([torch.randperm(n, generator=gen)[:k] for k in lens]).to(torch.int32)
    val = torch.rand(int(ptr[-1]), generator=gen) * 2 - 0.5
    Hd = H.double()
    G = Hd.T @ Hd
    Gbuf = torch.zeros(d * d + 1, device=gpu_device)
    Gbuf[1:] = G.float().flatten().to(gpu_device)
    for Gdev in (Gbuf[1:].view(d, d), G.float().to(gpu_device)):
        X = torch.full((rows, d), 7.0 if solver == als.SOLVER_DIRECT else 0.0, dtype=dtype, device=gpu_device)
        Y = als.Csr(rows, n, ptr.to(gpu_device), idx.to(gpu_device), val.to(gpu_device))
        als.als_solve_rows(ctx, Y, H.to(gpu_device), Gdev, als.make_params(alpha, lam, path=als.PATH_PRIMAL, solver=solver), X)
        als.als_status_sync(ctx)
        got = f64(X)
        for u, k in enumerate(lens):
            x = Hd[idx[ptr[u]:ptr[u + 1]].long()].numpy()
            A = alpha * G.numpy() + lam * np.eye(d) + x.T @ x
            ref = np.linalg.solve(A, x.T @ val[ptr[u]:ptr[u + 1]].double().numpy())
            cond = np.linalg.cond(A)
            tol = 4 * np.sqrt(d) * 2.0 ** -24 * cond + (1e-6 * cond if solver == als.SOLVER_CG else 0) + (2.0 ** -8 if dtype == torch.bfloat16 else 0)
            assert np.linalg.norm(got[u] - ref) <= tol * max(np.linalg.norm(ref), 1e-300), (k, tol)


@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_with_fewer_entries_than_the_table_has_rows(ctx, gpu_device, d, dtype):
    """Z holds one row per entry: every row class, a row range that starts inside the entries, repeated items, empty rows.
    Tolerances: the project's 1e-4 for fp32 tables and 1e-2 for bf16 ones, row by row."""
    say(f"entries < table rows, d={d} {dtype}")
    gen = torch.Generator().manual_seed(100 + d)
    lens = [3, 9, 0, 1, 2, 4, 5, 8, 9, 16, 17, 31, 32, 33, 48, 49, 64, 65, 80, 96, 97, 112, 128, 129, 200, 530, 0, 7, 40, 6]
    rows, n, lo, hi, alpha, lam = len(lens), 4099, 2, 28, 0.1, 1e-2
    ptr = torch.tensor([0] + lens).cumsum(0)
    nnz = int(ptr[-1])
    assert nnz < n
    H = (0.3 * torch.randn((n, d), generator=gen) * torch.linspace(1, 0.1, d)).to(dtype)
    idx = torch.randint(0, n, (nnz,), generator=gen).to(torch.int32)
    idx[20:24] = idx[20]
    val = torch.rand(nnz, generator=gen) + 0.5
    Hd = H.double()
    G = Hd.T @ Hd
    Hg, Gg = H.to(gpu_device), G.float().to(gpu_device)
    X = torch.full((rows, d), 3.0, dtype=dtype, device=gpu_device)
    Y = als.Csr(rows, n, ptr.to(gpu_device), idx.to(gpu_device), val.to(gpu_device))
    als.als_solve_rows(ctx, Y, Hg, Gg, als.make_params(alpha, lam), X, lo, hi)
    als.als_status_sync(ctx)
    got = f64(X)
    for u, k in enumerate(lens):
        if not lo <= u < hi:
            assert np.all(got[u] == 3.0)
            continue
        x = Hd[idx[ptr[u]:ptr[u + 1]].long()].numpy()
        ref = np.linalg.solve(alpha * G.numpy() + lam * np.eye(d) + x.T @ x, x.T @ val[ptr[u]:ptr[u + 1]].double().numpy())
        assert np.linalg.norm(got[u] - ref) <= (1e-4 if dtype == torch.float32 else 1e-2) * np.linalg.norm(ref), (u, k)
    # an indptr that claims more entries than nnz is reported; nothing beyond nnz is read or written
    short = als.Csr(rows, n, Y.indptr, Y.indices[:int(ptr[12])], Y.values[:int(ptr[12])])
    als.als_solve_rows(ctx, short, Hg, Gg, als.make_params(alpha, lam), X)
    with pytest.raises(als.AlsError):
        als.als_status_sync(ctx)


@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_topk_scores_are_summed_in_one_stated_order(ctx, gpu_device, d, dtype):
    """The bits of a score decide which of two close items comes first, so they are pinned: fp32 (and d = 16) one fused
    multiply-add per element in the order 16 j + 4 q + c (j outermost, then c, then q); bf16 with d >= 32 eight exact
    products at a time in storage order.  Entries are chosen so that fp64 holds every product and every sum before its
    rounding to fp32: twelve-bit mantissas for the chain, whole numbers of eight bits for the groups, the first group 2^8
    times the others so that its sum pushes the low bits of what follows out of fp32."""
    say(f"order of the sums of a score d={d} {dtype}")
    rng = np.random.default_rng(d)
    nq, n = 130, 64
    native = dtype == torch.bfloat16 and d >= 32
    if native:
        def entries(rows):
            x = rng.integers(128, 256, (rows, d)) * rng.choice([-1.0, 1.0], (rows, d))
            x[:, :8] *= 16
            return x
        groups = [list(range(i, i + 8)) for i in range(0, d, 8)]
    else:
        def entries(rows):
            x = torch.from_numpy(rng.integers(-2047, 2048, (rows, d)) * 2.0 ** rng.integers(-4, 5, (rows, d)))
            return x.to(dtype).double().numpy()
        groups = [[16 * j + 4 * q + c] for j in range(d // 16) for c in range(4) for q in range(4)]
    Q, H = entries(nq), entries(n)
    ref = np.zeros((nq, n))
    for g in groups:
        ref = (ref + Q[:, g] @ H[:, g].T).astype(np.float32).astype(np.float64)
    ids, sc = als.als_topk(ctx, torch.from_numpy(Q).to(dtype).to(gpu_device), torch.from_numpy(H).to(dtype).to(gpu_device), n)
    torch.cuda.synchronize()
    ids, sc = ids.cpu().numpy(), sc.cpu().numpy()
    for q in range(nq):
        best = np.lexsort((np.arange(n), -ref[q]))
        assert np.array_equal(ids[q], best)
        assert np.array_equal(sc[q].astype(np.float64), ref[q, best])


@pytest.mark.parametrize("d,dtype", [(16, torch.float32), (128, torch.float32), (128, torch.bfloat16)])
def test_rows_outside_the_entries_of_their_range_are_reported(ctx, gpu_device, d, dtype):
    """Z holds one row per entry between the first and the last indptr of the range.  With an indptr that is not monotone a
    row can reach beyond them although it stays within nnz: it is dropped and reported, Z is not read for it."""
    say(f"indptr not monotone d={d} {dtype}")
    gen = torch.Generator().manual_seed(d)
    n, alpha, lam = 300, 0.1, 1e-2
    H = (0.3 * torch.randn((n, d), generator=gen)).to(dtype).to(gpu_device)
    G = als.als_gramian(ctx, H)
    prm = als.make_params(alpha, lam)
    for ptr, lo, hi, dropped in (([0, 10, 4], 0, 2, [0]), ([0, 4, 12, 8, 12], 1, 3, [1]), ([0, 6, 2, 9, 12], 2, 4, [])):
        rows, idx = len(ptr) - 1, torch.randint(0, n, (ptr[-1] if ptr[-1] > 4 else 10,), generator=gen).to(torch.int32).to(gpu_device)
        Y = als.Csr(rows, n, torch.tensor(ptr, device=gpu_device), idx)
        X = torch.full((rows, d), 5.0, dtype=dtype, device=gpu_device)
        als.als_solve_rows(ctx, Y, H, G, prm, X, lo, hi)
        if dropped:
            with pytest.raises(als.AlsError) as e:
                als.als_status_sync(ctx)
            assert e.value.status == als.ALS_EINVAL
        als.als_status_sync(ctx)
        for u in range(rows):
            if u in dropped:
                continue  # what a dropped row holds is not stated
            if not lo <= u < hi:
                assert bool((X[u] == 5.0).all())
            elif ptr[u + 1] <= ptr[u]:
                assert bool((X[u] == 0.0).all())
            else:
                x = f64(H[idx[ptr[u]:ptr[u + 1]].long()])
                ref = np.linalg.solve(alpha * f64(G) + lam * np.eye(d) + x.T @ x, x.T @ np.ones(len(x)))
                assert np.linalg.norm(f64(X[u]) - ref) <= (1e-4 if dtype == torch.float32 else 1e-2) * np.linalg.norm(ref)


def _stale_hint_case(d, dtype, first, second, n, params, gpu_device):
    """Solve a matrix whose rows have `first` entries, rewrite it in place to `second` (the launch sizes that the first call
    left are those of the old content), solve again; the same with a fresh context, whose calls have no such sizes."""
    gen = torch.Generator().manual_seed(d)
    rows, nnz = len(first), int(first.sum())
    assert len(second) == rows and int(second.sum()) == nnz

    def ptr(lens):
        p = torch.zeros(rows + 1, dtype=torch.int64)
        p[1:] = torch.cumsum(lens, 0)
        return p
    idx = torch.randint(0, n, (nnz,), generator=gen).to(torch.int32).to(gpu_device)
    val = (torch.rand(nnz, generator=gen) + 0.5).to(gpu_device)
    H = (0.3 * torch.randn((n, d), generator=gen)).to(dtype).to(gpu_device)
    Y = als.Csr(rows, n, ptr(first).to(gpu_device), idx, val)
    out = []
    for warm in (True, False):
        c = als.Context(0)
        G = als.als_gramian(c, H)
        if warm:
            als.als_solve_rows(c, Y, H, G, params, torch.empty((rows, d), dtype=dtype, device=gpu_device))
            als.als_status_sync(c)
        Y.indptr.copy_(ptr(second))
        X = torch.full((rows, d), 7.0, dtype=dtype, device=gpu_device)
        als.als_solve_rows(c, Y, H, G, params, X)
        als.als_status_sync(c)
        out.append(X)
        c.close()
    assert torch.isfinite(out[0].float()).all()
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("what", ["rows", "segments"])
def test_primal_rows_beyond_a_launch_hint_that_is_too_small(gpu_device, d, dtype, what):
    """The grid-stride form of the primal kernels with several items per workgroup: 2048 (rows, segments) or 1024 (long rows)
    workgroups walk what lies beyond the hint.  The numbers do not depend on the form, bit for bit."""
    say(f"hint too small: primal {what} d={d} {dtype}")
    rows = 6400
    lens = torch.arange(rows) % 15 + 1  # 1 .. 15, 8 on average up to the cut of the last cycle
    if what == "rows":  # 100 rows of 512 entries, then every row
        second = lens.clone()
        second[-1] += 512 * 100 - int(lens.sum())
        first = torch.zeros(rows, dtype=torch.int64)
        first[::64] = 512
        _stale_hint_case(d, dtype, first, second, 3000, als.make_params(0.1, 1e-2, path=als.PATH_PRIMAL), gpu_device)
    else:  # no row longer than 8 entries, then 5120 of ten or more in two segments each
        first = torch.full((rows,), 8)
        second = torch.zeros(rows, dtype=torch.int64)
        second[:5120] = 9 + torch.arange(5120) % 3
        second[0] += 8 * rows - int(second.sum())
        _stale_hint_case(d, dtype, first, second, 3000, als.make_params(0.1, 1e-2, path=als.PATH_PRIMAL, split_nnz=8), gpu_device)


@pytest.mark.parametrize("d,dtype", [(16, torch.float32), (32, torch.bfloat16), (64, torch.float32), (128, torch.bfloat16)])
def test_long_rows_under_conjugate_gradients_beyond_a_launch_hint_that_is_too_small(gpu_device, d, dtype):
    """Long rows have two launches under this solver: 1024 workgroups walk the 5120 rows that a hint left out; without a hint each has a
    workgroup.  Bit for bit the same."""
    say(f"hint too small: long rows, conjugate gradients d={d} {dtype}")
    rows = 6400
    first = torch.full((rows,), 8)
    second = torch.zeros(rows, dtype=torch.int64)
    second[:5120] = 9 + torch.arange(5120) % 3
    second[0] += 8 * rows - int(second.sum())
    _stale_hint_case(d, dtype, first, second, 3000, als.make_params(0.1, 1e-2, path=als.PATH_PRIMAL, split_nnz=8, solver=als.SOLVER_CG), gpu_device)


@pytest.mark.parametrize("d,dtype", [(16, torch.float32), (32, torch.float32), (32, torch.bfloat16), (64, torch.float32),
                                     (128, torch.float32), (128, torch.bfloat16)])
def test_dual_rows_beyond_a_launch_hint_that_is_too_small(gpu_device, d, dtype):
    """The same for every dual class: 8192 workgroups walk the steps (of 16, 8 and 1 rows) that no hint announced; rows of 9 to 32 entries have
    one kernel, whose wavefronts walk about thirty steps of four rows each instead of four."""
    say(f"hint too small: dual classes d={d} {dtype}")
    counts = {3: 140_000, 7: 70_000, 13: 36_000}
    if d >= 32:
        counts[25] = 36_000
    if d >= 64:
        counts.update({40: 9000, 56: 9000})
    if d >= 128:
        counts.update({72: 9000, 88: 9000, 104: 9000, 120: 9000})
    lens = torch.cat([torch.full((c,), k) for k, c in counts.items()])
    lens = lens[torch.randperm(len(lens), generator=torch.Generator().manual_seed(1))]
    total = int(lens.sum())
    # empty rows bring the lists' capacity beyond the 2^17 steps of the common launch: 7/16 of a step per row for k <= 16 alone
    second = torch.cat([lens, torch.zeros(total // 500 + 120_000, dtype=torch.int64)])
    assert len(second) * 7 // 16 > 1 << 17
    first = torch.zeros(len(second), dtype=torch.int64)  # rows too long for the dual form, then none
    first[:total // 500] = 500
    first[0] += total % 500
    _stale_hint_case(d, dtype, first, second, 5000, als.make_params(0.1, 1e-2), gpu_device)


def _nearly_parallel(rows, d, dtype, gen):
    """Rows whose scores spread by less than the bound's margin: whole numbers, so that every score is exact."""
    x = 64 + torch.randint(0, 3, (rows, d), generator=gen).double()
    return x.to(dtype)


# tables just beyond the size from which the scan is kept (2^24 bytes) and one below it with many queries; queries beyond one
# workgroup of the scan (64)
@pytest.mark.parametrize("nq,n,d,dtype,k", [(70, 65_600, 64, torch.float32, 20), (130, 66_001, 128, torch.bfloat16, 64), (3, 262_200, 16, torch.float32, 1),
                                            (65, 131_100, 32, torch.float32, 33), (5, 524_300, 16, torch.bfloat16, 50), (600, 33_000, 64, torch.float32, 10)])
def test_topk_of_queries_that_are_left_to_the_scan(ctx, gpu_device, nq, n, d, dtype, k):
    """Queries whose scores hardly spread, queries without a bound (an infinite entry) and ordinary ones side by side, with
    and without exclusions.  The entries are whole numbers, the scores therefore exact: ids and scores are compared as they are."""
    say(f"topk scan nq={nq} n={n} d={d} {dtype} k={k}")
    gen = torch.Generator().manual_seed(n)
    H, Q = _nearly_parallel(n, d, dtype, gen), _nearly_parallel(nq, d, dtype, gen)
    Q[1::3] = torch.randint(-60, 61, Q[1::3].shape, generator=gen).to(dtype)  # spreads
    H[n // 2: n // 2 + 200, ::2] *= -1
    if nq > 3:
        Q[3, 0] = float("inf")
        Q[4] = 0
    S = (Q.double().to(gpu_device) @ H.double().to(gpu_device).T)
    if nq > 3:
        S[3] = torch.where(H[:, 0].to(gpu_device) > 0, float("inf"), -float("inf"))
    lens = torch.randint(0, 80, (nq,), generator=gen)
    ptr = torch.zeros(nq + 1, dtype=torch.int64)
    ptr[1:] = torch.cumsum(lens, 0)
    order = torch.sort(S, dim=1, descending=True, stable=True).indices[:, :k + 100]  # equal scores by ascending id
    idx = torch.cat([order[q, torch.randperm(k + 90, generator=gen)[:int(lens[q])].to(gpu_device)] for q in range(nq)]).to(torch.int32)
    Qd, Hd = Q.to(gpu_device), H.to(gpu_device)
    for ex in (False, True):
        csr = als.Csr(nq, n, ptr.to(gpu_device), idx) if ex else None
        ids, sc = als.als_topk(ctx, Qd, Hd, k, csr)
        torch.cuda.synchronize()
        for q in range(nq):
            r = order[q]
            if ex:
                r = r[~torch.isin(r, idx[int(ptr[q]):int(ptr[q + 1])].long())]
            r = r[:k]
            assert torch.equal(ids[q].long(), r), q
            assert torch.equal(sc[q].double(), S[q, r])


def test_topk_of_nearly_parallel_rows_takes_no_longer_than_a_scan(ctx, gpu_device):
    """1024 queries x 1M items: with one workgroup per query walking the table alone this took 75 times as long as on rows
    whose scores spread; the scan for all of them takes 7 times as long."""
    say("topk time on nearly parallel rows")
    gen = torch.Generator(device=gpu_device).manual_seed(1)
    ms = {}
    for name, mean, spread in (("wide", 0.0, 1.0), ("tight", 1.0, 1e-3)):
        H = mean + spread * torch.randn((1_000_000, 64), device=gpu_device, generator=gen)
        Q = mean + spread * torch.randn((1024, 64), device=gpu_device, generator=gen)
        als.als_topk(ctx, Q, H, 20)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(3):
            als.als_topk(ctx, Q, H, 20)
        e1.record()
        torch.cuda.synchronize()
        ms[name] = e0.elapsed_time(e1) / 3
    assert ms["tight"] <= 25 * ms["wide"], ms


def test_topk_of_more_queries_than_one_launch_holds(ctx, gpu_device):
    """2^24 + 70 queries of one workgroup of 256 threads each are more than 2^32 threads: they go in batches.  Whole numbers,
    so the scores are exact."""
    say("topk with more than 2^24 queries")
    nq, n, d = (1 << 24) + 70, 100, 16
    gen = torch.Generator(device=gpu_device).manual_seed(5)
    Q = torch.randint(-3, 4, (nq, d), device=gpu_device, generator=gen, dtype=torch.int8).to(torch.bfloat16)
    H = torch.randint(-3, 4, (n, d), device=gpu_device, generator=gen).to(torch.bfloat16)
    ids, sc = als.als_topk(ctx, Q, H, 1)
    torch.cuda.synchronize()
    for q0 in range(0, nq, 1 << 21):
        S = Q[q0:q0 + (1 << 21)].float() @ H.float().T
        best = S.max(dim=1).values
        assert torch.equal(sc[q0:q0 + (1 << 21), 0], best)
        first = torch.where(S == best[:, None], torch.arange(n, device=gpu_device), n).min(dim=1).values  # ties: smallest id
        assert torch.equal(ids[q0:q0 + (1 << 21), 0].long(), first)


def test_topk_on_a_nearly_full_card(gpu_device):
    """Where the workspace for all queries (about 0.3 GB) cannot be had, fewer are worked on together; the results are the same."""
    say("topk with 200 MB left on the card")
    nq, n, d, k = 8192, 4_000_000, 16, 20
    gen = torch.Generator(device=gpu_device).manual_seed(6)
    Q = torch.randn((nq, d), device=gpu_device, generator=gen).to(torch.bfloat16)
    H = torch.randn((n, d), device=gpu_device, generator=gen).to(torch.bfloat16)
    roomy = als.Context(0)
    want = als.als_topk(roomy, Q, H, k)
    torch.cuda.synchronize()
    roomy.close()
    c = als.Context(0)
    als.als_topk(c, Q[:1], H[:1000], k)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    filler = torch.empty(torch.cuda.mem_get_info()[0] - (200 << 20), dtype=torch.uint8, device=gpu_device)
    try:
        got = als.als_topk(c, Q, H, k)
        torch.cuda.synchronize()
    finally:
        del filler
        torch.cuda.empty_cache()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert c.lib.als_last_error(c.handle) == b""
    c.close()


@pytest.mark.parametrize("d,lo,hi", [(16, 9, 16), (32, 9, 16), (64, 9, 16), (128, 9, 16), (32, 17, 32), (64, 17, 32), (128, 17, 32)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("alpha", [0.1, 1e-4])
def test_rows_of_9_to_32_entries(ctx, gpu_device, d, lo, hi, dtype, alpha):
    """The 16-entry tiles of the two classes at every fill, steps of the list that are not full, entries that
    repeat (Z_I Z_I^T is singular then), labels of both signs and zero.  alpha = 1e-4: eigenvalues of S up to 1e4 apart.
    Tolerance: S is off by a unit of its trace at most, so t by a unit of S's largest eigenvalue, which is below 1 + k max |z|^2.  The
    unit is 2^-16 where the operands of S are cut (fp32, d >= 32) and 2^-20 where they are not (d = 16).  bf16 tables: the result is
    rounded (2^-9 of every entry, 2^-8 allowed), and with d >= 32 the reference takes Z rounded as the library does; the 2^-17 that the two
    Z differ by before that rounding lets one entry in 250 fall on the other side of a tie, 2^-13 of |z|^2 in S."""
    say(f"rows of {lo} to {hi} entries d={d} {dtype} alpha={alpha}")
    gen = torch.Generator().manual_seed(d + 1)
    n, lam = 700, 1e-2
    H = (torch.randn((n, d), generator=gen) * 0.3 / np.sqrt(d)).to(dtype)
    lens = torch.cat([torch.arange(lo, hi + 1), torch.randint(lo, hi + 1, (43,), generator=gen), torch.tensor([lo, hi, 3])])
    ptr = torch.zeros(len(lens) + 1, dtype=torch.int64)
    ptr[1:] = torch.cumsum(lens, 0)
    idx = torch.randint(0, n, (int(ptr[-1]),), generator=gen).to(torch.int32)
    idx[ptr[20] + 3:ptr[20] + lo] = idx[ptr[20]]
    val = torch.randn(int(ptr[-1]), generator=gen)
    val[ptr[5]:ptr[6]] = 0
    G = (H.double().T @ H.double()).float()
    B = alpha * G.double().numpy() + lam * np.eye(d)
    X = torch.empty((len(lens), d), device=gpu_device, dtype=dtype)
    als.als_solve_rows(ctx, als.Csr(len(lens), n, ptr.to(gpu_device), idx.to(gpu_device), val.to(gpu_device)), H.to(gpu_device),
                       G.to(gpu_device), als.make_params(alpha, lam), X)
    als.als_status_sync(ctx)
    got, bf16 = f64(X), dtype == torch.bfloat16
    unit = 2.0 ** -20 if d == 16 else 2.0 ** -13 if bf16 else 2.0 ** -16
    L = np.linalg.cholesky(B)
    Z = np.linalg.solve(L, f64(H).T).T
    if bf16 and d >= 32:
        Z = f64(torch.tensor(Z).to(torch.bfloat16))
    worst = 0.0
    for r in range(len(lens)):
        z, y = Z[idx[ptr[r]:ptr[r + 1]].numpy()], val[ptr[r]:ptr[r + 1]].double().numpy()
        ref = np.linalg.solve(L.T, z.T @ np.linalg.solve(np.eye(len(z)) + z @ z.T, y))
        z2 = np.max(np.sum(z * z, axis=1))
        bound = (2.0 ** -8 if bf16 else 0.0) + (1 if bf16 else 4) * unit * (1 + len(z) * z2)
        error = np.linalg.norm(got[r] - ref)
        worst = max(worst, error / (bound * max(np.linalg.norm(ref), 1e-30)))
        assert bound < 0.1 and error <= bound * np.linalg.norm(ref), (r, len(z), bound)
    say(f"largest error, of its bound: {worst:.3f}")


@pytest.mark.parametrize("d,dtype", [(32, torch.float32), (64, torch.bfloat16)])
@pytest.mark.parametrize("most", [8192, 512 * 256])
def test_rows_are_sorted_alike_on_both_sides_of_a_line(ctx, gpu_device, d, dtype, most):
    """8192 rows are the most that one workgroup sorts into the lists by itself, 512 per compute unit the most that are sorted two
    a thread.  One row more, rows of every class (empty, each side of the class boundaries, beyond the split threshold) in one
    call, and the same rows in two ranges: which list place a row gets does not enter its result, so the bits are the same."""
    say(f"lists d={d} {dtype} {most}")
    ks = [0, 1, 4, 5, 8, 9, 16, 17, 32, 33, 48, 64, 65, 3, 2, 7]
    k = torch.tensor(ks, device=gpu_device).repeat(most // 16 + 1)[:most + 1]
    k[[5, 1024, 4096, most - 1, most]] = torch.tensor([513, 700, 1025, 2000, 512], device=gpu_device)
    n, nnz = 3000, int(k.sum())
    indptr = torch.zeros(most + 2, dtype=torch.int64, device=gpu_device)
    indptr[1:] = torch.cumsum(k, 0)
    gen = torch.Generator(device=gpu_device).manual_seed(d)
    Y = als.Csr(most + 1, n, indptr, torch.randint(0, n, (nnz,), device=gpu_device, generator=gen).to(torch.int32),
                torch.rand(nnz, device=gpu_device, generator=gen) + 0.5)
    H = (0.1 * torch.randn((n, d), device=gpu_device, generator=gen)).to(dtype)
    G = als.als_gramian(ctx, H)
    prm = als.make_params(0.1, 1e-2)
    whole, parts = (torch.full((most + 1, d), 7.0, dtype=dtype, device=gpu_device) for _ in range(2))
    als.als_solve_rows(ctx, Y, H, G, prm, whole)
    als.als_solve_rows(ctx, Y, H, G, prm, parts, 0, most)
    als.als_solve_rows(ctx, Y, H, G, prm, parts, most, most + 1)
    als.als_status_sync(ctx)
    assert torch.equal(whole, parts)
    assert not whole[k == 0].any()


@pytest.mark.parametrize("d,dtype", [(32, torch.float32), (64, torch.float32), (128, torch.float32), (32, torch.bfloat16), (128, torch.bfloat16)])
@pytest.mark.parametrize("walked", [False, True])
def test_places_past_the_end_of_a_list_raise_no_flag(ctx, gpu_device, d, dtype, walked):
    """alpha = 0 and a tiny lambda: |z|^2 about 1e9, where a system of one entry repeated is singular in fp32.  Rows of 9 to 16 and
    of 17 and 18 distinct entries are regular; lists of every length modulo four, by the launch that small calls share and (300 000
    empty rows more) by the launches of their own.  fp32 rows are compared too: S is off by 2^-16 of its trace at most."""
    say(f"past the end of a list d={d} {dtype} walked={walked}")
    gen = torch.Generator().manual_seed(d)
    n, lam = 4000, 1e-10
    H = (torch.randn((n, d), generator=gen) * 0.3 / np.sqrt(d)).to(dtype)
    G = torch.zeros((d, d), device=gpu_device)
    some = 17_000 if walked else 4
    for more in range(4):
        lens = torch.cat([torch.full((some + more,), 17), torch.tensor([18]), torch.full((1 + more,), 9 + 2 * more),
                          torch.zeros(300_000 if walked else 0, dtype=torch.int64)])
        ptr = torch.zeros(len(lens) + 1, dtype=torch.int64)
        ptr[1:] = torch.cumsum(lens, 0)
        nnz = int(ptr[-1])
        start = torch.repeat_interleave(torch.randint(0, n - 18, (len(lens),), generator=gen), lens)
        idx = (start + torch.arange(nnz) - torch.repeat_interleave(ptr[:-1], lens)).to(torch.int32)  # distinct in a row
        X = torch.empty((len(lens), d), device=gpu_device, dtype=dtype)
        Y = als.Csr(len(lens), n, ptr.to(gpu_device), idx.to(gpu_device))
        als.als_solve_rows(ctx, Y, H.to(gpu_device), G, als.make_params(0.0, lam), X)
        als.als_status_sync(ctx)
        got = f64(X)
        assert np.isfinite(got).all()
        if dtype == torch.float32:
            for r in range(some, some + 2 * more + 2):
                v = f64(H)[idx[ptr[r]:ptr[r + 1]].numpy()]
                s = lam * np.eye(len(v)) + v @ v.T
                ref, ev = v.T @ np.linalg.solve(s, np.ones(len(v))), np.linalg.eigvalsh(s)
                assert np.linalg.norm(got[r] - ref) <= 4 * 2.0 ** -16 * np.trace(s) / ev[0] * np.linalg.norm(ref), (r, len(v))


def _triangular_solves_in_fp32(S, y):
    """S t = y for many small systems by Cholesky's factor and two substitutions, every multiply-add rounded once to fp32."""
    n, L, t = S.shape[-1], S.astype(np.float64), y.astype(np.float64)
    fp32 = lambda x: x.astype(np.float32).astype(np.float64)
    inv = np.empty_like(t)
    for c in range(n):
        inv[:, c] = fp32(1.0 / np.sqrt(L[:, c, c]))
        L[:, :, c] = fp32(L[:, :, c] * inv[:, c, None])
        L[:, :, c + 1:] = fp32(L[:, :, c + 1:] - L[:, :, c, None] * L[:, None, c + 1:, c])
    for c in range(n):
        t[:, c] = fp32(t[:, c] * inv[:, c])
        t[:, c + 1:] = fp32(t[:, c + 1:] - L[:, c + 1:, c] * t[:, c, None])
    for c in reversed(range(n)):
        t[:, c] = fp32(t[:, c] * inv[:, c])
        t[:, :c] = fp32(t[:, :c] - L[:, c, :c] * t[:, c, None])
    return t


@pytest.mark.parametrize("k", [9, 12, 15, 16])
@pytest.mark.parametrize("scale", [0.25, 1.0, 4.0])
def test_small_systems_are_solved_no_less_exactly_than_by_triangular_solves(ctx, gpu_device, k, scale):
    """alpha = 0, lambda = 1 and entries that are few bits long: Z = V and S = I + V V^T are exact, so what is left of the error is the
    solve's (conditions 2 to 300).  Compared with triangular solves whose multiply-adds round once.  A model of both forms of the solve on
    the CPU: refined 0.64 to 0.80 of the triangular error, not refined 1.0 to 1.12."""
    say(f"precision of small systems k={k} scale={scale}")
    d, rows, gen = 16, 600, np.random.default_rng(k)
    v = gen.integers(-16, 17, (rows, k, d)) / 16 * scale
    y = gen.integers(-64, 65, (rows, k)) / 64
    S = np.eye(k) + v @ v.transpose(0, 2, 1)
    assert (S.astype(np.float32) == S).all()
    ref = np.einsum("bid,bi->bd", v, np.linalg.solve(S, y[:, :, None])[:, :, 0])
    tri = np.zeros((rows, d))
    t = _triangular_solves_in_fp32(S, y)
    for e in range(k):
        tri = (tri + v[:, e] * t[:, e, None]).astype(np.float32).astype(np.float64)
    Y = als.Csr(rows, rows * k, torch.arange(0, rows * k + 1, k, device=gpu_device), torch.arange(rows * k, device=gpu_device, dtype=torch.int32),
                torch.tensor(y.reshape(-1), dtype=torch.float32, device=gpu_device))
    V = torch.tensor(v.reshape(-1, d), dtype=torch.float32, device=gpu_device)
    X = torch.empty((rows, d), device=gpu_device)
    als.als_solve_rows(ctx, Y, V, torch.zeros((d, d), device=gpu_device), als.make_params(0.0, 1.0), X)
    als.als_status_sync(ctx)
    error = lambda x: np.median(np.linalg.norm(x - ref, axis=1) / np.linalg.norm(ref, axis=1))
    say(f"error {error(f64(X)):.3e}, triangular {error(tri):.3e}")
    assert error(f64(X)) <= 0.9 * error(tri)


def _fastest_call(ctx, Y, H, G, X, repeats=20):
    """us of als_solve_rows, the fastest of several calls."""
    times = []
    for _ in range(repeats):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        als.als_solve_rows(ctx, Y, H, G, als.make_params(0.1, 1e-2), X)
        end.record()
        end.synchronize()
        times.append(1e3 * start.elapsed_time(end))
    als.als_status_sync(ctx)
    return min(times)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_empty_rows_cost_no_more_in_one_workgroup_than_in_many(ctx, gpu_device, dtype):
    """8192 rows are sorted by one workgroup, 8193 by seventeen; with nearly all of them empty, d = 128, zeroing is most of the work.  It took
    six times as long in one workgroup when every thread wrote its rows element by element; half again as long is allowed."""
    say(f"empty rows in one workgroup {dtype}")
    d, n = 128, 1000
    H = torch.randn((n, d), device=gpu_device).to(dtype)
    G, best = als.als_gramian(ctx, H), []
    for rows in (8192, 8193):
        X = torch.full((rows, d), 7.0, device=gpu_device, dtype=dtype)
        indptr = torch.zeros(rows + 1, dtype=torch.int64, device=gpu_device)
        indptr[-1] = 3
        best.append(_fastest_call(ctx, als.Csr(rows, n, indptr, torch.arange(3, dtype=torch.int32, device=gpu_device)), H, G, X))
        assert not X[:-1].any() and X[-1].any()
    assert best[0] <= 1.5 * best[1], best


def test_long_rows_are_cut_as_fast_in_one_workgroup_as_in_many(ctx, gpu_device):
    """8192 rows of 600 entries, two segments each, d = 16: 147 us in one workgroup that reserved places and divided in 64 bits row by row, 95
    by several; 103 as it is, and a quarter more than by several is allowed."""
    say("long rows in one workgroup")
    d, n, k, best = 16, 3000, 600, []
    gen = torch.Generator(device=gpu_device).manual_seed(1)
    H = torch.randn((n, d), device=gpu_device, generator=gen)
    G = als.als_gramian(ctx, H)
    idx = torch.randint(0, n, (8193 * k,), device=gpu_device, generator=gen).to(torch.int32)
    for rows in (8192, 8193):
        X = torch.empty((rows, d), device=gpu_device)
        Y = als.Csr(rows, n, torch.arange(0, rows * k + 1, k, device=gpu_device), idx[:rows * k].clone())
        best.append(_fastest_call(ctx, Y, H, G, X))
    say(f"us {best}")
    assert best[0] <= 1.25 * best[1], best


@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_classes_in_launches_of_their_own_and_in_a_common_one(ctx, gpu_device, d, dtype):
    """300 003 rows have lists for launches of their own (walked lists, tiles kept in registers), 15 000 of them share one launch (single
    steps, 16 < k <= 32 in fp32 with a second gather): the same labelled rows both ways, bit for bit.  Some rows are compared with fp64."""
    say(f"own and common launches d={d} {dtype}")
    rows, part, n, alpha, lam = 300_003, 15_000, 5000, 0.1, 1e-2
    gen = torch.Generator(device=gpu_device).manual_seed(d)
    rnd = lambda lo, hi, size: torch.randint(lo, hi, (size,), device=gpu_device, generator=gen)
    lens = torch.where(rnd(0, 4, rows) == 0, rnd(17, 33, rows), rnd(0, 17, rows))
    lens = torch.where(rnd(0, 40, rows) == 0, rnd(33, 160, rows), lens)
    indptr = torch.zeros(rows + 1, dtype=torch.int64, device=gpu_device)
    indptr[1:] = torch.cumsum(lens, 0)
    nnz = int(indptr[-1])
    Y = als.Csr(rows, n, indptr, rnd(0, n, nnz).to(torch.int32), torch.randn(nnz, device=gpu_device, generator=gen))
    H = (torch.randn((n, d), device=gpu_device, generator=gen) * 0.3 / np.sqrt(d)).to(dtype)
    G, prm = als.als_gramian(ctx, H), als.make_params(alpha, lam)
    whole, parts = (torch.full((rows, d), 7.0, device=gpu_device, dtype=dtype) for _ in range(2))
    als.als_solve_rows(ctx, Y, H, G, prm, whole)
    for r0 in range(0, rows, part):
        als.als_solve_rows(ctx, Y, H, G, prm, parts, r0, min(rows, r0 + part))
    als.als_status_sync(ctx)
    assert torch.equal(whole, parts)
    B, h = alpha * f64(G) + lam * np.eye(d), f64(H)
    for r in range(0, rows, 3001):
        at = slice(int(indptr[r]), int(indptr[r + 1]))
        v, y = h[Y.indices[at].cpu().numpy()], f64(Y.values[at])
        ref = np.linalg.solve(B + v.T @ v, v.T @ y)
        # the entries of S are off by 2^-16 |z|^2 (fp32) or, as Z is rounded, 2^-8 |z|^2 (bf16), and S has no eigenvalue below 1
        z2 = np.max(np.sum(v * np.linalg.solve(B, v.T).T, axis=1), initial=0.0)
        unit = 2.0 ** -16 if dtype == torch.float32 else 2.0 ** -8
        assert np.linalg.norm(f64(whole[r]) - ref) <= unit * (1 + len(v) * z2) * np.linalg.norm(ref), (r, len(v))


@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rows_of_tables_with_a_stride(ctx, gpu_device, d, dtype):
    """Tables whose rows are further apart than d: the same bits as without, empty rows zeroed one by one and in runs, and neither what
    lies between the rows nor rows outside the range written (a range that starts and ends inside a wavefront's 64 rows)."""
    say(f"strided tables d={d} {dtype}")
    rows, n, r0, r1 = 1500, 300, 3, 1497
    gen = torch.Generator(device=gpu_device).manual_seed(d)
    k = torch.randint(0, 40, (rows,), device=gpu_device, generator=gen)
    k[torch.rand(rows, device=gpu_device, generator=gen) < 0.4] = 0
    k[400:700] = 0
    k[[10, 800]] = 600
    indptr = torch.zeros(rows + 1, dtype=torch.int64, device=gpu_device)
    indptr[1:] = torch.cumsum(k, 0)
    Y = als.Csr(rows, n, indptr, torch.randint(0, n, (int(indptr[-1]),), device=gpu_device, generator=gen).to(torch.int32))
    H = (0.2 * torch.randn((n, d), device=gpu_device, generator=gen)).to(dtype)
    wide_h = torch.full((n, d + 16), float("nan"), device=gpu_device, dtype=dtype)
    wide_h[:, :d] = H
    wide_x = torch.full((rows, d + 8), 7.0, device=gpu_device, dtype=dtype)
    X = torch.full((rows, d), 7.0, device=gpu_device, dtype=dtype)
    G, prm = als.als_gramian(ctx, H), als.make_params(0.1, 1e-2)
    als.als_solve_rows(ctx, Y, H, G, prm, X, r0, r1)
    als.als_solve_rows(ctx, Y, wide_h[:, :d], G, prm, wide_x[:, :d], r0, r1)
    als.als_status_sync(ctx)
    assert torch.equal(wide_x[:, :d], X) and (wide_x[:, d:] == 7).all()
    assert (X[:r0] == 7).all() and (X[r1:] == 7).all() and torch.equal((X[r0:r1] == 0).all(dim=1), k[r0:r1] == 0)


@pytest.mark.parametrize("d,dtype", [(64, torch.float32), (128, torch.float32), (32, torch.bfloat16), (64, torch.bfloat16), (128, torch.bfloat16)])
@pytest.mark.parametrize("rows", [1, 4, 5, 15, 16, 17, 35])
def test_rows_that_leave_their_kernel_as_solutions(ctx, gpu_device, d, dtype, rows):
    """Launches of their own take X = R L^-1 along, sixteen rows at a time: `rows` rows of each class, which do not fill the last sixteen,
    in a strided table, against the launch that small calls share and its pass over the lists, bit for bit."""
    say(f"solved in their kernel d={d} {dtype} rows={rows}")
    gen = torch.Generator(device=gpu_device).manual_seed(rows)
    n, few = 700, rows * 5
    lens = torch.cat([torch.full((rows,), k) for k in (2, 7, 13, min(d, 25), min(d, 45))] + [torch.zeros(320_000, dtype=torch.int64)])
    lens = lens.to(gpu_device)
    indptr = torch.zeros(len(lens) + 1, dtype=torch.int64, device=gpu_device)
    indptr[1:] = torch.cumsum(lens, 0)
    nnz = int(indptr[-1])
    Y = als.Csr(len(lens), n, indptr, torch.randint(0, n, (nnz,), device=gpu_device, generator=gen).to(torch.int32),
                torch.rand(nnz, device=gpu_device, generator=gen) + 0.5)
    H = (torch.randn((n, d), device=gpu_device, generator=gen) * 0.3 / np.sqrt(d)).to(dtype)
    G, prm = als.als_gramian(ctx, H), als.make_params(0.1, 1e-2)
    own = torch.full((len(lens), d + 16), 7.0, device=gpu_device, dtype=dtype)
    common = torch.full((len(lens), d), 7.0, device=gpu_device, dtype=dtype)
    als.als_solve_rows(ctx, Y, H, G, prm, own[:, :d])
    als.als_solve_rows(ctx, Y, H, G, prm, common, 0, few)
    als.als_status_sync(ctx)
    assert torch.equal(own[:few, :d], common[:few]) and (own[:, d:] == 7).all()
    assert not own[few:, :d].any() and (common[few:] == 7).all() and torch.isfinite(common[:few]).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("alpha", [0.1, 1e-4])
def test_rows_of_33_to_48_entries_one_and_four_per_wavefront(ctx, gpu_device, d, dtype, alpha):
    """20 000 rows take the launch of four rows per wavefront once a call has seen them, and before that, like a few of them, the launch that
    small calls share, where each has a wavefront: the same bits for every length, entries that repeat and labels of both signs and
    zero.  Tolerance as for rows of 9 to 32 entries."""
    say(f"rows of 33 to 48 entries d={d} {dtype} alpha={alpha}")
    rows, n, lam = 20_000, 900, 1e-2
    gen = torch.Generator(device=gpu_device).manual_seed(d)
    lens = 33 + torch.randint(0, 16, (rows,), device=gpu_device, generator=gen)
    lens[:16] = 33 + torch.arange(16, device=gpu_device)
    indptr = torch.zeros(rows + 1, dtype=torch.int64, device=gpu_device)
    indptr[1:] = torch.cumsum(lens, 0)
    idx = torch.randint(0, n, (int(indptr[-1]),), device=gpu_device, generator=gen).to(torch.int32)
    idx[int(indptr[20]) + 3:int(indptr[21])] = idx[int(indptr[20])]
    val = torch.randn(len(idx), device=gpu_device, generator=gen)
    val[int(indptr[5]):int(indptr[6])] = 0
    Y = als.Csr(rows, n, indptr, idx, val)
    H = (torch.randn((n, d), device=gpu_device, generator=gen) * 0.3 / np.sqrt(d)).to(dtype)
    G, prm = als.als_gramian(ctx, H), als.make_params(alpha, lam)
    first, whole, parts = (torch.full((rows, d), 7.0, device=gpu_device, dtype=dtype) for _ in range(3))
    als.als_solve_rows(ctx, Y, H, G, prm, first)
    als.als_status_sync(ctx)
    ran = _launches(ctx, lambda: als.als_solve_rows(ctx, Y, H, G, prm, whole))
    assert ran["dual_k48"] == 1 and ran["dual_k16"] == 1, ran  # the class, and the common launch for what else there is
    for r0, r1 in ((0, 1), (1, 4), (4, 40), (40, 1500)):
        als.als_solve_rows(ctx, Y, H, G, prm, parts, r0, r1)
    als.als_status_sync(ctx)
    assert torch.equal(first, whole) and torch.equal(whole[:1500], parts[:1500]) and (parts[1500:] == 7).all()
    bf16, h = dtype == torch.bfloat16, f64(H)
    L = np.linalg.cholesky(alpha * f64(G) + lam * np.eye(d))
    Z = np.linalg.solve(L, h.T).T
    if bf16:
        Z = f64(torch.tensor(Z).to(torch.bfloat16))
    unit = 2.0 ** -13 if bf16 else 2.0 ** -16
    for r in list(range(24)) + [1499, 9999, rows - 1]:
        at = slice(int(indptr[r]), int(indptr[r + 1]))
        z, y = Z[idx[at].cpu().numpy()], f64(val[at])
        ref = np.linalg.solve(L.T, z.T @ np.linalg.solve(np.eye(len(z)) + z @ z.T, y))
        bound = (2.0 ** -8 if bf16 else 0.0) + (1 if bf16 else 4) * unit * (1 + len(z) * np.max(np.sum(z * z, axis=1)))
        assert bound < 0.5 and np.linalg.norm(f64(whole[r]) - ref) <= bound * np.linalg.norm(ref), (r, len(z), bound)


@pytest.mark.parametrize("d,dtype", [(32, torch.float32), (64, torch.float32), (128, torch.float32), (32, torch.bfloat16), (128, torch.bfloat16)])
def test_places_past_the_end_of_walked_lists_raise_no_flag(ctx, gpu_device, d, dtype):
    """The same with lists of 24 000 rows of 17 entries and 400 000 empty rows: the lists' capacities follow entries and rows, and go
    beyond the 2^17 steps of the common launch, so that the launches of their own run."""
    say(f"past the end of a walked list d={d} {dtype}")
    gen = torch.Generator().manual_seed(d)
    n, lam = 4000, 1e-10
    H = (torch.randn((n, d), generator=gen) * 0.3 / np.sqrt(d)).to(dtype)
    G = torch.zeros((d, d), device=gpu_device)
    some = 24_000
    for more in range(4):
        lens = torch.cat([torch.full((some + more,), 17), torch.tensor([18]), torch.full((1 + more,), 9 + 2 * more),
                          torch.zeros(400_000, dtype=torch.int64)])
        ptr = torch.zeros(len(lens) + 1, dtype=torch.int64)
        ptr[1:] = torch.cumsum(lens, 0)
        nnz = int(ptr[-1])
        start = torch.repeat_interleave(torch.randint(0, n - 18, (len(lens),), generator=gen), lens)
        idx = (start + torch.arange(nnz) - torch.repeat_interleave(ptr[:-1], lens)).to(torch.int32)  # distinct in a row
        X = torch.empty((len(lens), d), device=gpu_device, dtype=dtype)
        Y = als.Csr(len(lens), n, ptr.to(gpu_device), idx.to(gpu_device))
        ran = _launches(ctx, lambda: als.als_solve_rows(ctx, Y, H.to(gpu_device), G, als.make_params(0.0, lam), X))
        assert ran["dual_k16"] == 1 and ran["dual_k32"] == 1, ran
        als.als_status_sync(ctx)
        assert torch.isfinite(X).all()
        got = f64(X[:some + 20])
        if dtype == torch.float32:
            for r in range(some, some + 2 * more + 2):
                v = f64(H)[idx[ptr[r]:ptr[r + 1]].numpy()]
                s = lam * np.eye(len(v)) + v @ v.T
                ref, ev = v.T @ np.linalg.solve(s, np.ones(len(v))), np.linalg.eigvalsh(s)
                assert np.linalg.norm(got[r] - ref) <= 4 * 2.0 ** -16 * np.trace(s) / ev[0] * np.linalg.norm(ref), (r, len(v))


@pytest.mark.parametrize("d,dtype", [(64, torch.float32), (128, torch.float32), (32, torch.bfloat16), (64, torch.bfloat16), (128, torch.bfloat16)])
@pytest.mark.parametrize("rows", [1, 4, 5, 15, 16, 17, 35])
def test_rows_solved_in_launches_of_their_own_and_in_the_common_one(ctx, gpu_device, d, dtype, rows):
    """Launches of their own take X = R L^-1 along, sixteen rows at a time: `rows` rows of each class, which do not fill the last sixteen,
    in a strided table, against the launch that small calls share and its pass over the lists, bit for bit.  320 000 rows too long for the
    dual form, or empty, bring the lists' capacities, which follow rows and entries, beyond the 2^17 steps of the common launch."""
    say(f"own launches and the common one d={d} {dtype} rows={rows}")
    gen = torch.Generator(device=gpu_device).manual_seed(rows)
    n, few = 700, rows * 5
    lens = torch.cat([torch.full((rows,), k) for k in (2, 7, 13, min(d, 25), min(d, 45))]
                     + [torch.full((4000,), 500), torch.zeros(316_000, dtype=torch.int64)])
    lens = lens.to(gpu_device)
    indptr = torch.zeros(len(lens) + 1, dtype=torch.int64, device=gpu_device)
    indptr[1:] = torch.cumsum(lens, 0)
    nnz = int(indptr[-1])
    Y = als.Csr(len(lens), n, indptr, torch.randint(0, n, (nnz,), device=gpu_device, generator=gen).to(torch.int32),
                torch.rand(nnz, device=gpu_device, generator=gen) + 0.5)
    H = (torch.randn((n, d), device=gpu_device, generator=gen) * 0.3 / np.sqrt(d)).to(dtype)
    G, prm = als.als_gramian(ctx, H), als.make_params(0.1, 1e-2)
    own = torch.full((len(lens), d + 16), 7.0, device=gpu_device, dtype=dtype)
    common = torch.full((len(lens), d), 7.0, device=gpu_device, dtype=dtype)
    for _ in range(2):  # without and with a hint
        ran = _launches(ctx, lambda: als.als_solve_rows(ctx, Y, H, G, prm, own[:, :d]))
        assert all(ran[name] == 1 for name in ["dual_k4", "dual_k8", "dual_k16", "dual_k32"] + ["dual_k48"] * (d >= 64)), ran
        als.als_status_sync(ctx)
    # (the rows in a matrix of their own: of the large one the entries would bring the capacities along)
    small = als.Csr(few, n, indptr[:few + 1].clone(), Y.indices[:int(indptr[few])].clone(), Y.values[:int(indptr[few])].clone())
    ran = _launches(ctx, lambda: als.als_solve_rows(ctx, small, H, G, prm, common[:few]))
    assert ran["dual_k16"] == 1 and ran["dual_k4"] == ran["dual_k8"] == ran["dual_k32"] == ran["dual_k48"] == 0, ran
    als.als_status_sync(ctx)
    assert torch.equal(own[:few, :d], common[:few]) and (own[:, d:] == 7).all()
    assert not own[few + 4000:, :d].any() and torch.isfinite(own.float()).all() and not (own[:few + 4000, :d] == 7).all(dim=1).any()

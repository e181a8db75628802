"""The work that a user of this library has it do, as cases that can be timed and compared.

Four kinds of call, each through the public entry points of ``paper_2112_02194_amd.binding``:

``epoch``   one training epoch (both half-epochs and both Gramians) of a link matrix, in place
``foldin``  rows that were not trained are embedded against a fixed item table (``als_solve_rows`` with the
            Gramian that a serving program keeps)
``topk``    exact retrieval of the best items for a block of embedded rows
``loss``    the value of the objective, as watched between epochs

Matrices come from the repository's own recipes (``synth``: c1 to c5), tables are drawn on the GPU from the seed.
A program keeps one context for its whole life, and so does this file.
"""
from __future__ import annotations

import math

import torch

from paper_2112_02194_amd import binding as als
from synth import CONFIGS, make_problem

DEV = "cuda:0"
# entries per row of each recipe (c1 drops duplicates, which brings its drawn 27.8 down)
MEAN_DEGREE = {"c1": 20.2, "c2": 30.0, "c3": 20.0, "c4": 6.0, "c5": 25.0}
FOLD_DEGREE = 15.0  # three quarters of a row's 20 links are given, the rest is held out

_context = None


def context() -> als.Context:
    global _context
    if _context is None:
        _context = als.Context(0)
    return _context


# --------------------------------------------------------------------------- the cases

def listed():
    def epoch(name, recipe, rows, cols, d, dtype, values=False):
        return {"name": name, "kind": "epoch", "recipe": recipe, "rows": rows, "cols": cols, "d": d, "dtype": dtype,
                "values": values}

    return [
        # the smallest training job: every kernel is short, launches and host work count
        epoch("epoch_c1", "c1", 2000, 1500, 16, "f32"),
        # an ordinary job of odd sizes with graded labels (ratings, dwell times) and hubs
        epoch("epoch_labels", "c2", 50_021, 30_011, 32, "f32", values=True),
        # 1M nodes, heavy-tailed degrees up to 5000
        epoch("epoch_c2", "c2", 1_000_000, 1_000_000, 64, "f32"),
        # the headline: 10M nodes with host locality and very popular columns
        epoch("epoch_c3", "c3", 10_000_000, 10_000_000, 128, "f32"),
        # many short rows: table passes and gathers of a few entries
        epoch("epoch_c4", "c4", 50_000_000, 50_000_000, 128, "f32"),
        # bf16 tables, power-law degrees up to 1e5 (half the nodes of the full recipe: three of them fit the card)
        epoch("epoch_c5", "c5", 50_000_000, 50_000_000, 128, "bf16"),
        # serving: a small batch of new users against a table in production
        {"name": "foldin_batch", "kind": "foldin", "rows": 256, "items": 1_000_003, "d": 128, "dtype": "f32", "values": False},
        # the evaluation protocol: all held-out rows of a trained model at once
        {"name": "foldin_eval", "kind": "foldin", "rows": 300_007, "items": 3_000_000, "d": 128, "dtype": "bf16", "values": False},
        # serving: one page of users against a small catalogue, links already known left out
        {"name": "topk_page", "kind": "topk", "queries": 64, "items": 30_000, "d": 64, "dtype": "f32", "k": 20, "exclude": True},
        # evaluation: a block of rows against 1M items (Recall@20)
        {"name": "topk_eval", "kind": "topk", "queries": 4096, "items": 1_000_000, "d": 64, "dtype": "f32", "k": 20, "exclude": False},
        # the same against a large bf16 table with exclusions (Recall@50)
        {"name": "topk_large", "kind": "topk", "queries": 4096, "items": 10_000_000, "d": 128, "dtype": "bf16", "k": 50, "exclude": True},
        # watching convergence on the 1M-node job
        {"name": "loss_c2", "kind": "loss", "recipe": "c2", "rows": 1_000_000, "cols": 1_000_000, "d": 64, "dtype": "f32",
         "values": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["epoch", "epoch", "epoch", "foldin", "foldin", "topk", "topk", "loss"])
    d = rng.choice([16, 32, 64, 64, 128, 128])
    dtype = rng.choice(["f32", "f32", "bf16"])
    if kind in ("epoch", "loss"):
        recipe = rng.choice(["c1", "c2", "c3", "c4", "c5"])
        rows = _log_int(rng, 1000, 3_000_000)
        # the host recipe is a square link matrix; the others also stand for user x item matrices
        cols = rows if recipe == "c3" else min(3_000_000, max(1000, int(rows * math.exp(rng.uniform(-1.0, 1.0)))))
        return {"kind": kind, "recipe": recipe, "rows": rows, "cols": cols, "d": d, "dtype": dtype,
                "values": rng.random() < 0.3}
    if kind == "foldin":
        return {"kind": kind, "rows": _log_int(rng, 1, 300_000), "items": _log_int(rng, 10_000, 3_000_000), "d": d,
                "dtype": dtype, "values": rng.random() < 0.3}
    queries = _log_int(rng, 1, 8192)
    items = _log_int(rng, 5000, min(10_000_000, 4_000_000_000 // queries))
    return {"kind": kind, "queries": queries, "items": items, "d": d, "dtype": dtype, "k": rng.choice([10, 20, 50]),
            "exclude": rng.random() < 0.5}


# --------------------------------------------------------------------------- inputs

def _torch_dtype(case):
    return {"f32": torch.float32, "bf16": torch.bfloat16}[case["dtype"]]


def _initial_table(rows, d, dtype, gen):
    """N(0, 0.1 / sqrt(d)), the initialisation of a training run."""
    out = torch.empty((rows, d), dtype=dtype, device=DEV)
    out.normal_(0.0, 0.1 / math.sqrt(d), generator=gen)
    return out


def _trained_table(rows, d, dtype, gen, scales_gen):
    """Rows as training leaves them: a decaying spectrum in a rotated basis (the same one for both sides of a model)
    and norms that differ from row to row."""
    scale = 0.3 / math.sqrt(d) * torch.arange(1, d + 1, device=DEV, dtype=torch.float32) ** -0.5
    basis, _ = torch.linalg.qr(torch.randn((d, d), device=DEV, generator=scales_gen))
    mix = scale[:, None] * basis
    out = torch.empty((rows, d), dtype=dtype, device=DEV)
    for r0 in range(0, rows, 1 << 20):
        n = min(1 << 20, rows - r0)
        x = torch.randn((n, d), device=DEV, generator=gen) @ mix
        out[r0:r0 + n] = x * torch.exp(0.5 * torch.randn((n, 1), device=DEV, generator=gen))
    return out


def _links(rows, items, mean, values, gen):
    """Given links of new rows: four of five inside one neighbourhood of about a hundred items, the others popular
    items; distinct within a row."""
    u = torch.rand(rows, device=DEV, generator=gen, dtype=torch.float64)
    deg = (1 + torch.floor(torch.log(u) / math.log(1.0 - 1.0 / mean))).clamp_(1, 1500).to(torch.int64)
    owner = torch.repeat_interleave(torch.arange(rows, device=DEV), deg)
    n = owner.numel()
    base = torch.randint(0, max(1, items - 100), (rows,), device=DEV, generator=gen)
    near = base[owner] + torch.randint(0, min(100, items), (n,), device=DEV, generator=gen)
    rank = torch.exp(torch.rand(n, device=DEV, generator=gen, dtype=torch.float64) * math.log(items)).to(torch.int64)
    popular = (rank * 2654435761) % items
    ids = torch.where(torch.rand(n, device=DEV, generator=gen) < 0.8, near, popular)
    key = torch.unique(owner * items + ids)
    owner = torch.div(key, items, rounding_mode="floor")
    indptr = torch.zeros(rows + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(owner, minlength=rows), 0, out=indptr[1:])
    vals = None
    if values:
        vals = torch.rand(key.numel(), device=DEV, generator=gen) + 0.5
    return als.Csr(rows, items, indptr, (key - owner * items).to(torch.int32), vals)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1_000_003 * seed + 17)
    dtype, d, kind = _torch_dtype(case), case["d"], case["kind"]
    state = {"kind": kind, "ctx": context()}
    if kind in ("epoch", "loss"):
        recipe = case["recipe"]
        p = make_problem(recipe, device=DEV, rows=case["rows"], cols=case["cols"], d=d, seed=CONFIGS[recipe]["seed"] + seed,
                         values="uniform" if case["values"] else "ones", tables=False)
        state["Y"] = als.Csr(p.rows, p.cols, p.indptr, p.indices, p.values)
        state["Yt"] = als.Csr(p.cols, p.rows, p.t_indptr, p.t_indices, p.t_values)
        state["W"] = _initial_table(p.rows, d, dtype, gen)
        state["H"] = _initial_table(p.cols, d, dtype, gen)
        state["params"] = als.make_params(p.alpha, p.lam)
        if kind == "loss":
            state.pop("Yt")
    elif kind == "foldin":
        H = _trained_table(case["items"], d, dtype, gen, gen)
        G = torch.zeros((d, d), dtype=torch.float64, device=DEV)
        for r0 in range(0, case["items"], 1 << 20):
            x = H[r0:r0 + (1 << 20)].double()
            G += x.T @ x
        state.update(H=H, G=G.float(), Y=_links(case["rows"], case["items"], FOLD_DEGREE, case["values"], gen),
                     X=torch.zeros((case["rows"], d), dtype=dtype, device=DEV), params=als.make_params(0.1, 1e-2))
    else:
        shared = torch.Generator(device=DEV)
        shared.manual_seed(seed)
        state["H"] = _trained_table(case["items"], d, dtype, gen, shared)
        shared.manual_seed(seed)
        state["Q"] = _trained_table(case["queries"], d, dtype, gen, shared)
        state["k"] = case["k"]
        state["exclude"] = _links(case["queries"], case["items"], FOLD_DEGREE, False, gen) if case["exclude"] else None
    torch.cuda.synchronize()
    torch.cuda.empty_cache()  # the generators' temporaries: the library takes its workspace from the driver
    return state


# --------------------------------------------------------------------------- one pass

def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind == "epoch":
        als.als_epoch(ctx, state["Y"], state["Yt"], state["W"], state["H"], state["params"])
        return {"W": state["W"], "H": state["H"]}
    if kind == "foldin":
        return als.als_solve_rows(ctx, state["Y"], state["H"], state["G"], state["params"], state["X"])
    if kind == "topk":
        ids, scores = als.als_topk(ctx, state["Q"], state["H"], state["k"], state["exclude"])
        return {"ids": ids, "scores": scores}
    return als.als_loss(ctx, state["Y"], state["W"], state["H"], state["params"])


# --------------------------------------------------------------------------- what a pass cannot do without

def _solve_flops(rows, k, d):
    """Rows with k entries each, by the cheaper of the two forms of the row system (k x k or d x d)."""
    dual = k * (k + 1) * d + k ** 3 / 3.0 + 4 * k * d
    primal = k * d * (d + 1) + d ** 3 / 3.0 + 2 * k * d + 2 * d * d
    return rows * min(dual, primal)


def work(case):
    kind, d = case["kind"], case["d"]
    es = 4 if case["dtype"] == "f32" else 2
    if kind in ("epoch", "loss"):
        m, n = case["rows"], case["cols"]
        nnz = m * min(MEAN_DEGREE[case["recipe"]], n)
        csr = nnz * (8 if case["values"] else 4)
        gram = (m + n) * d * (d + 1)
        if kind == "loss":
            return {"bytes": csr + 8 * m + (m + n) * d * es, "flops": nnz * (2 * d + 2) + gram}
        return {"bytes": 2 * csr + 8 * (m + n) + 2 * (m + n) * d * es,
                "flops": gram + _solve_flops(m, nnz / m, d) + _solve_flops(n, nnz / n, d)}
    if kind == "foldin":
        m, n = case["rows"], case["items"]
        nnz = m * FOLD_DEGREE
        touched = min(nnz, n)  # item rows that the batch refers to, at most
        return {"bytes": nnz * (8 if case["values"] else 4) + 8 * m + touched * d * es + m * d * es + d * d * 4,
                "flops": _solve_flops(m, FOLD_DEGREE, d) + 2 * touched * d * d + d ** 3 / 3.0}
    m, n = case["queries"], case["items"]
    ex = m * (8 + 4 * FOLD_DEGREE) if case["exclude"] else 0
    return {"bytes": (m + n) * d * es + m * case["k"] * 8 + ex, "flops": 2.0 * m * n * d}


def tolerance(case):
    """Measured on cut-down cases of every kind against the same computation in 64 bits and against the other form of
    the row systems (every row by its d x d equations); stated: about four times the largest difference seen.

    fp32 tables: d = 16 8e-7; d >= 32 up to 2.1e-5 after two epochs (the k x k systems are formed from operands cut to
    16 bits, hi + lo), single entries 8.4e-5.  bf16 tables: 4e-3, single entries 4e-2 (the results' own rounding and
    that of the transformed table).  Objective 7e-7.  Top-k scores 1.8e-7, single ones 7e-7, 8e-5 of the ids in another
    order (scores closer than their rounding)."""
    if case["kind"] == "loss":
        return {"rel": 3e-6}
    if case["kind"] == "topk":
        return {"rel": 8e-7, "max": 3e-6, "differ": 4e-4}
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 1e-1}
    return {"rel": 4e-6, "max": 4e-5} if case["d"] == 16 else {"rel": 6e-5, "max": 3e-4}

"""The work that users of this library have it do, as measurable cases.

`listed()` names twelve of them at the sizes of this repository's own configurations and benchmark; `draw` gives others
of the same kinds over the ranges those stand for.  Every case is one call, or one training loop, through the Python
binding, on tables, indices and plans that the caller's program already holds on the GPU.

A case describes the schema (`schema`: "star", "union" or "onehot", with its sizes) and the call (`call`):

  train        `iters` steps of batch gradient descent of `m` models from zero weights, with the loss of every step
  lmm, tmm     T X and T^T Y with `cx` operand columns
  gram         T^T T
  kmeans       one Lloyd iteration with `k` centroids
  materialize  the join written out

A star schema is an entity table `r_S` x `c_S` and the joined tables of `dims`, written as "ROWSxCOLS:KEYS" separated by
spaces; KEYS is "u" (uniform foreign keys) or "z" (Zipf 1.1).  `missing` is the share of the target rows whose key finds
no row in the last joined table.
"""
import math

import torch

import paper_2502_01985_amd as il

DEV = "cuda:0"


def listed():
    return [
        # The smallest call: a two-table join that fits a cache, where the launch and the host path count.
        {"name": "train_small", "schema": "star", "r_S": 10_000, "c_S": 4, "dims": "1000x8:u", "missing": 0.0,
         "call": "train", "model": "linear", "m": 1, "bf16": False, "iters": 20},
        # Scoring every row of a join with one trained model.
        {"name": "predict_star", "schema": "star", "r_S": 1_000_000, "c_S": 20, "dims": "100000x200:u", "missing": 0.0,
         "call": "lmm", "cx": 1, "bf16": False},
        # The transposed multiply with a block of right-hand sides: gradients of 16 models, sketches, block solvers.
        {"name": "gradient_star_16", "schema": "star", "r_S": 1_000_000, "c_S": 20, "dims": "100000x200:u", "missing": 0.0,
         "call": "tmm", "cx": 16, "bf16": False},
        # Odd sizes: rows that are not float4-aligned, unmatched keys, a few models at once.
        {"name": "train_ragged", "schema": "star", "r_S": 333_333, "c_S": 13, "dims": "9001x33:z 41003x75:u",
         "missing": 0.1, "call": "train", "model": "logistic", "m": 3, "bf16": False, "iters": 10},
        # Logistic regression over a three-dimension star schema with one skewed key: the ordinary large training.
        {"name": "train_star3", "schema": "star", "r_S": 5_000_000, "c_S": 10,
         "dims": "100000x50:u 50000x100:z 10000x40:u", "missing": 0.0,
         "call": "train", "model": "logistic", "m": 1, "bf16": False, "iters": 10},
        # The Gram matrix of two stacked sources with shared columns and partly matched entities.
        {"name": "gram_union", "schema": "union", "rows": 2_000_000, "cols": 64, "shared": 32, "overlap": 0.3,
         "call": "gram"},
        # The Gram matrix of a star join (normal equations, PCA).
        {"name": "gram_star", "schema": "star", "r_S": 1_000_000, "c_S": 20, "dims": "100000x200:u", "missing": 0.0,
         "call": "gram"},
        # A hyper-parameter sweep: 256 models at once, in float32 and with bfloat16 inputs.
        {"name": "sweep_f32", "schema": "star", "r_S": 1_000_000, "c_S": 20, "dims": "100000x200:u", "missing": 0.0,
         "call": "train", "model": "linear", "m": 256, "bf16": False, "iters": 5},
        {"name": "sweep_bf16", "schema": "star", "r_S": 1_000_000, "c_S": 20, "dims": "100000x200:u", "missing": 0.0,
         "call": "train", "model": "linear", "m": 256, "bf16": True, "iters": 5},
        # Clustering the rows of a join: a left multiply, the nearest centroid, a transposed multiply.
        {"name": "kmeans_star", "schema": "star", "r_S": 1_000_000, "c_S": 20, "dims": "100000x200:u", "missing": 0.0,
         "call": "kmeans", "k": 10},
        # Sparse tables of one-hot encoded attributes (the shape of the paper's Movie data set).
        {"name": "train_onehot", "schema": "onehot", "r_T": 1_000_000, "dims": "6040x9510 3710x3840", "attributes": 20,
         "call": "train", "model": "logistic", "m": 1, "bf16": False, "iters": 10},
        # The join itself, for a user who is told to materialize: the largest output.
        {"name": "join_star3", "schema": "star", "r_S": 5_000_000, "c_S": 10,
         "dims": "100000x50:u 50000x100:z 10000x40:u", "missing": 0.0, "call": "materialize"},
    ]


# ------------------------------------------------------------------------------------------------- drawn cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _star(rng, most_dims, r_S, zipf):
    rows = _log(rng, *r_S)
    dims = []
    for _ in range(rng.randint(1, most_dims)):
        keys = "z" if zipf and rng.random() < 0.3 else "u"
        cols = _log(rng, 4, 100) if most_dims > 1 else _log(rng, 8, 200)
        dims.append("%dx%d:%s" % (min(rows, _log(rng, 1_000, 100_000)), cols, keys))
    return {"schema": "star", "r_S": rows, "c_S": rng.randint(3, 24), "dims": " ".join(dims),
            "missing": rng.choice([0.0, 0.0, 0.1])}


def draw(rng):
    kind = rng.choice(["train", "multi", "operator", "operator", "sweep", "gram_star", "gram_union", "kmeans", "onehot", "join"])
    if kind == "train":       # one or a few models on a star join, small to large
        return {**_star(rng, 1, (5_000, 1_000_000), False), "call": "train", "model": rng.choice(["linear", "logistic"]),
                "m": rng.randint(1, 4), "bf16": False, "iters": 10}
    if kind == "multi":       # logistic regression on up to three joined tables, skewed keys among them
        return {**_star(rng, 3, (50_000, 5_000_000), True), "call": "train", "model": "logistic",
                "m": rng.choice([1, 1, 2, 3]), "bf16": False, "iters": 5}
    if kind == "operator":
        return {**_star(rng, 2, (10_000, 1_000_000), True), "call": rng.choice(["lmm", "tmm"]), "cx": rng.randint(1, 16),
                "bf16": False}
    if kind == "sweep":
        return {**_star(rng, 1, (50_000, 1_000_000), False), "call": "train", "model": "linear",
                "m": rng.choice([32, 48, 64, 100, 128, 200, 256]), "bf16": rng.random() < 0.5, "iters": 5}
    if kind == "gram_star":
        return {**_star(rng, 2, (20_000, 1_000_000), False), "call": "gram"}
    if kind == "gram_union":
        cols = rng.randint(8, 64)
        return {"schema": "union", "rows": _log(rng, 20_000, 2_000_000), "cols": cols, "shared": rng.randint(0, cols // 2),
                "overlap": round(rng.uniform(0.0, 0.6), 2), "call": "gram"}
    if kind == "kmeans":
        return {**_star(rng, 1, (20_000, 1_000_000), False), "call": "kmeans", "k": rng.randint(2, 16)}
    if kind == "onehot":
        r_T = _log(rng, 50_000, 1_000_000)
        dims = ["%dx%d" % (_log(rng, 1_000, 6_000), _log(rng, 500, 9_500)) for _ in range(rng.randint(1, 2))]
        return {"schema": "onehot", "r_T": r_T, "dims": " ".join(dims), "attributes": rng.randint(4, 20), "call": "train",
                "model": "logistic", "m": 1, "bf16": False, "iters": 10}
    return {**_star(rng, 3, (50_000, 2_000_000), True), "call": "materialize"}


# ------------------------------------------------------------------------------------------------------ inputs
def _dims(case):
    out = []
    for text in case["dims"].split():
        size, _, keys = text.partition(":")
        rows, cols = size.split("x")
        out.append((int(rows), int(cols), keys))
    return out


def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)


def _keys(gen, n, rows, kind):
    if kind != "z":
        return torch.randint(0, rows, (n,), generator=gen, device=DEV, dtype=torch.int32)
    cdf = torch.cumsum(torch.arange(1, rows + 1, device=DEV, dtype=torch.float64) ** -1.1, 0)
    u = torch.rand(n, generator=gen, device=DEV, dtype=torch.float64) * cdf[-1]
    rank = torch.searchsorted(cdf, u).clamp_(max=rows - 1)
    return torch.randperm(rows, generator=gen, device=DEV)[rank].to(torch.int32)


def _schema(case, gen):
    """(sources, r_T, c_T): (table or CSR, row index or None, column map) for each source."""
    if case["schema"] == "union":
        rows, cols, shared = case["rows"], case["cols"], case["shared"]
        S1, S2 = _normal(gen, rows, cols), _normal(gen, rows, cols)
        n_match = int(round(case["overlap"] * rows))
        order2, order1 = (torch.randperm(rows, generator=gen, device=DEV) for _ in range(2))
        new = torch.sort(order2[n_match:]).values
        r_T, c_T = rows + new.numel(), 2 * cols - shared
        idx1 = torch.full((r_T,), -1, device=DEV, dtype=torch.int32)
        idx1[:rows] = torch.arange(rows, device=DEV, dtype=torch.int32)
        idx2 = torch.full((r_T,), -1, device=DEV, dtype=torch.int32)
        idx2[order1[:n_match]] = order2[:n_match].to(torch.int32)
        idx2[rows:] = new.to(torch.int32)
        S2[order2[:n_match], :shared] = 0.0          # a shared cell of a matched entity comes from the first source
        return [(S1, idx1, list(range(cols))), (S2, idx2, list(range(cols - shared, c_T)))], r_T, c_T
    sources, at = [], 0
    if case["schema"] == "onehot":
        r_T = case["r_T"]
        for rows, cols, _ in _dims(case):
            a = min(case["attributes"], cols)
            edges = torch.linspace(0, cols, a + 1, device=DEV, dtype=torch.float64).to(torch.int64)
            width = edges[1:] - edges[:-1]
            pick = (torch.rand((rows, a), generator=gen, device=DEV, dtype=torch.float64) * width).to(torch.int64)
            col = (edges[:-1] + torch.minimum(pick, width - 1)).to(torch.int32)
            val = torch.ones((rows, a), device=DEV)
            val[:, -1] = _normal(gen, rows)
            rowptr = (torch.arange(rows + 1, device=DEV, dtype=torch.int64) * a).to(torch.int32)
            table = il.CSR(rowptr, col.reshape(-1).contiguous(), val.reshape(-1).contiguous(), (rows, cols))
            sources.append((table, _keys(gen, r_T, rows, "u"), list(range(at, at + cols))))
            at += cols
        return sources, r_T, at
    r_T, dims = case["r_S"], _dims(case)
    sources.append((_normal(gen, r_T, case["c_S"]), None, list(range(case["c_S"]))))
    at = case["c_S"]
    for i, (rows, cols, keys) in enumerate(dims):
        fk = _keys(gen, r_T, rows, keys)
        if case["missing"] and i == len(dims) - 1:
            fk[torch.rand(r_T, generator=gen, device=DEV) < case["missing"]] = -1
        sources.append((_normal(gen, rows, cols), fk, list(range(at, at + cols))))
        at += cols
    return sources, r_T, at


def _dense64(sources):
    """The tables in 64 bits, sparse ones written out."""
    out = []
    for D, _, _ in sources:
        if isinstance(D, il.CSR):
            full = torch.zeros(D.shape, device=DEV, dtype=torch.float64)
            row = torch.repeat_interleave(torch.arange(D.shape[0], device=DEV), (D.rowptr[1:] - D.rowptr[:-1]).long())
            full[row, D.col.long()] = D.val.double()
            out.append(full)
        else:
            out.append(D.double())
    return out


def _rows64(sources, tables, c_T, lo, hi):
    """Rows lo..hi of the target table in 64 bits, by its definition."""
    T = torch.zeros((hi - lo, c_T), device=DEV, dtype=torch.float64)
    for (_, idx, cols), D in zip(sources, tables):
        first, last = cols[0], cols[-1] + 1           # every column map here is a block of target columns
        if idx is None:
            T[:, first:last] += D[lo:hi]
        else:
            at = idx[lo:hi].long()
            part = D[at.clamp(min=0)]
            part[at < 0] = 0.0
            T[:, first:last] += part
    return T


def _chunks(r_T, c_T):
    step = max(1, int(2e8 // c_T))
    return [(lo, min(r_T, lo + step)) for lo in range(0, r_T, step)]


def _operands(case, gen, sources, r_T, c_T):
    """The call's own inputs: what a program holds beside the tables."""
    s = {}
    call = case["call"]
    if call == "lmm":
        s["X"] = _normal(gen, c_T, case["cx"])
    elif call == "tmm":
        s["Y"] = _normal(gen, r_T, case["cx"])
    elif call == "kmeans":
        s["C0"] = _normal(gen, c_T, case["k"])
    elif call == "train":
        w = torch.randn(c_T, generator=gen, device=DEV, dtype=torch.float64) / math.sqrt(c_T)
        z = torch.zeros(r_T, device=DEV, dtype=torch.float64)
        for D, idx, cols in sources:                  # labels of a linear model plus noise
            wk = w[cols[0]:cols[-1] + 1]
            if isinstance(D, il.CSR):
                rows = torch.repeat_interleave(torch.arange(D.shape[0], device=DEV), (D.rowptr[1:] - D.rowptr[:-1]).long())
                p = torch.zeros(D.shape[0], device=DEV, dtype=torch.float64).index_add_(0, rows, D.val.double() * wk[D.col.long()])
            else:
                p = (D @ wk.float().unsqueeze(1)).squeeze(1).double()
            z += p if idx is None else torch.where(idx >= 0, p[idx.long().clamp(min=0)], 0.0)
        z += 0.1 * torch.randn(r_T, generator=gen, device=DEV, dtype=torch.float64)
        s["y"] = (z >= 0).float() if case["model"] == "logistic" else z.float()
        m = case["m"]
        if m > 1:                                     # learning rates log-spaced up to 0.5
            s["lr"] = torch.logspace(-3.0, math.log10(0.5), m, device=DEV, dtype=torch.float32)
        else:
            s["lr"] = torch.full((1,), 0.5 if case["model"] == "logistic" else 0.1, device=DEV)
    return s


def _max_cx(case):
    return {"lmm": case.get("cx"), "tmm": case.get("cx"), "train": case.get("m"), "kmeans": case.get("k")}.get(case["call"]) or 1


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    sources, r_T, c_T = _schema(case, gen)
    s = _operands(case, gen, sources, r_T, c_T)
    s["case"], s["plan"] = case, il.ilargi_plan_create(sources, r_T, c_T, max_cx=_max_cx(case))
    s["precision"] = il.BF16_IN_F32_ACC if case.get("bf16") else il.F32
    call = case["call"]
    if call == "lmm":
        s["out"] = torch.empty((r_T, case["cx"]), device=DEV)
    elif call == "tmm":
        s["out"] = torch.empty((c_T, case["cx"]), device=DEV)
    elif call == "gram":
        s["out"] = torch.empty((c_T, c_T), device=DEV)
    elif call == "materialize":
        s["out"] = torch.empty((r_T, c_T), device=DEV)
    elif call == "kmeans":
        s["assign"] = torch.empty(r_T, device=DEV, dtype=torch.int32)
        s["counts"] = torch.empty(case["k"], device=DEV, dtype=torch.int32)
    return s


def run(state):
    case, plan = state["case"], state["plan"]
    call = case["call"]
    if call == "lmm":
        return il.ilargi_lmm(plan, state["X"], out=state["out"], precision=state["precision"])
    if call == "tmm":
        return il.ilargi_tmm(plan, state["Y"], out=state["out"], precision=state["precision"])
    if call == "gram":
        return il.ilargi_crossprod(plan, out=state["out"])
    if call == "materialize":
        return il.ilargi_materialize(plan, out=state["out"])
    if call == "kmeans":
        C = state["C0"].clone()
        il.ilargi_kmeans_step(plan, C, state["assign"], state["counts"])
        return {"C": C, "assign": state["assign"], "counts": state["counts"]}
    W = torch.zeros((plan.c_T, case["m"]), device=DEV)
    losses = torch.empty((case["iters"], case["m"]), device=DEV)
    model = il.LOGISTIC if case["model"] == "logistic" else il.LINEAR
    for t in range(case["iters"]):
        il.ilargi_gd_step(plan, model, W, state["y"], state["lr"], losses[t], precision=state["precision"])
    return {"W": W, "losses": losses}


def _sizes(case):
    """(r_T, c_T, [(rows, cols, stored entries, whether a row index is read)])."""
    if case["schema"] == "union":
        rows, cols = case["rows"], case["cols"]
        r_T = 2 * rows - int(round(case["overlap"] * rows))
        # the first source's index is the identity on its rows; only the second one's has to be read
        return r_T, 2 * cols - case["shared"], [(rows, cols, None, False), (rows, cols, None, True)]
    if case["schema"] == "onehot":
        tabs = [(r, c, r * min(case["attributes"], c), True) for r, c, _ in _dims(case)]
        return case["r_T"], sum(t[1] for t in tabs), tabs
    tabs = [(case["r_S"], case["c_S"], None, False)] + [(r, c, None, True) for r, c, _ in _dims(case)]
    return case["r_S"], sum(t[1] for t in tabs), tabs


def work(case):
    r_T, c_T, tabs = _sizes(case)
    table_bytes = sum(4 * r * c if nnz is None else 8 * nnz + 4 * (r + 1) for r, c, nnz, _ in tabs)
    index_bytes = 4 * r_T * sum(1 for t in tabs if t[3])
    cells = sum(r * c if nnz is None else nnz for r, c, nnz, _ in tabs)
    call = case["call"]
    read = table_bytes + index_bytes
    if call == "materialize":
        return {"bytes": read + 4 * r_T * c_T, "flops": 0}
    if call == "gram":
        # the tables' own blocks (one triangle) and the cross blocks after the segment sums of the narrower table
        flops = sum(r * c * (c + 1) for r, c, _, _ in tabs)
        for i in range(len(tabs)):
            for j in range(i):
                flops += 2 * min(tabs[i][0], tabs[j][0]) * tabs[i][1] * tabs[j][1] + r_T * min(tabs[i][1], tabs[j][1])
        return {"bytes": read + 4 * c_T * c_T, "flops": flops}
    cx = _max_cx(case)
    product = 2 * cells * cx + r_T * cx * (len(tabs) - 1)   # the tables' products and the rows' sums
    if call in ("lmm", "tmm"):
        return {"bytes": read + 4 * (r_T + c_T) * cx, "flops": product}
    if call == "kmeans":
        return {"bytes": read + 8 * c_T * cx + 4 * r_T, "flops": 2 * product}
    per_step = read + 4 * r_T + 8 * c_T * cx + 8 * cx
    return {"bytes": case["iters"] * per_step, "flops": case["iters"] * 2 * product}


def tolerance(case):
    if case["call"] == "materialize":
        return "exact"
    if case.get("bf16"):
        return {"rel": 2.5e-3}                        # measured against 64 bits: 6e-4 (weights after 5 steps)
    if case["call"] == "kmeans":
        # sums alone are 7e-8 off; a row between two equally near centroids may go to either, which moves a centroid by
        # its share of the cluster
        return {"rel": 2e-4, "max": 5e-3, "differ": 1e-4}
    return {"rel": 1e-6}                              # measured against 64 bits: 4e-8 to 2.2e-7


def exact(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    sources, r_T, c_T = _schema(case, gen)
    s = _operands(case, gen, sources, r_T, c_T)
    tables = _dense64(sources)
    rows = lambda lo, hi: _rows64(sources, tables, c_T, lo, hi)  # noqa: E731
    chunks = _chunks(r_T, c_T)
    call = case["call"]
    if call == "lmm":
        X = s["X"].double()
        return torch.cat([rows(lo, hi) @ X for lo, hi in chunks])
    if call == "materialize":
        return torch.cat([rows(lo, hi) for lo, hi in chunks])
    if call == "tmm":
        return sum(rows(lo, hi).t() @ s["Y"][lo:hi].double() for lo, hi in chunks)
    if call == "gram":
        total = torch.zeros((c_T, c_T), device=DEV, dtype=torch.float64)
        for lo, hi in chunks:
            T = rows(lo, hi)
            total += T.t() @ T
        return total
    if call == "kmeans":
        C, k = s["C0"].double(), case["k"]
        assign, sums = torch.empty(r_T, device=DEV, dtype=torch.int32), torch.zeros((c_T, k), device=DEV, dtype=torch.float64)
        for lo, hi in chunks:
            T = rows(lo, hi)
            a = torch.argmin((C * C).sum(0) - 2 * (T @ C), dim=1)
            assign[lo:hi] = a.to(torch.int32)
            sums += T.t() @ torch.nn.functional.one_hot(a, k).double()
        counts = torch.bincount(assign.long(), minlength=k)
        return {"C": torch.where(counts > 0, sums / counts.clamp(min=1), C), "assign": assign, "counts": counts.to(torch.int32)}
    m, y, lr = case["m"], s["y"].double().unsqueeze(1), s["lr"].double()
    W, losses = torch.zeros((c_T, m), device=DEV, dtype=torch.float64), []
    for _ in range(case["iters"]):
        G = torch.zeros((c_T, m), device=DEV, dtype=torch.float64)
        loss = torch.zeros(m, device=DEV, dtype=torch.float64)
        for lo, hi in chunks:
            T = rows(lo, hi)
            Z = T @ W
            if case["model"] == "logistic":
                loss += (torch.nn.functional.softplus(Z) - y[lo:hi] * Z).sum(0) / r_T
                E = torch.sigmoid(Z) - y[lo:hi]
            else:
                E = Z - y[lo:hi]
                loss += (E * E).sum(0) / (2 * r_T)
            G += T.t() @ E
        losses.append(loss)
        W = W - lr * G / r_T
    return {"W": W, "losses": torch.stack(losses)}

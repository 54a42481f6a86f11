"""Iterations over entity tables of few columns (a lane per row, the gradient on the matrix cores), against 64 bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def il():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01985_amd as mod
    return mod


def _step(il, sources, r_T, c_T, m, model, gen, y=None, infinite=None):
    """One step from random weights against float64; returns what it gave and what it should have."""
    W = torch.randn(c_T, m, generator=gen, device="cuda") / 4
    if infinite is not None:
        W[infinite] = float("inf")
    y = (torch.rand(r_T, generator=gen, device="cuda") < 0.5).float() if y is None else y
    lr = torch.linspace(0.1, 0.4, m, device="cuda")
    Wd = W.double()
    z = torch.zeros(r_T, m, dtype=torch.float64, device="cuda")
    for D, idx, cols in sources:
        p = D.double() @ Wd[cols]
        z += p if idx is None else torch.where((idx >= 0).unsqueeze(1), p[idx.clamp(min=0).long()], 0.0)
    e = (z if model == "linear" else z.sigmoid()) - y.double().unsqueeze(1)
    G = torch.zeros(c_T, m, dtype=torch.float64, device="cuda")
    for D, idx, cols in sources:
        if idx is None:
            G[cols] += D.double().t() @ e
        else:
            ok = (idx >= 0).cpu()
            Z = torch.zeros(len(D), m, dtype=torch.float64).index_add_(0, idx.cpu()[ok].long(), e.cpu()[ok])
            G[cols] += D.double().t() @ Z.cuda()
    per_row = 0.5 * e * e if model == "linear" else torch.nn.functional.softplus(z) - y.double().unsqueeze(1) * z
    plan = il.ilargi_plan_create(sources, r_T, c_T, max_cx=m)
    out = []
    for _ in range(2):
        got, loss = W.clone(), torch.empty(m, device="cuda")
        il.ilargi_gd_step(plan, il.LINEAR if model == "linear" else il.LOGISTIC, got, y, lr, loss)
        out.append((got, loss))
    assert torch.equal(out[0][0].view(torch.int32), out[1][0].view(torch.int32))
    assert torch.equal(out[0][1].view(torch.int32), out[1][1].view(torch.int32))
    return W, out[0][0], out[0][1], lr.double() / r_T * G, per_row.mean(0)


@pytest.mark.parametrize("c", [1, 2, 3, 4, 7, 10, 12, 13, 15, 16, 17, 20, 21, 24])
@pytest.mark.parametrize("r_T,tables,m", [
    (20_033, [(50, 3)], 1),
    (40_001, [(900, 7), (30, 2)], 2),
    (70_003, [(3_000, 5), (200, 4), (7, 2), (1, 1)], 3),
    (300_001, [(90, 6)], 4),                               # several steps a wavefront, the last of one row
])
@pytest.mark.parametrize("model", ["linear", "logistic"])
def test_iteration_a_lane_per_row(il, r_T, tables, m, c, model):
    gen = torch.Generator(device="cuda").manual_seed(r_T + 10 * c)
    sources, at = [(torch.randn(r_T, c, generator=gen, device="cuda"), None, list(range(2, 2 + c)))], 2 + c   # two columns nobody feeds
    for rows, cols in tables:
        idx = torch.randint(0, rows, (r_T,), generator=gen, device="cuda", dtype=torch.int32)
        idx[torch.rand(r_T, generator=gen, device="cuda") < 0.1] = -1
        sources.append((torch.randn(rows, cols, generator=gen, device="cuda"), idx, list(range(at, at + cols))))
        at += cols
    W, got, loss, step, want = _step(il, sources, r_T, at, m, model, gen)
    # sums of r_T products in float32: a few units of 2^-24 by the 2-norm; and the rounding of the weight
    assert (got.double() - (W.double() - step)).norm() <= 2e-6 * step.norm() + 2.0 ** -24 * W.double().norm()
    assert (loss.double() - want).norm() <= 2e-6 * want.norm()


@pytest.mark.parametrize("m", [1, 3])
@pytest.mark.parametrize("case", ["prefix", "infinite label beyond the table", "infinite weight", "infinite value", "scattered columns", "shared columns"])
def test_iteration_a_lane_per_row_at_its_edges(il, case, m):
    gen = torch.Generator(device="cuda").manual_seed(3)
    r_T, c, rows = 50_001, 9, 400
    idx = torch.randint(0, rows, (r_T,), generator=gen, device="cuda", dtype=torch.int32)
    R = (torch.randn(rows, 5, generator=gen, device="cuda"), idx, list(range(c, c + 5)))
    d_rows = 33_333 if case in ("prefix", "infinite label beyond the table", "infinite weight") else r_T
    first = None
    if d_rows < r_T:                                       # the table feeds the first rows only
        first = torch.arange(r_T, device="cuda", dtype=torch.int32)
        first[d_rows:] = -1
    S = torch.randn(d_rows, c, generator=gen, device="cuda")
    y = (torch.rand(r_T, generator=gen, device="cuda") < 0.5).float()
    cols, infinite = list(range(c)), None
    if case == "infinite weight":                          # in the last model: rows that the table does not feed have no part in it
        infinite = (4, m - 1)
        idx[:d_rows] = -1
    if case == "infinite label beyond the table":
        y[r_T - 5] = float("inf")
    elif case == "infinite value":
        S[777, 4] = float("inf")
    elif case == "scattered columns":
        cols = cols[::-1]                                  # no block: another kernel
    elif case == "shared columns":
        R = (R[0], R[1], list(range(c - 2, c + 3)))
    W, got, loss, step, want = _step(il, [(S, first, cols), R], r_T, c + 5, m, "linear", gen, y, infinite)
    finite = step.isfinite()
    if case == "infinite label beyond the table":          # the entity table's weights stay out of it
        assert bool(finite[:c].all()) and torch.equal(got.isfinite()[:c], finite[:c]) and not bool(got[c:].isfinite().any())
    elif case == "infinite weight":
        assert bool(finite[c:].all()) and bool(finite[:, :m - 1].all()) and not bool(finite[:c, m - 1].any())
        assert torch.equal(got.isfinite(), finite)
    elif case == "infinite value":
        assert torch.equal(got.isfinite(), finite)
        return
    assert (got.double() - (W.double() - step))[finite].norm() <= 2e-6 * step[finite].norm() + 2.0 ** -24 * W.double()[finite].norm()

"""Segment sums in fixed point in LDS, and the assembly of gathers alone that forms them, against 64-bit sums."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# A run's sums are rounded to float32 once, up to 256 of them are added in pairs of parts, and the table's product adds
# thousands of rows in float32: a few units of 2^-24 by the 2-norm.
REL = 1e-6


@pytest.fixture(scope="module")
def il():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01985_amd as mod
    return mod


def _sources(r_T, rows, kinds, missing, gen, shift=0):
    sources, at = [], 0
    for r, kind in zip(rows, kinds):
        idx = torch.randint(0, r, (r_T + shift,), generator=gen, device="cuda", dtype=torch.int32)
        if kind == "sorted":
            idx = idx.sort()[0]
        elif kind == "hot":
            idx[torch.rand(r_T + shift, generator=gen, device="cuda") < 0.7] = r // 2
        idx[torch.rand(r_T + shift, generator=gen, device="cuda") < missing] = -1
        sources.append((torch.randn(r, 5, generator=gen, device="cuda"), idx[shift:], list(range(at, at + 5))))
        at += 5
    return sources, at


def _exact_tmm(sources, Y):
    # (on the CPU: atomic additions of doubles to one popular row take seconds on the GPU)
    out, Y = [], Y.double().cpu()
    for D, idx, _ in sources:
        idx = idx.cpu().long()
        ok = idx >= 0
        Z = torch.zeros(len(D), Y.shape[1], dtype=torch.float64).index_add_(0, idx[ok], Y[ok])
        out.append((D.double().cpu().unsqueeze(2) * Z.unsqueeze(1)).sum(0))
    return torch.cat(out).cuda()


def _close(got, want):
    """Each operand column by itself: what is large in one does not hide the others."""
    assert torch.equal(got.isfinite(), want.isfinite())
    for g, w in zip(got.double().reshape(-1, got.shape[-1]).t(), want.reshape(-1, got.shape[-1]).t()):
        ok = w.isfinite()
        assert (g - w)[ok].norm() <= REL * w[ok].norm()


@pytest.mark.parametrize("r_T,rows,kinds,cx", [
    (2_500_000, [20_160], ["uniform"], 1),                            # one full range ...
    (2_500_003, [20_161], ["uniform"], 1),                            # ... and a key more, rows beyond the last four
    (2_500_001, [2_000, 3], ["uniform", "hot"], 1),
    (1_500_002, [100_000, 50_001, 9_999], ["uniform", "hot", "uniform"], 1),
    (2_500_001, [30_000, 20_000], ["sorted", "uniform"], 1),          # four rows of a key side by side
    (1_500_003, [10_080, 5_000], ["uniform", "sorted"], 2),
    (2_500_001, [3_000, 6_721], ["hot", "uniform"], 3),
    (1_500_001, [3_000, 5_041, 1], ["sorted", "uniform", "uniform"], 4),
])
@pytest.mark.parametrize("values", ["normal", "late", "outlier", "odd", "tiny"])
def test_segment_sums_in_fixed_point(il, r_T, rows, kinds, cx, values):
    gen = torch.Generator(device="cuda").manual_seed(r_T + cx)
    shift = 1 if values == "late" else 0                              # row indices and operand off a multiple of 16 bytes
    sources, c_T = _sources(r_T, rows, kinds, 0.1, gen, shift)
    Y = torch.randn(r_T * cx + shift, generator=gen, device="cuda")[shift:].reshape(r_T, cx)
    if values == "late":
        Y[: r_T // 2] = 0.0                                           # nothing to see in a run's first rows
    elif values == "outlier":
        Y[r_T // 3, 0] = 3e9
    elif values == "odd":
        Y[r_T // 3, 0], Y[7, cx - 1], Y[r_T - 1, 0] = float("inf"), float("nan"), float("-inf")
    elif values == "tiny":
        Y *= 1e-36
    plan = il.ilargi_plan_create(sources, r_T, c_T, max_cx=cx)
    got = il.ilargi_tmm(plan, Y)
    _close(got, _exact_tmm(sources, Y))
    assert torch.equal(il.ilargi_tmm(plan, Y).view(torch.int32), got.view(torch.int32))


@pytest.mark.parametrize("r_T,rows,kinds,m", [
    (100_000, [250], ["uniform"], 1),
    (100_003, [40, 30], ["hot", "uniform"], 4),
    (600_001, [13_419], ["uniform"], 1),                              # as many keys as LDS holds ...
    (540_002, [6_711, 6_707], ["uniform", "hot"], 1),
    (600_001, [3_351], ["uniform"], 4),                               # ... of four models
    (600_001, [3_355], ["uniform"], 4),                               # ... and a few more
    (600_003, [1_500, 3_000, 10], ["uniform", "uniform", "uniform"], 3),
    (300_001, [1_000, 400, 3, 1], ["uniform", "hot", "uniform", "uniform"], 2),
    (2_600_001, [300], ["sorted"], 4),
    (700_000, [5_000, 300], ["sorted", "uniform"], 1),
])
@pytest.mark.parametrize("model", ["linear", "logistic"])
@pytest.mark.parametrize("values", ["normal", "outlier", "odd"])
def test_assembly_of_gathers_with_their_segment_sums(il, r_T, rows, kinds, m, model, values):
    gen = torch.Generator(device="cuda").manual_seed(r_T + m)
    sources, c_T = _sources(r_T, rows, kinds, 0.1, gen)
    W = torch.randn(c_T, m, generator=gen, device="cuda") / 4
    y = (torch.rand(r_T, generator=gen, device="cuda") < 0.5).float()
    if values == "outlier":
        y[r_T // 2] = 3e5
    elif values == "odd":
        y[r_T // 2] = float("inf")
    lr = torch.linspace(0.1, 0.4, m, device="cuda")
    Wd = W.double()
    z = torch.zeros(r_T, m, dtype=torch.float64, device="cuda")
    for D, idx, cols in sources:
        p = (D.double().unsqueeze(2) * Wd[cols].unsqueeze(0)).sum(1)
        z += torch.where((idx >= 0).unsqueeze(1), p[idx.clamp(min=0).long()], 0.0)
    e = (z if model == "linear" else z.sigmoid()) - y.double().unsqueeze(1)
    want = Wd - lr.double() / r_T * _exact_tmm(sources, e)
    per_row = 0.5 * e * e if model == "linear" else torch.nn.functional.softplus(z) - y.double().unsqueeze(1) * z
    plan = il.ilargi_plan_create(sources, r_T, c_T, max_cx=m)
    first, loss, again, loss2 = W.clone(), torch.empty(m, device="cuda"), W.clone(), torch.empty(m, device="cuda")
    which = il.LINEAR if model == "linear" else il.LOGISTIC
    il.ilargi_gd_step(plan, which, first, y, lr, loss)
    il.ilargi_gd_step(plan, which, again, y, lr, loss2)
    if values != "odd":
        # the step's own error, and the rounding of the updated weight to float32
        for got, w, w0 in zip(first.double().t(), want.t(), Wd.t()):                 # each model by itself
            assert (got - w).norm() <= REL * (w - w0).norm() + 2.0 ** -24 * w.norm()
        _close(loss, per_row.mean(0))
    else:
        assert torch.equal(first.isfinite(), want.isfinite())
    assert torch.equal(first.view(torch.int32), again.view(torch.int32)) and torch.equal(loss.view(torch.int32), loss2.view(torch.int32))


def _one_hot(il, r_T, rows, kinds, gen):
    """Tables with a column for every row: a cell of T^T Y is one key's sum."""
    sources, c_T = _sources(r_T, rows, kinds, 0.1, gen)
    out, at = [], 0
    for (_, idx, _), r in zip(sources, rows):
        ints = torch.arange(r + 1, device="cuda", dtype=torch.int32)
        out.append((il.CSR(ints, ints[:r].contiguous(), torch.ones(r, device="cuda"), (r, r)), idx, list(range(at, at + r))))
        at += r
    return out, at


def _sums_by_key(sources, Y):
    Y, out = Y.double().cpu(), []
    for D, idx, _ in sources:
        idx = idx.cpu().long()
        ok = idx >= 0
        out.append(torch.zeros(D.shape[0], Y.shape[1], dtype=torch.float64).index_add_(0, idx[ok], Y[ok]))
    return torch.cat(out)


def _each_sum_close(got, want, size):
    # a run's sum of a key is rounded a few times at most (once for each walk that found rows of it, and as often in adding
    # these), and up to 256 runs are added in pairs of parts: sixteen roundings of what the key's values come to in magnitude
    got = got.double().cpu()
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf()) and torch.equal(got[want.isinf()], want[want.isinf()])
    ok = want.isfinite()
    # (and where floats end, half of the smallest for each run)
    assert bool(((got - want).abs() <= 2.0 ** -20 * size + 256 * 2.0 ** -150)[ok].all())


@pytest.mark.parametrize("r_T,rows,kinds,cx", [
    (2_500_001, [20_160], ["uniform"], 1),                            # one full range ...
    (2_500_002, [20_161], ["sorted"], 1),                             # ... and a key more
    (1_500_002, [100_000, 50_001, 9_999], ["uniform", "hot", "uniform"], 1),
    (1_500_003, [10_080, 5_000], ["uniform", "sorted"], 2),
    (2_500_001, [3_000, 6_721], ["hot", "uniform"], 3),
    (1_500_001, [3_000, 5_041, 1], ["sorted", "uniform", "uniform"], 4),
])
@pytest.mark.parametrize("values", ["columns", "outliers", "small ones", "keys", "zeros", "wide", "smallest", "odd", "odd among small ones", "odd everywhere"])
def test_every_sum_by_itself(il, r_T, rows, kinds, cx, values):
    gen = torch.Generator(device="cuda").manual_seed(r_T + cx)
    sources, c_T = _one_hot(il, r_T, rows, kinds, gen)
    key = sources[0][1].clamp(min=0).long()
    Y = torch.randn(r_T, cx, generator=gen, device="cuda")
    u = torch.rand(r_T, generator=gen, device="cuda")
    if values == "columns":
        Y *= torch.tensor([1.0, 1e-9, 1e9, 1e-15][-cx:], device="cuda")
    elif values == "outliers":                                        # with a key and without one
        Y[r_T // 3], Y[r_T // 2, 0], Y[r_T - 2, cx - 1] = 1e12, 3e-20, -1e30
        sources[0][1][r_T - 2] = -1
    elif values in ("small ones", "odd among small ones"):            # more than a list in LDS holds, fewer than one in memory
        Y *= torch.where(u < 0.03, 1e-12 * u, 1.0).unsqueeze(1)
        if values != "small ones":
            Y[(u < 0.03) & (key % 5 == 0)] = float("inf")
            Y[(u < 0.01) & (key % 5 == 1)] = float("nan")
    elif values == "keys":                                            # values of a size of each key's own
        Y *= (10.0 ** (-4.0 * (key % 5))).unsqueeze(1)
    elif values == "zeros":
        Y[u < 0.9] = 0.0
        Y[: r_T // 2] = 0.0
    elif values == "wide":
        Y *= torch.exp2(200.0 * u - 100.0).unsqueeze(1)
    elif values == "smallest":
        Y *= torch.where(key % 3 == 0, 1e-39, 1.0).unsqueeze(1)
    elif values == "odd":
        Y[r_T // 3, 0], Y[r_T // 2, cx - 1], Y[r_T - 1] = float("inf"), float("nan"), float("-inf")
    elif values == "odd everywhere":
        Y[(u < 0.2) & (key % 7 == 3)] = float("inf")
        Y[(u > 0.9) & (key % 7 == 5)] = float("nan")
        Y[(u > 0.5) & (key % 11 == 5)] = float("-inf")
    plan = il.ilargi_plan_create(sources, r_T, c_T, max_cx=cx)
    got = il.ilargi_tmm(plan, Y)
    _each_sum_close(got, _sums_by_key(sources, Y), _sums_by_key(sources, Y.abs()))
    assert torch.equal(il.ilargi_tmm(plan, Y).view(torch.int32), got.view(torch.int32))


@pytest.mark.parametrize("r_T,rows,kinds,m", [
    (600_001, [13_419], ["uniform"], 1),                              # as many keys as LDS holds
    (100_003, [40, 30], ["hot", "uniform"], 4),
    (600_003, [1_500, 3_000, 10], ["uniform", "uniform", "uniform"], 2),
    (300_001, [1_000, 400, 3, 1], ["uniform", "hot", "uniform", "uniform"], 2),
    (2_600_001, [300], ["sorted"], 3),
])
@pytest.mark.parametrize("case", ["a model that diverges", "keys", "labels of some rows", "small labels", "infinite labels"])
def test_every_model_and_key_by_itself(il, r_T, rows, kinds, m, case):
    gen = torch.Generator(device="cuda").manual_seed(r_T + m)
    sources, c_T = _one_hot(il, r_T, rows, kinds, gen)
    key = sources[0][1].clamp(min=0).long()
    W = torch.zeros(c_T, m, device="cuda")
    y = torch.randn(r_T, generator=gen, device="cuda")
    if case == "a model that diverges":
        W[:, m - 1] = 1e14 * torch.randn(c_T, generator=gen, device="cuda")
    elif case == "keys":
        y *= 10.0 ** (-4.0 * (key % 5))
    elif case == "labels of some rows":
        y[::100_000] = 1e20
    elif case == "small labels":
        u = torch.rand(r_T, generator=gen, device="cuda")
        y *= torch.where(u < 0.03, 1e-15 * u, 1.0)
        y[(u < 0.01) & (key % 5 == 0)] = float("-inf")
    elif case == "infinite labels":
        y[(torch.rand(r_T, generator=gen, device="cuda") < 0.2) & (key % 7 == 3)] = float("inf")
    lr = torch.full((m,), 1e-3 * r_T, device="cuda")
    z, size = torch.zeros(r_T, m, dtype=torch.float64, device="cuda"), y.double().abs().unsqueeze(1).expand(r_T, m).clone()
    for D, idx, cols in sources:
        p = torch.where((idx >= 0).unsqueeze(1), W[cols].double()[idx.clamp(min=0).long()], 0.0)
        z += p
        size += p.abs()
    e = z - y.double().unsqueeze(1)
    scale = lr.double().cpu() / r_T
    want = W.double().cpu() - scale * _sums_by_key(sources, e)
    plan = il.ilargi_plan_create(sources, r_T, c_T, max_cx=m)
    got, loss, again = W.clone(), torch.empty(m, device="cuda"), W.clone()
    il.ilargi_gd_step(plan, il.LINEAR, got, y, lr, loss)
    il.ilargi_gd_step(plan, il.LINEAR, again, y, lr, loss)
    # (the residual's own rounding and that of the updated weight among the sixteen)
    _each_sum_close(got, want, scale * _sums_by_key(sources, size) + W.double().abs().cpu())
    assert torch.equal(got.view(torch.int32), again.view(torch.int32))

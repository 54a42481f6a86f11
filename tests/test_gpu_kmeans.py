"""KMeans over entity tables of few columns and large target tables (a lane per row), against 64 bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def il():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01985_amd as mod
    return mod


def _schema(r_T, c, tables, missing, gen, d_rows=None, at=0):
    d_rows = r_T if d_rows is None else d_rows
    idx = None
    if d_rows < r_T:                                          # the entity table feeds the first rows only
        idx = torch.arange(r_T, device="cuda", dtype=torch.int32)
        idx[d_rows:] = -1
    sources = [(torch.randn(d_rows, c, generator=gen, device="cuda"), idx, list(range(at, at + c)))]
    at += c
    for rows, cols in tables:
        idx = torch.randint(0, rows, (r_T,), generator=gen, device="cuda", dtype=torch.int32)
        idx[torch.rand(r_T, generator=gen, device="cuda") < missing] = -1
        sources.append((torch.randn(rows, cols, generator=gen, device="cuda"), idx, list(range(at, at + cols))))
        at += cols
    return sources, at


def _target(sources, r_T, c_T):
    T = torch.zeros(r_T, c_T, dtype=torch.float64, device="cuda")
    for D, idx, cols in sources:
        if idx is None:
            T[:, cols] = D.double()
        else:
            T[:, cols] = torch.where((idx >= 0).unsqueeze(1), D.double()[idx.clamp(min=0).long()], 0.0)
    return T


def _check(T, C, Cd, assign, counts):
    k = C.shape[1]
    a = assign.long()
    assert int(a.min()) >= 0 and int(a.max()) < k and torch.equal(torch.bincount(a, minlength=k).int(), counts)
    Cn = C.double()
    dist = (Cn * Cn).sum(0) - 2.0 * (T @ Cn)
    # rounding of a score: 2^-24 of its terms, a few dozen of them; rows closer to the boundary may go either way
    slack = 1e-5 * ((Cn * Cn).sum(0).max() + 2.0 * (T.abs() @ Cn.abs()).max(1).values)
    ok = T.isfinite().all(1)
    assert bool((dist.gather(1, a.unsqueeze(1)).squeeze(1) <= dist.min(1).values + slack)[ok].all())
    one = torch.nn.functional.one_hot(a, k).double()
    sums = torch.nan_to_num(T, 0.0, 0.0, 0.0).t() @ one
    want = torch.where(counts > 0, sums / counts.clamp(min=1), Cn)
    cells = torch.isfinite(Cd)
    assert (Cd.double() - want)[cells].norm() <= 2e-6 * want.norm()
    return cells


@pytest.mark.parametrize("c", [1, 2, 3, 8, 12, 13, 15, 16, 17, 20])
@pytest.mark.parametrize("r_T,tables,k", [
    (131_072, [(500, 8)], 3),
    (131_137, [(3_000, 5), (7, 30)], 10),                     # a last step of one row
    (150_001, [(100, 9), (50, 4), (3, 2), (1, 7)], 7),
    (200_000, [(9_000, 40)], 16),
    (140_003, [(64, 3)], 13),
])
def test_kmeans_a_lane_per_row(il, r_T, tables, k, c):
    gen = torch.Generator(device="cuda").manual_seed(c * 100 + k)
    sources, c_T = _schema(r_T, c, tables, 0.1, gen)
    T = _target(sources, r_T, c_T)
    C = torch.randn(c_T, k, generator=gen, device="cuda")
    plan = il.ilargi_plan_create(sources, r_T, c_T, max_cx=k)
    out = []
    for _ in range(2):
        Cd, assign, counts = C.clone(), torch.full((r_T,), -7, device="cuda", dtype=torch.int32), torch.zeros(k, device="cuda", dtype=torch.int32)
        il.ilargi_kmeans_step(plan, Cd, assign, counts)
        out.append((Cd, assign, counts))
    assert bool(_check(T, C, *out[0]).all())
    assert all(torch.equal(x, y) for x, y in zip(*out))
    Cd = C.clone()
    il.ilargi_kmeans_step(plan, Cd)                           # without the optional outputs
    assert torch.equal(Cd, out[0][0])


@pytest.mark.parametrize("case", ["prefix", "empty", "inf row", "nan row", "inf centroid", "alone", "last"])
def test_kmeans_a_lane_per_row_at_its_edges(il, case):
    gen = torch.Generator(device="cuda").manual_seed(5)
    r_T, c, k = 131_200, 18, 6
    tables = [] if case == "alone" else [(400, 11)]
    sources, c_T = _schema(r_T, c, tables, 0.0, gen, d_rows=100_001 if case == "prefix" else None)
    if case == "last":                                        # the entity table's columns are the target's last ones
        sources, c_T = _schema(r_T, c, tables, 0.0, gen, at=11)
        c_T = 11 + c
        sources = [(sources[0][0], None, list(range(11, 11 + c))), (sources[1][0], sources[1][1], list(range(11)))]
    if case in ("inf row", "nan row"):
        sources[0][0][70_000, 3] = float("inf") if case == "inf row" else float("nan")
    T = _target(sources, r_T, c_T)
    C = torch.randn(c_T, k, generator=gen, device="cuda")
    if case == "empty":
        C[:, 2] = 1e6                                         # nobody's centroid stays where it is
    if case == "inf centroid":
        C[1, 4] = float("inf")
    plan = il.ilargi_plan_create(sources, r_T, c_T, max_cx=k)
    Cd, assign, counts = C.clone(), torch.empty(r_T, device="cuda", dtype=torch.int32), torch.zeros(k, device="cuda", dtype=torch.int32)
    il.ilargi_kmeans_step(plan, Cd, assign, counts)
    if case == "inf centroid":
        keep = [0, 1, 2, 3, 5]
        assert int(counts[4]) == 0 and int(counts.sum()) == r_T
        again = il.ilargi_plan_create(sources, r_T, c_T, max_cx=5)
        C5, a5, n5 = C[:, keep].contiguous(), torch.empty_like(assign), torch.zeros(5, device="cuda", dtype=torch.int32)
        il.ilargi_kmeans_step(again, C5, a5, n5)
        assert torch.equal(torch.tensor(keep, device="cuda", dtype=torch.int32)[a5.long()], assign) and torch.equal(counts[keep], n5)
        return
    cells = _check(T, C, Cd, assign, counts)
    if case in ("inf row", "nan row"):                        # only in its own cluster's centroid
        assert int((~cells).sum()) == 1 and not bool(cells[3, int(assign[70_000])])
    else:
        assert bool(cells.all())
    if case == "empty":
        assert torch.equal(Cd[:, 2], C[:, 2])


@pytest.mark.parametrize("k", [3, 10, 16])
def test_infinite_centroids_and_rows_that_the_table_does_not_feed(il, k):
    gen = torch.Generator(device="cuda").manual_seed(k)
    r_T, c, d_rows = 140_001, 18, 70_003
    sources, c_T = _schema(r_T, c, [(400, 11)], 0.1, gen, d_rows=d_rows)
    T = _target(sources, r_T, c_T)
    C = torch.randn(c_T, k, generator=gen, device="cuda")
    C[1, 0] = float("inf")                                    # infinitely far from every row that does not have the column
    C[2, k - 1] = float("-inf")
    keep = list(range(1, k - 1))
    plan = il.ilargi_plan_create(sources, r_T, c_T, max_cx=k)
    Cd, assign, counts = C.clone(), torch.empty(r_T, device="cuda", dtype=torch.int32), torch.zeros(k, device="cuda", dtype=torch.int32)
    il.ilargi_kmeans_step(plan, Cd, assign, counts)
    Cn = C[:, keep].double()
    terms = (Cn * Cn).sum(0), 2.0 * (T[d_rows:] @ Cn)
    dist, a = terms[0] - terms[1], assign[d_rows:].long()
    assert int(a.min()) >= 1 and int(a.max()) <= k - 2
    # rounding of a score: 2^-24 of its terms, a few dozen of them
    slack = 1e-5 * (terms[0].max() + 2.0 * (T[d_rows:].abs() @ Cn.abs()).max(1).values)
    assert bool((dist.gather(1, (a - 1).unsqueeze(1)).squeeze(1) <= dist.min(1).values + slack).all())

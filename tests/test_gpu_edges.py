"""Kernels at the sizes where they can go wrong: edges of tiles, remainders, the smallest and largest of their ranges."""
import numpy as np
import pytest

import datagen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def il():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01985_amd as mod
    return mod


def _blocks(seed, r_T, widths, rows=None, missing=0.0, gap=0, shuffle=False, overlap=0):
    """Tables side by side (block k starts where k - 1 ends, plus `gap` unfed or minus `overlap` shared columns);
    the first is the entity table."""
    rng = datagen.rng_for(seed)
    sources, at = [], 0
    for k, c in enumerate(widths):
        r = r_T if k == 0 else (rows or max(1, r_T // 3))
        D = rng.standard_normal((r, c)).astype(np.float32)
        D[rng.random(D.shape) < 0.05] = -0.0
        idx = None
        if k > 0:
            idx = rng.integers(0, r, r_T).astype(np.int32)
            idx[rng.random(r_T) < missing] = -1
        cm = np.arange(at, at + c, dtype=np.int32)
        if shuffle:
            cm = rng.permutation(cm).astype(np.int32)
            cm[::5] = -1
        sources.append(datagen.Source(D, idx, cm))
        at += c + gap - overlap
    c_T = max(int(s.col_map.max()) for s in sources) + 1 + gap
    return datagen.Schema(sources, r_T, c_T)


@pytest.mark.parametrize("r_T,widths,kw", [
    (1, (1, 1), {}),                                              # one row, tile of four
    (5, (3, 8), {"missing": 0.5}),
    (1_023, (10, 50, 100, 40), {"missing": 0.1}),                 # column blocks that start on half a float4
    (4_097, (7, 33, 75), {}),                                     # nothing aligned, a last tile of few rows
    (3_001, (21, 200), {}),                                       # float4 source rows at an odd target column
    (2_050, (4, 8), {"gap": 3}),                                  # columns nobody feeds
    (2_049, (12, 20, 9), {"shuffle": True}),                      # scattered and dropped columns
    (2_047, (9, 9, 9), {"overlap": 7, "missing": 0.2}),           # columns with up to three feeders
    (300, (700, 1_200, 1_684), {}),                               # the widest target table a tile holds
    (300, (700, 1_201, 1_684), {}),                               # one column more: the row-wise kernel
])
@pytest.mark.parametrize("shift", [0, 1])
def test_materialize_any_column_block(il, r_T, widths, kw, shift):
    sch = _blocks(77 + r_T, r_T, widths, **kw)
    plan = il.ilargi_plan_create(il.schema_to_device(sch), sch.r_T, sch.c_T)
    flat = torch.full((sch.r_T * sch.c_T + 8,), 7.0, device="cuda")
    T = flat[shift:shift + sch.r_T * sch.c_T].view(sch.r_T, sch.c_T)      # a table that starts on any float
    il.ilargi_materialize(plan, T)
    want = oracle.Target(sch).T32
    assert np.array_equal(T.cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert torch.all(flat[:shift] == 7.0) and torch.all(flat[shift + sch.r_T * sch.c_T:] == 7.0)

"""Many models at once over a two-table star join: the update from the blocks that both tables' passes leave, against 64 bits."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("r_T,c_S,r_R,c_R,m", [
    (60_001, 4, 3_000, 20, 68),               # the fewest columns of the kernel, a slab of four
    (60_001, 20, 9_001, 64, 100),             # a slab that is not full
    (60_001, 12, 4_100, 100, 128),
    (90_000, 24, 30_000, 200, 256),           # hundreds of blocks of both tables
    (60_001, 8, 3_000, 256, 260),             # wider than the column reduce's registers
    (60_001, 8, 3_000, 63, 130),              # operands that are no whole float4s: launches of their own
])
@pytest.mark.parametrize("model", ["linear", "logistic"])
@pytest.mark.parametrize("drop", [False, True])
def test_update_from_the_blocks_of_both_tables(r_T, c_S, r_R, c_R, m, model, drop):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_01985_amd as il
    gen = torch.Generator(device="cuda").manual_seed(m)
    S, R = torch.randn(r_T, c_S, generator=gen, device="cuda"), torch.randn(r_R, c_R, generator=gen, device="cuda")
    fk = torch.randint(0, r_R, (r_T,), generator=gen, device="cuda", dtype=torch.int32)
    c_T = c_S + c_R + 1                                                  # a column that nobody feeds
    s_cols, r_cols = list(range(c_R, c_R + c_S)), list(range(c_R))
    if drop:
        r_cols[1] = -1
    plan = il.ilargi_plan_create([(S, None, s_cols), (R, fk, r_cols)], r_T, c_T, max_cx=m)
    W = torch.randn(c_T, m, generator=gen, device="cuda") / 8
    y = (torch.rand(r_T, generator=gen, device="cuda") < 0.5).float()
    lr = torch.logspace(-2, -0.5, m, device="cuda")
    Wd, Sd, Rd = W.double(), S.double(), R.double()
    fed = [j for j in range(c_R) if r_cols[j] >= 0]
    z = Sd @ Wd[s_cols] + (Rd[:, fed] @ Wd[fed])[fk.long()]
    e = (z if model == "linear" else z.sigmoid()) - y.double().unsqueeze(1)
    G = torch.zeros(c_T, m, dtype=torch.float64, device="cuda")
    G[s_cols] = Sd.t() @ e
    G[fed] = Rd[:, fed].t() @ torch.zeros(r_R, m, dtype=torch.float64, device="cuda").index_add_(0, fk.long(), e)
    step = lr.double() / r_T * G
    per_row = 0.5 * e * e if model == "linear" else torch.nn.functional.softplus(z) - y.double().unsqueeze(1) * z
    out = []
    for _ in range(2):
        got, loss = W.clone(), torch.empty(m, device="cuda")
        il.ilargi_gd_step(plan, il.LINEAR if model == "linear" else il.LOGISTIC, got, y, lr, loss)
        out.append((got, loss))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    # sums of r_T products in float32: a few units of 2^-24 by the 2-norm; and the rounding of the weight
    assert (out[0][0].double() - (Wd - step)).norm() <= 2e-6 * step.norm() + 2.0 ** -24 * Wd.norm()
    assert (out[0][1].double() - per_row.mean(0)).norm() <= 2e-6 * per_row.mean(0).norm()
    assert torch.equal(out[0][0][c_T - 1], W[c_T - 1])

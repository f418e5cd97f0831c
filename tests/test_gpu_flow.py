"""The one-launch factorisation (flow.hip) against the step schedule.

Both apply the same operations to every element in the same order, so l,
log|Σ|, the quadratic form and the whole factor are compared bit for bit (the
step schedule is taken when near_tiles is given), and l with the oracle at the
binary64 bound.  Sizes: one block, around its edges (half block, block, block
plus one), storage tiles of one to four blocks with all-padding blocks in the
last tile, and enough blocks that every workgroup takes several.  A repeated
location makes a pivot fail in the first or second half of a diagonal block,
in the first block or a later one; both schedules report the same column.
"""
import numpy as np
import pytest

import geoinputs
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

STEPS = 1 << 30  # near_tiles beyond every tile count: the step schedule, one panel per pass
THETA = (1.0, 0.1, 0.5)


@pytest.fixture(scope="module")
def g():
    import paper_1708_02835_amd as pkg
    pkg.lib()
    return pkg


@pytest.fixture(scope="module")
def ctx(g):
    c = g.Context(0)
    yield c
    c.close()


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def both(g, ctx, x, y, z, **o):
    return [g.loglik_eval(ctx, x, y, z, THETA, g.gl_opts_default(near_tiles=near, **o)) for near in (0, STEPS)]


@pytest.mark.parametrize("n,tile", [(1, 128), (64, 128), (127, 128), (128, 128), (129, 128), (193, 256), (385, 512),
                                    (641, 384), (1025, 512), (1601, 256), (4999, 128)])
def test_flow_equals_step_schedule(g, ctx, n, tile):
    print(f"flow n={n} tile={tile}", flush=True)
    x, y = geoinputs.jittered_grid(n, 5)
    z = geoinputs.normal_vector(n, 5)
    xd, yd, zd = dev(x), dev(y), dev(z)
    a, b = both(g, ctx, xd, yd, zd, tile=tile, keep_factor=1)
    try:
        assert a["status"] == b["status"] == g.GL_OK
        assert (a["loglik"], a["logdet"], a["quad"]) == (b["loglik"], b["logdet"], b["quad"])
        assert torch.equal(g.gl_factor_to_dense(ctx, a["factor"]), g.gl_factor_to_dense(ctx, b["factor"]))
        # the kept inverses of the diagonal blocks, through the variances
        t = torch.linspace(0.05, 0.95, 9, dtype=torch.float64, device="cuda")
        u, v = (g.krige_predict(ctx, r["factor"], t, t.flip(0).contiguous(), return_variance=True) for r in (a, b))
        assert torch.equal(u[0], v[0]) and torch.equal(u[1], v[1])
    finally:
        g.gl_factor_release(ctx, a["factor"])
        g.gl_factor_release(ctx, b["factor"])
    if n <= 1025:
        ref = oracle.loglik(x, y, z, THETA)
        assert abs(a["loglik"] - ref[0]) <= 1e-10 * abs(ref[0])


@pytest.mark.parametrize("first,tile", [(20, 128), (90, 128), (300, 128), (353, 256), (1500, 512)])
def test_flow_reports_the_failing_column(g, ctx, first, tile):
    # forty repeated locations: the pivots from `first` on vanish in exact arithmetic, so one of them fails
    n = first + 200
    x, y = geoinputs.jittered_grid(n, 6)
    x[first:first + 40], y[first:first + 40] = x[:40].copy()[:40], y[:40].copy()[:40]
    if first < 40:
        x[first:first + 40], y[first:first + 40] = x[0], y[0]
    z = geoinputs.normal_vector(n, 6)
    a, b = both(g, ctx, dev(x), dev(y), dev(z), tile=tile)
    assert a["status"] == b["status"] and a["info"] == b["info"]
    assert a["status"] == g.GL_NOT_SPD and first < a["info"] <= first + 40
    # and the workspace serves the next evaluation
    xs, ys = geoinputs.jittered_grid(n, 7)
    a, b = both(g, ctx, dev(xs), dev(ys), dev(z), tile=tile)
    assert a["status"] == g.GL_OK and a["loglik"] == b["loglik"]


@pytest.mark.parametrize("n,tile,bad", [(100, 128, None), (129, 128, None), (900, 256, None), (1300, 512, None),
                                        (900, 256, 40), (900, 256, 700)])
@pytest.mark.parametrize("prec", [1, 3])
def test_mixed_call_that_stays_binary64_takes_one_launch(g, ctx, prec, n, tile, bad):
    """tol_64 = 0 keeps every tile binary64; tile 0, factored for the thresholds,
    is generated again: the bits of GL_FP64 in Morton order, and its failing
    column where a location is repeated (in the first tile or a later one)."""
    x, y = geoinputs.jittered_grid(n, 6)
    z = geoinputs.normal_vector(n, 6)
    if bad is not None:
        x[bad + 1], y[bad + 1] = x[bad], y[bad]
    xd, yd, zd = dev(x), dev(y), dev(z)
    a = g.loglik_eval(ctx, xd, yd, zd, THETA, g.gl_opts_default(precision=prec, tile=tile, tol_64=0.0))
    b = g.loglik_eval(ctx, xd, yd, zd, THETA, g.gl_opts_default(tile=tile, reorder=1))
    assert (a["status"], a["info"]) == (b["status"], b["info"])
    if b["status"] == g.GL_OK:
        assert (a["loglik"], a["logdet"], a["quad"]) == (b["loglik"], b["logdet"], b["quad"])

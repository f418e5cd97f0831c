"""The one-launch backward solve (back.hip) behind kriging, against the oracle:
sizes around one column block (half a block, a block, a block plus one), ragged
last tiles of every storage tile size with all-padding blocks, and a chain of
many blocks.  The bound is that of the kriging parity tests, 1e-9 of the largest
measurement, far above the rounding of either side (κ(Σ) is below 1e4 here, so
a solve is good to about 1e-12)."""
import numpy as np
import pytest

import geoinputs
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


@pytest.mark.parametrize("n,tile", [(1, 128), (64, 128), (65, 256), (127, 384), (128, 128), (129, 128), (129, 512),
                                    (385, 256), (641, 512), (900, 384), (1601, 128)])
def test_backward_solve_through_kriging(n, tile):
    import paper_1708_02835_amd as g
    theta = (1.3, 0.1, 0.5)
    x, y = geoinputs.jittered_grid(n, 8)
    z = geoinputs.normal_vector(n, 8)
    xn, yn = geoinputs.uniform_points(33, 8)
    print(f"back n={n} tile={tile}", flush=True)
    with g.Context(0) as ctx:
        r = g.loglik_eval(ctx, dev(x), dev(y), dev(z), theta, g.gl_opts_default(tile=tile, keep_factor=1))
        assert r["status"] == g.GL_OK
        first = g.krige_predict(ctx, r["factor"], dev(xn), dev(yn))
        again = g.krige_predict(ctx, r["factor"], dev(xn), dev(yn))
        assert torch.equal(first, again)
        got = first.cpu().numpy()
        g.gl_factor_release(ctx, r["factor"])
    want, info = oracle.krige(x, y, z, xn, yn, theta)
    assert info == 0
    assert np.max(np.abs(got - want)) <= 1e-9 * np.max(np.abs(z))


@pytest.mark.parametrize("n,tile,m", [(1, 128, 1), (128, 128, 64), (129, 256, 63), (385, 512, 65), (700, 384, 130),
                                      (900, 128, 1061)])
def test_variances_at_block_edges(n, tile, m):
    """The one-launch right-hand-side solve (64 of them per block row): against
    the oracle at the variance parity bound, 1e-15 κ(Σ) and at least 1e-10."""
    import paper_1708_02835_amd as g
    theta = (1.3, 0.1, 0.5)
    x, y = geoinputs.jittered_grid(n, 9)
    z = geoinputs.normal_vector(n, 9)
    xn, yn = geoinputs.uniform_points(m, 9)
    print(f"variances n={n} tile={tile} m={m}", flush=True)
    with g.Context(0) as ctx:
        r = g.loglik_eval(ctx, dev(x), dev(y), dev(z), theta, g.gl_opts_default(tile=tile, keep_factor=1))
        assert r["status"] == g.GL_OK
        pred, var = g.krige_predict(ctx, r["factor"], dev(xn), dev(yn), return_variance=True)
        pred, var = pred.cpu().numpy(), var.cpu().numpy()
        g.gl_factor_release(ctx, r["factor"])
    want, wvar, info = oracle.krige(x, y, z, xn, yn, theta, return_variance=True)
    assert info == 0
    tol = max(1e-10, 1e-15 * np.linalg.cond(oracle.cov_symmetric(x, y, theta)))
    assert np.max(np.abs(pred - want)) <= 1e-9 * np.max(np.abs(z))
    assert np.max(np.abs(var - wvar)) <= tol * theta[0]


@pytest.mark.parametrize("metric,t3", [(0, 0.5), (0, 1.0), (1, 0.8)])
def test_grouped_kriging_sums_equal_single_ones(metric, t3):
    """2,050 new locations over two chunks of observed points take the kernel
    that sums four at a time, half of them the one that sums one: the same
    order per location, so the same bits."""
    import paper_1708_02835_amd as g
    n, m = 4097, 2050
    x, y = geoinputs.jittered_grid(n, 10)
    xn, yn = geoinputs.uniform_points(m, 10)
    z = geoinputs.normal_vector(n, 10)
    theta = (1.3, 300.0 if metric else 0.03, t3)
    if metric:
        x, y, xn, yn = -100 + 15 * x, 30 + 15 * y, -100 + 15 * xn, 30 + 15 * yn
    o = dict(metric=metric, radius=6371.0)
    print(f"grouped kriging metric={metric} t3={t3}", flush=True)
    with g.Context(0) as ctx:
        r = g.loglik_eval(ctx, dev(x), dev(y), dev(z), theta, g.gl_opts_default(keep_factor=1, **o))
        assert r["status"] == g.GL_OK
        whole = g.krige_predict(ctx, r["factor"], dev(xn), dev(yn))
        h = m // 2
        parts = [g.krige_predict(ctx, r["factor"], dev(xn[a:a + h]), dev(yn[a:a + h])) for a in (0, h)]
        assert torch.equal(whole, torch.cat(parts))
        g.gl_factor_release(ctx, r["factor"])

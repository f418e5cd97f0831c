"""Cross-validation folds factored together (one launch for many folds) against
each fold on its own, kept factor and prediction: the same operations in the
same order, so the same bits.  More folds than lanes of a wavefront (the launch
looks its problems up 64 at a time), folds of very different size with more
than one tile size, a fold of one location, folds that do not fit together, and
a fold whose covariance is not positive definite."""
import numpy as np
import pytest

import geoinputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

THETA = (1.3, 0.1, 0.5)


def dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


@pytest.fixture(scope="module")
def g():
    import paper_1708_02835_amd as g
    return g


def inputs(n, seed):
    x, y = geoinputs.jittered_grid(n, seed)
    return x, y, geoinputs.normal_vector(n, seed)


def one_by_one(g, ctx, x, y, z, folds, k, **o):
    """Prediction of every location from the folds other than its own (NaN where the factorisation fails)."""
    pred = np.full(len(x), np.nan)
    for f in range(k):
        known, miss = folds != f, folds == f
        r = g.loglik_eval(ctx, dev(x[known]), dev(y[known]), dev(z[known]), THETA, g.gl_opts_default(keep_factor=1, **o))
        if r["status"] == g.GL_OK:
            pred[miss] = g.krige_predict(ctx, r["factor"], dev(x[miss]), dev(y[miss])).cpu().numpy()
            g.gl_factor_release(ctx, r["factor"])
    return pred


def sizes(n, counts, seed):
    folds = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    assert len(folds) == n
    return np.random.Generator(np.random.PCG64(seed)).permutation(folds)


CASES = [("many", 350, [5] * 70, 128, 0), ("one location", 260, [1, 130, 129], 128, 0),
         ("uneven", 1300, [1100, 150, 50], 256, 0), ("automatic tile", 2500, [2300, 150, 50], 0, 0),
         ("ragged", 1025, [205] * 5, 384, 0), ("wide tile", 700, [234, 233, 233], 512, 0),
         ("no room", 900, [300] * 3, 128, 8 << 20)]


@pytest.mark.parametrize("name,n,counts,tile,budget", CASES, ids=[c[0] for c in CASES])
def test_folds_together_equal_folds_alone(g, name, n, counts, tile, budget):
    x, y, z = inputs(n, 31)
    k = len(counts)
    folds = sizes(n, counts, 32)
    print(f"cv {name} n={n} k={k} tile={tile}", flush=True)
    with g.Context(0, budget) if budget else g.Context(0) as ctx:
        pred = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
        mse, st = g.krige_cv(ctx, dev(x), dev(y), dev(z), THETA, folds, g.gl_opts_default(tile=tile), pred=pred)
        assert st == g.GL_OK
        again, _ = g.krige_cv(ctx, dev(x), dev(y), dev(z), THETA, folds, g.gl_opts_default(tile=tile))
        assert list(mse) == list(again)
        want = one_by_one(g, ctx, x, y, z, folds, k, tile=tile)
    got = pred.cpu().numpy()
    assert np.array_equal(got, want)
    for f in range(k):
        ref = float(np.mean((want[folds == f] - z[folds == f]) ** 2))
        assert abs(mse[f] - ref) <= 1e-12 * ref


def test_failing_folds_are_reported_and_leave_the_others(g):
    """Location 0 repeated in fold 1: Σ of every fold that observes both is
    singular, only fold 1, which holds one of them out, is factored."""
    n, k = 600, 3
    x, y, z = inputs(n, 33)
    folds = (np.arange(n) % k).astype(np.int32)
    x[1], y[1] = x[0], y[0]
    folds[1] = 1
    with g.Context(0) as ctx:
        pred = torch.full((n,), 7.5, dtype=torch.float64, device="cuda")
        mse, st = g.krige_cv(ctx, dev(x), dev(y), dev(z), THETA, folds, g.gl_opts_default(tile=128), pred=pred)
        want = one_by_one(g, ctx, x, y, z, folds, k, tile=128)
    got = pred.cpu().numpy()
    failed = [f for f in range(k) if np.isnan(want[folds == f]).any()]
    assert st == (g.GL_NOT_SPD if failed else g.GL_OK) and 1 not in failed
    for f in range(k):
        if f in failed:
            assert np.isnan(mse[f]) and np.all(got[folds == f] == 7.5)
        else:
            assert np.array_equal(got[folds == f], want[folds == f])

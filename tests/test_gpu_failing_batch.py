"""A problem whose Σ is not positive definite beside healthy ones in one launch:
the healthy results are those of single calls, bit for bit, and the failing one
reports its own column.  The failing problem has far more 128×128 blocks left
than a launch has workgroups (512), so workgroups that stopped with it would be
missing for the others, and every workspace held another θ's values before.
Σ fails through sixty repeated locations, whose pivots come out as rounding
noise of either sign (a single repeat would leave it to one rounding)."""
import math
import time

import numpy as np
import pytest

import geoinputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

THETA, EARLIER = (1.0, 0.1, 0.5), (1.7, 0.06, 1.5)
DUP = 60


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


def field(n, seed, bad=None):
    """bad: the DUP locations from there on repeat the DUP before them."""
    x, y = geoinputs.jittered_grid(n, seed)
    if bad is not None:
        x[bad:bad + DUP], y[bad:bad + DUP] = x[bad - DUP:bad].copy(), y[bad - DUP:bad].copy()
    return dev(x), dev(y), dev(geoinputs.normal_vector(n, seed))


def test_queue_serves_the_requests_beside_a_failing_one(g, ctx):
    data = [field(6400, 41, bad=DUP), field(6000, 42), field(6300, 43), field(2500, 44)]
    sets = [g.gl_dataset_register(ctx, *d) for d in data]
    q = g.lq_create(ctx)
    order = [1, 0, 2, 3, 0, 1, 2, 0, 3, 1, 0, 2] * 2  # ticks of several requests, a failing one in most
    try:
        for theta in (EARLIER, THETA):
            res = [g.lq_wait(q, t, int(60e6)) for t in [g.lq_submit(q, sets[i], theta) for i in order]]
    finally:
        g.lq_destroy(q)
        for s in sets:
            g.gl_dataset_release(ctx, s)
    ref = [g.loglik_eval(ctx, *d, THETA, g.gl_opts_default(tile=256)) for d in data]
    assert ref[0]["status"] == g.GL_NOT_SPD and DUP < ref[0]["info"] <= 2 * DUP
    for i, r in zip(order, res):
        assert (r["status"], r["info"]) == (ref[i]["status"], ref[i]["info"]), i
        if i == 0:
            assert r["loglik"] == -math.inf
        else:
            assert (r["loglik"], r["logdet"], r["quad"]) == (ref[i]["loglik"], ref[i]["logdet"], ref[i]["quad"]), i


def test_cross_validation_computes_the_folds_beside_failing_ones(g, ctx):
    """Folds 0 and 1 hold out one copy each of every repeated location, folds 2
    and 3 observe both."""
    n, k = 8000, 4
    x, y, z = field(n, 45, bad=DUP)
    folds = (np.arange(n) % k).astype(np.int32)
    folds[:DUP], folds[DUP:2 * DUP] = 0, 1
    o = g.gl_opts_default(tile=128)
    g.krige_cv(ctx, *field(n, 46), EARLIER, folds, o)
    pred = torch.full((n,), 7.5, dtype=torch.float64, device="cuda")
    mse, st = g.krige_cv(ctx, x, y, z, THETA, folds, o, pred=pred)
    assert st == g.GL_NOT_SPD
    for f in range(k):
        known, miss = (torch.as_tensor(m).cuda() for m in (folds != f, folds == f))
        r = g.loglik_eval(ctx, x[known], y[known], z[known], THETA, g.gl_opts_default(tile=128, keep_factor=1))
        if f >= 2:
            assert r["status"] == g.GL_NOT_SPD
            assert np.isnan(mse[f]) and bool((pred[miss] == 7.5).all())
            continue
        want = g.krige_predict(ctx, r["factor"], x[miss], y[miss])
        g.gl_factor_release(ctx, r["factor"])
        assert torch.equal(pred[miss], want), f
        # the same squares summed in another order
        assert abs(mse[f] - float(((want - z[miss]) ** 2).mean())) <= 1e-12 * mse[f]


def test_independent_blocks_report_the_first_failing_block(g, ctx):
    """Block 0 fails near its end, block 1 at its start, block 2 not at all."""
    block = 48 * 128
    parts = [field(block, 47, bad=6000), field(block, 48, bad=DUP), field(block, 49)]
    x, y, z = (torch.cat(c) for c in zip(*parts))
    r = g.loglik_eval(ctx, x, y, z, THETA, g.gl_opts_default(tile=128, ind_tiles=48))
    ref = g.loglik_eval(ctx, *parts[0], THETA, g.gl_opts_default(tile=128))
    assert ref["status"] == g.GL_NOT_SPD and 6000 < ref["info"] <= 6000 + DUP
    assert (r["status"], r["info"]) == (g.GL_NOT_SPD, ref["info"])


def test_failure_half_way_ends_the_evaluation(g, ctx):
    """The blocks before column n/2 are half of the work: a failure there leaves the
    other half out (the sums of the blocks after it would be a quarter more)."""
    n = 40000
    times = []
    for bad in (None, n // 2):
        x, y, z = field(n, 50, bad=bad)
        for _ in range(2):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            r = g.loglik_eval(ctx, x, y, z, THETA)
            t = time.perf_counter() - t0
        times.append(t)
    assert r["status"] == g.GL_NOT_SPD and n // 2 < r["info"] <= n // 2 + DUP
    print(f"healthy {times[0]:.4f} s, failing {times[1]:.4f} s", flush=True)
    assert times[1] < 0.65 * times[0]

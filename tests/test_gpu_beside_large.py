"""Work beside a large factorisation gets onto the chip while it runs: a small
request of the queue beside a large one on a stream of its own or beside a batch
of large ones, and a kernel of another stream beside a direct call.  Each arrives in the first tenth of the
large work and has to be done in less than half (a third) of its time: alone it
takes less than a hundredth of it, kept out it waits for nearly all of it."""
import threading
import time

import numpy as np
import pytest

import geoinputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

THETA = (1.0, 0.1, 0.5)
LARGE = 40000


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


def field(n, seed):
    return [torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()
            for a in (*geoinputs.jittered_grid(n, seed), geoinputs.normal_vector(n, seed))]


def test_small_request_beside_a_large_one(g, ctx):
    sets = [g.gl_dataset_register(ctx, *field(n, 51)) for n in (LARGE, 1000)]
    q = g.lq_create(ctx)
    try:
        for s in sets:  # workspaces and streams exist from here on
            assert g.lq_wait(q, g.lq_submit(q, s, THETA), int(60e6))["status"] == g.GL_OK
        t0 = time.perf_counter()
        large = g.lq_submit(q, sets[0], THETA)
        time.sleep(0.02)
        t1 = time.perf_counter()
        assert g.lq_wait(q, g.lq_submit(q, sets[1], THETA), int(60e6))["status"] == g.GL_OK
        t2 = time.perf_counter()
        assert g.lq_wait(q, large, int(60e6))["status"] == g.GL_OK
        t3 = time.perf_counter()
        print(f"small {t2 - t1:.4f} s, large {t3 - t0:.4f} s", flush=True)
        assert t2 - t1 < 0.5 * (t3 - t0)
    finally:
        g.lq_destroy(q)
        for s in sets:
            g.gl_dataset_release(ctx, s)


@pytest.mark.parametrize("delay", [0.0, 0.03])
def test_small_request_beside_a_batch_of_large_ones(g, ctx, delay):
    """Submitted with them, or while they run."""
    sets = [g.gl_dataset_register(ctx, *field(n, 53)) for n in (14000, 1000)]
    q = g.lq_create(ctx)

    def batch():
        t0 = time.perf_counter()
        large = [g.lq_submit(q, sets[0], THETA) for _ in range(16)]
        time.sleep(delay)
        t1 = time.perf_counter()
        small = g.lq_wait(q, g.lq_submit(q, sets[1], THETA), int(60e6))
        t2 = time.perf_counter()
        res = [g.lq_wait(q, t, int(60e6)) for t in large]
        return t2 - t1, time.perf_counter() - t0, [small] + res

    try:
        batch()  # workspaces exist from here on
        small, all_of_them, res = batch()
    finally:
        g.lq_destroy(q)
        for s in sets:
            g.gl_dataset_release(ctx, s)
    print(f"small {small:.4f} s, batch {all_of_them:.4f} s", flush=True)
    assert all(r["status"] == g.GL_OK for r in res)
    assert len({r["loglik"] for r in res[1:]}) == 1
    assert small < 0.3 * all_of_them


def test_kernel_of_another_stream_runs_beside_a_large_evaluation(g, ctx):
    """The first of several streams' kernels to end: a stream may share the
    evaluation's hardware queue (a process has four), others then do not."""
    x, y, z = field(LARGE, 52)
    a = torch.ones(1 << 20, device="cuda")
    sides = [torch.cuda.Stream() for _ in range(6)]

    def launch(factor):
        out = []
        for s in sides:
            with torch.cuda.stream(s):
                out.append((a * factor, torch.cuda.Event()))
                out[-1][1].record()
        return out

    g.loglik_eval(ctx, x, y, z, THETA)
    launch(2)
    torch.cuda.synchronize()
    took = []

    def evaluate():
        t0 = time.perf_counter()
        g.loglik_eval(ctx, x, y, z, THETA)
        took.append(time.perf_counter() - t0)

    th = threading.Thread(target=evaluate)
    th.start()
    time.sleep(0.02)
    t1 = time.perf_counter()
    launched = launch(3)
    while not any(e.query() for _, e in launched):
        time.sleep(1e-4)
    t2 = time.perf_counter()
    th.join()
    torch.cuda.synchronize()
    print(f"kernel {t2 - t1:.4f} s, evaluation {took[0]:.4f} s", flush=True)
    assert all(float(b[0]) == 3.0 for b, _ in launched)
    assert t2 - t1 < 0.5 * took[0]

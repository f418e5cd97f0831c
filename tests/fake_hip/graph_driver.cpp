// Which schedule a replayed evaluation graph holds, checked on the CPU (built
// against the HIP stand-in of this folder by tests/test_graph_key.py, with the
// capture functions of this file).  Test infrastructure only.  A capture runs its
// commands at once, a replay none; the one-launch factorisation is a stand-in
// that counts its calls.  Prints "ok" when everything holds.
#include <stdio.h>

#include <vector>

#include "engine.hpp"

static int captures = 0, replays = 0, one_launch = 0;
static int object;
hipError_t count_begin(hipStream_t, hipStreamCaptureMode)
{
    ++captures;
    return hipSuccess;
}
hipError_t count_end(hipStream_t, hipGraph_t *g)
{
    *g = reinterpret_cast<hipGraph_t>(&object);
    return hipSuccess;
}
hipError_t count_instantiate(hipGraphExec_t *e, hipGraph_t, void *, char *, size_t)
{
    *e = reinterpret_cast<hipGraphExec_t>(&object);
    return hipSuccess;
}
hipError_t count_launch(hipGraphExec_t, hipStream_t)
{
    ++replays;
    return hipSuccess;
}

namespace gl {
int flow_factorize(Work &w, hipStream_t s, bool)
{
    ++one_launch;
    for (int64_t k = 0; k < w.nt; ++k) {
        launch_potrf(w.tiles, w.b, k, w.n, w.info, w.logsum, w.dinv_k(k), s);
        launch_fwd_diag(w.tiles, w.b, k, w.n, w.v, w.quad, w.dinv_k(k), w.info, s);
    }
    return GL_OK;
}
}  // namespace gl

int main()
{
    gl_context *ctx = nullptr;
    if (gl_context_create(0, 0, &ctx) != GL_OK) return 2;
    const int64_t n = 300;  // tiles of 128, and as many near tiles by default
    std::vector<double> x(n), y(n, 0.0), z(n, 0.5);
    int failures = 0;
    // near_tiles of each call; captures and one-launch factorisations after it
    const int calls[][3] = {{0, 1, 1}, {0, 1, 1}, {128, 2, 1}, {128, 2, 1}, {0, 3, 2}, {64, 4, 2}, {128, 5, 2}, {0, 6, 3}};
    int k = 0;
    for (const auto &c : calls) {
        gl_opts o;
        gl_opts_default(&o);
        o.graph = 1;
        o.near_tiles = c[0];
        gl_result r;
        const int st = loglik_eval(ctx, x.data(), y.data(), z.data(), n, gl_theta{2.0, 0.1, 0.5}, &o, &r, nullptr);
        ++k;
        if (st != GL_OK || captures != c[1] || one_launch != c[2] || replays != k) {
            fprintf(stderr, "call %d (near_tiles %d): status %d, %d captures, %d one-launch, %d replays\n", k, c[0], st,
                    captures, one_launch, replays);
            ++failures;
        }
    }
    gl_context_destroy(ctx);
    if (failures) return 1;
    printf("ok\n");
    return 0;
}

// Kriging variances in a build without the kernels that solve for them (the HIP
// stand-in of this folder, built by tests/test_solve_launchers.py): an error, not
// the unsolved right-hand sides' values.  Test infrastructure only.
#include <stdio.h>

#include <vector>

#include "geolik.h"

int main()
{
    gl_context *ctx = nullptr;
    if (gl_context_create(0, 0, &ctx) != GL_OK) return 2;
    const int64_t n = 200;
    std::vector<double> x(n), y(n, 0.0), z(n, 0.5);
    for (int64_t i = 0; i < n; ++i) x[i] = (double)i;
    gl_opts o;
    gl_opts_default(&o);
    o.keep_factor = 1;
    gl_result r;
    if (loglik_eval(ctx, x.data(), y.data(), z.data(), n, gl_theta{2.0, 0.1, 0.5}, &o, &r, nullptr) != GL_OK) return 2;
    double xn[2] = {0.5, 1.5}, yn[2] = {0, 0}, zn[2], var[2];
    const int st = krige_predict(ctx, r.factor, xn, yn, 2, zn, var, nullptr);
    gl_context_destroy(ctx);
    printf("%d\n", st);
    return 0;
}

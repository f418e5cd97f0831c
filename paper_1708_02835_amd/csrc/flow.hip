// The one-launch factorisation (flow.hpp) with workgroups that stay, and the choice
// between it and turns.hip.
#define FLOW_LEAVE false
#include "flow.hpp"

namespace gl {

namespace {

// Sums of the parts over the block columns, in order: thread per right-hand side.
__global__ void flow_rhs_sum_kernel(const double *__restrict__ part, int nb, int groups, int64_t m, double theta1,
                                    double *__restrict__ var)
{
    const int64_t k = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (k >= m) return;
    double q = 0.0;
#pragma unroll 8
    for (int j = 0; j < nb; ++j) q += part[((int64_t)j * groups + (k >> 6)) * 64 + (k & 63)];
    var[k] = theta1 - q;
}

}  // namespace

int flow_factorize(Work &w, hipStream_t s, bool solve)
{
    return (double)w.n * w.n * w.n / 3.0 <= FLOW_LONG ? flow_launch(w, s, solve) : flow_launch_turns(w, s, solve);
}

void launch_flow_batched(int b, const BatchReq *d, int count, int64_t blocks, int64_t pads, double flops, hipStream_t s)
{
    if (flops <= FLOW_LONG) flow_launch_batched(b, d, count, blocks, pads, s);
    else flow_launch_batched_turns(b, d, count, blocks, pads, s);
}

int64_t flow_rhs_scratch(int64_t n, int64_t m)
{
    const int64_t groups = ceil_div(m, 64);
    return 8 * (1 + groups) + ceil_div(n, FB) * groups * 64;
}

void launch_flow_rhs(const Work &w, double *st, int64_t m, double theta1, double *scratch, double *var, hipStream_t s)
{
    const int nb = (int)ceil_div(w.n, FB), groups = (int)ceil_div(m, 64);
    launch_fill(scratch, 8 * (1 + groups), 0.0, s);
    int *words = reinterpret_cast<int *>(scratch);
    double *part = scratch + 8 * (1 + groups);
    if (64.0 * groups * w.n * w.n <= FLOW_LONG) flow_launch_rhs(w, st, groups, words, part, s);
    else flow_launch_rhs_turns(w, st, groups, words, part, s);
    flow_rhs_sum_kernel<<<groups, 64, 0, s>>>(part, nb, groups, m, theta1, var);
}

}  // namespace gl

// Whole evaluations of many independent problems in fused launches (see
// batch.hpp): fills the prefix offsets of the descriptors, copies them to the
// device and enqueues the launches.
#include <algorithm>

#include "batch.hpp"

namespace gl {

int enqueue_whole(BatchReq *d, BatchReq *dev, int count, int b, hipStream_t s, int *launches)
{
    std::sort(d, d + count, [](const BatchReq &x, const BatchReq &y) { return x.n > y.n; });
    int64_t o_stage = 0, o_gen = 0, o_flow = 0, pads = 0;
    double flops = 0.0;
    bool euclid = true;
    for (int i = 0; i < count; ++i) {
        BatchReq &q = d[i];
        const int64_t nb = ceil_div(q.n, 128);
        const int64_t next = i + 1 < count ? ceil_div(d[i + 1].n, 128) : 0;
        q.is_new = q.finishing = 1;
        q.o_stage = o_stage;
        q.o_gen = o_gen;
        q.o_flow = o_flow;
        o_stage += ceil_div(q.npad, 256);
        o_gen += tile_count(q.nt);
        // columns with nb .. next + 1 blocks left, in i + 1 factorisations each
        o_flow += (i + 1) * (tile_count(nb) - tile_count(next));
        pads += q.npad / 128 - nb;
        flops += (double)q.n * q.n * q.n / 3.0;
        euclid = euclid && q.geo.metric == GL_EUCLIDEAN;
    }
    if (o_flow + pads > INT32_MAX) return GL_EINVAL;
    GL_HIP_TRY(hipMemcpyAsync(dev, d, count * sizeof(BatchReq), hipMemcpyHostToDevice, s));
    launch_stage_batched(dev, count, o_stage, s);
    launch_gen_batched(b, dev, count, o_gen, euclid, s);
    if (launch_flow_batched) {
        launch_flow_batched(b, dev, count, o_flow, pads, flops, s);
    } else {
        for (int i = 0; i < count; ++i) {
            const BatchReq &q = d[i];
            for (int64_t k = 0; k < q.nt; ++k) {
                double *dinv = q.dinv + k * 64 * b;
                launch_potrf(q.tiles, b, k, q.n, q.info, q.logsum, dinv, s);
                launch_trsm(q.tiles, b, q.nt, k, dinv, q.info, s);
                launch_fwd_diag(q.tiles, b, k, q.n, q.v, q.quad, dinv, q.info, s);
                launch_fwd_update(q.tiles, b, q.nt, k, q.v, q.info, s);
                launch_trailing(q.tiles, b, q.nt, k, k + 1, q.nt - 1, q.info, false, false, s);
            }
        }
    }
    launch_final_batched(dev, count, s);
    GL_HIP_TRY(hipGetLastError());
    if (launches) *launches = 4;
    return GL_OK;
}

}  // namespace gl

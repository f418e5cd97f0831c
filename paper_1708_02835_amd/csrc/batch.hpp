// Descriptors of the fused multi-request launches used by the serving loop and
// the independent-blocks approximation.  One launch covers the same phase of
// many requests; each request's work is given by exclusive prefix offsets and
// runs the same per-request code as a single evaluation, so a request's
// arithmetic does not depend on what else is in the launch.
#pragma once

#include "common.hpp"

namespace gl {

struct BatchReq {
    double *tiles, *x, *y, *v, *dinv, *logsum, *quad;
    int64_t *info;
    DevResult *res;
    const double *sx, *sy, *sz;  // dataset (sources of the staging copy)
    gl_theta th;
    Geom geo;
    int64_t n, nt, npad, k;      // k: unused by the whole-evaluation launches (0)
    int64_t o_stage, o_gen, o_flow;
    int32_t is_new, finishing;   // generates / reduces in this launch (1)
    int32_t stride;              // of the progress words, in ints
    int32_t *words;              // flow_words() ints, cleared with the staging
};

// Progress words of one whole factorisation (flow.hpp): a ticket and three words
// per 128-column block, each on a cache line of its own from one block on.
__host__ __device__ inline int flow_stride(int64_t n) { return n >= 128 ? 16 : 1; }
__host__ __device__ inline int64_t flow_words(int64_t n, int stride) { return (2 + 3 * ((n + 127) / 128)) * stride; }

// Largest request index r with offset(r) <= g (ranges may be empty), 64
// requests looked at a time, by whole wavefronts (one after the other, the scan
// bound launches of many small requests: 1,000 cross-validation folds of 999
// locations 31.0 -> 24.0 ms, 49 blocks of 2,048 3.41 -> 3.37 ms).
#define GL_BATCH_FIND(d, count, g, field)                                           \
    ([&]() {                                                                        \
        const int l_ = threadIdx.x & 63;                                            \
        int r_ = 0;                                                                 \
        for (int q_ = 0; q_ < (count); q_ += 64) {                                  \
            const unsigned long long m_ =                                           \
                __ballot(q_ + l_ < (count) && (d)[q_ + l_].field <= (g));           \
            if (m_ == 0) break;                                                     \
            r_ = q_ + 63 - __clzll(m_);                                             \
        }                                                                           \
        return __builtin_amdgcn_readfirstlane(r_);                                  \
    }())

// Launchers (b = 128, 256, 384, 512); grids come from the totals of the prefix
// offsets.
void launch_stage_batched(const BatchReq *d, int count, int64_t blocks, hipStream_t s);
// euclid: every request that generates in this launch uses the Euclidean distance.
void launch_gen_batched(int b, const BatchReq *d, int count, int64_t tiles, bool euclid, hipStream_t s);
// Factorisations and forward solves of all requests, sorted by falling size:
// `blocks` 128×128 blocks in all, `pads` all-padding diagonal blocks and `flops`, the sum of
// n³/3 (flow.hip; weak: not part of builds without device code).
void launch_flow_batched(int b, const BatchReq *d, int count, int64_t blocks, int64_t pads, double flops, hipStream_t s)
    __attribute__((weak));
// v <- L⁻ᵀ v for every request whose factorisation succeeded, in one launch (back.hip); d as after
// enqueue_whole (its words are used again), longest: the largest n.
void launch_backward_batched(int b, const BatchReq *d, int count, int64_t longest, hipStream_t s);
void launch_final_batched(const BatchReq *d, int count, hipStream_t s);

// The whole evaluations of d[0..count) (count >= 1): staging and Σ generation,
// the factorisations and forward solves, the final sums.  The caller sets
// the fields up to k, words and stride, with dinv that of step 0; d is sorted
// and its offsets filled in, the array is copied to dev (device, count
// entries) on s and the launches follow.  d must stay valid until the copy
// has been consumed (pinned memory: until the stream passes it).  Builds
// without device code run the factorisations one after the other by steps.
int enqueue_whole(BatchReq *d, BatchReq *dev, int count, int b, hipStream_t s, int *launches);

}  // namespace gl

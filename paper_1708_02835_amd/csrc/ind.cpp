// Independent-blocks (IND) approximation, Sec. 6.8: the tiles outside the
// diagonal super tiles of s×s tiles are annihilated, so Σ is block diagonal
// with blocks of s·b consecutive locations and l(θ) is the sum of the exact
// log-likelihoods of the blocks.  Nothing outside the blocks is generated or
// factored: the blocks are independent factorisations of s tile columns each
// (the last one possibly shorter), all in one launch (enqueue_whole).
//
// Kriging under the same approximation (the exact-versus-IND prediction
// comparison of the paper's experiments, with Eq. (5)): applied to the
// covariance of all locations, observed and held-out alike, the blocks are
// independent fields, so each held-out value is predicted from the observed
// values of its own block, Z_M = Σ_MO Σ_OO⁻¹ Z_O, through the block's factor
// (backward substitution of w = L⁻¹ Z_O).
//
// The folds of an exact cross-validation are such a set of independent
// problems too (cv_folds).
#include <algorithm>
#include <vector>

#include "batch.hpp"
#include "engine.hpp"

namespace gl {

// Sums the per-block results in block order; info of the first failing block,
// as a global 1-based column.
__global__ void ind_total_kernel(const DevResult *__restrict__ r, int64_t nblk, int64_t block,
                                 DevResult *__restrict__ out)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double l = 0.0, ld = 0.0, q = 0.0;
    int64_t info = 0;
    for (int64_t i = 0; i < nblk; ++i) {
        if (info == 0 && r[i].info != 0) info = i * block + r[i].info;
        l += r[i].loglik;
        ld += r[i].logdet;
        q += r[i].quad;
    }
    out->info = info;
    out->loglik = info ? -INFINITY : l;
    out->logdet = info ? NAN : ld;
    out->quad = info ? NAN : q;
}

// The blocks of one IND factorisation: one descriptor per block (factor
// tiles, padded coordinates, w = L⁻¹ Z of the block in v), the locations the
// blocks were cut from (input or Morton order) and the per-block results.
struct IndPlan {
    int b = 0;
    int64_t nblk = 0;
    std::vector<BatchReq> proto;
    std::vector<int64_t> start, nb, ntb;
    std::vector<size_t> off;            // of each block's part of the workspace, in doubles
    size_t morton = 0, doubles = 0;     // of the reordered inputs; whole workspace
    const double *sx = nullptr, *sy = nullptr;
    const BatchReq *desc = nullptr;     // device descriptors
    const DevResult *res = nullptr;     // per-block results (device)
};

static size_t word_doubles(int64_t n) { return (size_t)(flow_words(n, flow_stride(n)) + 1) / 2; }

static size_t desc_doubles(int64_t nblk) { return ((size_t)nblk * sizeof(BatchReq) + 15) / 16 * 2; }

// Workspace of one factorisation of n locations: tiles, x, y, v, logsum,
// quad, dinv, progress words.
static size_t block_doubles(int64_t n, int b)
{
    const int64_t nt = ceil_div(n, b), np = nt * b;
    const size_t d = (size_t)tile_count(nt) * b * b + 3 * np + 2 * nt + 64 * np + word_doubles(n);
    return d + (d & 1);
}

// The blocks [start[i], start[i] + count[i]) of n locations (each count >= 1)
// and the layout of their workspace, in doubles: descriptors | per-block
// results, info | per block: its workspace | reordered inputs, keys
static void ind_layout(int b, const std::vector<int64_t> &start, const std::vector<int64_t> &count, int64_t n,
                       bool reorder, IndPlan &p)
{
    p.b = b;
    p.nblk = (int64_t)start.size();
    p.start = start;
    p.nb = count;
    size_t off = desc_doubles(p.nblk) + 16 * (size_t)p.nblk;
    for (int64_t i = 0; i < p.nblk; ++i) {
        p.off.push_back(off);
        p.ntb.push_back(ceil_div(count[i], b));
        off += block_doubles(count[i], b);
    }
    p.morton = off;
    if (reorder) off += 3 * (size_t)n + (n & 1) + (size_t)npow2_of(n) + 4;
    p.doubles = off;
}

// The context's workspace, grown to `bytes`.
static int ind_workspace(gl_context *ctx, size_t bytes)
{
    if (bytes <= ctx->ind_cap) return GL_OK;
    const size_t old = ctx->ind_cap;
    if (ctx->used.load() - old + bytes > ctx->budget) return GL_ENOMEM;
    if (ctx->ind_buf) hipFree(ctx->ind_buf);
    ctx->ind_buf = nullptr;
    ctx->ind_cap = 0;
    ctx->used -= old;
    if (hipMalloc(&ctx->ind_buf, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return GL_ENOMEM;
    }
    ctx->ind_cap = bytes;
    ctx->used += bytes;
    return GL_OK;
}

// Enqueues the factorisation of the blocks of p (ind_layout) in the workspace
// `base` and the fixed-order sum of the per-block results into ctx->res_h (all
// on s).  With reorder the locations are first put in Morton order.  block:
// uniform block length (the likelihood's), for the reported column.
static int ind_factor(gl_context *ctx, const double *x, const double *y, const double *z, int64_t n, gl_theta th,
                      const gl_opts &o, int64_t block, bool reorder, double *base, hipStream_t s, IndPlan &p)
{
    const int64_t nblk = p.nblk;
    const int b = p.b;
    BatchReq *ddesc = reinterpret_cast<BatchReq *>(base);
    DevResult *bres = reinterpret_cast<DevResult *>(base + desc_doubles(nblk));
    int64_t *binfo = reinterpret_cast<int64_t *>(base + desc_doubles(nblk) + 8 * nblk);
    const double *sx = x, *sy = y, *sz = z;
    if (reorder) {
        double *xo = base + p.morton, *yo = xo + n, *zo = yo + n;
        uint64_t *keys = reinterpret_cast<uint64_t *>(zo + n + (n & 1));
        launch_morton_order(x, y, z, n, n, keys, xo, yo, zo, nullptr, s);  // unpadded output
        sx = xo;
        sy = yo;
        sz = zo;
    }
    std::vector<BatchReq> proto(nblk);
    for (int64_t i = 0; i < nblk; ++i) {
        BatchReq &d = proto[i];
        const int64_t npb = p.ntb[i] * b;
        double *q = base + p.off[i];
        d.tiles = q;
        q += (size_t)tile_count(p.ntb[i]) * b * b;
        d.x = q;
        d.y = q + npb;
        d.v = q + 2 * npb;
        q += 3 * npb;
        d.logsum = q;
        d.quad = q + p.ntb[i];
        q += 2 * p.ntb[i];
        d.dinv = q;
        q += 64 * npb;
        d.words = reinterpret_cast<int32_t *>(q);
        d.stride = flow_stride(p.nb[i]);
        d.info = binfo + 8 * i;
        d.res = bres + i;
        d.sx = sx + p.start[i];
        d.sy = sy + p.start[i];
        d.sz = sz + p.start[i];
        d.th = th;
        d.geo = geom_of(o);
        d.n = p.nb[i];
        d.nt = p.ntb[i];
        d.npad = npb;
    }
    // The descriptors go to pinned host memory owned by the context, which the
    // asynchronous copy reads until the stream passes it; the previous call's
    // copy is waited for before the memory is rewritten or replaced.
    const size_t entries = (size_t)nblk;
    if (ctx->ind_done) GL_HIP_TRY(hipEventSynchronize(ctx->ind_done));
    else GL_HIP_TRY(hipEventCreateWithFlags(&ctx->ind_done, hipEventDisableTiming));
    if (entries > ctx->ind_host_cap) {
        if (ctx->ind_host) GL_HIP_TRY(hipHostFree(ctx->ind_host));
        ctx->ind_host = nullptr;
        ctx->ind_host_cap = 0;
        GL_HIP_TRY(hipHostMalloc(reinterpret_cast<void **>(&ctx->ind_host), entries * sizeof(BatchReq),
                                 hipHostMallocDefault));
        ctx->ind_host_cap = entries;
    }
    std::copy(proto.begin(), proto.end(), ctx->ind_host);
    const int rc = enqueue_whole(ctx->ind_host, ddesc, (int)nblk, b, s, nullptr);
    if (rc != GL_OK) return rc;
    GL_HIP_TRY(hipEventRecord(ctx->ind_done, s));
    ind_total_kernel<<<1, 64, 0, s>>>(bres, nblk, block, ctx->res_h);
    GL_HIP_TRY(hipGetLastError());
    p.proto = std::move(proto);
    p.sx = sx;
    p.sy = sy;
    p.desc = ddesc;
    p.res = bres;
    return GL_OK;
}

int ind_eval(gl_context *ctx, const double *x, const double *y, const double *z, int64_t n, gl_theta th,
             const gl_opts &o, gl_result *res, hipStream_t s)
{
    const int b = pick_tile(n, o.tile);
    const int64_t block = o.ind_tiles * (int64_t)b;
    std::vector<int64_t> start, count;
    for (int64_t a = 0; a < n; a += block) {
        start.push_back(a);
        count.push_back(std::min(block, n - a));
    }
    IndPlan p;
    ind_layout(b, start, count, n, o.reorder != 0, p);
    int rc = ind_workspace(ctx, p.doubles * sizeof(double));
    if (rc == GL_OK)
        rc = ind_factor(ctx, x, y, z, n, th, o, block, o.reorder != 0, static_cast<double *>(ctx->ind_buf), s, p);
    if (rc != GL_OK) return res->status = rc;
    GL_HIP_TRY(hipStreamSynchronize(s));
    fill_result(res, *ctx->res_h, p.b);
    return res->status;
}

int ind_krige(gl_context *ctx, const double *x, const double *y, const double *z, const int64_t *kcount,
              const double *xnew, const double *ynew, const int64_t *mcount, int64_t nblocks, gl_theta th,
              const gl_opts &o, int b, double *znew, hipStream_t s)
{
    // blocks that observe something are factored; the others predict 0
    std::vector<int64_t> start, count, kstart(nblocks + 1, 0), mstart(nblocks + 1, 0), slot(nblocks, -1);
    for (int64_t B = 0; B < nblocks; ++B) {
        kstart[B + 1] = kstart[B] + kcount[B];
        mstart[B + 1] = mstart[B] + mcount[B];
        if (kcount[B] > 0) {
            slot[B] = (int64_t)start.size();
            start.push_back(kstart[B]);
            count.push_back(kcount[B]);
        }
    }
    const int64_t n = kstart[nblocks];
    IndPlan p;
    if (!start.empty()) {
        ind_layout(b, start, count, n, false, p);
        int rc = ind_workspace(ctx, p.doubles * sizeof(double));
        if (rc == GL_OK)
            rc = ind_factor(ctx, x, y, z, n, th, o, o.ind_tiles * (int64_t)b, false,
                            static_cast<double *>(ctx->ind_buf), s, p);
        if (rc != GL_OK) return rc;
        GL_HIP_TRY(hipStreamSynchronize(s));
        if (ctx->res_h->info != 0) return GL_NOT_SPD;
        // X = L⁻ᵀ w within each block, in place
        launch_backward_batched(p.b, p.desc, (int)p.nblk, *std::max_element(p.nb.begin(), p.nb.end()), s);
    }
    // each block's held-out values from its own observed values
    int64_t part_len = 1;
    for (int64_t B = 0; B < nblocks; ++B)
        if (mcount[B] > 0 && kcount[B] > 0) part_len = std::max(part_len, mcount[B] * krige_chunks(kcount[B]));
    double *part = nullptr;
    if (hipMallocAsync(reinterpret_cast<void **>(&part), (size_t)part_len * sizeof(double), s) != hipSuccess) {
        (void)hipGetLastError();
        return GL_ENOMEM;
    }
    for (int64_t B = 0; B < nblocks; ++B) {
        if (mcount[B] == 0) continue;
        double *out = znew + mstart[B];
        if (kcount[B] == 0) {
            launch_fill(out, mcount[B], 0.0, s);
            continue;
        }
        const int64_t nchunk = krige_chunks(kcount[B]);
        launch_krige(x + kstart[B], y + kstart[B], kcount[B], p.proto[slot[B]].v, th, geom_of(o), xnew + mstart[B],
                     ynew + mstart[B], mcount[B], part, nchunk, s);
        launch_krige_reduce(part, mcount[B], nchunk, out, s);
    }
    GL_HIP_TRY(hipGetLastError());
    GL_HIP_TRY(hipFreeAsync(part, s));
    return GL_OK;
}

size_t cv_fold_bytes(int64_t n, int64_t nk, int b)
{
    const int64_t nm = n - nk;
    // index list, known x, y, z | missing x, y, z, prediction, kriging sums | mse, result
    const size_t own = n + 3 * nk + (4 + krige_chunks(nk)) * (size_t)nm + 1 + 8;
    return (block_doubles(nk, b) + desc_doubles(1) + 16 + own) * sizeof(double);
}

int cv_folds(gl_context *ctx, const double *x, const double *y, const double *z, int64_t n, gl_theta th,
             const gl_opts &o, int b, const int32_t *fold_h, const int64_t *count, int32_t f0, int32_t f1, double *mse_h,
             double *pred_out, hipStream_t s)
{
    const int32_t G = f1 - f0;
    std::vector<int64_t> kstart(G + 1, 0), mstart(G + 1, 0), kcount(G);
    size_t part_len = 0;
    for (int32_t g = 0; g < G; ++g) {
        const int64_t nm = count[f0 + g], nk = n - nm;
        kcount[g] = nk;
        kstart[g + 1] = kstart[g] + nk;
        mstart[g + 1] = mstart[g] + nm;
        part_len = std::max(part_len, (size_t)nm * krige_chunks(nk));
    }
    const int64_t K = kstart[G], M = mstart[G];
    // each fold's known locations, then each fold's missing ones, all in input order
    std::vector<int64_t> order((size_t)(K + M));
    {
        std::vector<int64_t> a(kstart.begin(), kstart.end() - 1), m(mstart.begin(), mstart.end() - 1);
        for (int64_t i = 0; i < n; ++i)
            for (int32_t g = 0; g < G; ++g) {
                if (fold_h[i] == f0 + g) order[(size_t)(K + m[g]++)] = i;
                else order[(size_t)a[g]++] = i;
            }
    }
    IndPlan p;
    ind_layout(b, std::vector<int64_t>(kstart.begin(), kstart.end() - 1), kcount, K, false, p);
    const size_t own = (size_t)(K + M) + 3 * K + 4 * M + part_len + G;
    const size_t bytes = (p.doubles + own) * sizeof(double);
    if (ctx->used.load() + bytes > ctx->budget) return GL_ENOMEM;
    double *base = nullptr;
    if (hipMalloc(reinterpret_cast<void **>(&base), bytes) != hipSuccess) {
        (void)hipGetLastError();
        return GL_ENOMEM;
    }
    ctx->used += bytes;
    double *kx = base + p.doubles, *ky = kx + K, *kz = ky + K;
    double *mx = kz + K, *my = mx + M, *mz = my + M, *pred = mz + M, *part = pred + M, *dmse = part + part_len;
    int64_t *idx = reinterpret_cast<int64_t *>(dmse + G);
    std::vector<DevResult> res(G);
    std::vector<double> mse(G);
    auto run = [&]() -> int {
        GL_HIP_TRY(hipMemcpyAsync(idx, order.data(), order.size() * sizeof(int64_t), hipMemcpyHostToDevice, s));
        launch_gather3(x, y, z, idx, K, kx, ky, kz, s);
        launch_gather3(x, y, z, idx + K, M, mx, my, mz, s);
        const int rc = ind_factor(ctx, kx, ky, kz, K, th, o, 0, false, base, s, p);
        if (rc != GL_OK) return rc;
        launch_backward_batched(b, p.desc, G, *std::max_element(kcount.begin(), kcount.end()), s);
        for (int32_t g = 0; g < G; ++g) {
            const int64_t nm = mstart[g + 1] - mstart[g], nchunk = krige_chunks(kcount[g]);
            double *out = pred + mstart[g];
            launch_krige(kx + kstart[g], ky + kstart[g], kcount[g], p.proto[g].v, th, geom_of(o), mx + mstart[g],
                         my + mstart[g], nm, part, nchunk, s);
            launch_krige_reduce(part, nm, nchunk, out, s);
            launch_mse(out, mz + mstart[g], nm, dmse + g, s);
        }
        GL_HIP_TRY(hipMemcpyAsync(res.data(), p.res, G * sizeof(DevResult), hipMemcpyDeviceToHost, s));
        GL_HIP_TRY(hipMemcpyAsync(mse.data(), dmse, G * sizeof(double), hipMemcpyDeviceToHost, s));
        GL_HIP_TRY(hipStreamSynchronize(s));
        int status = GL_OK;
        for (int32_t g = 0; g < G; ++g) {
            const bool ok = res[g].info == 0;
            mse_h[f0 + g] = ok ? mse[g] : NAN;
            if (!ok) status = GL_NOT_SPD;
            if (ok && pred_out)
                launch_scatter(pred + mstart[g], idx + K + mstart[g], mstart[g + 1] - mstart[g], pred_out, s);
        }
        GL_HIP_TRY(hipGetLastError());
        return status;
    };
    const int rc = run();
    (void)hipStreamSynchronize(s);  // `base` and the host arrays are read until here
    (void)hipFree(base);
    ctx->used -= bytes;
    return rc;
}

}  // namespace gl

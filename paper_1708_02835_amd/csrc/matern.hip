// Σ(θ) generation kernels (Alg. 1 steps 3-4, Alg. 2 step 2, Alg. 3 steps 3-6):
// the distance matrix is never stored; each element is evaluated from the two
// locations and written once.
#include "batch.hpp"
#include "common.hpp"
#include "matern_device.hpp"
#include "mfma.hpp"

namespace gl {

// Decode a packed lower-triangle tile index t into (i, j), i >= j.
__device__ inline void tile_from_index(int64_t t, int64_t &i, int64_t &j)
{
    int64_t r = (int64_t)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while (r * (r + 1) / 2 > t) --r;
    while ((r + 1) * (r + 2) / 2 <= t) ++r;
    i = r;
    j = t - r * (r + 1) / 2;
}

// All b×b entries of tile (i, j) of the packed lower storage, by one workgroup
// or, where there are few tiles, by `parts` of them with a range of columns
// each.  Rows and columns at or beyond n are padding: 1 on the global
// diagonal, 0 elsewhere, so the padded matrix is block-diagonal with an
// identity tail and the likelihood terms of the first n rows are unchanged.
// Diagonal tiles are written in full (both triangles).  Stores are coalesced:
// consecutive threads write consecutive rows of one column (two columns at
// once for 128-row tiles).  When norm2 is not NULL, the tile's squared
// Frobenius norm is written to norm2[t] by a fixed-order block reduction
// (parts = 1).
// MODE (checked by the launchers): GEN_ANY any distance and smoothness;
// GEN_EUCLID Euclidean distance, so the kernel carries no great-circle
// trigonometry; GEN_CLOSED Euclidean distance and smoothness 1/2, 3/2 or
// 5/2, so it carries no Bessel evaluator either.  Fewer registers let more
// waves share a CU; the values are the same, bit for bit, in every mode.
enum { GEN_ANY = 0, GEN_EUCLID = 1, GEN_CLOSED = 2 };
constexpr int GEN_WAVES(int mode) { return mode == GEN_ANY ? 2 : 4; }  // workgroups per CU: bounds the registers

// Columns are split until this many workgroups (four per CU) share the tiles,
// down to 16 columns each: n = 400 has 10 tiles of 128, 46 µs with one
// workgroup each.
constexpr int64_t GEN_BLOCKS = 1024;
static int gen_parts(int64_t tiles, int b)
{
    int parts = 1;
    while (tiles * parts < GEN_BLOCKS && b / (2 * parts) >= 16 && b % (2 * parts) == 0) parts *= 2;
    return parts;
}

// Great-circle terms of one location: longitude, latitude and the cosine of
// the latitude, in the operations of gcd_dist.
template <int MODE>
struct GenPoint {
    double x, y, c;
    __device__ void set(double px, double py, const Geom &geo)
    {
        x = px;
        y = py;
        c = MODE == GEN_ANY && geo.metric ? cos(py * (M_PI / 180.0)) : 0.0;
    }
    __device__ double to(const GenPoint &o, const Geom &geo) const
    {
        if constexpr (MODE == GEN_ANY)
            if (geo.metric) return gcd_dist_cos(x, y, c, o.x, o.y, o.c, geo.radius);
        return dist2d(x, y, o.x, o.y);
    }
};

template <int B, int MODE>
__device__ __forceinline__ void gen_tiles_body(double *__restrict__ tiles, const double *__restrict__ x,
                                               const double *__restrict__ y, int64_t n, gl_theta th, Geom geo,
                                               double *__restrict__ norm2, int64_t t, int part, int parts)
{
    int64_t ti, tj;
    tile_from_index(t, ti, tj);
    const MaternSetup ms = matern_setup(th.theta1, th.theta2, th.theta3);
    const int cols = B / parts, c0 = part * cols;
    __shared__ GenPoint<MODE> pc[B];  // the column locations
    for (int c = threadIdx.x; c < cols; c += 256) {
        const int64_t gc = tj * B + c0 + c;
        pc[c].set(gc < n ? x[gc] : 0.0, gc < n ? y[gc] : 0.0, geo);
    }
    const BesselTab *tabp = nullptr;
    if constexpr (MODE == GEN_CLOSED) {
        __syncthreads();
    } else {
        __shared__ BesselTab tab;
        bessel_tab_init(ms, tab);  // ends with the barrier the staging needs too
        tabp = &tab;
    }
    double *T = tiles + t * (int64_t)B * B;
    constexpr int RPT = (B + 255) / 256;      // rows per thread
    constexpr int CPT = B < 256 ? 256 / B : 1;  // columns side by side
    const int r0 = threadIdx.x % (256 / CPT), cs = threadIdx.x / (256 / CPT);
    GenPoint<MODE> pr[RPT];
    int64_t gr[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = r0 + 256 * q;
        gr[q] = ti * B + r;
        const bool ok = (r < B) && gr[q] < n;
        pr[q].set(ok ? x[gr[q]] : 0.0, ok ? y[gr[q]] : 0.0, geo);
    }
    double ss = 0.0;
    for (int c = cs; c < cols; c += CPT) {
        const int64_t gc = tj * B + c0 + c;
        const bool colok = gc < n;
        const GenPoint<MODE> p = pc[c];
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int r = r0 + 256 * q;
            if (r >= B) continue;
            double v;
            if (colok && gr[q] < n) {
                const double d = pr[q].to(p, geo);
                if constexpr (MODE == GEN_CLOSED) v = matern_eval_closed(ms, d);
                else v = matern_eval(ms, d, tabp);
            } else {
                v = (gr[q] == gc) ? 1.0 : 0.0;
            }
            T[(int64_t)(c0 + c) * B + r] = v;
            ss += v * v;
        }
    }
    if (norm2) {
        __shared__ double red[4];
        double w = wave_sum(ss);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
        __syncthreads();
        if (threadIdx.x == 0) norm2[t] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

template <int B, int MODE>
__global__ __launch_bounds__(256, GEN_WAVES(MODE)) void gen_tiles_kernel(double *__restrict__ tiles,
                                                        const double *__restrict__ x,
                                                        const double *__restrict__ y, int64_t n,
                                                        gl_theta th, Geom geo, double *__restrict__ norm2)
{
    gen_tiles_body<B, MODE>(tiles, x, y, n, th, geo, norm2, blockIdx.x, blockIdx.y, gridDim.y);
}

template <int B>
static void launch_gen_tiles_b(double *tiles, const double *x, const double *y, int64_t n, int64_t nt,
                               gl_theta th, Geom geo, double *norm2, hipStream_t s)
{
    dim3 grid((unsigned)tile_count(nt), norm2 ? 1 : gen_parts(tile_count(nt), B));
    if (geo.metric != GL_EUCLIDEAN)
        gen_tiles_kernel<B, GEN_ANY><<<grid, 256, 0, s>>>(tiles, x, y, n, th, geo, norm2);
    else if (matern_setup(th.theta1, th.theta2, th.theta3).kind != 0)
        gen_tiles_kernel<B, GEN_CLOSED><<<grid, 256, 0, s>>>(tiles, x, y, n, th, geo, norm2);
    else
        gen_tiles_kernel<B, GEN_EUCLID><<<grid, 256, 0, s>>>(tiles, x, y, n, th, geo, norm2);
}

void launch_gen_tiles(double *tiles, const double *x, const double *y, int64_t n, int b, int64_t nt,
                      gl_theta th, Geom geo, double *norm2, hipStream_t s)
{
    switch (b) {
    case 128: launch_gen_tiles_b<128>(tiles, x, y, n, nt, th, geo, norm2, s); break;
    case 256: launch_gen_tiles_b<256>(tiles, x, y, n, nt, th, geo, norm2, s); break;
    case 384: launch_gen_tiles_b<384>(tiles, x, y, n, nt, th, geo, norm2, s); break;
    default: launch_gen_tiles_b<512>(tiles, x, y, n, nt, th, geo, norm2, s); break;
    }
}

// The same, with θ read from device memory (replayed hipGraphs: the graph
// stays valid while θ changes between replays).
template <int B, int MODE>
__global__ __launch_bounds__(256, GEN_WAVES(MODE)) void gen_tiles_dev_kernel(double *__restrict__ tiles, const double *__restrict__ x,
                                                            const double *__restrict__ y, int64_t n,
                                                            const gl_theta *__restrict__ thp, Geom geo)
{
    gen_tiles_body<B, MODE>(tiles, x, y, n, *thp, geo, nullptr, blockIdx.x, blockIdx.y, gridDim.y);
}

template <int B>
static void launch_gen_tiles_dev_b(double *tiles, const double *x, const double *y, int64_t n, int64_t nt,
                                   const gl_theta *thp, Geom geo, hipStream_t s)
{
    dim3 grid((unsigned)tile_count(nt), gen_parts(tile_count(nt), B));
    if (geo.metric == GL_EUCLIDEAN) gen_tiles_dev_kernel<B, GEN_EUCLID><<<grid, 256, 0, s>>>(tiles, x, y, n, thp, geo);
    else gen_tiles_dev_kernel<B, GEN_ANY><<<grid, 256, 0, s>>>(tiles, x, y, n, thp, geo);
}

void launch_gen_tiles_dev(double *tiles, const double *x, const double *y, int64_t n, int b, int64_t nt,
                          const gl_theta *thp, Geom geo, hipStream_t s)
{
    switch (b) {
    case 128: launch_gen_tiles_dev_b<128>(tiles, x, y, n, nt, thp, geo, s); break;
    case 256: launch_gen_tiles_dev_b<256>(tiles, x, y, n, nt, thp, geo, s); break;
    case 384: launch_gen_tiles_dev_b<384>(tiles, x, y, n, nt, thp, geo, s); break;
    default: launch_gen_tiles_dev_b<512>(tiles, x, y, n, nt, thp, geo, s); break;
    }
}

template <int B, int MODE>
__global__ __launch_bounds__(256, GEN_WAVES(MODE)) void gen_batched_kernel(const BatchReq *__restrict__ d, int count)
{
    const int64_t g = blockIdx.x;
    const int r = GL_BATCH_FIND(d, count, g, o_gen);
    const BatchReq &q = d[r];
    gen_tiles_body<B, MODE>(q.tiles, q.x, q.y, q.n, q.th, q.geo, nullptr, g - q.o_gen, 0, 1);
}

template <int B>
static void launch_gen_batched_b(const BatchReq *d, int count, int64_t tiles, bool euclid, hipStream_t s)
{
    if (euclid) gen_batched_kernel<B, GEN_EUCLID><<<(unsigned)tiles, 256, 0, s>>>(d, count);
    else gen_batched_kernel<B, GEN_ANY><<<(unsigned)tiles, 256, 0, s>>>(d, count);
}

void launch_gen_batched(int b, const BatchReq *d, int count, int64_t tiles, bool euclid, hipStream_t s)
{
    if (tiles <= 0) return;
    switch (b) {
    case 128: launch_gen_batched_b<128>(d, count, tiles, euclid, s); break;
    case 256: launch_gen_batched_b<256>(d, count, tiles, euclid, s); break;
    case 384: launch_gen_batched_b<384>(d, count, tiles, euclid, s); break;
    default: launch_gen_batched_b<512>(d, count, tiles, euclid, s); break;
    }
}

// Dense column-major n1×n2 covariance between two point sets: out[i + j*ld].
// Block: 256 rows × 64 columns, which spreads the setup (the Bessel
// constants) over 64 elements per thread.
constexpr int DENSE_COLS = 64;

template <int MODE>
__global__ __launch_bounds__(256, GEN_WAVES(MODE)) void gen_dense_kernel(const double *__restrict__ x1,
                                                        const double *__restrict__ y1, int64_t n1,
                                                        const double *__restrict__ x2,
                                                        const double *__restrict__ y2, int64_t n2,
                                                        gl_theta th, Geom geo, int cols, double *__restrict__ out,
                                                        int64_t ld)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t j0 = (int64_t)blockIdx.y * cols;
    const MaternSetup ms = matern_setup(th.theta1, th.theta2, th.theta3);
    __shared__ GenPoint<MODE> pc[DENSE_COLS];
    const int m = (int)min((int64_t)cols, n2 - j0);
    if ((int)threadIdx.x < m) pc[threadIdx.x].set(x2[j0 + threadIdx.x], y2[j0 + threadIdx.x], geo);
    const BesselTab *tabp = nullptr;
    if constexpr (MODE == GEN_CLOSED) {
        __syncthreads();
    } else {
        __shared__ BesselTab tab;
        bessel_tab_init(ms, tab);
        tabp = &tab;
    }
    if (i >= n1) return;
    GenPoint<MODE> p;
    p.set(x1[i], y1[i], geo);
    for (int c = 0; c < m; ++c) {
        const double d = p.to(pc[c], geo);
        if constexpr (MODE == GEN_CLOSED) out[i + (j0 + c) * ld] = matern_eval_closed(ms, d);
        else out[i + (j0 + c) * ld] = matern_eval(ms, d, tabp);
    }
}

void launch_gen_dense(const double *x1, const double *y1, int64_t n1, const double *x2,
                      const double *y2, int64_t n2, gl_theta th, Geom geo, double *out, int64_t ld,
                      hipStream_t s)
{
    int cols = DENSE_COLS;
    while (cols > 4 && ceil_div(n1, 256) * ceil_div(n2, cols) < GEN_BLOCKS) cols /= 2;
    dim3 grid((unsigned)ceil_div(n1, 256), (unsigned)ceil_div(n2, cols));
    if (geo.metric != GL_EUCLIDEAN)
        gen_dense_kernel<GEN_ANY><<<grid, 256, 0, s>>>(x1, y1, n1, x2, y2, n2, th, geo, cols, out, ld);
    else if (matern_setup(th.theta1, th.theta2, th.theta3).kind != 0)
        gen_dense_kernel<GEN_CLOSED><<<grid, 256, 0, s>>>(x1, y1, n1, x2, y2, n2, th, geo, cols, out, ld);
    else
        gen_dense_kernel<GEN_EUCLID><<<grid, 256, 0, s>>>(x1, y1, n1, x2, y2, n2, th, geo, cols, out, ld);
}

// Kriging, Eq. (5): Z1_k = Σ_j C(||s_new,k - s_j||) v_j with v = Σ22⁻¹ Z2.
// Σ12 is generated on the fly.  Workgroup (k/K, chunk) sums the chunk's
// KRIGE_CHUNK observed points for new points k .. k + K - 1 into
// part[k * nchunk + chunk]: K > 1 reads an observed point and sets the
// evaluator up once for K new ones, where that leaves enough workgroups.
constexpr int KRIGE_CHUNK = 4096;

template <int K, int MODE>
__global__ __launch_bounds__(256, GEN_WAVES(MODE)) void krige_kernel(const double *__restrict__ x,
                                                                     const double *__restrict__ y, int64_t n,
                                                                     const double *__restrict__ v, gl_theta th,
                                                                     Geom geo, const double *__restrict__ xn,
                                                                     const double *__restrict__ yn, int64_t m,
                                                                     double *__restrict__ part, int64_t nchunk)
{
    const int64_t k0 = (int64_t)blockIdx.x * K;
    const int64_t c = blockIdx.y;
    const MaternSetup ms = matern_setup(th.theta1, th.theta2, th.theta3);
    const BesselTab *tabp = nullptr;
    if constexpr (MODE != GEN_CLOSED) {
        __shared__ BesselTab tab;
        bessel_tab_init(ms, tab);
        tabp = &tab;
    }
    GenPoint<MODE> pk[K];
    double acc[K];
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const int64_t k = min(k0 + q, m - 1);
        pk[q].set(xn[k], yn[k], geo);
        acc[q] = 0.0;
    }
    const int64_t j0 = c * KRIGE_CHUNK;
    const int64_t j1 = min(n, j0 + KRIGE_CHUNK);
    for (int64_t j = j0 + threadIdx.x; j < j1; j += 256) {
        GenPoint<MODE> pj;
        pj.set(x[j], y[j], geo);
        const double vj = v[j];
#pragma unroll 1
        for (int q = 0; q < K; ++q) {
            const double d = pk[q].to(pj, geo);
            double e;
            if constexpr (MODE == GEN_CLOSED) e = matern_eval_closed(ms, d);
            else e = matern_eval(ms, d, tabp);
            acc[q] += e * vj;
        }
    }
    __shared__ double red[K][4];
#pragma unroll
    for (int q = 0; q < K; ++q) {
        const double w = wave_sum(acc[q]);
        if ((threadIdx.x & 63) == 0) red[q][threadIdx.x >> 6] = w;
    }
    __syncthreads();
    if ((int)threadIdx.x < K && k0 + threadIdx.x < m) {
        const double *r = red[threadIdx.x];
        part[(k0 + threadIdx.x) * nchunk + c] = (r[0] + r[1]) + (r[2] + r[3]);
    }
}

__global__ void krige_reduce_kernel(const double *__restrict__ part, int64_t m, int64_t nchunk,
                                    double *__restrict__ out)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= m) return;
    double s = 0.0;
    for (int64_t c = 0; c < nchunk; ++c) s += part[k * nchunk + c];
    out[k] = s;
}

template <int K>
static void launch_krige_k(const double *x, const double *y, int64_t n, const double *v, gl_theta th, Geom geo,
                           const double *xn, const double *yn, int64_t m, double *part, int64_t nchunk, hipStream_t s)
{
    dim3 grid((unsigned)ceil_div(m, K), (unsigned)nchunk);
    if (geo.metric != GL_EUCLIDEAN)
        krige_kernel<K, GEN_ANY><<<grid, 256, 0, s>>>(x, y, n, v, th, geo, xn, yn, m, part, nchunk);
    else if (matern_setup(th.theta1, th.theta2, th.theta3).kind != 0)
        krige_kernel<K, GEN_CLOSED><<<grid, 256, 0, s>>>(x, y, n, v, th, geo, xn, yn, m, part, nchunk);
    else
        krige_kernel<K, GEN_EUCLID><<<grid, 256, 0, s>>>(x, y, n, v, th, geo, xn, yn, m, part, nchunk);
}

void launch_krige(const double *x, const double *y, int64_t n, const double *v, gl_theta th, Geom geo,
                  const double *xn, const double *yn, int64_t m, double *part, int64_t nchunk,
                  hipStream_t s)
{
    if (m * nchunk >= 4 * GEN_BLOCKS) launch_krige_k<4>(x, y, n, v, th, geo, xn, yn, m, part, nchunk, s);
    else launch_krige_k<1>(x, y, n, v, th, geo, xn, yn, m, part, nchunk, s);
}

void launch_krige_reduce(const double *part, int64_t m, int64_t nchunk, double *out, hipStream_t s)
{
    krige_reduce_kernel<<<(unsigned)ceil_div(m, 256), 256, 0, s>>>(part, m, nchunk, out);
}

int64_t krige_chunks(int64_t n) { return ceil_div(n, KRIGE_CHUNK); }

// Right-hand sides of the kriging variances (Eq. 4), transposed: tile (c, i)
// of st (b×b column-major) holds C(||s_new,r - s_p||) for new location
// c·b + r and observed location i·b + p; zero where either is padding.  One
// workgroup per tile; stores are coalesced along r.
template <int B, int MODE>
__global__ __launch_bounds__(256, GEN_WAVES(MODE)) void gen_rhs_kernel(double *__restrict__ st,
                                                                       const double *__restrict__ x,
                                                                       const double *__restrict__ y, int64_t n,
                                                                       int64_t nt, const double *__restrict__ xn,
                                                                       const double *__restrict__ yn, int64_t m,
                                                                       gl_theta th, Geom geo)
{
    const int64_t t = blockIdx.x;
    const int64_t c = t / nt, i = t % nt;
    const MaternSetup ms = matern_setup(th.theta1, th.theta2, th.theta3);
    __shared__ GenPoint<MODE> pc[B];  // the observed locations
    for (int p = threadIdx.x; p < B; p += 256) {
        const int64_t gp = i * B + p;
        pc[p].set(gp < n ? x[gp] : 0.0, gp < n ? y[gp] : 0.0, geo);
    }
    const BesselTab *tabp = nullptr;
    if constexpr (MODE == GEN_CLOSED) {
        __syncthreads();
    } else {
        __shared__ BesselTab tab;
        bessel_tab_init(ms, tab);
        tabp = &tab;
    }
    double *T = st + t * (int64_t)B * B;
    constexpr int RPT = (B + 255) / 256;
    constexpr int CPT = B < 256 ? 256 / B : 1;
    const int r0 = threadIdx.x % (256 / CPT), cs = threadIdx.x / (256 / CPT);
    GenPoint<MODE> pr[RPT];
    bool rok[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
        const int r = r0 + 256 * q;
        const int64_t kn = c * B + r;
        rok[q] = (r < B) && kn < m;
        pr[q].set(rok[q] ? xn[kn] : 0.0, rok[q] ? yn[kn] : 0.0, geo);
    }
    for (int p = cs; p < B; p += CPT) {
        const bool pok = i * B + p < n;
        const GenPoint<MODE> o = pc[p];
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int r = r0 + 256 * q;
            if (r >= B) continue;
            double v = 0.0;
            if (pok && rok[q]) {
                const double d = pr[q].to(o, geo);
                if constexpr (MODE == GEN_CLOSED) v = matern_eval_closed(ms, d);
                else v = matern_eval(ms, d, tabp);
            }
            T[(int64_t)p * B + r] = v;
        }
    }
}

template <int B>
static void launch_gen_rhs_b(double *st, const double *x, const double *y, int64_t n, int64_t nt, const double *xn,
                             const double *yn, int64_t m, int64_t chunks, gl_theta th, Geom geo, hipStream_t s)
{
    const unsigned grid = (unsigned)(chunks * nt);
    if (geo.metric != GL_EUCLIDEAN)
        gen_rhs_kernel<B, GEN_ANY><<<grid, 256, 0, s>>>(st, x, y, n, nt, xn, yn, m, th, geo);
    else if (matern_setup(th.theta1, th.theta2, th.theta3).kind != 0)
        gen_rhs_kernel<B, GEN_CLOSED><<<grid, 256, 0, s>>>(st, x, y, n, nt, xn, yn, m, th, geo);
    else
        gen_rhs_kernel<B, GEN_EUCLID><<<grid, 256, 0, s>>>(st, x, y, n, nt, xn, yn, m, th, geo);
}

void launch_gen_rhs(double *st, const double *x, const double *y, int64_t n, int b, int64_t nt, const double *xn,
                    const double *yn, int64_t m, int64_t chunks, gl_theta th, Geom geo, hipStream_t s)
{
    switch (b) {
    case 128: launch_gen_rhs_b<128>(st, x, y, n, nt, xn, yn, m, chunks, th, geo, s); break;
    case 256: launch_gen_rhs_b<256>(st, x, y, n, nt, xn, yn, m, chunks, th, geo, s); break;
    case 384: launch_gen_rhs_b<384>(st, x, y, n, nt, xn, yn, m, chunks, th, geo, s); break;
    default: launch_gen_rhs_b<512>(st, x, y, n, nt, xn, yn, m, chunks, th, geo, s); break;
    }
}

}  // namespace gl

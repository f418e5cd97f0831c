// Backward solve X = L⁻ᵀ w in one launch (the second half of "dposv" in Alg. 3).
//
// One workgroup per 128-column block j of L, in descending order of j:
//   y_j = w_j - Σ_{i>j} L_ijᵀ x_i,   x_j = L_jj⁻ᵀ y_j
// It streams its block column from the last row up, every block into
// registers while the x_i it will meet is still being solved, so a step of the
// chain x_{j+1} -> x_j costs one publication, one product from registers and
// the diagonal solve, and the launch reads L once.  Kriging 1,000 points from a
// factor of n = 40,000 takes 2.3 ms with it, of which 1.35 ms is the time a copy
// needs for the 6.4 GB of L (28.8 ms with a diagonal and an update kernel per
// tile row, 165-345 µs for the diagonal alone: a 512-row substitution by one
// wave).
//
// Columns are taken from a ticket counter, so a workgroup only waits for
// columns that running workgroups hold.  x travels through agent-scope
// atomic stores and loads (write-through, past the XCDs' own L2s), which
// leaves the caches that L streams through alone: the count of solved blocks
// is raised after the stores of x have completed, and x is only loaded once
// the count covers it.
//
// The diagonal block is solved by the inverses of its two 64×64 blocks:
//   x_1 = D_1⁻ᵀ y_1,  x_0 = D_0⁻ᵀ (y_0 - L_10ᵀ x_1).
// Sums have a fixed order.
#include "batch.hpp"
#include "common.hpp"
#include "engine.hpp"
#include "mfma.hpp"

namespace gl {

namespace {

constexpr int KB = 128;  // column block

struct BackShared {
    // D_0⁻¹ (r >= c) at c·65 + r and D_1⁻¹ at r·65 + c, its diagonal at r·65 + 64: two triangles in one square
    double tri[64 * 65];
    double l10[64 * 65];  // L_10, column c at c·65
    double y[KB];
    double part[4][64];
    int word;
};

// Sum over the eight lanes of a group.
__device__ __forceinline__ double sum8(double v)
{
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    return v + __shfl_xor(v, 4, 64);
}

// The next column of one solve; words: ticket and number of solved columns, zero at first.
template <int B>
__device__ __forceinline__ void back_column(const double *__restrict__ tiles, const double *__restrict__ dinv, double *x,
                                            int nb, int *words, BackShared &sh)
{
    constexpr int S = B / KB;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int *solved = words + 1;
    if (tid == 0) sh.word = __hip_atomic_fetch_add(words, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int j = nb - 1 - __builtin_amdgcn_readfirstlane(sh.word);
    if (j < 0) return;
    // element (r, c) of block (i, j) at rows(i)[(128 j + c) B + r]
    auto rows = [&](int i) { return tiles + tile_offset(i / S, 0, B) + (i % S) * KB + (int64_t)j * KB * B; };
    {
        const double *dv = dinv + (int64_t)j * 2 * 64 * 64;
        const double *l = rows(j) + 64;
        for (int e = tid; e < 64 * 64; e += 256) {
            const int c = e >> 6, r = e & 63;
            if (r >= c) {
                sh.tri[c * 65 + r] = dv[e];
                sh.tri[r * 65 + (r == c ? 64 : c)] = dv[64 * 64 + e];
            }
            sh.l10[c * 65 + r] = l[(int64_t)c * B + r];
        }
    }
    // lane 8 g + q of wave w: columns 32 w + 8 p + g (p = 0..3), row pairs 2 q + 16 k (k = 0..7):
    // a load covers 128 contiguous bytes of eight columns
    const int q = lane & 7;
    const int64_t off = (int64_t)(wave * 32 + (lane >> 3)) * B + 2 * q;
    d2 l[4][8];
    auto load = [&](int i) {
        const double *src = rows(i) + off;
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int k = 0; k < 8; ++k) l[p][k] = *reinterpret_cast<const d2 *>(src + (int64_t)p * 8 * B + 16 * k);
    };
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int have = 0;  // blocks of x known to be solved: nb - have .. nb - 1
    if (nb - 1 > j) load(nb - 1);
    for (int i = nb - 1; i > j; --i) {
        if (have < nb - i) {
            for (;;) {
                have = __hip_atomic_load(solved, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (have >= nb - i) break;
                // columns far behind the chain poll less often
                if (i - j > 8) __builtin_amdgcn_s_sleep(16);
                else __builtin_amdgcn_s_sleep(1);
            }
            have = __builtin_amdgcn_readfirstlane(have);
            asm volatile("" ::: "memory");
        }
        const double *xi = x + (int64_t)i * KB + 2 * q;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const double x0 = __hip_atomic_load(xi + 16 * k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const double x1 = __hip_atomic_load(xi + 16 * k + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int p = 0; p < 4; ++p) acc[p] = fma(l[p][k][1], x1, fma(l[p][k][0], x0, acc[p]));
        }
        if (i - 1 > j) load(i - 1);
    }
    // the diagonal block
    double *xj = x + (int64_t)j * KB;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const double s = sum8(acc[p]);
        const int c = wave * 32 + p * 8 + (lane >> 3);
        if (q == 0) sh.y[c] = xj[c] - s;
    }
    __syncthreads();
    const int c = tid & 63, g = tid >> 6;
    auto total = [&] { return (sh.part[0][c] + sh.part[1][c]) + (sh.part[2][c] + sh.part[3][c]); };
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < 64; m += 4) {
        const int r = m + g;
        const double d = sh.tri[r * 65 + (r == c ? 64 : c)];
        s = fma(r >= c ? d : 0.0, sh.y[64 + r], s);
    }
    sh.part[g][c] = s;
    __syncthreads();
    if (tid < 64) sh.y[64 + c] = total();
    __syncthreads();
    s = 0.0;
#pragma unroll
    for (int m = 0; m < 64; m += 4) s = fma(sh.l10[c * 65 + m + g], sh.y[64 + m + g], s);
    sh.part[g][c] = s;
    __syncthreads();
    if (tid < 64) sh.y[c] -= total();
    __syncthreads();
    s = 0.0;
#pragma unroll
    for (int m = 0; m < 64; m += 4) {
        const int r = m + g;
        s = fma(r >= c ? sh.tri[c * 65 + r] : 0.0, sh.y[r], s);
    }
    sh.part[g][c] = s;
    __syncthreads();
    if (tid < KB)
        __hip_atomic_store(xj + tid, tid < 64 ? total() : sh.y[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // columns finish in order, each after the one before, so this is the only writer now
    if (tid == 0) __hip_atomic_store(solved, nb - j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int B>
__global__ __launch_bounds__(256, 2) void back_kernel(const double *__restrict__ tiles, const double *__restrict__ dinv,
                                                      double *x, int nb, int *words)
{
    __shared__ BackShared sh;
    back_column<B>(tiles, dinv, x, nb, words, sh);
}

__global__ void back_clear_kernel(const BatchReq *__restrict__ d, int count)
{
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r < count) d[r].words[0] = d[r].words[1] = 0;
}

// Workgroups count·i .. count·i + count - 1 hold a column of each solve: the
// chains run side by side.  Failed factorisations are passed over.
template <int B>
__global__ __launch_bounds__(256, 2) void back_batched_kernel(const BatchReq *__restrict__ d, int count)
{
    __shared__ BackShared sh;
    const BatchReq &q = d[blockIdx.x % count];
    const int nb = (int)((q.n + KB - 1) / KB);
    if ((int)(blockIdx.x / count) >= nb || *q.info != 0) return;
    back_column<B>(q.tiles, q.dinv, q.v, nb, q.words, sh);
}

}  // namespace

// v (n values, padded to whole tiles) <- L⁻ᵀ v; words: BACK_WORDS doubles of scratch.
void launch_backward(const double *tiles, const double *dinv, int b, int64_t n, double *v, double *words,
                     hipStream_t s)
{
    launch_fill(words, BACK_WORDS, 0.0, s);
    const int nb = (int)ceil_div(n, KB);
    int *w = reinterpret_cast<int *>(words);
    switch (b) {
    case 128: back_kernel<128><<<nb, 256, 0, s>>>(tiles, dinv, v, nb, w); break;
    case 256: back_kernel<256><<<nb, 256, 0, s>>>(tiles, dinv, v, nb, w); break;
    case 384: back_kernel<384><<<nb, 256, 0, s>>>(tiles, dinv, v, nb, w); break;
    default: back_kernel<512><<<nb, 256, 0, s>>>(tiles, dinv, v, nb, w); break;
    }
}

void launch_backward_batched(int b, const BatchReq *d, int count, int64_t longest, hipStream_t s)
{
    back_clear_kernel<<<(unsigned)ceil_div(count, 256), 256, 0, s>>>(d, count);
    const unsigned grid = (unsigned)(count * ceil_div(longest, KB));
    switch (b) {
    case 128: back_batched_kernel<128><<<grid, 256, 0, s>>>(d, count); break;
    case 256: back_batched_kernel<256><<<grid, 256, 0, s>>>(d, count); break;
    case 384: back_batched_kernel<384><<<grid, 256, 0, s>>>(d, count); break;
    default: back_batched_kernel<512><<<grid, 256, 0, s>>>(d, count); break;
    }
}

}  // namespace gl

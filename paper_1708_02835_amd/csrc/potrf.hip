// Diagonal-tile Cholesky factorisation (the POTRF task of the tile algorithm,
// Sec. 5.2 and Alg. 2 step 3).
//
// One workgroup of 256 threads factors the b×b tile A_kk = L_kk L_kkᵀ in place
// (lower triangle), right-looking over 64-column panels s:
//   1. the 64×64 diagonal block D is copied to LDS, factored and inverted by
//      16-column panels (factor_invert_64).  D⁻¹ is also written to `dinv`
//      for the panel TRSM and the forward solve of this step;
//   2. the rows below the block are solved on the matrix cores as
//      P = A[s+64:, s:s+64] · D⁻ᵀ, each wave owning whole 16-row groups;
//   3. the trailing lower triangle A[s+64:, s+64:] -= P Pᵀ is updated on the
//      matrix cores in 32×32 blocks shared by the four waves.
// Applying inverted 64×64 diagonal blocks instead of substituting element by
// element is the usual GPU form of the blocked triangular solve; its rounding
// stays within the spread of other binary64 orderings (see the parity tests).
// A non-positive (or NaN) pivot stores the 1-based global column in *info and
// stops; every later kernel of the factorisation then returns immediately.
// The tile's contribution 2 Σ log L_rr over rows r < n goes to logsum[k].
// At b = 128 the whole tile stays in LDS between the steps (potrf_tile128).
// The kernel runs beside the bulk trailing updates, so it starts only when a
// CU has room for its registers and LDS: its footprint is kept at what the
// general path needs (a fully unrolled block read raised the registers and
// made some calls wait out a whole trailing launch).
#include "common.hpp"
#include "mfma.hpp"
#include "potrf64.hpp"

namespace gl {

// b = 128: the whole lower tile fits in LDS (three 64×64 blocks: D0, the
// rows below it, D1), so it is read once, both panels are factored there and
// only the results go back; the steps and their arithmetic are those of
// potrf_general below (a panel solve and one trailing update between the two
// diagonal blocks), without the global-memory round trips between them.
__device__ __forceinline__ void potrf_tile128(double *__restrict__ tiles, int64_t k, int64_t n,
                                              int64_t *__restrict__ info, double *__restrict__ logsum,
                                              double *__restrict__ dinv)
{
    constexpr int B = 128;
    double *A = tiles + tile_offset(k, k, B);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    __shared__ double D0[PB][PB + 1];  // D0[c][r] = A[r][c]: first diagonal block, then L0
    __shared__ double Pn[PB][PB + 1];  // Pn[c][r] = A[64 + r][c]: rows below, then the panel P
    __shared__ double D1[PB][PB + 1];  // D1[c][r] = A[64 + r][64 + c]: second diagonal block
    __shared__ double Xi[PB][PB + 1];
    __shared__ double red[4];
    __shared__ int fail;

    for (int e = tid; e < PB * PB; e += 256) {
        const int c = e >> 6, r = e & 63;
        D0[c][r] = A[(int64_t)c * B + r];
        Pn[c][r] = A[(int64_t)c * B + PB + r];
        D1[c][r] = A[(int64_t)(PB + c) * B + PB + r];
    }
    if (tid == 0) fail = 0;
    __syncthreads();
    if (!factor_invert_64(D0, Xi, &fail, k * B, info)) return;
    for (int e = tid; e < PB * PB; e += 256) {
        const int c = e >> 6, r = e & 63;
        if (r >= c) A[(int64_t)c * B + r] = D0[c][r];
        dinv[c * PB + r] = r >= c ? Xi[c][r] : 0.0;
    }
    {
        // panel P = A[64:128, 0:64] · D0⁻ᵀ, wave w owning rows 16w..16w+15; each
        // wave reads its own rows of Pn before writing them
        const int r0 = wave * 16;
        double y[PB / 4];
#pragma unroll
        for (int kk = 0; kk < PB / 4; ++kk) y[kk] = Pn[4 * kk + (lane >> 4)][r0 + (lane & 15)];
        d4 acc[4];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            acc[cb] = (d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kk = 0; kk < 4 * cb + 4; ++kk)  // D0⁻¹ is lower triangular
                acc[cb] = mfma_f64(Xi[4 * kk + (lane >> 4)][cb * 16 + (lane & 15)], y[kk], acc[cb]);
        }
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c = cb * 16 + mfma_row(lane, q), r = r0 + mfma_col(lane);
                A[(int64_t)c * B + PB + r] = acc[cb][q];
                Pn[c][r] = acc[cb][q];
            }
    }
    __syncthreads();
    // D1 -= P Pᵀ, lower triangle, in 32×32 blocks (0,0), (1,0), (1,1), K = 64 in two halves
    if (wave < 3) {
        const int bi = wave == 0 ? 0 : 1, bj = wave == 2 ? 1 : 0;
        const int ra = bi * 32 + (lane & 15), rc = bj * 32 + (lane & 15);
        const int rr = bi * 32 + mfma_col(lane), cc = bj * 32;
        d4 c00, c01, c10, c11;  // start from the negated block
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int col = cc + mfma_row(lane, q);
            c00[q] = -D1[col][rr];
            c01[q] = -D1[col + 16][rr];
            c10[q] = -D1[col][rr + 16];
            c11[q] = -D1[col + 16][rr + 16];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            double a0[8], a1[8], b0[8], b1[8];
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const int col = 32 * h + 4 * kk + (lane >> 4);
                a0[kk] = Pn[col][ra];
                a1[kk] = Pn[col][ra + 16];
                b0[kk] = Pn[col][rc];
                b1[kk] = Pn[col][rc + 16];
            }
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                c00 = mfma_f64(b0[kk], a0[kk], c00);
                c01 = mfma_f64(b1[kk], a0[kk], c01);
                c10 = mfma_f64(b0[kk], a1[kk], c10);
                c11 = mfma_f64(b1[kk], a1[kk], c11);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int col = cc + mfma_row(lane, q);
            D1[col][rr] = -c00[q];
            D1[col + 16][rr] = -c01[q];
            D1[col][rr + 16] = -c10[q];
            D1[col + 16][rr + 16] = -c11[q];
        }
    }
    __syncthreads();
    if (!factor_invert_64(D1, Xi, &fail, k * B + PB, info)) return;
    for (int e = tid; e < PB * PB; e += 256) {
        const int c = e >> 6, r = e & 63;
        if (r >= c) A[(int64_t)(PB + c) * B + PB + r] = D1[c][r];
        dinv[PB * PB + c * PB + r] = r >= c ? Xi[c][r] : 0.0;
    }
    // 2 Σ log L_rr over the rows that are not padding
    double acc = 0.0;
    if (tid < B && k * B + tid < n) acc = log(tid < PB ? D0[tid][tid] : D1[tid - PB][tid - PB]);
    double w = wave_sum(acc);
    if (lane == 0) red[wave] = w;
    __syncthreads();
    if (tid == 0) logsum[k] = 2.0 * ((red[0] + red[1]) + (red[2] + red[3]));
}

template <int B>
__device__ __forceinline__ void potrf_general(double *__restrict__ tiles, int64_t k, int64_t n,
                                              int64_t *__restrict__ info, double *__restrict__ logsum,
                                              double *__restrict__ dinv)
{
    double *A = tiles + tile_offset(k, k, B);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    __shared__ double Ds[PB][PB + 1];  // Ds[c][r] = D[r][c]
    __shared__ double Xi[PB][PB + 1];  // Xi[c][r] = (D⁻¹)[r][c]
    __shared__ double red[4];
    __shared__ int fail;

    for (int s = 0; s < B; s += PB) {
        for (int e = tid; e < PB * PB; e += 256) {
            const int c = e >> 6, r = e & 63;
            Ds[c][r] = A[(int64_t)(s + c) * B + s + r];
        }
        if (tid == 0) fail = 0;
        __syncthreads();
        if (!factor_invert_64(Ds, Xi, &fail, k * B + s, info)) return;
        // L block back to the tile, D⁻¹ to the step's inverse buffer
        double *dv = dinv + (int64_t)(s / PB) * PB * PB;
        for (int e = tid; e < PB * PB; e += 256) {
            const int c = e >> 6, r = e & 63;
            if (r >= c) A[(int64_t)(s + c) * B + s + r] = Ds[c][r];
            dv[c * PB + r] = r >= c ? Xi[c][r] : 0.0;
        }
        // panel rows below: P = A[s+64:, s:s+64] · D⁻ᵀ
        const int R = B - s - PB;
        for (int rb = wave; rb < R / 16; rb += 4) {
            const int r0 = s + PB + rb * 16;
            double y[PB / 4];
#pragma unroll
            for (int kk = 0; kk < PB / 4; ++kk)
                y[kk] = A[(int64_t)(s + 4 * kk + (lane >> 4)) * B + r0 + (lane & 15)];
            d4 acc[4];
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                acc[cb] = (d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int kk = 0; kk < 4 * cb + 4; ++kk)  // D⁻¹ is lower triangular
                    acc[cb] = mfma_f64(Xi[4 * kk + (lane >> 4)][cb * 16 + (lane & 15)], y[kk], acc[cb]);
            }
            // result row q of lane l: column cb*16 + l/16 + 4q; lane % 16: row
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    A[(int64_t)(s + cb * 16 + mfma_row(lane, q)) * B + r0 + mfma_col(lane)] = acc[cb][q];
        }
        __syncthreads();
        // trailing lower triangle in 32×32 blocks, K = 64 in two halves
        if (R > 0) {
            const int nb = R / 32;
            const int nblk = nb * (nb + 1) / 2;
            const int t0 = s + PB;
            for (int blk = wave; blk < nblk; blk += 4) {
                int bi = (int)((sqrt(8.0 * blk + 1.0) - 1.0) * 0.5);
                while (bi * (bi + 1) / 2 > blk) --bi;
                while ((bi + 1) * (bi + 2) / 2 <= blk) ++bi;
                const int bj = blk - bi * (bi + 1) / 2;
                const int ra = t0 + bi * 32 + (lane & 15);  // C rows
                const int rc = t0 + bj * 32 + (lane & 15);  // C columns
                const int rr = t0 + bi * 32 + mfma_col(lane);
                const int cc = t0 + bj * 32;
                d4 c00, c01, c10, c11;  // start from the negated block
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t col = cc + mfma_row(lane, q);
                    c00[q] = -A[col * B + rr];
                    c01[q] = -A[(col + 16) * B + rr];
                    c10[q] = -A[col * B + rr + 16];
                    c11[q] = -A[(col + 16) * B + rr + 16];
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    double a0[8], a1[8], b0[8], b1[8];
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk) {
                        const int64_t col = s + 32 * h + 4 * kk + (lane >> 4);
                        a0[kk] = A[col * B + ra];
                        a1[kk] = A[col * B + ra + 16];
                        b0[kk] = A[col * B + rc];
                        b1[kk] = A[col * B + rc + 16];
                    }
                    // operands swapped: result row = C column, lane % 16 = C row
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk) {
                        c00 = mfma_f64(b0[kk], a0[kk], c00);
                        c01 = mfma_f64(b1[kk], a0[kk], c01);
                        c10 = mfma_f64(b0[kk], a1[kk], c10);
                        c11 = mfma_f64(b1[kk], a1[kk], c11);
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t col = cc + mfma_row(lane, q);
                    A[col * B + rr] = -c00[q];
                    A[(col + 16) * B + rr] = -c01[q];
                    A[col * B + rr + 16] = -c10[q];
                    A[(col + 16) * B + rr + 16] = -c11[q];
                }
            }
        }
        __syncthreads();
    }

    // 2 Σ log L_rr over the rows that are not padding
    // (summed by 128-row blocks, each as potrf_tile128 sums its rows)
    double total = 0.0;
    for (int s = 0; s < B; s += 128) {
        const int r = s + tid;
        double acc = 0.0;
        if (tid < 128 && k * B + r < n) acc = log(A[(int64_t)r * B + r]);
        const double w = wave_sum(acc);
        __syncthreads();
        if (lane == 0) red[wave] = w;
        __syncthreads();
        total += 2.0 * ((red[0] + red[1]) + (red[2] + red[3]));
    }
    if (tid == 0) logsum[k] = total;
}

template <int B>
__global__ __launch_bounds__(256, 2) void potrf_kernel(double *__restrict__ tiles, int64_t k, int64_t n,
                                                       int64_t *__restrict__ info,
                                                       double *__restrict__ logsum,
                                                       double *__restrict__ dinv)
{
    if (*info != 0) return;
    __builtin_amdgcn_s_setprio(3);  // critical path of the step schedule
    if constexpr (B == 128) potrf_tile128(tiles, k, n, info, logsum, dinv);
    else potrf_general<B>(tiles, k, n, info, logsum, dinv);
}

void launch_potrf(double *tiles, int b, int64_t k, int64_t n, int64_t *info, double *logsum,
                  double *dinv, hipStream_t s)
{
    switch (b) {
    case 128: potrf_kernel<128><<<1, 256, 0, s>>>(tiles, k, n, info, logsum, dinv); break;
    case 256: potrf_kernel<256><<<1, 256, 0, s>>>(tiles, k, n, info, logsum, dinv); break;
    case 384: potrf_kernel<384><<<1, 256, 0, s>>>(tiles, k, n, info, logsum, dinv); break;
    default: potrf_kernel<512><<<1, 256, 0, s>>>(tiles, k, n, info, logsum, dinv); break;
    }
}

}  // namespace gl

// Cholesky factor and inverse of one 64×64 block held in LDS, by the four
// waves of a 256-thread workgroup: the serial heart of every diagonal-tile
// factorisation.
#pragma once

#include "mfma.hpp"

namespace gl {

constexpr int PB = 64;  // diagonal block edge

// 1/sqrt(p) for a pivot p > 0.  The generic binary64 square root and division
// are long dependent sequences on the critical chain of the column loop below;
// here the hardware reciprocal square root y (about 2^-23 relative error) is
// refined by one third-order step, y (1 + e/2 + 3e²/8) with e = 1 - p y², whose
// remainder 5e³/16 is below 2^-67: four dependent operations instead of the
// seven of two Newton steps.
__device__ __forceinline__ double pivot_rsqrt(double p)
{
    const double y = __builtin_amdgcn_rsq(p);
    const double e = fma(-(p * y), y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// sqrt(p): p / sqrt(p) with one residual correction.
__device__ __forceinline__ double pivot_sqrt(double p)
{
    const double inv = pivot_rsqrt(p), g = p * inv;
    return fma(fma(-g, g, p), 0.5 * inv, g);
}

// v with lane l's value (l a constant) replaced by the wave-uniform x.
__device__ __forceinline__ double writelane_f64(double x, int l, double v)
{
    const long long xb = __double_as_longlong(x), vb = __double_as_longlong(v);
    int lo = (int)(vb & 0xffffffffll), hi = (int)(vb >> 32);
    asm("v_writelane_b32 %0, %1, %2" : "+v"(lo) : "s"((int)(xb & 0xffffffffll)), "i"(l));
    asm("v_writelane_b32 %0, %1, %2" : "+v"(hi) : "s"((int)(xb >> 32)), "i"(l));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Factor the 64×64 block D held in Ds (Ds[c][r] = D[r][c], lower triangle
// valid) as D = L Lᵀ in place and write X = L⁻¹ to Xi (Xi[c][r] = X[r][c]; the
// 16×16 blocks above the diagonal are not written), by 16-column panels P:
//   (a) wave 0 factors the whole panel, lane l owning row 16P + l: column c is
//       scaled by its pivot's reciprocal root and each later column j takes
//       -L_rc L_jc with L_jc broadcast from lane j through scalar registers
//       (no LDS round trip and no separate solve of the rows below).  From
//       the second panel on, lanes 48..63 have no row of the block left and
//       carry identity rows instead: the same recurrence turns them into the
//       rows of X_PPᵀ, so the diagonal blocks' inverses cost nothing (wave 1
//       repeats the first panel with identity rows for X_00).  The identity
//       rows live above the diagonal of Ds, where a lane finds them with the
//       address pattern of a matrix row: rows 0..15 of panel P, rows 16..31
//       of panel 2 for X_00;
//   (b) the next panel's blocks take -L_IP L_JPᵀ on the matrix cores, one wave
//       per block, and (a) goes on.
// While wave 0 factors panel P, the other waves update the columns beyond it
// with panel P - 1, correct the diagonal of panel P - 1 and build the block
// columns of X: wave J + 1 owns column J, X_IJ = -X_II Σ_{M=J}^{I-1} L_IM X_MJ.
// A 16x16x4 result has the lane layout of a B operand, so the owner keeps X_MJ
// and the sums in registers.
// Bound by (a): per panel about 360 instructions of the updates and 16 links
// of the chain broadcast - reciprocal root - scale - update, then an LDS round
// trip of (b).  Alone on a CU a block takes 17,200
// cycles (7.2 µs; 26,000 with the rows below solved through the inverse, square
// roots in the column loop and a scalar copy of every mask).
// A non-positive (or NaN) pivot stores the 1-based global column (col0 +
// local column + 1) of the first one in *info and the function returns false
// on every thread, otherwise true.  *fail must be 0 on entry (before a
// barrier).  Called by all 256 threads; ends with a barrier.
__device__ __forceinline__ bool factor_invert_64(double (*Ds)[PB + 1], double (*Xi)[PB + 1], int *fail, int64_t col0,
                                                 int64_t *info)
{
    // opaque to the compiler, so that the many lane-derived addresses below are
    // computed here and not hoisted into a caller's loop and spilled
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15;
    const int q = lane >> 4;
    __shared__ double pivots[PB];

    // X_PP[i][j] as panel P leaves it
    auto xdiag = [&](int P, int i, int j) { return P ? Ds[16 * P + i][j] : Ds[32 + i][16 + j]; };
    // Σ over 16 of L_IM X, L_IM from Ds, X in B layout
    auto mul_l = [&](int I, int M, d4 x, d4 t) {
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) t = mfma_f64(Ds[16 * M + 4 * kc + q][16 * I + r16], x[kc], t);
        return t;
    };
    // block (I, J) of X to Xi
    auto put_x = [&](int I, int J, d4 x) {
#pragma unroll
        for (int r = 0; r < 4; ++r) Xi[16 * J + r16][16 * I + q + 4 * r] = x[r];
    };
    // X_IJ = -X_II T
    auto close = [&](int I, int J, d4 t) {
        d4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) x = mfma_f64(-xdiag(I, r16, 4 * kc + q), t[kc], x);
        put_x(I, J, x);
        return x;
    };
    // X_PP in B layout, also to Xi
    auto diag_x = [&](int P) {
        d4 x;
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) x[kc] = xdiag(P, 4 * kc + q, r16);
        put_x(P, P, x);
        return x;
    };
    // L_cc of panel P from its pivots
    auto diag_l = [&](int P) {
        if (lane < 16) Ds[16 * P + lane][16 * P + lane] = pivot_sqrt(pivots[16 * P + lane]);
    };
    // block (I, J) -= L_IP L_JPᵀ (result row: block column, lane % 16: block row)
    auto update = [&](int I, int J, int P) {
        d4 c;
#pragma unroll
        for (int r = 0; r < 4; ++r) c[r] = Ds[16 * J + q + 4 * r][16 * I + r16];
#pragma unroll
        for (int kc = 0; kc < 4; ++kc) {
            const int m = 16 * P + 4 * kc + q;
            c = mfma_f64(-Ds[m][16 * J + r16], Ds[m][16 * I + r16], c);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) Ds[16 * J + q + 4 * r][16 * I + r16] = c[r];
    };

    {
        const int m = tid >> 4, i = tid & 15;
        const double v = m == i ? 1.0 : 0.0;
        Ds[16 + m][i] = v;
        Ds[32 + m][i] = v;
        Ds[48 + m][i] = v;
        Ds[32 + m][16 + i] = v;
    }
    __syncthreads();
    d4 x0 = {0.0, 0.0, 0.0, 0.0}, x1 = x0, t2 = x0, t3 = x0;  // the owner's X_JJ, X_J+1,J and open sums
    bool ok = true;
    for (int P = 0; P < 4; ++P) {
        const int p0 = 16 * P;
        const bool factoring = wave == 0 || (P == 0 && wave == 1);
        // the lane's row: of the matrix, of an identity, or (no row left) row 63 again
        double *mine = &Ds[p0][min(p0 + lane, PB - 1)];
        if (lane >= 48 && P > 0) mine = &Ds[p0][lane - 48];
        if (lane >= 48 && P == 0 && wave == 1) mine = &Ds[32][16 + lane - 48];
        double a[16];
        if (factoring) {
#pragma unroll
            for (int m = 0; m < 16; ++m) a[m] = mine[m * (PB + 1)];
        }
        if (P == 0) __syncthreads();  // both have read panel 0 before either writes it back
        if (factoring) {
            double pv = 1.0;  // lane c < 16: pivot c
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                const double piv = readlane_f64(a[c], c);
                pv = writelane_f64(piv, c, pv);
                a[c] *= pivot_rsqrt(piv);
#pragma unroll
                for (int j = c + 1; j < 16; ++j) a[j] = fma(-a[c], readlane_f64(a[c], j), a[j]);
            }
            // lanes with the same row write the same values
#pragma unroll
            for (int m = 0; m < 16; ++m) mine[m * (PB + 1)] = a[m];
            if (lane < 16) pivots[p0 + lane] = pv;
            const unsigned long long bad = __ballot(!(pv > 0.0));
            if (ok && bad && wave == 0) {
                ok = false;
                if (lane == 0) {
                    *fail = 1;
                    *info = col0 + p0 + __ffsll(bad);
                }
            }
        } else if (P == 1) {
            if (wave == 2) {
                update(2, 2, 0);
                update(3, 2, 0);
            } else if (wave == 3) {
                update(3, 3, 0);
                diag_l(0);
            }
        } else if (P == 2) {
            if (wave == 1) {
                x0 = diag_x(0);
                t2 = mul_l(2, 0, x0, t2);
                x1 = close(1, 0, mul_l(1, 0, x0, (d4){0.0, 0.0, 0.0, 0.0}));
            } else if (wave == 2) {
                diag_l(1);
            } else {
                update(3, 3, 1);
            }
        } else if (P == 3) {
            if (wave == 1) {
                t2 = mul_l(2, 1, x1, t2);
                t3 = mul_l(3, 1, x1, mul_l(3, 0, x0, t3));
            } else if (wave == 2) {
                x0 = diag_x(1);
                t2 = mul_l(2, 1, x0, t2);
                t3 = mul_l(3, 1, x0, t3);
            } else {
                diag_l(2);
                t3 = mul_l(3, 2, diag_x(2), t3);
            }
        }
        __syncthreads();
        if (P < 3) {
            if (wave < 3 - P) update(P + 1 + wave, P + 1, P);
            __syncthreads();
        }
    }
    if (wave == 0) {
        diag_x(3);
        diag_l(3);
    }
    if (wave == 1 || wave == 2) t3 = mul_l(3, 2, close(2, wave - 1, t2), t3);
    if (wave > 0) close(3, wave - 1, t3);
    __syncthreads();
    return *fail == 0;
}

}  // namespace gl

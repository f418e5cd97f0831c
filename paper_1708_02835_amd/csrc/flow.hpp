// The whole tiled Cholesky factorisation and forward solve (Alg. 2 steps 3-6)
// in one launch.
//
// The matrix is cut into 128×128 blocks (a storage tile of b = 128 s holds s×s
// of them).  One task computes one block of L from start to end, left-looking:
//   block (i, j), i > j:  -T = -A_ij + Σ_{k<j} L_ik L_jkᵀ,  L_ij = T L_jj⁻ᵀ,
//                         v_i -= L_ij w_j
//   block (j, j):         the same sum, its Cholesky factor, the inverses of its
//                         two 64×64 diagonal blocks, w_j = L_jj⁻¹ v_j and the
//                         block's parts of log|Σ| and wᵀw
// with the accumulators of the sum in registers throughout, so a block of A is
// read once and a block of L written once whatever the number of panels (the
// step schedule reads and writes it once per one or two panels), and nothing
// waits at a kernel boundary: a block starts its sum as soon as its first
// panels exist and follows the frontier.
//
// Workgroups take tasks from a ticket counter in column order, diagonal block
// first, a few each in a long launch.  Every task depends only on tasks with smaller tickets, and a ticket
// is only held by a running workgroup, so the smallest unfinished task can
// always proceed: no co-residency of the grid is assumed, and every wait ends.
// Progress words: prog[i] = 64-column halves of row i's blocks that are final
// (they finish in column order, since each block needs the one before),
// ready[j] = 1 once L_jj's first 64 columns and D_0⁻¹ are final, 2 with the
// second half, 3 with w_j, vdone[i] = blocks whose part of v_i is subtracted.
// What a word announces is stored through the XCD's cache to the agent's
// coherence point (agent-scope stores), the word follows once those stores are
// acknowledged, and a reader invalidates its caches after it has seen the word.
// A pivot that is not positive stores its column in *info; workgroups that
// wait see it and leave the task (and the launch, if it has no other problem).
//
// The chain is diagonal block j -> block (j + 1, j) -> the last panel of
// diagonal block j + 1, with block (j + 2, j), which block (j + 2, j + 1) needs,
// close behind.  Their workgroups ask the other workgroup on their CU to stand
// still meanwhile (see CuClaim); blocks near the diagonal announce their first
// half early, so that diagonal block j + 1 has only 64 columns left to add when
// the second arrives; and the forward solve stays off the chain.
//
// Four waves of 32 rows × 128 columns: a wave then holds whole rows of T, and
// since a 16x16x4 result has the lane layout of a B operand, the triangular
// solve of its rows runs from registers, without an exchange.  The diagonal
// block gives wave w the 16-row blocks w and 7 - w, nine of the 36 lower
// blocks each.
//
// The sequence of operations on every element is that of the step schedule
// (potrf.hip, trsm.hip, trailing.hip, solve.hip), so both give the same bits.
//
// Bound by the matrix cores from about n = 12,000 up (69 TFLOP/s of 78.6 at
// n = 40,000 and 100,000) and by the chain below: 36.5 µs per 128 columns at
// n = 1,600, of which the two 64×64 factors take 16, the panel and update between
// them 5.7, L_j+1,j 4.5 after the second half of L_jj and the last 64 columns of
// the next diagonal block 7 (46.6 before the claims, the early halves and the
// forward solve off the chain).  At n = 8,100, where the chain shares the CUs with
// the other blocks, a step takes 55 µs (71 before).  Whole evaluations, step
// schedule and this: n = 400 480 and 164 µs, n = 1,600 1.49 and 0.49 ms, n = 8,100
// 11.2 and 3.8 ms, n = 40,000 371 and 311 ms.
#pragma once

#include <algorithm>

#include "batch.hpp"
#include "common.hpp"
#include "engine.hpp"
#include "mfma.hpp"
#include "potrf64.hpp"

namespace gl {

// The same launches with workgroups that leave (turns.hip); see FLOW_LONG.
int flow_launch_turns(Work &w, hipStream_t s, bool solve);
void flow_launch_batched_turns(int b, const BatchReq *d, int count, int64_t blocks, int64_t pads, hipStream_t s);
void flow_launch_rhs_turns(const Work &w, double *st, int groups, int *words, double *part, hipStream_t s);

namespace {

constexpr int FB = 128;      // block edge
constexpr int FK = 16;       // columns per staged chunk
constexpr int FP = FB + 16;  // LDS pitch of a staged chunk (bank spread, as trailing.hip)
constexpr int CHAIN = 2;     // blocks below the diagonal that count as the chain's
constexpr bool LEAVE = FLOW_LEAVE;  // the including file's form, see FLOW_LONG
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

struct FlowProb {
    double *tiles, *v, *dinv, *logsum, *quad;
    int64_t *info;
    int *words;   // ticket, then prog, ready and vdone, `stride` ints apart
    int64_t n;
    int nb, pad;  // blocks with rows below n; all-padding blocks after them
    int stride, solve;
};

struct FlowShared {
    double buf[4 * FK * FP];  // K loop: two chunks of both operands
    double v[FB], w[FB];
    double part[4][PB];
    double red[4];
    int fail, word;
};

template <class T>
__device__ __forceinline__ T peek(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// A store to the coherence point; words are posted after settle().
template <class T>
__device__ __forceinline__ void post(T *p, T x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
constexpr int BUF_AGENT = 16;  // the same for a buffer store (sc1)

// Workgroups in the serial phase of a chain task, per CU.  Another workgroup's
// binary64 matrix instructions hold the SIMD's pipe for 64 cycles each, which
// stretched a diagonal block from 25 to 95 µs, so workgroups in the K loop of
// other tasks wait while their CU is claimed (standing still for some 30 µs,
// one of 512).  A claimant waits for nobody who might stand still: for none, or
// in its solve for diagonal block j, which has already announced its first half.
__device__ int flow_cu_claims[8 * 256];
struct CuClaim {
    int *count;
    __device__ __forceinline__ CuClaim()
    {
        // HW_ID bits 8..15: CU, shader array and engine; XCC_ID: the XCD
        const int cu = __builtin_amdgcn_s_getreg(4 | (8 << 6) | (7 << 11));
        const int xcd = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (2 << 11));
        count = flow_cu_claims + xcd * 256 + cu;
    }
    __device__ __forceinline__ void take() const { add(1); }
    __device__ __forceinline__ void drop() const { add(-1); }
    __device__ __forceinline__ bool held() const { return peek(count) > 0; }
    __device__ __forceinline__ void add(int d) const
    {
        if (threadIdx.x == 0) (void)__hip_atomic_fetch_add(count, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
};

// Waits until min(*a, *b) >= want and returns it; -1 when the factorisation
// has failed (info, if not NULL).  Called by every thread; one polls.  Where
// workgroups leave, those that come after a failure look at info first: a block
// would otherwise sum all that is final before it meets a word that will not come
// (n = 40,000 failing at column 20,000: 247 ms, with the look 158).
__device__ __forceinline__ int await(const int *a, const int *b, int want, const int64_t *info, FlowShared &sh)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        int x;
        if constexpr (LEAVE) {
            for (;;) {
                const int64_t failed = info ? peek(info) : 0;
                x = min(peek(a), peek(b));
                if (failed != 0) x = -1;
                if (failed != 0 || x >= want) break;
                __builtin_amdgcn_s_sleep(1);
            }
        } else {
            while ((x = min(peek(a), peek(b))) < want) {
                if (info && peek(info) != 0) {
                    x = -1;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        sh.word = x;
    }
    __syncthreads();
    return sh.word;
}

// Every wave's stores so far have been acknowledged when this returns, those at
// agent scope from the coherence point: a word posted now announces them.
__device__ __forceinline__ void settle()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// The thread index as a value the compiler knows nothing about: addresses
// derived from it are computed where they are used, not once outside the task
// loop and spilled.
__device__ __forceinline__ int thread_index()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// 64×64 column-major block (ld) to LDS, column m's row c at m·64 + (c ^ 16 (m & 1)):
// the two 16-lane halves of an operand read fall in different banks.  src is as
// its doubles are, 8-byte aligned: a workspace's dinv follows nt (nt + 1) / 2 norms.
typedef double d2_any __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ void stage64(const double *__restrict__ src, int64_t ld, double *dst)
{
    const int tid = thread_index();
    d2 r[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int e = 2 * tid + 512 * q;
        r[q] = *reinterpret_cast<const d2_any *>(src + (e >> 6) * ld + (e & 63));
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int e = 2 * tid + 512 * q;
        *reinterpret_cast<d2 *>(dst + (e & ~63) + ((e & 63) ^ ((e >> 2) & 16))) = r[q];
    }
}
__device__ __forceinline__ double staged(const double *s, int m, int c) { return s[m * 64 + (c ^ ((m & 1) << 4))]; }

// acc += rows of A times rows of B over the columns [c0, c1) (multiples of
// FK), A of 64 NA and B of 128 rows, ld B; wave w has the NA 16-row blocks from
// NA w.  Between chunks the workgroup stands still while `cu` is claimed, if
// `yields`.
template <int B, int NA>
__device__ __forceinline__ void accumulate(const double *__restrict__ Ap, const double *__restrict__ Bp, int c0, int c1,
                                           d4 (*acc)[8], double *buf, const CuClaim &cu, bool yields)
{
    auto As = reinterpret_cast<double(*)[FK][FP]>(buf);
    auto Bs = reinterpret_cast<double(*)[FK][FP]>(buf + 2 * FK * FP);
    const int tid = thread_index();
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = tid >> 4;
    const int le = (tid & 15) * 2;
    const int row0 = wave * 16 * NA + (lane & 15);
    d2 ra[4], rb[4];
    auto load = [&](int col) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q < 2 * NA) ra[q] = *reinterpret_cast<const d2 *>(Ap + (int64_t)(col + lc) * B + le + 32 * q);
            rb[q] = *reinterpret_cast<const d2 *>(Bp + (int64_t)(col + lc) * B + le + 32 * q);
        }
    };
    auto store = [&](int cur) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q < 2 * NA) *reinterpret_cast<d2 *>(&As[cur][lc][le + 32 * q]) = ra[q];
            *reinterpret_cast<d2 *>(&Bs[cur][lc][le + 32 * q]) = rb[q];
        }
    };
    load(c0);
    store(0);
    __syncthreads();
    int cur = 0;
    for (int c = c0; c < c1; c += FK, cur ^= 1) {
        bool held = false;
        if (yields) held = cu.held();
        if (c + FK < c1) load(c + FK);
#pragma unroll
        for (int kk = 0; kk < FK; kk += 4) {
            const double *arow = As[cur][kk + (lane >> 4)];
            const double *brow = Bs[cur][kk + (lane >> 4)];
            const double a0 = arow[row0], a1 = NA > 1 ? arow[row0 + 16] : 0.0;
            double bv[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) bv[b] = brow[b * 16 + (lane & 15)];
            // operands swapped: result row = block column, lane % 16 = block row
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                acc[0][b] = mfma_f64(bv[b], a0, acc[0][b]);
                if (NA > 1) acc[1][b] = mfma_f64(bv[b], a1, acc[1][b]);
            }
        }
        // the staging of the next chunk stays after this chunk's products
        __builtin_amdgcn_sched_barrier(0);
        if (held)
            while (cu.held()) __builtin_amdgcn_s_sleep(16);
        if (c + FK < c1) store(cur ^ 1);
        __syncthreads();
    }
}

// The same for the lower half of a diagonal block, A == B: wave w has the
// 16-row blocks w and 7 - w, columns up to the diagonal.  [c0, c1) is in whole
// 64s, staged four chunks at a time: with nine products per wave and four
// columns, a chunk is computed faster than its loads come back.
template <int B>
__device__ __forceinline__ void accumulate_diag(const double *__restrict__ Ap, int c0, int c1, d4 (*acc)[8], double *buf)
{
    auto As = reinterpret_cast<double(*)[FP]>(buf);
    const int tid = thread_index();
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lc = tid >> 4;
    const int le = (tid & 15) * 2;
    const int ra0 = wave * 16 + (lane & 15), ra1 = (7 - wave) * 16 + (lane & 15);
    d2 ra[4][4];
    auto load = [&](int col) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                ra[g][q] = *reinterpret_cast<const d2 *>(Ap + (int64_t)(col + FK * g + lc) * B + le + 32 * q);
    };
    load(c0);
    for (int c = c0; c < c1; c += 4 * FK) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<d2 *>(&As[FK * g + lc][le + 32 * q]) = ra[g][q];
        __syncthreads();
        if (c + 4 * FK < c1) load(c + 4 * FK);
#pragma unroll 4
        for (int kk = 0; kk < 4 * FK; kk += 4) {
            const double *arow = As[kk + (lane >> 4)];
            const double a0 = arow[ra0], a1 = arow[ra1];
            double bv[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) bv[b] = arow[b * 16 + (lane & 15)];
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                if (b < 4 && b <= wave) acc[0][b] = mfma_f64(bv[b], a0, acc[0][b]);
                if (b < 4 || b <= 7 - wave) acc[1][b] = mfma_f64(bv[b], a1, acc[1][b]);
            }
        }
        __syncthreads();
    }
}

// X = T D⁻ᵀ for 16-row groups held as -T in acc[.][h .. h+3] (in place), D⁻¹
// lower triangular, read by inv(m, c) = D⁻¹[c][m].
template <int NA, int H, class F>
__device__ __forceinline__ void solve64(d4 (*acc)[8], F &&inv)
{
    const int lane = thread_index() & 63;
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][H + b] = -acc[a][H + b];
#pragma unroll
    for (int cb = 3; cb >= 0; --cb) {
        d4 x[NA];
#pragma unroll
        for (int a = 0; a < NA; ++a) x[a] = (d4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int mb = 0; mb <= cb; ++mb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double dv = inv(16 * mb + 4 * r + (lane >> 4), 16 * cb + (lane & 15));
#pragma unroll
                for (int a = 0; a < NA; ++a) x[a] = mfma_f64(dv, acc[a][H + mb][r], x[a]);
            }
#pragma unroll
        for (int a = 0; a < NA; ++a) acc[a][H + cb] = x[a];
    }
}

// -T of the second 64 columns takes X_0 L_10ᵀ, L_10 staged in s.
template <int NA>
__device__ __forceinline__ void carry64(d4 (*acc)[8], const double *s)
{
    const int lane = thread_index() & 63;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double l = staged(s, 16 * mb + 4 * r + (lane >> 4), 16 * cb + (lane & 15));
#pragma unroll
                for (int a = 0; a < NA; ++a) acc[a][4 + cb] = mfma_f64(l, acc[a][mb][r], acc[a][4 + cb]);
            }
}

// Block (i, j), i > j.  False when the factorisation has failed.
template <int B>
__device__ __forceinline__ bool flow_off(const FlowProb &p, int i, int j, FlowShared &sh)
{
    constexpr int S = B / FB;
    const int tid = thread_index();
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // row panels: column c of rows 128 i .. at rows(i) + c·B
    const double *Ai = p.tiles + tile_offset(i / S, 0, B) + (i % S) * FB;
    const double *Bj = p.tiles + tile_offset(j / S, 0, B) + (j % S) * FB;
    double *C = const_cast<double *>(Ai) + (int64_t)j * FB * B;
    const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(C, (short)0, FB * B * 8, 0x00020000);
    const int cvo = (mfma_row(lane, 0) * B + wave * 32 + mfma_col(lane)) * 8;
    int *prog = p.words + 2 * p.stride, *ready = prog + (p.nb + j) * p.stride, *vdone = prog + (2 * p.nb + i) * p.stride;
    const bool chain = i <= j + CHAIN;
    const CuClaim cu;

    d4 acc[2][8];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[a][b][r] = -__builtin_bit_cast(
                    double, __builtin_amdgcn_raw_buffer_load_b64(crs, cvo, ((b * 16 + 4 * r) * B + a * 16) * 8, 0));
    for (int k = 0; k < 2 * j;) {
        const int have = await(prog + i * p.stride, prog + j * p.stride, k + 1, p.info, sh);
        if (have < 0) return false;
        const int e = min(have, 2 * j);
        const bool last = chain && e == 2 * j;  // nothing left to wait for
        if (last) cu.take();
        accumulate<B, 2>(Ai, Bj, k * PB, e * PB, acc, sh.buf, cu, !last);
        if (last) cu.drop();
        k = e;
    }
    // first 64 columns, then the second
    const double *Ljj = Bj + (int64_t)j * FB * B;
    const double *dv = p.dinv + (int64_t)j * 2 * PB * PB;
    double *s0 = sh.buf, *s1 = sh.buf + PB * PB;
    if (await(ready, ready, 1, p.info, sh) < 0) return false;
    if (chain) cu.take();
    stage64(dv, PB, s0);
    stage64(Ljj + PB, B, s1);
    __syncthreads();
    solve64<2, 0>(acc, [&](int m, int c) { return staged(s0, m, c); });
    auto put = [&](int h) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = h; b < h + 4; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const double x = acc[a][b][r];
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), crs, cvo,
                                                          ((b * 16 + 4 * r) * B + a * 16) * 8, BUF_AGENT);
                }
    };
    put(0);
    if (chain) {
        settle();
        if (tid == 0) post(prog + i * p.stride, 2 * j + 1);
    }
    carry64<2>(acc, s1);
    if (await(ready, ready, 2, p.info, sh) < 0) {
        if (chain) cu.drop();
        return false;
    }
    stage64(dv + PB * PB, PB, s0);
    __syncthreads();
    solve64<2, 4>(acc, [&](int m, int c) { return staged(s0, m, c); });
    put(4);
    settle();
    if (tid == 0) post(prog + i * p.stride, 2 * j + 2);
    if (chain) cu.drop();
    if (!p.solve) return true;
    if (await(ready, ready, 3, p.info, sh) < 0) return false;
    if (await(vdone, vdone, j, p.info, sh) < 0) return false;
    if (tid < FB) sh.w[tid] = peek(p.v + (int64_t)j * FB + tid);
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) s = fma(acc[a][b][r], sh.w[b * 16 + mfma_row(lane, r)], s);
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        double *vi = p.v + (int64_t)i * FB + wave * 32 + a * 16 + lane;
        if (lane < 16) post(vi, peek(vi) - s);
    }
    settle();
    if (tid == 0) post(vdone, j + 1);
    return true;
}

// Block (j, j).  False when the factorisation fails or has failed.
template <int B>
__device__ __forceinline__ bool flow_diag(const FlowProb &p, int j, FlowShared &sh)
{
    constexpr int S = B / FB;
    const int tid = thread_index();
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double *Aj = p.tiles + tile_offset(j / S, 0, B) + (j % S) * FB;
    double *C = const_cast<double *>(Aj) + (int64_t)j * FB * B;
    double *vj = p.v + (int64_t)j * FB;
    double *dv = p.dinv + (int64_t)j * 2 * PB * PB;
    int *prog = p.words + 2 * p.stride, *ready = prog + (p.nb + j) * p.stride, *vdone = prog + (2 * p.nb + j) * p.stride;
    const CuClaim cu;
    const int64_t rows = p.n - (int64_t)j * FB;  // rows that are not padding
    const int q = lane >> 4, r16 = lane & 15;
    const int rb0 = wave, rb1 = 7 - wave;  // 16-row blocks of this wave

    d4 acc[2][8];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[a][b][r] = -C[(int64_t)(b * 16 + mfma_row(lane, r)) * B + (a ? rb1 : rb0) * 16 + r16];
    for (int k = 0; k < 2 * j;) {
        const int have = await(prog + j * p.stride, prog + j * p.stride, k + 1, p.info, sh);
        if (have < 0) return false;
        const int e = min(have, 2 * j);
        if (e == 2 * j) cu.take();
        accumulate_diag<B>(Aj, k * PB, e * PB, acc, sh.buf);
        k = e;
    }
    if (j == 0) cu.take();
    auto X = reinterpret_cast<double(*)[PB + 1]>(sh.buf);                  // D_0, then X_10, then D_1⁻¹
    auto Y = reinterpret_cast<double(*)[PB + 1]>(sh.buf + PB * (PB + 1));  // D_0⁻¹, then D_1
#pragma unroll
    for (int b = 0; b < 4; ++b)
        if (b <= wave) {
#pragma unroll
            for (int r = 0; r < 4; ++r) X[b * 16 + mfma_row(lane, r)][rb0 * 16 + r16] = -acc[0][b][r];
        }
    if (tid == 0) sh.fail = 0;
    __syncthreads();
    if (!factor_invert_64(X, Y, &sh.fail, (int64_t)j * FB, p.info)) {
        if (tid == 0) __threadfence();
        cu.drop();
        return false;
    }
    // the rows below by 16-row blocks, one per wave; L_00, D_0⁻¹ and they go out
    solve64<1, 0>(&acc[1], [&](int m, int c) { return Y[m][c]; });
    for (int e = tid; e < PB * PB; e += 256) {
        const int c = e >> 6, r = e & 63;
        if (r >= c) post(C + (int64_t)c * B + r, X[c][r]);
        post(dv + e, r >= c ? Y[c][r] : 0.0);
    }
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) post(C + (int64_t)(b * 16 + mfma_row(lane, r)) * B + rb1 * 16 + r16, acc[1][b][r]);
    double lg = wave == 0 ? X[lane][lane] : 1.0;
    __syncthreads();
    // X_10 to LDS, -D_1 += X_10 X_10ᵀ
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) X[b * 16 + mfma_row(lane, r)][(3 - wave) * 16 + r16] = acc[1][b][r];
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
        if (cb <= 3 - wave) {
#pragma unroll
            for (int mb = 0; mb < 4; ++mb)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[1][4 + cb] = mfma_f64(X[16 * mb + 4 * r + q][16 * cb + r16], acc[1][mb][r], acc[1][4 + cb]);
        }
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
        if (cb <= 3 - wave) {
#pragma unroll
            for (int r = 0; r < 4; ++r) Y[16 * cb + mfma_row(lane, r)][(3 - wave) * 16 + r16] = -acc[1][4 + cb][r];
        }
    settle();
    if (tid == 0) post(ready, 1);
    if (!factor_invert_64(Y, X, &sh.fail, (int64_t)j * FB + PB, p.info)) {
        if (tid == 0) __threadfence();
        cu.drop();
        return false;
    }
    for (int e = tid; e < PB * PB; e += 256) {
        const int c = e >> 6, r = e & 63;
        if (r >= c) post(C + (int64_t)(PB + c) * B + PB + r, Y[c][r]);
        post(dv + PB * PB + e, r >= c ? X[c][r] : 0.0);
    }
    settle();
    if (tid == 0) post(ready, 2);
    cu.drop();
    if (!p.solve) return true;
    // off the chain: w_0 = D_0⁻¹ v_0, w_1 = D_1⁻¹ (v_1 - L_10 w_0), each product
    // over four thread groups
    const int vr = tid & 63, vg = tid >> 6;
    if (wave == 1) lg = Y[lane][lane];
    lg = tid < FB && tid < rows ? log(lg) : 0.0;
    if (await(vdone, vdone, j, p.info, sh) < 0) return false;
    double d0[16], l10[16];
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        d0[m] = dv[(4 * m + vg) * PB + vr];
        l10[m] = C[(int64_t)(4 * m + vg) * B + PB + vr];
    }
    if (tid < FB) sh.v[tid] = peek(vj + tid);
    __syncthreads();
    auto total = [&] { return (sh.part[0][vr] + sh.part[1][vr]) + (sh.part[2][vr] + sh.part[3][vr]); };
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < 16; ++m) s = fma(d0[m], sh.v[4 * m + vg], s);
    sh.part[vg][vr] = s;
    __syncthreads();
    if (tid < PB) sh.w[vr] = total();
    __syncthreads();
    s = 0.0;
#pragma unroll
    for (int m = 0; m < 16; ++m) s = fma(l10[m], sh.w[4 * m + vg], s);
    sh.part[vg][vr] = s;
    __syncthreads();
    if (tid < PB) sh.v[PB + vr] -= total();
    __syncthreads();
    s = 0.0;
#pragma unroll
    for (int m = 0; m < PB; m += 4) s = fma(m + vg <= vr ? X[m + vg][vr] : 0.0, sh.v[PB + m + vg], s);
    sh.part[vg][vr] = s;
    __syncthreads();
    if (tid < PB) sh.w[PB + vr] = total();
    __syncthreads();
    const double w = tid < FB ? sh.w[tid] : 0.0;
    if (tid < FB) post(vj + tid, w);
    // the block's parts, added in block order (the storage tile's first block starts the sums)
    double part = wave_sum(lg);
    if (lane == 0 && wave < 2) sh.red[wave] = part;
    part = wave_sum(tid < rows ? w * w : 0.0);
    if (lane == 0 && wave < 2) sh.red[2 + wave] = part;
    __syncthreads();
    if (tid == 0) {
        const int t = j / S;
        double ls = 2.0 * (sh.red[0] + sh.red[1]), qs = sh.red[2] + sh.red[3];
        if (j % S) {
            ls = peek(p.logsum + t) + ls;
            qs = peek(p.quad + t) + qs;
        }
        post(p.logsum + t, ls);
        post(p.quad + t, qs);
    }
    settle();
    if (tid == 0) post(ready, 3);
    return true;
}

// Block column j of a factorisation of m block columns and the row's offset
// below the diagonal, from its index u in column order (column c: m - c blocks).
__device__ __forceinline__ int flow_column(int u, int m, int &below)
{
    const double a = 2.0 * m + 1.0;
    int j = (int)((a - sqrt(a * a - 8.0 * u)) * 0.5);
    j = max(j, 0);
    while (j > 0 && j * m - j * (j - 1) / 2 > u) --j;
    while ((j + 1) * m - (j + 1) * j / 2 <= u) ++j;
    below = u - (j * m - j * (j - 1) / 2);
    return j;
}

template <int B>
__device__ __forceinline__ bool flow_task(const FlowProb &p, int i, int j, FlowShared &sh)
{
    if (i == j) {
        __builtin_amdgcn_s_setprio(3);  // the critical chain
        return flow_diag<B>(p, j, sh);
    }
    if (i <= j + CHAIN) __builtin_amdgcn_s_setprio(2);
    else __builtin_amdgcn_s_setprio(0);
    return flow_off<B>(p, i, j, sh);
}

// A diagonal block that is all padding: L is the identity Σ has there.
__device__ __forceinline__ void flow_pad(double *dinv, int j)
{
    double *dv = dinv + (int64_t)j * 2 * PB * PB;
    for (int e = threadIdx.x; e < 2 * PB * PB; e += 256) dv[e] = ((e >> 6) & 63) == (e & 63) ? 1.0 : 0.0;
}

// Workgroups stay until the last ticket, up to two per CU, or (LEAVE, in turns.hip)
// end after FLOW_TURNS tickets.  Two workgroups fill a CU's registers and LDS, so
// those that stay keep everything else out for the whole launch; as the others end,
// the dispatcher lets other streams in: a small evaluation, a second large one, a
// kernel of another library.  They leave in launches of more than FLOW_LONG
// operations (5 ms).  A request of 1,000 points beside an evaluation of n = 40,000:
// 255 ms where they stay, 5 with two tickets each, 15 with four, 38 with eight; the
// evaluation itself takes 314 ms either way.  (Without workgroups to spare it takes
// 333: they are dealt to the XCDs in turn, and an XCD that is ahead runs out of its
// share.  Those left over find no ticket.)
// The two forms are compiled apart, so that the code of the one that stays keeps
// its place: with both in one code object n = 8,100 took 4.1 ms instead of 3.85
// (3.9 and 3.64 in the kernel) by the same instructions 256 bytes further on, after
// some generator kernels and not after others.  What does it is not known
// (instruction cache misses are few, 3e-5 of the requests, also on a first call).
constexpr double FLOW_LONG = 0.35e12;
constexpr int FLOW_TURNS = 2;
static unsigned flow_grid(int64_t tasks)
{
    return (unsigned)std::min<int64_t>(tasks, LEAVE ? tasks / FLOW_TURNS + tasks / 16 + 512 : 512);
}

// The next ticket; beyond every total when the workgroup has had its turns.
__device__ __forceinline__ int flow_ticket(int *counter, FlowShared &sh, int *turns)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        if (LEAVE && (*turns)-- == 0) sh.word = INT32_MAX;
        else sh.word = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(sh.word);
}

template <int B>
__global__ __launch_bounds__(256, 2) void flow_kernel(FlowProb p)
{
    __shared__ FlowShared sh;
    const int total = p.nb * (p.nb + 1) / 2;
    int *turns = nullptr;
    if constexpr (LEAVE) {
        __shared__ int left;
        turns = &left;
        if (threadIdx.x == 0) left = FLOW_TURNS;
    }
    for (;;) {
        const int t = flow_ticket(p.words, sh, turns);
        if (t >= total + p.pad) return;
        if (t >= total) {
            flow_pad(p.dinv, p.nb + t - total);
            continue;
        }
        int below;
        const int j = flow_column(t, p.nb, below);
        if (!flow_task<B>(p, j + below, j, sh)) return;
    }
}

__device__ __forceinline__ FlowProb flow_prob(const BatchReq &q, int S)
{
    FlowProb p;
    p.tiles = q.tiles;
    p.v = q.v;
    p.dinv = q.dinv;
    p.logsum = q.logsum;
    p.quad = q.quad;
    p.info = q.info;
    p.words = q.words;
    p.n = q.n;
    p.nb = (int)((q.n + FB - 1) / FB);
    p.pad = (int)q.nt * S - p.nb;
    p.stride = q.stride;
    p.solve = 1;
    return p;
}

// Many factorisations, sorted by falling size.  Their columns are aligned at
// the end (the largest starts alone, the others join when as many columns are
// left), so the serial tails of all of them run together; a column takes the
// diagonal blocks of all active factorisations first, then their next blocks.
// While factorisations 0..a are active every column counts a + 1 times the
// blocks of the largest, and o_flow of factorisation a is the number of blocks
// before it joins.
template <int B>
__global__ __launch_bounds__(256, 2) void flow_batched_kernel(const BatchReq *__restrict__ d, int count, int total,
                                                              int pads)
{
    __shared__ FlowShared sh;
    const int lane = threadIdx.x & 63;
    int *turns = nullptr;
    if constexpr (LEAVE) {
        __shared__ int left;
        turns = &left;
        if (threadIdx.x == 0) left = FLOW_TURNS;
    }
    for (;;) {
        const int t = flow_ticket(d[0].words, sh, turns);
        if (t >= total + pads) return;
        if (t >= total) {
            int r = t - total;
            for (int q = 0; q < count; ++q) {
                const FlowProb p = flow_prob(d[q], B / FB);
                if (r < p.pad) {
                    flow_pad(p.dinv, p.nb + r);
                    break;
                }
                r -= p.pad;
            }
            continue;
        }
        int active = 0;
        for (int q0 = 0; q0 < count; q0 += 64) {
            const int q = q0 + lane;
            const unsigned long long in = __ballot(q < count && d[min(q, count - 1)].o_flow <= t);
            active += __popcll(in);
            if (in != ~0ull) break;
        }
        active = __builtin_amdgcn_readfirstlane(active);
        const BatchReq &last = d[active - 1];
        const int u = t - (int)last.o_flow;
        int below;
        const int c = flow_column(u / active, (int)((last.n + FB - 1) / FB), below);
        const FlowProb p = flow_prob(d[u % active], B / FB);
        const int j = c + p.nb - (int)((last.n + FB - 1) / FB);
        // a block of a failed factorisation is left where it meets a word that
        // will not come; the other problems' blocks still want this workgroup
        (void)flow_task<B>(p, j + below, j, sh);
    }
}

// Right-hand sides of the kriging variances (Eq. 4), U = Sᵀ L⁻ᵀ by blocks of 64
// of them: a right-hand side is one more row below L, so block (R, j) is
// computed as a block of L is, and waits for its own row only.  64 rows
// instead of 128 halve the chain along a row and fill the chip with 1,000
// right-hand sides.  Each block also leaves its part of Σ U², so U is not read
// again.  n = 16,000, 1,000 right-hand sides: the whole kriging call 10.7 -> 5.7
// ms against two launches per tile row, whose diagonal solves had 16 workgroups.
template <int B>
__global__ __launch_bounds__(256, 2) void flow_rhs_kernel(const double *__restrict__ tiles,
                                                          const double *__restrict__ dinv,
                                                          double *__restrict__ st, int nb, int64_t nt,
                                                          int groups, int *words, double *__restrict__ part)
{
    constexpr int S = B / FB, RS = B / 64;
    __shared__ FlowShared sh;
    int *turns = nullptr;
    if constexpr (LEAVE) {
        __shared__ int left;
        turns = &left;
        if (threadIdx.x == 0) left = FLOW_TURNS;
    }
    for (;;) {
        const int t = flow_ticket(words, sh, turns);
        if (t >= nb * groups) return;
        const int j = t / groups, R = t % groups;
        const int tid = thread_index();
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        int *prog = words + 16 * (1 + R);
        const CuClaim cu;
        double *A = st + (R / RS) * nt * B * B + (R % RS) * 64;
        double *C = A + (int64_t)j * FB * B;
        const double *Bj = tiles + tile_offset(j / S, 0, B) + (j % S) * FB;
        const double *dv = dinv + (int64_t)j * 2 * PB * PB;
        double *s0 = sh.buf, *s1 = sh.buf + PB * PB;
        const int64_t at = (int64_t)mfma_row(lane, 0) * B + wave * 16 + mfma_col(lane);
        d4 acc[1][8];
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[0][b][r] = -C[at + (int64_t)(b * 16 + 4 * r) * B];
        for (int c = 0; c < j;) {
            const int e = min(await(prog, prog, c + 1, nullptr, sh), j);
            accumulate<B, 1>(A, Bj, c * FB, e * FB, acc, sh.buf, cu, false);
            c = e;
        }
        __syncthreads();
        stage64(dv, PB, s0);
        stage64(Bj + (int64_t)j * FB * B + PB, B, s1);
        __syncthreads();
        solve64<1, 0>(acc, [&](int m, int c) { return staged(s0, m, c); });
        carry64<1>(acc, s1);
        __syncthreads();
        stage64(dv + PB * PB, PB, s0);
        __syncthreads();
        solve64<1, 4>(acc, [&](int m, int c) { return staged(s0, m, c); });
        double q = 0.0;
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double x = acc[0][b][r];
                post(C + at + (int64_t)(b * 16 + 4 * r) * B, x);
                q = fma(x, x, q);
            }
        settle();
        if (tid == 0) post(prog, j + 1);
        q += __shfl_xor(q, 16, 64);
        q += __shfl_xor(q, 32, 64);
        if (lane < 16) part[((int64_t)j * groups + R) * 64 + wave * 16 + lane] = q;
    }
}

}  // namespace

static int flow_launch(Work &w, hipStream_t s, bool solve)
{
    FlowProb p;
    p.tiles = w.tiles;
    p.v = w.v;
    p.dinv = w.dinv;
    p.logsum = w.logsum;
    p.quad = w.quad;
    p.info = w.info;
    p.n = w.n;
    p.nb = (int)ceil_div(w.n, FB);
    p.pad = (int)(w.npad / FB) - p.nb;
    p.solve = solve;
    // the words take the place of the sort keys, which the staging is done
    // with (and clears); a cache line each where the keys leave room
    p.words = reinterpret_cast<int *>(w.keys);
    p.stride = flow_stride(w.n);
    const int64_t bytes = flow_words(w.n, p.stride) * (int64_t)sizeof(int);
    if (bytes > (npow2_of(w.n) + 4) * (int64_t)sizeof(uint64_t)) return GL_EINVAL;
    const unsigned grid = flow_grid((int64_t)p.nb * (p.nb + 1) / 2 + p.pad);
    switch (w.b) {
    case 128: flow_kernel<128><<<grid, 256, 0, s>>>(p); break;
    case 256: flow_kernel<256><<<grid, 256, 0, s>>>(p); break;
    case 384: flow_kernel<384><<<grid, 256, 0, s>>>(p); break;
    default: flow_kernel<512><<<grid, 256, 0, s>>>(p); break;
    }
    GL_HIP_TRY(hipGetLastError());
    return GL_OK;
}

static void flow_launch_batched(int b, const BatchReq *d, int count, int64_t blocks, int64_t pads, hipStream_t s)
{
    const unsigned grid = flow_grid(blocks + pads);
    switch (b) {
    case 128: flow_batched_kernel<128><<<grid, 256, 0, s>>>(d, count, (int)blocks, (int)pads); break;
    case 256: flow_batched_kernel<256><<<grid, 256, 0, s>>>(d, count, (int)blocks, (int)pads); break;
    case 384: flow_batched_kernel<384><<<grid, 256, 0, s>>>(d, count, (int)blocks, (int)pads); break;
    default: flow_batched_kernel<512><<<grid, 256, 0, s>>>(d, count, (int)blocks, (int)pads); break;
    }
}

static void flow_launch_rhs(const Work &w, double *st, int groups, int *words, double *part, hipStream_t s)
{
    const int nb = (int)ceil_div(w.n, FB);
    const unsigned grid = flow_grid((int64_t)nb * groups);
    switch (w.b) {
    case 128: flow_rhs_kernel<128><<<grid, 256, 0, s>>>(w.tiles, w.dinv, st, nb, w.nt, groups, words, part); break;
    case 256: flow_rhs_kernel<256><<<grid, 256, 0, s>>>(w.tiles, w.dinv, st, nb, w.nt, groups, words, part); break;
    case 384: flow_rhs_kernel<384><<<grid, 256, 0, s>>>(w.tiles, w.dinv, st, nb, w.nt, groups, words, part); break;
    default: flow_rhs_kernel<512><<<grid, 256, 0, s>>>(w.tiles, w.dinv, st, nb, w.nt, groups, words, part); break;
    }
}

}  // namespace gl

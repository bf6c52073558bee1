// fp64 building blocks on 64 x 64 blocks, shared by the inverse (invert.hip) and the closed-form
// recovery of pruned rows (reconstruct.hip): the one-wavefront Cholesky factorisation + inverse of a
// diagonal block, by one wavefront or by a workgroup of four, and products of 64 x 64 tiles on the fp64
// matrix core (v_mfma_f64_16x16x4_f64).
#pragma once

#include "common.h"

namespace obc_dense64 {

constexpr int NB = 64;   // block-column width and GEMM tile edge
typedef double doublex4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double readlane_f64(double v, int l)
{
    long long b = __double_as_longlong(v);
    unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// 1 / sqrt(x) in full fp64: hardware estimate and two Newton steps
__device__ __forceinline__ double rsqrt_f64(double x)
{
    double r = __builtin_amdgcn_rsq(x);
    r = r * (1.5 - 0.5 * x * r * r);
    r = r * (1.5 - 0.5 * x * r * r);
    return r;
}

// Factor the bs x bs (bs <= 64) diagonal block at A (leading dimension lda) in place (lower
// triangle), and write the inverse of that triangular factor to Linv (NB x NB, row-major, zeros
// above the diagonal).  A block smaller than 64 is padded with the identity.
//
// One wavefront, the block in LDS, worked on in 16 x 16 sub-blocks.  For each of the four block
// columns: the diagonal sub-block is factored and its factor inverted in registers (lane i < 16
// holds row i; values cross lanes with v_readlane), the sub-blocks below are multiplied by that
// inverse and the trailing sub-blocks updated, both on the fp64 matrix core
// (v_mfma_f64_16x16x4: lane l supplies a(i = l % 16, k = l / 16) and b(k = l / 16, j = l % 16)
// and holds c(4 r + l / 16, l % 16) in accumulator register r).  The off-diagonal sub-blocks of
// L^-1 then follow from  T_is = -T_ii sum_{s <= k < i} L_ik T_ks.
//
// LDS of one diagonal-block factorisation (doubles): the block, the inverse of its factor, one sub-block
constexpr int PL = NB + 1;
constexpr int SB = 16;                        // sub-block edge
constexpr int POTRF_LDS = 2 * NB * PL + SB * (SB + 1);

// The factorisation runs on ONE wavefront; its LDS accesses are ordered with this (all earlier LDS
// operations of the wavefront are complete and none later is moved before it).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// The part of potrf_wave after the block has been parked in LDS: expects the block at lds[i * PL + j]
// (lower triangle; identity where the block is padded, zeros above the diagonal) and zeros in the
// NB * PL doubles after it, all visible to the calling wavefront.
__device__ __forceinline__ void potrf_wave_core(double *__restrict__ A, int lda, int bs, double *__restrict__ Linv,
                                                int *status, int err, double *lds);

__device__ __forceinline__ void potrf_wave(double *__restrict__ A, int lda, int bs, double *__restrict__ Linv,
                                           int *status, int err, double *lds)
{
    double *Ls = lds;                         // the block; becomes L (lower triangle)
    double *Ts = lds + NB * PL;               // L^-1
    const int lane = threadIdx.x & 63;
    // the block's rows are requested in batches of 16 (all in flight at once: each batch is one trip
    // to memory, and the block is on the factorisation's serial chain), then parked in LDS
#pragma unroll 1
    for (int i0 = 0; i0 < NB; i0 += 16) {
        double v[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = i0 + r;
            v[r] = (i == lane) ? 1.0 : 0.0;
            if (i < bs && lane <= i) v[r] = A[(int64_t)i * lda + lane];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            Ls[(i0 + r) * PL + lane] = v[r];
            Ts[(i0 + r) * PL + lane] = 0.0;
        }
    }
    wave_lds_sync();

    potrf_wave_core(A, lda, bs, Linv, status, err, lds);
}

__device__ __forceinline__ void potrf_wave_core(double *__restrict__ A, int lda, int bs, double *__restrict__ Linv,
                                                int *status, int err, double *lds)
{
    double *Ls = lds;
    double *Ts = lds + NB * PL;
    double *Xs = lds + 2 * NB * PL;
    const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    bool bad = false;
#pragma unroll
    for (int s = 0; s < NB / SB; ++s) {
        const int o = SB * s;
        // (an opaque copy of the lane index per block column: otherwise the lane masks below are
        // shared by the four unrolled block columns and stay live in scalar registers throughout)
        int l16s = l16;
        asm volatile("" : "+v"(l16s));
        // ---- diagonal sub-block: row (o + l16) in registers (lanes >= 16 duplicate lanes < 16)
        double row[SB], rj[SB], t[SB];
#pragma unroll
        for (int c = 0; c < SB; ++c) row[c] = Ls[(o + l16) * PL + o + c];
#pragma unroll
        for (int j = 0; j < SB; ++j) {
            double pj = readlane_f64(row[j], j);
            if (!(pj > 0.0) || !(pj < __builtin_inf())) { bad = true; pj = 1.0; }
            const double r = rsqrt_f64(pj);
            rj[j] = r;                                          // 1 / L[j][j]
            const double cj = row[j] * r;
            row[j] = (l16s == j) ? pj * r : (l16s > j ? cj : 0.0);
            const double mine = (l16s > j) ? cj : 0.0;          // L[l16][j] below the diagonal
#pragma unroll
            for (int c = j + 1; c < SB; ++c) {
                const double lcj = readlane_f64(cj, c);         // L[c][j]
                row[c] = fma(-mine, lcj, row[c]);
                // pin the update here: left to itself the compiler defers it to the column's
                // turn and keeps every L[c][j] alive in scalar registers until then
                asm volatile("" : "+v"(row[c]));
            }
        }
        // ---- inverse of the 16 x 16 factor, lane c computes column c:
        //      t[i] = (delta_ic - sum_{k<i} L[i][k] t[k]) / L[i][i]
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            double acc = (l16s == i) ? 1.0 : 0.0;
            // the lane to read from, made to depend on the previous row's result: otherwise
            // the lane reads of all rows are issued up front and overflow the scalar registers
            int sel = i;
            if (i > 0) asm volatile("" : "+s"(sel) : "v"(t[i > 0 ? i - 1 : 0]));
#pragma unroll
            for (int k = 0; k < i; ++k) acc = fma(-readlane_f64(row[k], sel), t[k], acc);
            t[i] = acc * rj[i];
        }
        if (lane < SB) {
#pragma unroll
            for (int c = 0; c < SB; ++c) {
                Ls[(o + lane) * PL + o + c] = row[c];
                Ts[(o + c) * PL + o + lane] = t[c];
            }
        }
        wave_lds_sync();
        // ---- sub-blocks below: L_is = A_is T_ss^T
        doublex4 P[NB / SB];
#pragma unroll
        for (int ib = s + 1; ib < NB / SB; ++ib) {
            doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kc = 0; kc < SB / 4; ++kc) {
                const double av = Ls[(SB * ib + l16) * PL + o + 4 * kc + lg];
                const double bv = Ts[(o + l16) * PL + o + 4 * kc + lg];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
            }
            P[ib] = acc;
        }
        wave_lds_sync();
#pragma unroll
        for (int ib = s + 1; ib < NB / SB; ++ib)
#pragma unroll
            for (int r = 0; r < 4; ++r) Ls[(SB * ib + 4 * r + lg) * PL + o + l16] = P[ib][r];
        wave_lds_sync();
        // ---- trailing sub-blocks: A_ij -= L_is L_js^T  (s < j <= i)
#pragma unroll
        for (int ib = s + 1; ib < NB / SB; ++ib)
#pragma unroll
            for (int jb = s + 1; jb <= ib; ++jb) {
                doublex4 acc;
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] = Ls[(SB * ib + 4 * r + lg) * PL + SB * jb + l16];
#pragma unroll
                for (int kc = 0; kc < SB / 4; ++kc) {
                    const double av = -Ls[(SB * ib + l16) * PL + o + 4 * kc + lg];
                    const double bv = Ls[(SB * jb + l16) * PL + o + 4 * kc + lg];
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) Ls[(SB * ib + 4 * r + lg) * PL + SB * jb + l16] = acc[r];
            }
        wave_lds_sync();
    }
    // ---- off-diagonal sub-blocks of T = L^-1, block column by block column, top to bottom
#pragma unroll
    for (int s = 0; s + 1 < NB / SB; ++s)
#pragma unroll
        for (int ib = s + 1; ib < NB / SB; ++ib) {
            doublex4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kb = s; kb < ib; ++kb)
#pragma unroll
                for (int kc = 0; kc < SB / 4; ++kc) {
                    const double av = Ls[(SB * ib + l16) * PL + SB * kb + 4 * kc + lg];
                    const double bv = Ts[(SB * kb + 4 * kc + lg) * PL + SB * s + l16];
                    x = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, x, 0, 0, 0);
                }
#pragma unroll
            for (int r = 0; r < 4; ++r) Xs[(4 * r + lg) * (SB + 1) + l16] = x[r];
            wave_lds_sync();
            doublex4 y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kc = 0; kc < SB / 4; ++kc) {
                const double av = -Ts[(SB * ib + l16) * PL + SB * ib + 4 * kc + lg];
                const double bv = Xs[(4 * kc + lg) * (SB + 1) + l16];
                y = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, y, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) Ts[(SB * ib + 4 * r + lg) * PL + SB * s + l16] = y[r];
            wave_lds_sync();
        }
    // results to memory, 16 rows per batch (all LDS reads of a batch in flight at once)
#pragma unroll 1
    for (int i0 = 0; i0 < NB; i0 += 16) {
        double lv[16], tv[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            lv[r] = Ls[(i0 + r) * PL + lane];
            tv[r] = Ts[(i0 + r) * PL + lane];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = i0 + r;
            if (i < bs && lane <= i) A[(int64_t)i * lda + lane] = lv[r];
            Linv[i * NB + lane] = (lane <= i) ? tv[r] : 0.0;
        }
    }
    if (lane == 0 && bad) obc_latch(status, err);
}

// ---- 64 x 64 tile products -------------------------------------------------------------------
// 64 x 64 x (K <= 64) products with the whole contraction staged in LDS at once: every operand is
// requested from memory before any is waited for, so a product costs one trip to memory instead of
// one per 16-wide slab.  Operand tiles sit k-major in LDS, S[k * PL + i], padded like the
// factorisation's block (PL = 65) so that both can use the same memory.

// 16 elements per thread of a rows x cols piece of a row-major matrix (element e = tid + 256 h is
// (e / 64, e % 64): consecutive threads read along a row); zero outside the piece
__device__ __forceinline__ void tile_fetch(double (&r)[16], const double *__restrict__ p, int64_t ld, int rows, int cols)
{
#pragma unroll
    for (int h = 0; h < 16; ++h) {
        const int e = threadIdx.x + h * 256;
        const int row = e >> 6, col = e & 63;
        r[h] = (row < rows && col < cols) ? p[(int64_t)row * ld + col] : 0.0;
    }
}
// park a fetched piece in LDS: element (row, col) at S[row][col], or transposed at S[col][row]
template <bool TRANSPOSE>
__device__ __forceinline__ void tile_park(double *S, const double (&r)[16])
{
#pragma unroll
    for (int h = 0; h < 16; ++h) {
        const int e = threadIdx.x + h * 256;
        const int row = e >> 6, col = e & 63;
        S[TRANSPOSE ? col * PL + row : row * PL + col] = r[h];
    }
}
// acc(i, j) (+)= sum_k As[k][i] Bs[k][j] over all 64 k; wave (wm, wn) of the 2 x 2 owns 32 x 32 outputs.
// v_mfma_f64_16x16x4: lane l supplies a(i = l % 16, k = l / 16) and b(k = l / 16, j = l % 16) and
// holds c(4 r + l / 16, l % 16) in accumulator register r.
template <bool ACCUMULATE = false>
__device__ __forceinline__ void tile_mma(doublex4 (&acc)[2][2], const double *As, const double *Bs)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1, kl = lane >> 4, il = lane & 15;
    if (!ACCUMULATE) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[a][b] = doublex4{0.0, 0.0, 0.0, 0.0};
    }
#pragma unroll
    for (int kk = 0; kk < NB; kk += 4) {
        const double a0 = As[(kk + kl) * PL + wm * 32 + il], a1 = As[(kk + kl) * PL + wm * 32 + 16 + il];
        const double b0 = Bs[(kk + kl) * PL + wn * 32 + il], b1 = Bs[(kk + kl) * PL + wn * 32 + 16 + il];
        acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
        acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
        acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
    }
}
// visit the calling thread's 16 accumulator entries: f(row, col, value)
template <typename F>
__device__ __forceinline__ void tile_each(doublex4 (&acc)[2][2], F f)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                f(wm * 32 + a * 16 + 4 * r + (lane >> 4), wn * 32 + b * 16 + (lane & 15), (double)acc[a][b][r]);
}
// set them: acc(row, col) = f(row, col)
template <typename F>
__device__ __forceinline__ void tile_fill(doublex4 (&acc)[2][2], F f)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[a][b][r] = f(wm * 32 + a * 16 + 4 * r + (lane >> 4), wn * 32 + b * 16 + (lane & 15));
}

template <typename F>
__device__ __forceinline__ void tile_each2(doublex4 (&x)[2][2], doublex4 (&y)[2][2], F f)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                f(wm * 32 + a * 16 + 4 * r + (lane >> 4), wn * 32 + b * 16 + (lane & 15), (double)x[a][b][r], (double)y[a][b][r]);
}

// The diagonal-block factorisation of potrf_wave for a whole workgroup of four wavefronts, block
// already in LDS (layout and contract of potrf_wave_core; the factor is not written out).  The 64
// dependent column steps stay on wavefront 0, everything else moves off its chain:
//  * wavefront 0 factors a whole 16-column panel at a time -- lane l holds row (16 s + l) of the
//    panel, so the sub-blocks below the diagonal one come out of the same instructions as the
//    diagonal sub-block (no product with its inverse);
//  * the inverse of diagonal sub-block s - 1 is computed by wavefront 1 while wavefront 0 factors
//    panel s;
//  * the trailing sub-block updates of a panel are dealt to all four wavefronts, the three block
//    columns of the off-diagonal part of L^-1 to three of them, the final stores to all.
// LDS: POTRF_LDS doubles as for potrf_wave, then two more 16 x 17 scratch sub-blocks, then 2 x 16
// reciprocal pivots.
// rsqrt_f64 (hardware estimate and two Newton steps) one operation at a time, so that the caller can
// place the nine dependent operations among independent work: stage 0 .. 8, result in r after stage 8
__device__ __forceinline__ void rsqrt_stage(int st, double x, double &r, double &a)
{
    switch (st) {
    case 0: r = __builtin_amdgcn_rsq(x); break;
    case 1: case 5: a = r * r; break;
    case 2: case 6: a = x * a; break;
    case 3: case 7: a = fma(-0.5, a, 1.5); break;
    case 4: case 8: r = r * a; break;
    default: break;
    }
}

constexpr int POTRF_WG_LDS = POTRF_LDS + 2 * SB * (SB + 1) + 2 * SB;

__device__ __forceinline__ void potrf_wg_core(double *__restrict__ Linv, int *status, int err, double *lds)
{
    double *Ls = lds;
    double *Ts = lds + NB * PL;
    double *Xs0 = lds + 2 * NB * PL;
    double *Rj = lds + POTRF_LDS + 2 * SB * (SB + 1);
    const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bool bad = false;

    // inverse of the 16 x 16 factor at sub-block o (rows in LDS, reciprocal pivots in rjs), lane c
    // computes column c:  t[i] = (delta_ic - sum_{k<i} L[i][k] t[k]) / L[i][i]
    auto invert_diag = [&](int o, const double *rjs) {
        double row[SB], t[SB];
#pragma unroll
        for (int c = 0; c < SB; ++c) row[c] = Ls[(o + l16) * PL + o + c];
#pragma unroll
        for (int i = 0; i < SB; ++i) {
            double acc = (l16 == i) ? 1.0 : 0.0;
            // the lane to read from, made to depend on the previous row's result: otherwise
            // the lane reads of all rows are issued up front and overflow the scalar registers
            int sel = i;
            if (i > 0) asm volatile("" : "+s"(sel) : "v"(t[i > 0 ? i - 1 : 0]));
#pragma unroll
            for (int k = 0; k < i; ++k) acc = fma(-readlane_f64(row[k], sel), t[k], acc);
            t[i] = acc * rjs[i];
        }
        if (lane < SB) {
#pragma unroll
            for (int c = 0; c < SB; ++c) Ts[(o + c) * PL + o + lane] = t[c];
        }
    };

#pragma unroll
    for (int s = 0; s < NB / SB; ++s) {
        const int o = SB * s;
        if (wave == 0) {
            // ---- panel s: row (o + lane) in registers
            int ls = lane;
            asm volatile("" : "+v"(ls));   // (an opaque copy per panel: keeps the lane masks out of scalar registers)
            const bool has = o + lane < NB;
            double row[SB], rj[SB];
#pragma unroll
            for (int c = 0; c < SB; ++c) row[c] = has ? Ls[(o + lane) * PL + o + c] : 0.0;
            // The pivot of column j + 1 is known as soon as column j has updated row entry j + 1: its
            // reciprocal square root (a chain of dependent fp64 operations) is started right there,
            // among the remaining updates of column j, instead of after them.
            double pj = readlane_f64(row[0], 0);
            if (!(pj > 0.0) || !(pj < __builtin_inf())) { bad = true; pj = 1.0; }
            double r = rsqrt_f64(pj);
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                rj[j] = r;                                          // 1 / L[j][j]
                const double cj = row[j] * r;
                row[j] = (ls == j) ? pj * r : (ls > j ? cj : 0.0);
                const double mine = (ls > j) ? cj : 0.0;            // L[o + lane][j] below the diagonal
                double pn = 1.0, rn = 1.0, an = 0.0;
#pragma unroll
                for (int c = j + 1; c < SB; ++c) {
                    const double lcj = readlane_f64(cj, c);         // L[o + c][j]
                    row[c] = fma(-mine, lcj, row[c]);
                    // pin the update here: left to itself the compiler defers it to the column's
                    // turn and keeps every L[c][j] alive in scalar registers until then
                    asm volatile("" : "+v"(row[c]));
                    if (c == j + 1) {
                        pn = readlane_f64(row[c], c);
                        if (!(pn > 0.0) || !(pn < __builtin_inf())) { bad = true; pn = 1.0; }
                    }
                    rsqrt_stage(c - (j + 1), pn, rn, an);           // one operation of it per update
                }
#pragma unroll
                for (int st = (SB - 1 - j > 0 ? SB - 1 - j : 0); st < 9; ++st) rsqrt_stage(st, pn, rn, an);
                pj = pn;
                r = rn;
            }
            if (has) {
#pragma unroll
                for (int c = 0; c < SB; ++c) Ls[(o + lane) * PL + o + c] = row[c];
            }
            if (lane == 0) {
#pragma unroll
                for (int j = 0; j < SB; ++j) Rj[(s & 1) * SB + j] = rj[j];
            }
        } else if (wave == 1 && s > 0) {
            double rjs[SB];
#pragma unroll
            for (int i = 0; i < SB; ++i) rjs[i] = Rj[((s - 1) & 1) * SB + i];
            invert_diag(o - SB, rjs);
        }
        __syncthreads();                       // panel s (and the inverse of sub-block s - 1) in LDS
        // ---- trailing sub-blocks: A_ij -= L_is L_js^T  (s < j <= i), dealt to the four wavefronts
        int pair = 0;
#pragma unroll
        for (int ib = s + 1; ib < NB / SB; ++ib)
#pragma unroll
            for (int jb = s + 1; jb <= ib; ++jb, ++pair) {
                if ((pair & 3) != wave) continue;
                doublex4 acc;
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] = Ls[(SB * ib + 4 * r + lg) * PL + SB * jb + l16];
#pragma unroll
                for (int kc = 0; kc < SB / 4; ++kc) {
                    const double av = -Ls[(SB * ib + l16) * PL + o + 4 * kc + lg];
                    const double bv = Ls[(SB * jb + l16) * PL + o + 4 * kc + lg];
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) Ls[(SB * ib + 4 * r + lg) * PL + SB * jb + l16] = acc[r];
            }
        if (s + 1 < NB / SB) __syncthreads();
    }
    if (wave == 1) {
        double rjs[SB];
#pragma unroll
        for (int i = 0; i < SB; ++i) rjs[i] = Rj[((NB / SB - 1) & 1) * SB + i];
        invert_diag(NB - SB, rjs);
    }
    __syncthreads();
    // ---- off-diagonal sub-blocks of T = L^-1: block column s on wavefront s, top to bottom
    //      T_is = -T_ii sum_{s <= k < i} L_ik T_ks  (a wavefront only reads what it wrote itself,
    //      the factor and the diagonal sub-blocks)
#pragma unroll
    for (int s = 0; s + 1 < NB / SB; ++s) {
        if (wave != s) continue;
        double *Xs = Xs0 + s * SB * (SB + 1);
#pragma unroll
        for (int ib = s + 1; ib < NB / SB; ++ib) {
            doublex4 x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kb = s; kb < ib; ++kb)
#pragma unroll
                for (int kc = 0; kc < SB / 4; ++kc) {
                    const double av = Ls[(SB * ib + l16) * PL + SB * kb + 4 * kc + lg];
                    const double bv = Ts[(SB * kb + 4 * kc + lg) * PL + SB * s + l16];
                    x = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, x, 0, 0, 0);
                }
#pragma unroll
            for (int r = 0; r < 4; ++r) Xs[(4 * r + lg) * (SB + 1) + l16] = x[r];
            wave_lds_sync();
            doublex4 y = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kc = 0; kc < SB / 4; ++kc) {
                const double av = -Ts[(SB * ib + l16) * PL + SB * ib + 4 * kc + lg];
                const double bv = Xs[(4 * kc + lg) * (SB + 1) + l16];
                y = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, y, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) Ts[(SB * ib + 4 * r + lg) * PL + SB * s + l16] = y[r];
            wave_lds_sync();
        }
    }
    __syncthreads();
    // ---- L^-1 to memory (it also stays in LDS for the caller): 16 rows per wavefront
    {
        double tv[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) tv[r] = Ts[(wave * 16 + r) * PL + lane];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = wave * 16 + r;
            Linv[i * NB + lane] = (lane <= i) ? tv[r] : 0.0;
        }
    }
    if (threadIdx.x == 0 && bad) obc_latch(status, err);
}

}  // namespace obc_dense64

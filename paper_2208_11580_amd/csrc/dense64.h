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
//  * of a panel's trailing updates the next panel waits for those of its own block column, one per
//    wavefront; wavefronts 2 and 3 do the others beside it, and what of the off-diagonal part of L^-1
//    is known by then; while the last diagonal sub-block is inverted, the rest of it but the products
//    with that inverse.
// Bound by the columns' chain on wavefront 0: 4 x 4750 of 26 200 cycles for 64 columns (one column: two multiplications, a
// multiply-add, two ways through a lane read, nine operations of the reciprocal square root); 33 500 cycles with a panel's
// columns stored when it ends, its updates all waited for and the off-diagonal part at the end (a launch of the inverse at
// d = 576 26.0 -> 23 us).
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

// A 16-column panel, lane l's row of it in `own`; it goes to `out` column by column.  The pivot of column J + 1 is known as
// soon as column J has updated entry J + 1: its reciprocal square root (a chain of dependent fp64 operations) is started
// right there and goes on among the remaining updates.  (A column's entries as DPP operands of the updates, from a copy of
// the diagonal sub-block in every 16-lane row, take no lane reads, but v_fmac_f64 with DPP takes 16 cycles: 6500 cycles a
// panel.)
struct PanelWalk {
    double own[SB];
    double *out, *rj;      // the lane's row of the panel in LDS; the reciprocal pivots
    int lane;              // (an opaque copy of the lane index per panel keeps the lane masks out of scalar registers)
    bool bad;
};
template <int J, int C>
__device__ __forceinline__ void panel_updates(PanelWalk &w, double mo, double co, double pn, double &rn, double &an)
{
    if constexpr (C < SB) {
        // four at a time: a value read from a lane takes several instructions' time to reach the next one
        constexpr int N = C + 4 <= SB ? 4 : SB - C;
        double l[4];
#pragma unroll
        for (int i = 0; i < N; ++i) l[i] = readlane_f64(co, C + i);          // L[C + i][J]
#pragma unroll
        for (int i = 0; i < N; ++i) w.own[C + i] = fma(mo, l[i], w.own[C + i]);
        // pin the updates here: left to itself the compiler defers them to the columns' turns and keeps every L[.][J]
        // alive in scalar registers until then
        if constexpr (N == 4) asm volatile("" : "+v"(w.own[C]), "+v"(w.own[C + 1]), "+v"(w.own[C + 2]), "+v"(w.own[C + 3]));
        else {
#pragma unroll
            for (int i = 0; i < N; ++i) asm volatile("" : "+v"(w.own[C + i]));
        }
        constexpr int st = (C - J - 2) / 4 * 2;                              // two operations of the chain per group
        rsqrt_stage(st, pn, rn, an);
        rsqrt_stage(st + 1, pn, rn, an);
        panel_updates<J, C + N>(w, mo, co, pn, rn, an);
    }
}
template <int J>
__device__ __forceinline__ void panel_columns(PanelWalk &w, double pj, double r)
{
    if constexpr (J < SB) {
        const double co = w.own[J] * r, mo = (w.lane > J) ? -co : 0.0;     // - L[.][J] below the diagonal
        double pn = 1.0, rn = 1.0, an = 0.0;
        if constexpr (J + 1 < SB) {
            w.own[J + 1] = fma(mo, readlane_f64(co, J + 1), w.own[J + 1]);
            asm volatile("" : "+v"(w.own[J + 1]));
            pn = readlane_f64(w.own[J + 1], J + 1);
            asm volatile("" : "+v"(pn));                        // (checked by the vector ALU: no way through a scalar)
            if (!(pn > 0.0) || !(pn < __builtin_inf())) { w.bad = true; pn = 1.0; }
        }
        w.out[J] = (w.lane == J) ? pj * r : (w.lane > J ? co : 0.0);
        w.rj[J] = r;                                            // 1 / L[J][J], from every lane
        panel_updates<J, J + 2>(w, mo, co, pn, rn, an);
        if constexpr (J + 1 < SB) {
#pragma unroll
            for (int st = (SB - J - 2 + 3) / 4 * 2; st < 9; ++st) rsqrt_stage(st, pn, rn, an);
        }
        panel_columns<J + 1>(w, pn, rn);
    }
}

// rows I .. 15 of the inverse of a 16 x 16 factor, lane c computes column c:
// t[i] = (delta_ic - sum_{k<i} L[i][k] t[k]) / L[i][i];  row: row l % 16 of L; nt: -t
template <int I, int K>
__device__ __forceinline__ void inverse_row(double &acc, const double (&row)[SB], const double (&nt)[SB])
{
#define OBC_FM(v, m) "v_fmac_f64_dpp %0, %" #v ", %" #m " row_newbcast:%c[lane] row_mask:0xf bank_mask:0xf\n\t"
    if constexpr (K + 3 < I) {
        asm("s_nop 1\n\t" OBC_FM(1, 5) OBC_FM(2, 6) OBC_FM(3, 7) OBC_FM(4, 8)
            : "+&v"(acc) : "v"(row[K]), "v"(row[K + 1]), "v"(row[K + 2]), "v"(row[K + 3]), "v"(nt[K]), "v"(nt[K + 1]),
              "v"(nt[K + 2]), "v"(nt[K + 3]), [lane] "n"(I));
        inverse_row<I, K + 4>(acc, row, nt);
    } else if constexpr (K < I) {
        asm("s_nop 1\n\t" OBC_FM(1, 2) : "+&v"(acc) : "v"(row[K]), "v"(nt[K]), [lane] "n"(I));
        inverse_row<I, K + 1>(acc, row, nt);
    }
#undef OBC_FM
}
template <int I>
__device__ __forceinline__ void inverse_rows(double (&t)[SB], double (&nt)[SB], const double (&row)[SB], const double *rjs, int l16)
{
    if constexpr (I < SB) {
        double acc = (l16 == I) ? 1.0 : 0.0;
        inverse_row<I, 0>(acc, row, nt);
        t[I] = acc * rjs[I];
        nt[I] = -t[I];
        inverse_rows<I + 1>(t, nt, row, rjs, l16);
    }
}

// bs: live size of the block; sub-blocks that are padding only are left out
__device__ __forceinline__ void potrf_wg_core(double *__restrict__ Linv, int bs, int *status, int err, double *lds)
{
    double *Ls = lds;
    double *Ts = lds + NB * PL;
    double *Xs0 = lds + 2 * NB * PL;
    double *Rj = lds + POTRF_LDS + 2 * SB * (SB + 1);
    const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nblk = (bs + SB - 1) / SB;
    bool bad = false;
    if (threadIdx.x < NB && (int)threadIdx.x >= SB * nblk) Ts[threadIdx.x * PL + threadIdx.x] = 1.0;

    // inverse of the 16 x 16 factor of sub-block s
    auto invert_diag = [&](int s) {
        const int o = SB * s;
        double row[SB], t[SB], nt[SB], rjs[SB];
#pragma unroll
        for (int c = 0; c < SB; ++c) {
            row[c] = Ls[(o + l16) * PL + o + c];
            rjs[c] = Rj[(s & 1) * SB + c];
        }
        inverse_rows<0>(t, nt, row, rjs, l16);
        if (lane < SB) {
#pragma unroll
            for (int c = 0; c < SB; ++c) Ts[(o + c) * PL + o + lane] = t[c];
        }
    };
    // A_ij -= L_is L_js^T
    auto update = [&](int ib, int jb, int s) {
        doublex4 acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = Ls[(SB * ib + 4 * r + lg) * PL + SB * jb + l16];
#pragma unroll
        for (int kc = 0; kc < SB / 4; ++kc) {
            const double av = -Ls[(SB * ib + l16) * PL + SB * s + 4 * kc + lg];
            const double bv = Ls[(SB * jb + l16) * PL + SB * s + 4 * kc + lg];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) Ls[(SB * ib + 4 * r + lg) * PL + SB * jb + l16] = acc[r];
    };
    // Off-diagonal sub-blocks of T = L^-1:  T_is = -T_ii X_is,  X_is = sum_{s <= k < i} L_ik T_ks, which is parked in
    // the scratch sub-block of column s
    auto off_sum = [&](int ib, int s) {
        doublex4 x = {0.0, 0.0, 0.0, 0.0};
        for (int kb = s; kb < ib; ++kb)
#pragma unroll
            for (int kc = 0; kc < SB / 4; ++kc) {
                const double av = Ls[(SB * ib + l16) * PL + SB * kb + 4 * kc + lg];
                const double bv = Ts[(SB * kb + 4 * kc + lg) * PL + SB * s + l16];
                x = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, x, 0, 0, 0);
            }
        double *Xs = Xs0 + s * SB * (SB + 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) Xs[(4 * r + lg) * (SB + 1) + l16] = x[r];
        wave_lds_sync();
    };
    auto off_solve = [&](int ib, int s) {
        const double *Xs = Xs0 + s * SB * (SB + 1);
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
    };

    // Wavefront 0 goes from panel to panel.  Of panel s's updates it waits for those of block column s + 1 only, one per
    // wavefront; the others are done by wavefronts 2 and 3 beside panel s + 1, and so is sub-block (1, 0) of T.
#pragma unroll 1
    for (int s = 0; s < nblk; ++s) {
        const int o = SB * s;
        if (wave == 0) {
            PanelWalk w;
            w.lane = lane;
            asm volatile("" : "+v"(w.lane));
            w.bad = false;
            // (lanes beyond the block's last row write to its last sub-block column above the diagonal, which nobody reads)
            const bool has = o + lane < NB;
            w.out = has ? &Ls[(o + lane) * PL + o] : &Ls[(o + lane - NB) * PL + NB - SB];
            w.rj = Rj + (s & 1) * SB;
#pragma unroll
            for (int c = 0; c < SB; ++c) w.own[c] = has ? w.out[c] : 0.0;
            double pj = readlane_f64(w.own[0], 0);
            if (!(pj > 0.0) || !(pj < __builtin_inf())) { w.bad = true; pj = 1.0; }
            panel_columns<0>(w, pj, rsqrt_f64(pj));
            bad |= w.bad;
        } else if (wave == 1) {
            if (s > 0) invert_diag(s - 1);
        } else if (s == 1) {
            if (nblk > 2 && wave == 2) update(2, 2, 0);
            if (nblk > 3 && wave == 3) { update(3, 2, 0); update(3, 3, 0); }
        } else if (s == 2) {
            if (nblk > 3 && wave == 3) update(3, 3, 1);
        } else if (s == 3) {
            if (wave == 2) { off_sum(1, 0); off_solve(1, 0); }
        }
        __syncthreads();                       // panel s (and the inverse of sub-block s - 1) in LDS
        if (s + 1 < nblk) {
            if (s + 1 + wave < nblk) update(s + 1 + wave, s + 1, s);
            __syncthreads();
        }
    }
    if (nblk == NB / SB) {
        // everything of T's last row but the products with its diagonal sub-block, while that is inverted
        if (wave == 0) off_sum(3, 2);
        else if (wave == 1) invert_diag(3);
        else if (wave == 2) { off_sum(2, 1); off_solve(2, 1); off_sum(3, 1); }
        else { off_sum(2, 0); off_solve(2, 0); off_sum(3, 0); }
        __syncthreads();
        if (wave != 1) off_solve(3, wave == 0 ? 2 : wave == 2 ? 1 : 0);
    } else {
        if (wave == 1) invert_diag(nblk - 1);
        __syncthreads();
        // block column s on wavefront s, top to bottom (a wavefront only reads what it wrote itself, the factor and the
        // diagonal sub-blocks)
        for (int ib = wave + 1; ib < nblk; ++ib) {
            off_sum(ib, wave);
            off_solve(ib, wave);
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

// The panel kernel of the blocked row solver (see rows_blocked.hip for the scheme).  Included by
// one small translation unit per (threads, elements per thread, block size) variant.
#pragma once

#include <atomic>
#include <type_traits>

#include "rows_blocked.h"

namespace obc_blocked {

typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));

constexpr int kNmShift = 16;          // above any index
constexpr int kBeyond = 0x40000000;   // a byte offset beyond any row's matrix: the load returns 0

// Per-thread state of the panel: everything indexed by the owned element e (compact index
// tid + e*T) or by the step r inside the block.  All indices are compile-time constants (panel_step
// reaches the step's own vector by branches), so the arrays live in registers.
template <int EPT, int BR>
struct PanelRegs {
    double w[EPT], dg[EPT];
    // original index, ~index where it was pruned before, kGone: no live index.  N:M: the weights that its block
    // has given up are counted in the bits from kNmShift on (every thread counts for its own: in LDS the counters
    // were a read in the selection's chain).
    int og[EPT];
    float u[BR][EPT];   // u_r for the first BR steps of the block (0 before its step); later ones live in LDS
    // block pruning only: row j of the 4 x 4 diagonal block of the current inverse that element j
    // belongs to (entry k = A[j][4 (j / 4) + k]; the element's own slot is not used), and the first
    // position of the block being eliminated
    float ob[EPT][4];
    int p0;
};

// B: steps of the panel
template <int B>
struct PanelShared {
    static constexpr int PMAX = (B + 15) / 16 * 16;
    unsigned long long red_k[2][16];
    __attribute__((aligned(16))) float cvec[PMAX];
    float invd_s[PMAX];
    __attribute__((aligned(16))) float cold[UCAP];   // coefficients of the outer block's earlier vectors ...
    __attribute__((aligned(16))) float invd_old[UCAP];                            // ... and their 1 / a_r
    int live[16 * 16];   // survivors per (owned element, wave)
    // the step's scalars: the update of the weights, 1 / a_pp, the index's original position, whether
    // the pivot is usable
    double g, invapp;
    int o, ok;
    // What the steps' records are made of when the panel ends (original index, weight, 1 / a_pp): made
    // and stored in every step they would lengthen the chain that the whole workgroup waits for, and
    // the owner's wait for its fetched row would be one for its stores too.
    int rec_o[PMAX];
    double rec_w[PMAX], rec_invapp[PMAX];
};

// order-preserving map of a float onto unsigned integers
__device__ __forceinline__ unsigned score_bits(float f)
{
    unsigned u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// value of lane K of the caller's group of four lanes (DPP quad_perm broadcast); must be called
// with all four lanes active
template <int K>
__device__ __forceinline__ float quad_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), K * 0x55, 0xf, 0xf, false));
}
template <int K>
__device__ __forceinline__ double quad_bcast(double v)
{
    long long b = __double_as_longlong(v);
    unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, K * 0x55, 0xf, 0xf, false);
    unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), K * 0x55, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Block pruning (Sec. 4 "Block-Sparsity", eq. (5)), blocks of 4: the score w_P^T ((H^-1)_P)^-1 w_P of
// the block that the calling lane's element belongs to.  The block's four elements sit on four
// neighbouring lanes (positions 4b .. 4b+3 of the compact index space); every lane gathers the
// block's weights and its 4 x 4 piece of the inverse and runs the same elimination, so the four
// lanes get bit-identical scores.  NaN when a pivot is not positive.
__device__ __forceinline__ double quad_block_score(double w, double dg, const float (&ob)[4])
{
    double v[4], M[4][4];
    v[0] = quad_bcast<0>(w); v[1] = quad_bcast<1>(w); v[2] = quad_bcast<2>(w); v[3] = quad_bcast<3>(w);
    M[0][0] = quad_bcast<0>(dg); M[1][1] = quad_bcast<1>(dg);
    M[2][2] = quad_bcast<2>(dg); M[3][3] = quad_bcast<3>(dg);
    M[1][0] = (double)quad_bcast<1>(ob[0]);
    M[2][0] = (double)quad_bcast<2>(ob[0]); M[2][1] = (double)quad_bcast<2>(ob[1]);
    M[3][0] = (double)quad_bcast<3>(ob[0]); M[3][1] = (double)quad_bcast<3>(ob[1]);
    M[3][2] = (double)quad_bcast<3>(ob[2]);
    double s = 0.0;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double piv = M[k][k];
        bad = bad || !(piv > 0.0);
        const double ip = 1.0 / piv;
        s += v[k] * v[k] * ip;
#pragma unroll
        for (int i = k + 1; i < 4; ++i) {
            const double f = M[i][k] * ip;
            v[i] -= f * v[k];
#pragma unroll
            for (int j = k + 1; j <= i; ++j) M[i][j] -= f * M[j][k];
        }
    }
    return bad ? __builtin_nan("") : s;
}

// One DPP stage of an unsigned minimum: combine with the lane `row_shr` positions down the
// 16-lane row (lanes shifted in from outside the row contribute the identity).
template <int CTRL>
__device__ __forceinline__ unsigned dpp_umin_stage(unsigned v)
{
    const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(-1, (int)v, CTRL, 0xf, 0xf, false);
    return o < v ? o : v;
}

// minimum over each 16-lane row, valid in the row's last lane
__device__ __forceinline__ unsigned row16_umin(unsigned v)
{
    v = dpp_umin_stage<0x111>(v);   // row_shr:1
    v = dpp_umin_stage<0x112>(v);   // row_shr:2
    v = dpp_umin_stage<0x114>(v);   // row_shr:4
    v = dpp_umin_stage<0x118>(v);   // row_shr:8
    return v;
}

// the same over each N lanes (a power of two, 4 .. 16, whose values every group of N repeats; uniform result)
template <int N>
__device__ __forceinline__ unsigned lanes_umin(unsigned v)
{
    v = dpp_umin_stage<0x111>(v);
    v = dpp_umin_stage<0x112>(v);
    if constexpr (N > 4) v = dpp_umin_stage<0x114>(v);
    if constexpr (N > 8) v = dpp_umin_stage<0x118>(v);
    return (unsigned)__builtin_amdgcn_readlane((int)v, 15);
}

// minimum over the wavefront (uniform result)
__device__ __forceinline__ unsigned wave_umin(unsigned v)
{
    v = row16_umin(v);
    unsigned a0 = (unsigned)__builtin_amdgcn_readlane((int)v, 15), a1 = (unsigned)__builtin_amdgcn_readlane((int)v, 31);
    unsigned a2 = (unsigned)__builtin_amdgcn_readlane((int)v, 47), a3 = (unsigned)__builtin_amdgcn_readlane((int)v, 63);
    a0 = a1 < a0 ? a1 : a0;
    a2 = a3 < a2 ? a3 : a2;
    return a2 < a0 ? a2 : a0;
}

// acc[e] += sum_i c_i u_i[e], i < 4, for N elements: coefficient i is in lane L + i of every 16-lane row
// of c.  The coefficient is taken from its lane by the multiply-add itself (DPP row_newbcast): no lane
// read, no scalar register.  A DPP operand must not have been written by the vector ALU within two
// cycles; the compiler does not look into the block, so it waits itself.  (The sums are written before the last
// vector is read: without "&" one still to come, known to be 0, could share the register of a sum that starts at 0.)
template <int L, int N>
__device__ __forceinline__ void fma_bcast(float *acc, float c, const float *u0, const float *u1, const float *u2,
                                          const float *u3)
{
#define OBC_FB(acc, c, u, lane) "v_fmac_f32_dpp %" #acc ", %" #c ", %" #u " row_newbcast:%" #lane " row_mask:0xf bank_mask:0xf\n\t"
    if constexpr (N >= 3) {
        asm("s_nop 1\n\t" OBC_FB(0, 3, 4, 16) OBC_FB(1, 3, 5, 16) OBC_FB(2, 3, 6, 16) OBC_FB(0, 3, 7, 17)
                OBC_FB(1, 3, 8, 17) OBC_FB(2, 3, 9, 17) OBC_FB(0, 3, 10, 18) OBC_FB(1, 3, 11, 18)
                    OBC_FB(2, 3, 12, 18) OBC_FB(0, 3, 13, 19) OBC_FB(1, 3, 14, 19) OBC_FB(2, 3, 15, 19)
            : "+&v"(acc[0]), "+&v"(acc[1]), "+&v"(acc[2])
            : "v"(c), "v"(u0[0]), "v"(u0[1]), "v"(u0[2]), "v"(u1[0]), "v"(u1[1]), "v"(u1[2]), "v"(u2[0]), "v"(u2[1]),
              "v"(u2[2]), "v"(u3[0]), "v"(u3[1]), "v"(u3[2]), "n"(L), "n"(L + 1), "n"(L + 2), "n"(L + 3));
        if constexpr (N > 3) fma_bcast<L, N - 3>(acc + 3, c, u0 + 3, u1 + 3, u2 + 3, u3 + 3);
    } else if constexpr (N == 2) {
        asm("s_nop 1\n\t" OBC_FB(0, 2, 3, 11) OBC_FB(1, 2, 4, 11) OBC_FB(0, 2, 5, 12) OBC_FB(1, 2, 6, 12)
                OBC_FB(0, 2, 7, 13) OBC_FB(1, 2, 8, 13) OBC_FB(0, 2, 9, 14) OBC_FB(1, 2, 10, 14)
            : "+&v"(acc[0]), "+&v"(acc[1])
            : "v"(c), "v"(u0[0]), "v"(u0[1]), "v"(u1[0]), "v"(u1[1]), "v"(u2[0]), "v"(u2[1]), "v"(u3[0]), "v"(u3[1]),
              "n"(L), "n"(L + 1), "n"(L + 2), "n"(L + 3));
    } else {
        asm("s_nop 1\n\t" OBC_FB(0, 1, 2, 6) OBC_FB(0, 1, 3, 7) OBC_FB(0, 1, 4, 8) OBC_FB(0, 1, 5, 9)
            : "+&v"(acc[0])
            : "v"(c), "v"(u0[0]), "v"(u1[0]), "v"(u2[0]), "v"(u3[0]), "n"(L), "n"(L + 1), "n"(L + 2), "n"(L + 3));
    }
#undef OBC_FB
}

// The same for one owned element and the vectors R0 .. S - 1: coefficient r in lane r % 16 of c[r / 16].
template <int S, int R0, int NC, int BR>
__device__ __forceinline__ void fma_bcast_all(float &acc, const float (&c)[NC], const float (&u)[BR][1])
{
#define OBC_FB(op, lane) "v_fmac_f32_dpp %0, %1, %" #op " row_newbcast:%" #lane " row_mask:0xf bank_mask:0xf\n\t"
    if constexpr (R0 < S) {
        constexpr int N = S - R0 >= 8 ? 8 : S - R0 >= 4 ? 4 : S - R0 >= 2 ? 2 : 1, L = R0 % 16;
        const float ck = c[R0 / 16];
        if constexpr (N == 8)
            asm("s_nop 1\n\t" OBC_FB(2, 10) OBC_FB(3, 11) OBC_FB(4, 12) OBC_FB(5, 13) OBC_FB(6, 14) OBC_FB(7, 15)
                    OBC_FB(8, 16) OBC_FB(9, 17)
                : "+&v"(acc)
                : "v"(ck), "v"(u[R0][0]), "v"(u[R0 + 1][0]), "v"(u[R0 + 2][0]), "v"(u[R0 + 3][0]), "v"(u[R0 + 4][0]),
                  "v"(u[R0 + 5][0]), "v"(u[R0 + 6][0]), "v"(u[R0 + 7][0]), "n"(L), "n"(L + 1), "n"(L + 2), "n"(L + 3),
                  "n"(L + 4), "n"(L + 5), "n"(L + 6), "n"(L + 7));
        else if constexpr (N == 4)
            asm("s_nop 1\n\t" OBC_FB(2, 6) OBC_FB(3, 7) OBC_FB(4, 8) OBC_FB(5, 9)
                : "+&v"(acc)
                : "v"(ck), "v"(u[R0][0]), "v"(u[R0 + 1][0]), "v"(u[R0 + 2][0]), "v"(u[R0 + 3][0]), "n"(L), "n"(L + 1),
                  "n"(L + 2), "n"(L + 3));
        else if constexpr (N == 2)
            asm("s_nop 1\n\t" OBC_FB(2, 4) OBC_FB(3, 5)
                : "+&v"(acc)
                : "v"(ck), "v"(u[R0][0]), "v"(u[R0 + 1][0]), "n"(L), "n"(L + 1));
        else
            asm("s_nop 1\n\t" OBC_FB(2, 3) : "+&v"(acc) : "v"(ck), "v"(u[R0][0]), "n"(L));
        fma_bcast_all<S, R0 + N>(acc, c, u);
    }
#undef OBC_FB
}

// The least index v among the lanes of `among` that hold the minimum (uniform result).  It nearly always has
// one holder, whose index is read from its lane; among several the lowest lane's is the least where a thread
// owns one index, else they are compared (`least`).
template <int EPT, class Least>
__device__ __forceinline__ unsigned least_holder(bool holds, unsigned v, unsigned long long among, Least least)
{
    const unsigned long long b = __ballot(holds) & among;
    if (EPT > 1 && (b & (b - 1)) != 0) return least(holds ? v : ~0u);
    return (unsigned)__builtin_amdgcn_readlane((int)v, __builtin_ctzll(b));
}

struct PanelRow {
    const float *Acur;
    float *gU;
    int ld, swz, d, m, done, total, ndead, row, old, ldu;
    double qd, qo, qmax, iqd;
    float nm_inv;   // 1 / M
    // the row's matrix for raw buffer loads: resource, bytes between an element of a row and the next,
    // row_base of the thread's first index
    __amdgpu_buffer_rsrc_t rsrc;
    __amdgpu_buffer_rsrc_t ursrc;   // the row's vectors (u_index)
    int es, rb_tid;
    int nw;         // waves launched (one owned element per thread: as many as the live size needs)
    int mw;         // live size less the wave's first index
};

// byte offset of element (i, 0) of the row's matrix
__device__ __forceinline__ int row_base(int i, const PanelRow &pr)
{
    return pr.swz ? ((i >> 2) * pr.ld * 4 + (i & 3)) * 4 : i * pr.ld * 4;
}

// o / M for 0 <= o < 2^20: (o + 1/2) / M is at least 1 / (2 M) away from every integer, many times
// the rounding of this product (an integer division would be some twenty instructions of the step's
// dependent chain)
__device__ __forceinline__ int nm_block(int o, float nm_inv) { return (int)(((float)o + 0.5f) * nm_inv); }

// The score of owned element e as an order-preserving integer (all ones when it is no candidate) and,
// except in block pruning, its error (target - w).
template <int MODE, int EPT, int BR>
__device__ __forceinline__ unsigned candidate_key(const PanelArgs &a, const PanelRow &pr, const PanelRegs<EPT, BR> &st,
                                                  int e, double &er)
{
    float sc;
    er = 0.0;
    if constexpr (MODE == MODE_BLOCK) {
        sc = (float)quad_block_score(st.w[e], st.dg[e], st.ob[e]);
        if (st.og[e] == kGone) return ~0u;
    } else {
        if (st.og[e] == kGone) return ~0u;
        if (st.og[e] < 0) {
            sc = -__builtin_inff();   // dead indices go first, before any outlier
        } else {
            if (MODE == MODE_PRUNE && a.nm_m > 0 && (st.og[e] >> kNmShift) >= a.nm_m - a.nm_n) return ~0u;
            double tq = 0.0;
            if (MODE == MODE_QUANT) {
                double c = rint((st.w[e] - pr.qo) * pr.iqd);
                c = fmin(fmax(c, 0.0), pr.qmax);
                tq = pr.qo + pr.qd * c;
            }
            er = tq - st.w[e];
            sc = (float)(er * er) * __builtin_amdgcn_rcpf((float)st.dg[e]);
            // outlier heuristic: a weight whose error exceeds half a grid step sorts before every
            // non-outlier
            if (MODE == MODE_QUANT && a.outliers && fabs(er) > 0.5 * pr.qd) sc = outlier_first(sc);
        }
    }
    return sc == sc ? score_bits(sc) : ~0u;   // a NaN score is no candidate
}

// Where a thread owns two to four elements the steps of a panel are a loop over groups of four: one body of 20 .. 40 KB
// instead of 200 .. 400 KB of code that each wave would run through once.  What a step may do depends on its number
// only through uniform branches: the correction stops at the vectors in use, the new vector reaches its registers by a
// branch tree.  In ms, without a loop and as one: 3072 x 768 at 4 bit 15.59, 15.26, 768 x 768 pruned 4.21, 4.12, 203 x 1283
// at 4 bit 4.93, 4.90, 256 x 2304 at 4 bit 23.19, 23.10, 12 x 2048 pruned 5.88, 5.84; blocks of four within 1.2 % either way.
// From six elements on the loop holds all vectors' registers from the first step on, also next to the re-reading of
// earlier panels' vectors, and its branches cost more than the code.  In ms, as a loop and without: 100 x 4608 pruned
// 88.1, 86.7, at 4 bit 88.5, 86.3, 2:4 76.1, 75.0, in blocks of four 94.9, 93.4; 64 x 3072 in blocks of four 23.3, 22.7;
// 100 x 3072 at 4 bit 28.8, 28.1; 8 x 2600 pruned 10.21, 10.11.
// With one it is a step's latency that the branches lengthen, above all where a CU holds one row; corrections by whole
// groups of four and the select of their coefficients count there too.  In us, as a loop and without: 64 x 576 2:4
// 520, 503; 12 x 1000 pruned 1894, 1785; 64 x 768 at 4 bit 1318, 1273; in blocks of four 12 x 516 697, 626, 64 x 768 1216,
// 1132.  Results are bit for bit the same.
template <int EPT>
constexpr bool kStepLoop = EPT >= 2 && EPT <= 4;

// acc[e] += the correction by the register-held vectors from 4 K to 4 LAST - 1, four at a time, as far as the
// first 4 `quads` go (a group's vectors that are still to come are 0, and so are their coefficients).
template <int EPT, int BR, int K, int LAST, int NC>
__device__ __forceinline__ void correct_regs(float *acc, const float (&cv)[NC], const PanelRegs<EPT, BR> &st, int quads)
{
    if constexpr (K < LAST) {
        if (quads <= K) return;
        fma_bcast<4 * K % 16, EPT>(acc, cv[K / 4], st.u[4 * K], st.u[4 * K + 1], st.u[4 * K + 2], st.u[4 * K + 3]);
        correct_regs<EPT, BR, K + 1, LAST>(acc, cv, st, quads);
    }
}

// ... and by the LDS-held ones before step S
template <int T, int EPT, int BR, int BL, int L, int NC>
__device__ __forceinline__ void correct_lds(float (&acc)[EPT], const float (&cv)[NC], const float *ul, int S)
{
    if constexpr (L < BL) {
        if (BR + L >= S) return;
        float v[4][EPT];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < EPT; ++e) v[i][e] = ul[((L + i) * EPT + e) * T];
        fma_bcast<(BR + L) % 16, EPT>(acc, cv[(BR + L) / 16], v[0], v[1], v[2], v[3]);
        correct_lds<T, EPT, BR, BL, L + 4>(acc, cv, ul, S);
    }
}

// the calling thread's entries of the register-held vectors, element e, four per LDS write
template <int EPT, int BR, int K>
__device__ __forceinline__ void publish_regs(float *cvec, const PanelRegs<EPT, BR> &st, int e, int quads)
{
    if constexpr (K < BR / 4) {
        if (quads <= K) return;
        *reinterpret_cast<float4 *>(&cvec[4 * K]) =
            make_float4(st.u[4 * K][e], st.u[4 * K + 1][e], st.u[4 * K + 2][e], st.u[4 * K + 3][e]);
        publish_regs<EPT, BR, K + 1>(cvec, st, e, quads);
    }
}

// u[4 quad + SUB] = c, LO <= quad < HI: a branch tree down to the registers (a select per register would
// be as many instructions as a step has elsewhere)
template <int EPT, int BR, int SUB, int LO, int HI>
__device__ __forceinline__ void keep_regs(PanelRegs<EPT, BR> &st, const float (&c)[EPT], int quad)
{
    if constexpr (HI - LO == 1) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) asm volatile("v_mov_b32 %0, %1" : "=v"(st.u[4 * LO + SUB][e]) : "v"(c[e]));
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (quad < MID) keep_regs<EPT, BR, SUB, LO, MID>(st, c, quad);
        else keep_regs<EPT, BR, SUB, MID, HI>(st, c, quad);
    }
}

// One greedy step, the S-th of the block, S = 4 quad + SUB; IN_LDS: S >= BR, its vector is kept in LDS.  QUAD:
// quad where the steps are not a loop, else -1.
// OLD: the panel follows others of its outer block, whose vectors it finds in memory.  Returns 0 to
// continue, 1 when the row has no step left, 2 on a numeric failure.  Every thread of the workgroup
// returns the same value.
template <int MODE, int T, int EPT, int BR, int BL, bool OLD, int SUB, bool IN_LDS, int QUAD>
__device__ __forceinline__ int panel_step(const PanelArgs &a, const PanelRow &pr, PanelRegs<EPT, BR> &st,
                                          PanelShared<BR + BL> &sh, float *ul, int quad)
{
    // u_r[j] for r >= BR is kept at ul[(r - BR) * (T * EPT) + j]; only the owner of j touches it
    constexpr int CAP = T * EPT;
    static_assert(EPT > 1 || (QUAD >= 0 && BL == 0), "one owned element: all vectors in registers, no loop");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int S = 4 * quad + SUB;
    if (pr.done + S >= pr.total) return 1;

    // ---- (1) selection.  The error (target - w) is formed in fp64 (for OBQ it is a difference of
    // nearby numbers); the score itself, error^2 / a_jj, is only compared, so it is taken in fp32
    // with the hardware reciprocal (2 ulp): candidates closer than that count as tied.
    // A candidate is the pair (order-preserving bits of the score, index); the argmin with ties to
    // the lowest index is taken in two unsigned 32-bit minima: the least score, then the least
    // index among the candidates that have it.  All ones = no candidate.
    unsigned cs = ~0u, ci = ~0u;
    double cer = 0.0;   // error of the thread's best candidate
    if constexpr (MODE != MODE_BLOCK || SUB == 0) {   // (a block is chosen every fourth step)
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            double er;
            const unsigned b = candidate_key<MODE>(a, pr, st, e, er);
            if (b < cs) {   // (indices ascend with e)
                cs = b;
                ci = (unsigned)((MODE == MODE_BLOCK ? tid & ~3 : tid) + e * T);
                cer = er;
            }
        }
    }
    int p;
    if constexpr (MODE == MODE_BLOCK && SUB != 0) {
        __syncthreads();   // the previous step's readers of the shared step data are done
        p = st.p0 + SUB;
    } else {
        const unsigned ws = wave_umin(cs);
        const unsigned wi = least_holder<EPT>(cs == ws, ci, MODE == MODE_BLOCK ? 0x1111111111111111ull : ~0ull,
                                              [](unsigned v) { return wave_umin(v); });
        unsigned gs = ws;
        p = (int)wi;
        if (EPT > 1 || pr.nw > 1) {
            if (lane == 0) sh.red_k[SUB & 1][wave] = ((unsigned long long)ws << 32) | wi;
            __syncthreads();
            constexpr int NW2 = T <= 256 ? 4 : T <= 512 ? 8 : 16;
            const int l = lane & (NW2 - 1);
            const unsigned long long wk = l < pr.nw ? sh.red_k[SUB & 1][l] : ~0ull;
            gs = lanes_umin<NW2>((unsigned)(wk >> 32));
            p = (int)least_holder<EPT>((unsigned)(wk >> 32) == gs, (unsigned)wk, (1ull << NW2) - 1,
                                       [](unsigned v) { return lanes_umin<NW2>(v); });
        }
        if (gs == ~0u) return 2;
        if constexpr (MODE == MODE_BLOCK) st.p0 = p;
    }

    // ---- (2) fetch the owned part of row p of A0.  Only the lower triangle of A0 is kept up to
    // date (the matrix is symmetric): entry (p, j) is read as (max(p, j), min(p, j)), i.e. along
    // row p up to the diagonal and down column p below it.
    // Byte offsets: element (i, j), j <= i, lies at row_base(i) + j es, so both parts are affine in the
    // owned element; raw buffer loads take 32-bit offsets.
    const int ep = p / T, pt = p - ep * T;   // p's owner: element ep of thread pt
    float col[EPT];
    {
        const int along = tid * pr.es + row_base(p, pr), down = pr.rb_tid + p * pr.es;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            int off = tid <= p - e * T ? along + e * T * pr.es : down + e * T * pr.ld * 4;
            if (EPT > 1 && tid >= pr.m - e * T) off = kBeyond;   // indices beyond m: no memory access, 0
            col[e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(pr.rsrc, off, 0, 2));
        }
    }
    // the owner of p publishes the pivot's data and its entries of the earlier vectors of this block
    if (tid == pt) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            if (e != ep) continue;
            // entries p of the vectors kept in registers, four per LDS write
            publish_regs<EPT, BR, 0>(sh.cvec, st, e, IN_LDS ? BR / 4 : quad + (SUB > 0));
            const double ap = st.dg[e];
            // 1 / ap: the hardware's estimate and two Newton steps (a division's scaling and fix-up
            // steps would only lengthen the chain that everybody waits for)
            double invapp = __builtin_amdgcn_rcp(ap);
            invapp = fma(fma(-ap, invapp, 1.0), invapp, invapp);
            invapp = fma(fma(-ap, invapp, 1.0), invapp, invapp);
            const double wp = st.w[e];
            sh.g = (MODE == MODE_BLOCK ? wp : -cer) * invapp;
            sh.invapp = invapp;
            const int o = MODE == MODE_PRUNE && st.og[e] >= 0 ? st.og[e] & ((1 << kNmShift) - 1) : st.og[e];
            sh.o = o;
            sh.ok = (ap > 0.0) && (ap < __builtin_inf()) ? 1 : 0;
            sh.invd_s[S] = (float)invapp;
            sh.rec_o[S] = o;
            sh.rec_w[S] = wp;
            sh.rec_invapp[S] = invapp;
            // (keeps the elements' code apart: merged, it copies their vectors into common registers first, which
            // spill: 3072 x 768 at 4 bit 17.97 instead of 15.9 ms)
            if constexpr (EPT > 1) asm volatile("" ::"v"(wp));
        }
    }
    // coefficients of the earlier panels' vectors, which are in memory: one lane each
    if constexpr (OLD) {
        if (tid < pr.old) sh.cold[tid] = pr.gU[u_index(tid, p, pr.ldu)];
    }
    // entries p of the vectors kept in LDS: one lane each
    if constexpr (IN_LDS) {
        const int r = BR + tid;
        if (r < S) sh.cvec[r] = ul[(r - BR) * CAP + p];
    }
    __syncthreads();
    const double g = sh.g, invapp = sh.invapp;
    const int op = __builtin_amdgcn_readfirstlane(sh.o);
    const bool isdead = op < 0;
    // coefficients u_r[p] / a_r of this step: lane l has those of r = l % 16, l % 16 + 16, ..., from S on 0 (one
    // owned element: never used)
    constexpr int NC = QUAD >= 0 ? (4 * QUAD + SUB + 15) / 16 : ((IN_LDS ? BR + BL : BR) + 15) / 16;
    float cv[NC > 0 ? NC : 1];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        const int r = 16 * k + (lane & 15);
        const float c = __fmul_rn(sh.cvec[r], sh.invd_s[r]);
        cv[k] = EPT == 1 || r < S ? c : 0.f;
    }

    if (!__builtin_amdgcn_readfirstlane(sh.ok)) return 2;   // (after the reads above are on their way)

    // ---- (3) bring the fetched row up to date, keep it, update w and the diagonal.
    // The correction is summed on its own and subtracted once: its roundings are then relative to
    // the (small) correction instead of to the matrix entry, and the sum does not wait for the
    // fetched row.
    if constexpr (OLD) {
        // The earlier panels' vectors, panel by panel, exactly as their flush would have applied them:
        // entry (i, j), i >= j, gets sum_k (-u_k[i] / a_k) u_k[j], summed from zero in k order (which is
        // how the fp32 matrix instruction sums) and added once.  (Indices beyond m read what lies behind
        // the vector -- a row's UCAP vectors are longer than any index -- and only reach values that are
        // never used.)
        auto earlier = [&](auto ne) {
            constexpr int NE = decltype(ne)::value;      // the wave's elements that hold live indices
#pragma unroll 1
            for (int r0 = 0; r0 < pr.old; r0 += BR + BL) {
                float sum[NE];
#pragma unroll
                for (int e = 0; e < NE; ++e) sum[e] = 0.f;
#pragma unroll 1
                for (int r = r0; r < r0 + BR + BL; r += 4) {
                    const float4 o4 = *reinterpret_cast<const float4 *>(&sh.cold[r]);
                    const float4 i4 = *reinterpret_cast<const float4 *>(&sh.invd_old[r]);
                    // (half of the elements at a time: what is in flight has to find room in the registers)
                    constexpr int HE = (NE + 1) / 2;
#pragma unroll
                    for (int e0 = 0; e0 < NE; e0 += HE) {
                        uintx4 v[HE];
#pragma unroll
                        for (int e = 0; e < HE; ++e)
                            if (e0 + e < NE) v[e] = __builtin_amdgcn_raw_buffer_load_b128(pr.ursrc, tid * 16, ((r >> 2) * pr.ldu + (e0 + e) * T) * 16, 0);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float up = q == 0 ? o4.x : q == 1 ? o4.y : q == 2 ? o4.z : o4.w;
                            const float ni = -(q == 0 ? i4.x : q == 1 ? i4.y : q == 2 ? i4.z : i4.w), fp = __fmul_rn(up, ni);
#pragma unroll
                            for (int e = e0; e < e0 + HE && e < NE; ++e) {
                                const bool along = tid <= p - e * T;     // (p, j) with j <= p, else (j, p)
                                const float vq = __uint_as_float(v[e - e0][q]);
                                sum[e] = fmaf(along ? fp : up, along ? vq : __fmul_rn(vq, ni), sum[e]);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
#pragma unroll
                for (int e = 0; e < NE; ++e) col[e] = __fadd_rn(col[e], sum[e]);
            }
        };
        static_assert(EPT > 3, "every live size of the variant reaches the elements before the last two");
        if ((EPT - 2) * T >= pr.mw) earlier(std::integral_constant<int, EPT - 2>{});
        else if ((EPT - 1) * T >= pr.mw) earlier(std::integral_constant<int, EPT - 1>{});
        else earlier(std::integral_constant<int, EPT>{});
    }
    float c[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) c[e] = 0.f;
    if constexpr (EPT == 1) {
        fma_bcast_all<4 * QUAD + SUB, 0>(c[0], cv, st.u);
    } else if constexpr (!IN_LDS) {
        correct_regs<EPT, BR, 0, BR / 4>(c, cv, st, SUB == 0 ? quad : quad + 1);
    } else {
        correct_regs<EPT, BR, 0, BR / 4>(c, cv, st, BR / 4);
        correct_lds<T, EPT, BR, BL, 0>(c, cv, ul + tid, S);
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) c[e] = __fsub_rn(col[e], c[e]);
    if constexpr (QUAD >= 0) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) st.u[4 * QUAD + SUB][e] = c[e];
    } else if constexpr (!IN_LDS) {
        keep_regs<EPT, BR, SUB, 0, BR / 4>(st, c, quad);
    } else {
#pragma unroll
        for (int e = 0; e < EPT; ++e) ul[(S - BR) * CAP + tid + e * T] = c[e];
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        if constexpr (MODE == MODE_BLOCK) {
            // Lemma 1 on the element's row of its own 4 x 4 block: A[j][j'] -= u[j] u[j'] / a
            const float cs = c[e] * (float)invapp;
            st.ob[e][0] = fmaf(-cs, quad_bcast<0>(c[e]), st.ob[e][0]);
            st.ob[e][1] = fmaf(-cs, quad_bcast<1>(c[e]), st.ob[e][1]);
            st.ob[e][2] = fmaf(-cs, quad_bcast<2>(c[e]), st.ob[e][2]);
            st.ob[e][3] = fmaf(-cs, quad_bcast<3>(c[e]), st.ob[e][3]);
        }
        if (st.og[e] != kGone) {
            if (tid + e * T == p) {
                st.og[e] = kGone;
            } else {
                const double cd = (double)c[e];
                st.w[e] = fma(-cd, g, st.w[e]);
                st.dg[e] = fma(-(cd * cd), invapp, st.dg[e]);
            }
        }
    }
    if (MODE == MODE_PRUNE && a.nm_m > 0 && !isdead) {
        const int b = nm_block(op, pr.nm_inv), pw = p - (pr.m - pr.mw);   // p less the wave's first index
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            // (original indices ascend with the position: a block's weights lie within M - 1 positions of each other,
            // and few waves have an element there)
            if (EPT > 1 && (unsigned)(pw - e * T + a.nm_m - 1) >= 62u + 2 * a.nm_m) continue;
            if (st.og[e] >= 0 && nm_block(st.og[e] & ((1 << kNmShift) - 1), pr.nm_inv) == b) st.og[e] += 1 << kNmShift;
        }
    }
    if (MODE == MODE_BLOCK && a.trace && SUB == 3) {
        float *tr = a.trace + ((size_t)pr.row * a.out_ld + (pr.done + S) / 4) * pr.d;
#pragma unroll
        for (int e = 0; e < EPT; ++e)
            if (st.og[e] != kGone) tr[st.og[e]] = (float)st.w[e];
    }
    if (MODE == MODE_PRUNE && a.trace && !isdead) {
        float *tr = a.trace + ((size_t)pr.row * a.out_ld + (pr.done + S - pr.ndead)) * pr.d;
#pragma unroll
        for (int e = 0; e < EPT; ++e)
            if (st.og[e] >= 0) tr[st.og[e] & ((1 << kNmShift) - 1)] = (float)st.w[e];
    }
    return 0;
}

// Four steps from 4 quad on; returns the number of them done and sets *failed.
template <int MODE, int T, int EPT, int BR, int BL, bool OLD, bool IN_LDS, int QUAD = -1>
__device__ __forceinline__ int panel_quad(const PanelArgs &a, const PanelRow &pr, PanelRegs<EPT, BR> &st,
                                          PanelShared<BR + BL> &sh, float *ul, int quad, bool *failed)
{
    int rc = panel_step<MODE, T, EPT, BR, BL, OLD, 0, IN_LDS, QUAD>(a, pr, st, sh, ul, quad);
    if (rc == 0) {
        rc = panel_step<MODE, T, EPT, BR, BL, OLD, 1, IN_LDS, QUAD>(a, pr, st, sh, ul, quad);
        if (rc == 0) {
            rc = panel_step<MODE, T, EPT, BR, BL, OLD, 2, IN_LDS, QUAD>(a, pr, st, sh, ul, quad);
            if (rc == 0) {
                rc = panel_step<MODE, T, EPT, BR, BL, OLD, 3, IN_LDS, QUAD>(a, pr, st, sh, ul, quad);
                if (rc == 0) return 4;
                *failed = rc == 2;
                return 3;
            }
            *failed = rc == 2;
            return 2;
        }
        *failed = rc == 2;
        return 1;
    }
    *failed = rc == 2;
    return 0;
}

// all steps of a panel whose vectors are kept in registers, without a loop; returns the number of them done
template <int MODE, int T, int EPT, int BR, int BL, bool OLD, int QUAD>
__device__ __forceinline__ int panel_unrolled(const PanelArgs &a, const PanelRow &pr, PanelRegs<EPT, BR> &st,
                                              PanelShared<BR + BL> &sh, float *ul, bool *failed)
{
    if constexpr (QUAD < BR / 4) {
        const int n = panel_quad<MODE, T, EPT, BR, BL, OLD, false, QUAD>(a, pr, st, sh, ul, QUAD, failed);
        if (n < 4) return 4 * QUAD + n;
        return panel_unrolled<MODE, T, EPT, BR, BL, OLD, QUAD + 1>(a, pr, st, sh, ul, failed);
    } else {
        return BR;
    }
}

// OLD: an instance that can follow others of its outer block (a.old > 0).  At six elements a thread the
// panels that do not are instances without it: what re-reading the earlier vectors takes does not fit the
// registers next to a step's state (8 x 2600, 240 steps with a flush each 40, without it and with: pruned 2.03,
// 2.27 ms, in blocks, where nothing shares a flush, 2.14, 2.37; 128 x 2600 4.48, 4.70 and 4.66, 4.85).
template <int MODE, int T, int EPT, int BR, int BL, bool OLD>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(T == 256 ? (EPT == 1 ? 4 : 3) : T / 256)))
void panel_kernel(PanelArgs a)
{
    constexpr int B = BR + BL;
    static_assert(BR % 4 == 0 && BL % 4 == 0, "the vectors are used four at a time");
    static_assert(sizeof(PanelShared<B>) <= 160 * 1024 - kPanelDynLds && BL * T * EPT * sizeof(float) <= kPanelDynLds, "a CU's LDS");
    __shared__ PanelShared<B> sh;
    // dynamic LDS: BL vectors of T * EPT floats
    extern __shared__ __align__(16) uint8_t dyn_lds[];
    float *ul = reinterpret_cast<float *>(dyn_lds);

    // Rows of at most BMAX weights are through after one panel: it takes its state from the caller's
    // arrays and leaves nothing for a next one (one launch instead of a set-up and a panel, and no
    // workspace).  One wave per row.
    constexpr bool CAN_DIRECT = EPT == 1 && BL == 0 && T == 256;
    const bool direct = CAN_DIRECT && a.direct;

    const int row = blockIdx.x, tid = threadIdx.x;
    PanelRow pr;
    pr.row = row;
    pr.d = a.d;
    bool live0 = true;          // direct: the caller's mask
    if (direct) {
        live0 = tid < a.d && (MODE == MODE_BLOCK || !a.live_in || a.live_in[(size_t)row * a.d + tid] != 0);
        pr.m = a.d;
        pr.done = 0;
        pr.ndead = a.d - __popcll(__ballot(live0));
        pr.total = panel_total(MODE, a.d, a.d - pr.ndead, a.k_steps, a.stop_counts, row);
    } else {
        pr.m = a.ws.m[row];
        pr.done = a.ws.done[row];
        pr.total = a.ws.total[row];
        pr.ndead = a.ws.ndead[row];
        if (pr.done >= pr.total) {
            if (tid == 0) a.ws.nb[row] = 0;
            return;
        }
    }
    const int d = a.d, m = pr.m;
    pr.Acur = a.A_cur + (size_t)row * a.a_row_stride;
    pr.ld = a.ld;
    pr.swz = a.swz;
    pr.rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)pr.Acur, 0, (int)(a.swz ? ((size_t)d * d + 3) / 4 * 16 : (size_t)d * d * 4),
                                                0x00020000u);
    pr.es = a.swz ? 16 : 4;
    pr.rb_tid = row_base(tid, pr);
    pr.nw = blockDim.x >> 6;
    pr.mw = m - __builtin_amdgcn_readfirstlane(tid & ~63);
    pr.gU = a.ws.U + (size_t)row * UCAP * a.ws.ldu;
    pr.ldu = a.ws.ldu;
    pr.ursrc = __builtin_amdgcn_make_buffer_rsrc((void *)pr.gU, 0, UCAP * pr.ldu * 4, 0x00020000u);
    pr.old = a.old;
    double *gw = a.ws.w + (size_t)row * d;
    double *gd = a.ws.diag + (size_t)row * d;
    int *go = a.ws.orig + (size_t)row * d;

    PanelRegs<EPT, BR> st;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        int j = tid + e * T;
        if (direct) {
            st.og[e] = j < m ? (live0 ? j : ~j) : kGone;
            st.w[e] = live0 ? (double)a.W[(size_t)row * d + j] : 0.0;
            st.dg[e] = j < m ? (double)pr.Acur[(size_t)j * d + j] : 1.0;
        } else {
            st.og[e] = j < m ? go[j] : kGone;
            st.w[e] = st.og[e] != kGone ? gw[j] : 0.0;
            st.dg[e] = st.og[e] != kGone ? gd[j] : 1.0;
        }
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
#pragma unroll
        for (int r = 0; r < BR; ++r) st.u[r][e] = 0.f;
#pragma unroll
        for (int r = 0; r < BL; ++r) ul[r * (T * EPT) + tid + e * T] = 0.f;
    }
    for (int r = tid; r < a.old; r += blockDim.x) sh.invd_old[r] = a.ws.invd[(size_t)row * UCAP + r];
    if constexpr (MODE == MODE_BLOCK) {
        // the element's row of its 4 x 4 diagonal block, from the lower triangle of the matrix
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int j = tid + e * T, j0 = j & ~3;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int jj = j0 + k;
                const int hi = (jj <= j) ? j : jj, lo = (jj <= j) ? jj : j;
                const size_t off = pr.swz ? quad_index(hi, lo, pr.ld) : (size_t)hi * pr.ld + lo;
                st.ob[e][k] = (j < m) ? pr.Acur[off] : 0.f;
            }
        }
        if constexpr (OLD) {
            // ... and the outer block's earlier eliminations, as their flush would have applied them
            __syncthreads();
#pragma unroll 1
            for (int r0 = 0; r0 < a.old; r0 += B) {
#pragma unroll
                for (int e = 0; e < EPT; ++e) {
                    float sum[4] = {0.f, 0.f, 0.f, 0.f};
                    const int q = tid & 3;
#pragma unroll 2
                    for (int r = r0; r < r0 + B; ++r) {
                        const float u = pr.gU[u_index(r, tid + e * T, pr.ldu)], f = __fmul_rn(u, -sh.invd_old[r]);
                        // (all lanes read their neighbours before any of them chooses)
                        const float u0 = quad_bcast<0>(u), u1 = quad_bcast<1>(u), u2 = quad_bcast<2>(u), u3 = quad_bcast<3>(u);
                        const float f1 = quad_bcast<1>(f), f2 = quad_bcast<2>(f), f3 = quad_bcast<3>(f);
                        sum[0] = fmaf(f, u0, sum[0]);      // (j, j0): j is the larger index
                        sum[1] = fmaf(q >= 1 ? f : f1, q >= 1 ? u1 : u, sum[1]);
                        sum[2] = fmaf(q >= 2 ? f : f2, q >= 2 ? u2 : u, sum[2]);
                        sum[3] = fmaf(q >= 3 ? f : f3, q >= 3 ? u3 : u, sum[3]);
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) st.ob[e][k] = __fadd_rn(st.ob[e][k], sum[k]);
                }
            }
        }
        st.p0 = 0;
    }
    pr.qd = 1.0;
    pr.qo = 0.0;
    pr.qmax = (double)a.maxq;
    pr.nm_inv = a.nm_m > 0 ? 1.0f / (float)a.nm_m : 0.f;
    if (MODE == MODE_PRUNE && a.nm_m > 0 && !direct) {
#pragma unroll
        for (int e = 0; e < EPT; ++e)
            if (st.og[e] >= 0) st.og[e] |= (int)a.ws.blk[(size_t)row * d + nm_block(st.og[e], pr.nm_inv)] << kNmShift;
    }
    if (MODE == MODE_QUANT) { pr.qd = (double)a.delta[row]; pr.qo = (double)a.offset[row]; }
    pr.iqd = 1.0 / pr.qd;
    __syncthreads();

    bool failed = false;
    int nbv = 0;
    bool more = true;
    if constexpr (!kStepLoop<EPT>) {
        nbv = panel_unrolled<MODE, T, EPT, BR, BL, OLD, 0>(a, pr, st, sh, ul, &failed);
        more = nbv == BR;
    } else {
#pragma unroll 1
        for (int quad = 0; more && quad < BR / 4; ++quad) {
            const int n = panel_quad<MODE, T, EPT, BR, BL, OLD, false>(a, pr, st, sh, ul, quad, &failed);
            nbv += n;
            more = n == 4;
        }
    }
    if constexpr (BL > 0) {
#pragma unroll 1
        for (int quad = BR / 4; more && quad < (BR + BL) / 4; ++quad) {
            const int n = panel_quad<MODE, T, EPT, BR, BL, OLD, true>(a, pr, st, sh, ul, quad, &failed);
            nbv += n;
            more = n == 4;
        }
    }
    __syncthreads();

    // ---- block epilogue.  Before the outer block's last panel the state stays in the present index
    // space; the last one drops the eliminated indices from it.
    if (!direct)
        for (int r = tid; r < nbv; r += blockDim.x) a.ws.invd[(size_t)row * UCAP + a.old + r] = sh.invd_s[r];
    float *Wo = a.W_out + (size_t)row * d;
    if (direct && tid < d) {
        if (st.og[0] != kGone || !live0) Wo[tid] = live0 ? (float)st.w[0] : 0.f;
        if (MODE == MODE_QUANT && (st.og[0] != kGone || !live0)) a.codes[(size_t)row * d + tid] = -1;
    }
    // the steps' records
    if (tid < nbv) {
        auto step_loss = [&](int r, double target) {
            const double er = target - sh.rec_w[r];
            return (float)(0.5 * er * er * sh.rec_invapp[r]);
        };
        const int op = sh.rec_o[tid];
        if (MODE == MODE_BLOCK) {
            Wo[op] = 0.f;
            if (tid % 4 == 3) {
                // the block's loss is the sum of its four single losses
                double acc = (double)step_loss(tid - 3, 0.0);
                for (int q = 2; q >= 0; --q) acc += (double)step_loss(tid - q, 0.0);
                const size_t t = (size_t)row * a.out_ld + (pr.done + tid) / 4;
                a.order[t] = op / 4;
                a.loss[t] = (float)acc;
            }
        } else if (op >= 0) {
            double code = 0.0, target = 0.0;
            if (MODE == MODE_QUANT) {
                code = rint((sh.rec_w[tid] - pr.qo) * pr.iqd);   // same expression as in the selection
                code = fmin(fmax(code, 0.0), pr.qmax);
                target = pr.qo + pr.qd * code;
            }
            const size_t t = (size_t)row * a.out_ld + (pr.done + tid - pr.ndead);
            a.order[t] = op;
            a.loss[t] = step_loss(tid, target);
            Wo[op] = (float)target;
            if (MODE == MODE_QUANT) a.codes[(size_t)row * d + op] = (int)code;
        }
    }
    if (direct) {
        if (failed && tid == 0) obc_latch(a.status, OBC_ERR_NUMERIC);
        return;
    }
    int jn[EPT];           // new index, or -1
    int live = 0;          // survivors at lower indices of the workgroup so far
    if (a.last) {
        constexpr int NW = T / 64;
        const int lane = tid & 63, wave = tid >> 6;
        static_assert(EPT * NW <= 16 * 16, "survivor counts");
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const unsigned long long bal = __ballot(st.og[e] != kGone);
            jn[e] = __popcll(bal & ((1ull << lane) - 1ull));
            if (lane == 0) sh.live[e * NW + wave] = __popcll(bal);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            int here = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const int n = w < pr.nw ? sh.live[e * NW + w] : 0;
                if (w < wave) here += n;
                if (w == wave) jn[e] += live + here;
                if (w >= wave) here += n;
            }
            live += here;
            if (st.og[e] == kGone) jn[e] = -1;
        }
    } else {
#pragma unroll
        for (int e = 0; e < EPT; ++e) jn[e] = tid + e * T < m ? tid + e * T : -1;
    }
    int *gmap = a.ws.map + (size_t)row * d;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int j = tid + e * T;
        if (jn[e] >= 0) {
            if (MODE == MODE_PRUNE && st.og[e] >= 0) {
                // N:M: all live weights of a block hold its count
                if (a.nm_m > 0)
                    a.ws.blk[(size_t)row * d + nm_block(st.og[e] & ((1 << kNmShift) - 1), pr.nm_inv)] = (uint8_t)(st.og[e] >> kNmShift);
                st.og[e] &= (1 << kNmShift) - 1;
            }
            gw[jn[e]] = st.w[e];
            gd[jn[e]] = st.dg[e];
            go[jn[e]] = st.og[e];
            gmap[jn[e]] = j;
            if (st.og[e] >= 0) Wo[st.og[e]] = (float)st.w[e];
            // this panel's vectors u_r, in the new index order (a row that ended within four of them has no use for them)
#pragma unroll
            for (int r = 0; r < B; r += 4)
                if (r < nbv) {
                    uintx4 v;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        v[q] = __float_as_uint(r < BR ? st.u[r < BR ? r + q : 0][e] : ul[(r + q - BR) * (T * EPT) + j]);
                    __builtin_amdgcn_raw_buffer_store_b128(v, pr.ursrc, jn[e] * 16, ((a.old + r) >> 2) * pr.ldu * 16, 0);
                }
        }
    }
    if constexpr (OLD) {
        // the earlier panels' vectors move to the new order in place: a group of them is read
        // whole before any of it is written
        if (a.last) {
#pragma unroll 1
            for (int r = 0; r < a.old; r += 4) {
                const int at = (r >> 2) * pr.ldu * 16;
                uintx4 v[EPT];
#pragma unroll
                for (int e = 0; e < EPT; ++e) v[e] = __builtin_amdgcn_raw_buffer_load_b128(pr.ursrc, tid * 16, at + e * T * 16, 0);
                __syncthreads();
#pragma unroll
                for (int e = 0; e < EPT; ++e)
                    if (jn[e] >= 0) __builtin_amdgcn_raw_buffer_store_b128(v[e], pr.ursrc, jn[e] * 16, at, 0);
            }
        }
    }
    if (tid == 0) {
        if (a.last) a.ws.m[row] = live;
        a.ws.done[row] = pr.done + nbv;
        a.ws.nb[row] = a.old + nbv;
        if (failed) {
            a.ws.total[row] = pr.done + nbv;   // the row stops here
            obc_latch(a.status, OBC_ERR_NUMERIC);
        }
    }
}


// A kernel's dynamic LDS limit is a per-device attribute: `done` remembers, one bit per device, where
// it has been raised for `fn`.  Safe from several host threads (raising it twice is harmless).
inline int panel_raise_lds_limit(const void *fn, std::atomic<unsigned long long> &done)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return -1;
    const unsigned long long bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return 0;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kPanelDynLds) != hipSuccess)
        return -1;
    done.fetch_or(bit, std::memory_order_release);
    return 0;
}

// With one owned element per thread a launch has as many waves as the largest live size needs: a
// step is bound by instruction issue, and a wave without live elements issues as many as the others.
template <int MODE, int T, int EPT, int BR, int BL, bool OLD>
int panel_launch(int R, hipStream_t st, const PanelArgs &a)
{
    const size_t lds = (size_t)BL * T * EPT * sizeof(float);
    auto kernel = panel_kernel<MODE, T, EPT, BR, BL, OLD>;
    static std::atomic<unsigned long long> raised{0};
    if (lds > 48 * 1024 && panel_raise_lds_limit((const void *)kernel, raised) != 0) return -1;
    hipLaunchKernelGGL(kernel, dim3(R), dim3(EPT == 1 ? a.threads : T), lds, st, a);
    return 0;
}

// NAME: launch_panel, or launch_panel_old where a variant has an instance of its own for OLD
#define OBC_DEFINE_PANEL(NAME, OLD, T, EPT, BR, BL)                                                     \
    int NAME##_##T##_##EPT##_##BR##_##BL(int mode, int R, hipStream_t st, const PanelArgs &a) \
    {                                                                                                   \
        return mode == MODE_PRUNE ? panel_launch<MODE_PRUNE, T, EPT, BR, BL, OLD>(R, st, a)     \
                                  : panel_launch<MODE_QUANT, T, EPT, BR, BL, OLD>(R, st, a);    \
    }

// The block-pruning instance of a variant, in a translation unit of its own.
#define OBC_DEFINE_PANEL_BLOCK(OLD, T, EPT, BR, BL)                                                     \
    int launch_panel_block_##T##_##EPT##_##BR##_##BL(int, int R, hipStream_t st,         \
                                                     const PanelArgs &a)                                \
    {                                                                                                   \
        return panel_launch<MODE_BLOCK, T, EPT, BR, BL, OLD>(R, st, a);                         \
    }

}  // namespace obc_blocked

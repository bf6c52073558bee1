// Row solver, blocked strategy: the greedy loops of Algorithm 1 / Algorithm 3 (arxiv 2208.11580)
// with the Lemma-1 eliminations applied to the row's private inverse in blocks of B steps.
//
// What a greedy step needs is small: the current diagonal of A, the current weights, and the
// current row p of A.  The first two are O(d) to maintain.  Row p can be formed on demand from
// the matrix as of the last block boundary, A0, and the eliminations done since:
//
//     A[p,:] = A0[p,:] - sum_r (u_r[p] / a_r) u_r        u_r = row p_r of A when p_r was chosen,
//                                                        a_r = its diagonal entry
//
// so inside a block nothing of size d^2 moves.  Every B steps the deferred eliminations are
// applied at once,  A0 <- A0 - U diag(1/a) U^T,  a dense rank-B contraction that runs on the fp32
// matrix cores and touches A once per B steps instead of once per step.  The result is the same
// sequence of exact OBS steps; only the order of fp32 roundings inside A differs from the
// rank-1 strategy.
//
// Where a CU only holds the vectors of a few steps (above 2304 columns) several panels share a flush:
// the later ones find the earlier ones' vectors in memory and apply them to the fetched row with the
// flush's own roundings, so that the results do not depend on the grouping.  Rows of at most 64
// weights are one panel, which starts from the caller's arrays.
//
// Two kernels alternate on the stream (host loop, no host synchronisation):
//
//   panel_kernel  one workgroup per row, B greedy steps.  Thread t owns the compact indices
//                 t, t+T, ...: their weights and diagonal (fp64) live in its registers, and of the B
//                 vectors u_r the first BR; the other BL lie in LDS.  Per step: score + workgroup
//                 argmin (barrier 1), the owner of p publishes its weight update, 1 / a_p and its
//                 entries of the vectors while every thread fetches its part of A0[p,:] (barrier 2),
//                 then the row is corrected, w / diag are updated and u_s is kept.  When the panel
//                 ends the steps' records and the vectors (for the flush) are written.
//   flush_kernel  A0_new = compact(A0 - U diag(1/a) U^T): tiles of 32 x 64 on the fp32 matrix cores, one
//                 wavefront each (only the lower triangle is kept).  The eliminated rows and columns are dropped
//                 while writing (out of place, two buffers), so the matrix shrinks with the live set and later
//                 blocks cost (m/d)^2 of the first.  A large first one is flush_first_kernel: strips of 128 or 256
//                 rows with the vectors in LDS.
//
// The first block reads the shared H^-1 directly, so no per-row copy of it is ever made.
// Already-pruned weights (quantization or pruning of survivors) are eliminated first, in index
// order, with no weight change and nothing recorded: 64 at a time by a block form of Lemma 1 as
// long as every row has that many left (see "bulk elimination" below), the rest as candidates
// with score -infinity inside the panel.
#include <type_traits>

#include "rows_blocked.h"

namespace {

using namespace obc_blocked;

// up to this width a call with a mask waits for nothing (it can be captured): its panels eliminate the
// pruned indices, and there is no bulk elimination
constexpr int kNoWaitMaxD = 192;

size_t carve(BlockedWs *ws, void *base, int R, int d)
{
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += obc_align_up(bytes, 256);
        return base ? (char *)base + o : (char *)nullptr;
    };
    size_t mat = (size_t)R * obc_align_up((size_t)d * d, 4) * sizeof(float);
    char *p0 = take(mat), *p1 = take(mat);
    const int ldu = (d + 3) & ~3;
    char *pu = take((size_t)R * UCAP * ldu * sizeof(float));
    char *pi = take((size_t)R * UCAP * sizeof(float));
    char *pm = take((size_t)R * d * sizeof(int));
    char *pw = take((size_t)R * d * sizeof(double));
    char *pd = take((size_t)R * d * sizeof(double));
    char *po = take((size_t)R * d * sizeof(int));
    char *s0 = take((size_t)R * sizeof(int)), *s1 = take((size_t)R * sizeof(int));
    char *s2 = take((size_t)R * sizeof(int)), *s3 = take((size_t)R * sizeof(int));
    char *s4 = take((size_t)R * sizeof(int));
    char *pb = take((size_t)R * d);
    const size_t bulk = d > kNoWaitMaxD ? (size_t)R * BMAX * BMAX * sizeof(double) : 0;
    char *pmb = take(bulk), *ptb = take(bulk);
    char *psc = take(256);
    if (ws) {
        ws->Mb = (double *)pmb; ws->Tb = (double *)ptb; ws->scal = (int *)psc;
        ws->Abuf[0] = (float *)p0; ws->Abuf[1] = (float *)p1; ws->U = (float *)pu; ws->ldu = ldu;
        ws->invd = (float *)pi; ws->map = (int *)pm; ws->w = (double *)pw;
        ws->diag = (double *)pd; ws->orig = (int *)po; ws->m = (int *)s0; ws->done = (int *)s1;
        ws->total = (int *)s2; ws->ndead = (int *)s3; ws->nb = (int *)s4; ws->blk = (uint8_t *)pb;
    }
    return off;
}

// ------------------------------------------------------------------------------------------ init
struct InitArgs {
    const float *W, *Hinv;
    const uint8_t *live_in;
    const int32_t *stop_counts;
    int d, k_steps, mode;
    BlockedWs ws;
    int32_t *codes;
    float *W_out;
};

__global__ __launch_bounds__(256) void blocked_init_kernel(InitArgs a)
{
    __shared__ int cnt;
    const int row = blockIdx.x, tid = threadIdx.x, d = a.d;
    if (tid == 0) cnt = 0;
    __syncthreads();
    int dead_local = 0;
    for (int j = tid; j < d; j += 256) {
        bool alive = (a.mode != MODE_BLOCK && a.live_in) ? a.live_in[(size_t)row * d + j] != 0 : true;
        a.ws.w[(size_t)row * d + j] = alive ? (double)a.W[(size_t)row * d + j] : 0.0;
        a.ws.diag[(size_t)row * d + j] = (double)a.Hinv[(size_t)j * d + j];
        a.ws.orig[(size_t)row * d + j] = alive ? j : ~j;
        a.ws.blk[(size_t)row * d + j] = 0;
        a.W_out[(size_t)row * d + j] = alive ? a.W[(size_t)row * d + j] : 0.f;   // rows that do no step keep W
        if (a.mode == MODE_QUANT) a.codes[(size_t)row * d + j] = -1;
        dead_local += alive ? 0 : 1;
    }
    atomicAdd(&cnt, dead_local);
    __syncthreads();
    if (tid == 0) {
        const int total = panel_total(a.mode, d, d - cnt, a.k_steps, a.stop_counts, row);
        a.ws.m[row] = d;
        a.ws.done[row] = 0;
        a.ws.total[row] = total;
        a.ws.ndead[row] = cnt;
        a.ws.nb[row] = 0;
    }
}

// p[0 .. n) = v with 16-byte streaming stores; the floats before the first 16-byte boundary and
// after the last one singly (p is 4-byte aligned)
__global__ __launch_bounds__(256) void fill_f32_kernel(float *p, size_t n, float v)
{
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    size_t head = ((16 - ((uintptr_t)p & 15)) & 15) / 4;
    if (head > n) head = n;
    const floatx4 v4 = {v, v, v, v};
    floatx4 *p4 = reinterpret_cast<floatx4 *>(p + head);
    const size_t n4 = (n - head) / 4, tail = (n - head) % 4;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n4; e += (size_t)gridDim.x * 256)
        __builtin_nontemporal_store(v4, p4 + e);
    if (blockIdx.x == 0) {
        if (threadIdx.x < head) p[threadIdx.x] = v;
        if (threadIdx.x < tail) p[head + n4 * 4 + threadIdx.x] = v;
    }
}

// ------------------------------------------------------------ bulk elimination of pruned indices
// Already-pruned indices (quantization or pruning of the survivors of an earlier pass) leave the
// inverse without any choice to make: they go in index order and change no weight.  For a set P of
// BMAX of them the eliminations collapse into one block step (the block form of Lemma 1, as in
// eq. (5)):  A <- A - A[:,P] (A[P,P])^-1 A[P,:] = A - U U^T  with  U = A[:,P] L^-T,  A[P,P] = L L^T.
// That needs no vectors kept on chip, so the rank of the update is BMAX whatever the width of the
// row -- the greedy panel manages 24 at 4608 -- and the flush that follows moves that much less.
// Three kernels per block: gather A[:,P] and A[P,P]; factor A[P,P] and invert the factor (fp64,
// one wavefront per row); U = L^-1 A[P,:] with the diagonal update and the compaction.  Every row
// does the same number of such blocks (the smallest count of pruned indices over the rows decides);
// what is left goes through the panel as before.
struct DeadArgs {
    const float *A_cur;
    size_t a_row_stride;
    int ld, swz, d;
    BlockedWs ws;
};

// out[0] = smallest number of up-front eliminations over the rows, out[1] = largest number of
// eliminations (up-front + greedy) any row does
__global__ __launch_bounds__(256) void min_ndead_kernel(const int *__restrict__ ndead, const int *__restrict__ total,
                                                        int R, int *out)
{
    __shared__ int red[256], redt[256];
    int v = 0x7fffffff, t = 0;
    for (int i = threadIdx.x; i < R; i += 256) {
        v = ndead[i] < v ? ndead[i] : v;
        t = total[i] > t ? total[i] : t;
    }
    red[threadIdx.x] = v;
    redt[threadIdx.x] = t;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            red[threadIdx.x] = red[threadIdx.x + w] < red[threadIdx.x] ? red[threadIdx.x + w] : red[threadIdx.x];
            redt[threadIdx.x] = redt[threadIdx.x + w] > redt[threadIdx.x] ? redt[threadIdx.x + w] : redt[threadIdx.x];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) { out[0] = red[0]; out[1] = redt[0]; }
}

// The block's pivots (the first BMAX pruned indices in compact order), the rows of the matrix at
// them (G, in the old compact order) and their principal submatrix (Mb, fp64).
__global__ __launch_bounds__(512) void dead_gather_kernel(DeadArgs a)
{
    __shared__ int pv[BMAX];
    __shared__ int wcnt[8];
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = a.ws.m[row];
    const int *orig = a.ws.orig + (size_t)row * a.d;
    int found = 0;                                       // pivots found so far (uniform)
    for (int c0 = 0; c0 < m && found < BMAX; c0 += 512) {
        const int j = c0 + tid;
        const bool dead = j < m && orig[j] < 0;
        const unsigned long long bal = __ballot(dead);
        if (lane == 0) wcnt[wave] = __popcll(bal);
        __syncthreads();
        int before = found, total = 0;
        for (int w = 0; w < 8; ++w) {
            if (w < wave) before += wcnt[w];
            total += wcnt[w];
        }
        const int rank = before + __popcll(bal & ((1ull << lane) - 1ull));
        if (dead && rank < BMAX) pv[rank] = j;
        found += total;
        __syncthreads();
    }
    // (the host only launches this while every row still has BMAX pruned indices)
    const float *Acur = a.A_cur + (size_t)row * a.a_row_stride;
    float *G = a.ws.U + ((size_t)row * UCAP + BMAX) * a.ws.ldu;
    for (int r = 0; r < BMAX; ++r) {
        const int p = pv[r];
        for (int j = tid; j < m; j += 512) {
            const int hi = (j <= p) ? p : j, lo = (j <= p) ? j : p;
            const size_t off = a.swz ? quad_index(hi, lo, a.ld) : (size_t)hi * a.ld + lo;
            G[(size_t)r * a.ws.ldu + j] = Acur[off];
        }
    }
    if (tid < BMAX) a.ws.invd[(size_t)row * UCAP + tid] = __int_as_float(pv[tid]);
    __syncthreads();                                     // G visible to the whole workgroup
    double *Mb = a.ws.Mb + (size_t)row * BMAX * BMAX;
    for (int e = tid; e < BMAX * BMAX; e += 512) {
        const int r = e / BMAX, s2 = e % BMAX;
        Mb[e] = (double)G[(size_t)r * a.ws.ldu + pv[s2]];
    }
}

// U = T G (T = L^-1 lower triangular, fp32 here), written in the new compact order; the diagonal
// loses sum_k U[k][j]^2; weights, diagonal, original indices and the index map are compacted.
// Only the owner of column j ever touches G[:, j], so once it has read the column it parks the
// column's new diagonal entry and new index there (rows 0..2) until the compaction.
__global__ __launch_bounds__(512) void dead_apply_kernel(DeadArgs a)
{
    __shared__ __align__(16) float Tl[BMAX][BMAX];       // T[k][r]
    __shared__ int pv[BMAX];
    const int row = blockIdx.x, tid = threadIdx.x, d = a.d;
    const int m = a.ws.m[row];
    const int ldu = a.ws.ldu;
    const double *Tb = a.ws.Tb + (size_t)row * BMAX * BMAX;
    for (int e = tid; e < BMAX * BMAX; e += 512) Tl[e / BMAX][e % BMAX] = (float)Tb[e];
    if (tid < BMAX) pv[tid] = __float_as_int(a.ws.invd[(size_t)row * UCAP + tid]);
    __syncthreads();
    float *U = a.ws.U + (size_t)row * UCAP * ldu;
    float *G = U + (size_t)BMAX * ldu;
    double *gw = a.ws.w + (size_t)row * d;
    double *gd = a.ws.diag + (size_t)row * d;
    int *go = a.ws.orig + (size_t)row * d;
    int *gmap = a.ws.map + (size_t)row * d;

#pragma unroll 1
    for (int j = tid; j < m; j += 512) {
        int below = 0;
        bool piv = false;
        for (int s2 = 0; s2 < BMAX; ++s2) {
            below += (pv[s2] < j) ? 1 : 0;
            piv = piv || (pv[s2] == j);
        }
        int jnew = -1;
        double newd = 0.0;
        if (!piv) {
            jnew = j - below;
            float g[BMAX];
#pragma unroll
            for (int r = 0; r < BMAX; ++r) g[r] = G[(size_t)r * ldu + j];
            double dsum = 0.0;
            float u4[4];
#pragma unroll
            for (int k = 0; k < BMAX; ++k) {
                float acc = 0.f;
#pragma unroll
                for (int r = 0; r <= k; ++r) acc = fmaf(Tl[k][r], g[r], acc);
                u4[k % 4] = acc;
                if (k % 4 == 3) *reinterpret_cast<float4 *>(U + u_index(k - 3, jnew, ldu)) = make_float4(u4[0], u4[1], u4[2], u4[3]);
                dsum += (double)acc * (double)acc;
                // one row of T at a time (otherwise its LDS reads are all issued up front)
                __builtin_amdgcn_sched_barrier(0);
            }
            newd = gd[j] - dsum;
        }
        const long long bits = __double_as_longlong(newd);
        G[j] = __int_as_float((int)(unsigned)bits);
        G[(size_t)ldu + j] = __int_as_float((int)(unsigned)((unsigned long long)bits >> 32));
        G[(size_t)2 * ldu + j] = __int_as_float(jnew);
    }
    // compaction: read the old entries, wait for everybody, write the new ones
    constexpr int EMAX = 10;                             // ceil(largest d / 512)
    double wv[EMAX], dv[EMAX];
    int ov[EMAX], jn[EMAX];
#pragma unroll
    for (int e = 0; e < EMAX; ++e) {
        const int j = tid + e * 512;
        jn[e] = -1;
        if (j >= m) continue;
        jn[e] = __float_as_int(G[(size_t)2 * ldu + j]);
        const unsigned lo = (unsigned)__float_as_int(G[j]), hi = (unsigned)__float_as_int(G[(size_t)ldu + j]);
        dv[e] = __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
        wv[e] = gw[j];
        ov[e] = go[j];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EMAX; ++e) {
        if (jn[e] < 0) continue;
        gw[jn[e]] = wv[e];
        gd[jn[e]] = dv[e];
        go[jn[e]] = ov[e];
        gmap[jn[e]] = tid + e * 512;
    }
    if (tid < BMAX) a.ws.invd[(size_t)row * UCAP + tid] = 1.f;
    if (tid == 0) {
        a.ws.m[row] = m - BMAX;
        a.ws.done[row] += BMAX;
        a.ws.nb[row] = BMAX;
    }
}

// ----------------------------------------------------------------------------------------- flush
struct FlushArgs {
    const float *A_old;
    size_t old_row_stride;   // 0 when every row still reads the shared H^-1
    int ld_old;
    int old_swz;             // layout of A_old: 0 plain row-major, 1 row-quad (A_new is always row-quad)
    float *A_new;
    size_t new_row_stride;
    int ld_new;
    int m;                   // live size after the flush of every row that still has steps to do
    int d, R;
    int strips;              // of 128 rows
    int keep;                // the new matrices stay in the caches
    int chunks;              // groups of K vectors that this flush applies (one panel each, or half of one above 72 steps)
    BlockedWs ws;
};

typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
constexpr unsigned kBufWord3 = 0x00020000u;   // raw buffer, 32-bit data format
constexpr int kFar = 0x40000000;              // byte offset beyond any matrix: "out of range"
// Cache policy bits of the matrix accesses (gfx950 buffer instructions: 1 = sc0, 2 = nt, 16 = sc1).
// The new matrix is written once and next read by another kernel: streaming stores keep it from
// displacing the vectors and the old matrix's lines in L2.
constexpr int kMatStorePolicy = 2 | 16;

// The stores go through the caches where all rows' new matrices together fit the 256 MB memory-side cache, in which the
// next panels find the rows that they fetch; larger ones only displace what is of use.  In us, with no limit, 640 MB, 256 MB
// and none through the caches: 64 x 576 2:4 459, 459, 459, 469; 203 x 1283 at 8 bit 4490, 4485, 4410, 4425; 768 x 768 pruned
// 3882, 3776, 3733, 3742; 256 x 2304 at 4 bit 22483, 21861, 21826, 21807; 64 x 3072 pruned 20227, 19720, 19615, 19653.
constexpr double kKeepBytes = 256e6;

// x[v] = x[v + 1] from Z on
template <int Z, int N>
__device__ __forceinline__ void close_from(float (&x)[N])
{
#pragma unroll
    for (int v = Z; v + 1 < N; ++v) x[v] = x[v + 1];
}

// the same from z on (uniform), by a branch to the group of four that z lies in; z is in groups LO .. HI - 1
template <int LO, int HI, int N>
__device__ __forceinline__ void close_gap(float (&x)[N], int z)
{
    if constexpr (HI - LO == 1) {
#pragma unroll
        for (int v = LO * 4; v < LO * 4 + 4; ++v)
            if (v + 1 < N) x[v] = v >= z ? x[v + 1] : x[v];
        if constexpr (LO * 4 + 4 < N) close_from<LO * 4 + 4, N>(x);
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (z < MID * 4) close_gap<LO, MID>(x, z);
        else close_gap<MID, HI>(x, z);
    }
}

// value of position P of the caller's 16-lane row
template <int P>
__device__ __forceinline__ float row16_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + P, 0xf, 0xf, false));
}

// A_new = compact(A_old - U diag(1/a) U^T) on the lower triangle, K vectors at a time from zero and `chunks` such
// groups (<= J) one after the other.  Every row that still has steps to do has exactly K x chunks deferred
// eliminations and the same live size (a row with fewer has finished and is skipped).
//
// A wave forms a tile of 32 rows x 64 columns by itself: no LDS, no barrier; the four waves of a workgroup take
// 128 rows of the same columns.  The product runs on v_mfma_f32_4x4x1 with one operand broadcast: its 16 blocks
// are 64 columns, one per lane, and the same four rows, so that a lane holds a column of the tile and the registers
// its rows.  What a row needs is then uniform over the wave: where it lay in the old matrix is a scalar, and the
// old matrix is read whole quads of rows at a time (16 bytes a lane, 1 KB a load) although the rows of a new quad
// lie in two or three old ones -- the eliminated rows are closed up in registers (QUADS).  (With 32x32x2 the two
// halves of a wave hold different rows; there the same entries were read singly, four loads over the same lines.)
// An operand is read 16 bytes at a time as well: four vectors of a column (U's layout).
//
// What bounds it: HBM (8 bytes per entry of the new triangle; without any product and operand the same loads and stores
// take 0.72 .. 0.8 of its time) and, not quite overlapped at four waves a SIMD, the matrix cores and the waves' start: some
// 4 us up to a tile's first entries, of 12 in all.  In us, by strips (the form of flush_first_kernel) and by tiles: 256 rows,
// 2208 columns left, 48 vectors 1285, 1115; 880, 64 vectors 234, 218; 3072 rows, 672, 48 vectors 1590, 1390; 64 rows, 384, 64
// vectors 29, 19; 256 rows, 2880, 2 x 40 vectors 2660, 2305.  Several tiles a wave are slower: each store then stands in
// front of the next tile's operands, whose wait is one for the store (1115 -> 1400).
template <int K, int J, bool QUADS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void flush_kernel(FlushArgs a)
{
    static_assert(K % 4 == 0 && K * J <= UCAP, "vectors come in groups of four");
    constexpr int NG = (K + 7) / 8;             // groups of 8 vectors (the last may be one of 4)
    constexpr int NB = J > 1 ? 2 : 3;           // groups in flight
    constexpr int NQ = 10;                      // quads of old rows that 32 rows may reach into
    constexpr int ND = (K + 31) / 32;
    // Workgroups are dealt round-robin to the 8 XCDs: all tiles of one row of the layer stay on one XCD, whose L2
    // holds its vectors.
    const int L = blockIdx.x, xcd = L & 7;
    const int per_row = a.strips * (a.strips + 1);
    const int ri = (L >> 3) / per_row, t = (L >> 3) - ri * per_row, row = ri * 8 + xcd;
    if (row >= a.R) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // strip s has 2 (s + 1) column tiles
    int strip = (int)((__builtin_sqrtf(4.f * t + 1.f) - 1.f) * 0.5f);
    if ((strip + 1) * (strip + 2) <= t) ++strip;
    if (strip * (strip + 1) > t) --strip;
    strip = __builtin_amdgcn_readfirstlane(strip);
    const int mn = a.m;
    const int r0 = strip * 128 + wave * 32, c0 = (t - strip * (strip + 1)) * 64;
    if (r0 >= mn || c0 > r0) return;
    const int nb = a.ws.nb[row], done = a.ws.done[row], total = a.ws.total[row];   // (waited for below)

    const int d = a.d, ldu = a.ws.ldu, ldo = a.ld_old, ldn = a.ld_new, swz = a.old_swz;
    __amdgpu_buffer_rsrc_t rmap = __builtin_amdgcn_make_buffer_rsrc((void *)(a.ws.map + (size_t)row * d), 0, mn * 4, kBufWord3);
    __amdgpu_buffer_rsrc_t ru = __builtin_amdgcn_make_buffer_rsrc((void *)(a.ws.U + (size_t)row * UCAP * ldu), 0,
                                                                  UCAP * ldu * 4, kBufWord3);
    __amdgpu_buffer_rsrc_t rinv = __builtin_amdgcn_make_buffer_rsrc((void *)(a.ws.invd + (size_t)row * UCAP), 0, UCAP * 4, kBufWord3);
    const int il = lane & 31, kl = lane >> 5;
    const int nr = mn - r0 < 32 ? mn - r0 : 32;          // rows of the tile
    const int jcol = c0 + lane;
    // lane l: old index of row l % 32, of column l (beyond the end 0)
    const int orow = __builtin_amdgcn_raw_buffer_load_b32(rmap, (r0 + il) * 4, 0, 0);
    const int jold = __builtin_amdgcn_raw_buffer_load_b32(rmap, jcol * 4, 0, 0);
    // -1 / a of the vectors: register q, position 4 g + i of a 16-lane row: vector 32 q + 8 g + i (upper lanes: + 4)
    float ninv[J][ND];
#pragma unroll
    for (int ch = 0; ch < J; ++ch)
#pragma unroll
        for (int q = 0; q < ND; ++q) {
            const int k = ch * K + 32 * q + 8 * ((lane & 15) >> 2) + (lane & 3) + 4 * kl;
            ninv[ch][q] = -__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rinv, k * 4, 0, 0));
        }
    // the operands of 8 vectors: rows (lower lanes the first four vectors, upper lanes the others), columns
    const int va = (kl * ldu + r0 + il) * 16, vb = jcol * 16, step = ldu * 16;
    uintx4 ua[NB], ub[NB][2];
    int at = 0;
    auto fetch = [&](int gg) {
        asm volatile("" : "+s"(at));                      // (a running offset; and not ahead of what stands before it)
        const int b = gg % NB;
        const bool half = K % 8 && gg % NG == NG - 1;
        ua[b] = __builtin_amdgcn_raw_buffer_load_b128(ru, va, at, 0);
        ub[b][0] = __builtin_amdgcn_raw_buffer_load_b128(ru, vb, at, 0);
        if (!half) ub[b][1] = __builtin_amdgcn_raw_buffer_load_b128(ru, vb, at + step, 0);
        at += half ? step : 2 * step;
    };
#pragma unroll
    for (int g = 0; g < NB && g < NG * J; ++g) fetch(g);
    __builtin_amdgcn_sched_barrier(0);
    const int chunks = J == 1 ? 1 : a.chunks;
    if (nb != K * chunks || done >= total) return;

    // ---- the old entries
    __amdgpu_buffer_rsrc_t rold = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(a.A_old + (size_t)row * a.old_row_stride), 0, swz ? (d + 3) / 4 * d * 16 : d * d * 4, kBufWord3);
    constexpr int NX = QUADS ? NQ * 4 : 32;
    float x[NX];
    const int o_first = __builtin_amdgcn_readfirstlane(orow), o_last = __builtin_amdgcn_readlane(orow, nr - 1);
    const int quad0 = o_first >> 2;
    const bool fits = QUADS && o_last - quad0 * 4 < NQ * 4;
    const int colo = jcol < mn ? jold * (QUADS || swz ? 16 : 4) : kFar;
    // row by row: from the plain layout whole lines, from the quads 4 of every 16 bytes
    auto rows_singly = [&](int om) {
#pragma unroll
        for (int v = 0; v < 32; ++v) {
            const int o = __builtin_amdgcn_readlane(om, v), lim = v < nr ? o : -1;     // columns up to the diagonal
            const int ro = QUADS || swz ? ((o >> 2) * ldo * 4 + (o & 3)) * 4 : o * ldo * 4;
            x[v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rold, jold > lim ? kFar : colo, ro, 0));
            if (v % 4 == 3) __builtin_amdgcn_sched_barrier(0);     // (their offsets do not all fit the scalar registers)
        }
    };
    if constexpr (QUADS) {
        // (a column's quads from the one with its diagonal entry on; no branches, which would hold up the loads)
        const int lo = (jold >> 2) - quad0;
        int n = (fits ? (o_last >> 2) - quad0 + 1 : 0) - lo;
        n = n < 0 ? 0 : n;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int off = (unsigned)(q - lo) < (unsigned)n ? colo : kFar;
            const uintx4 v = __builtin_amdgcn_raw_buffer_load_b128(rold, off, (quad0 + q) * ldo * 16, 0);
            x[4 * q] = __uint_as_float(v.x); x[4 * q + 1] = __uint_as_float(v.y);
            x[4 * q + 2] = __uint_as_float(v.z); x[4 * q + 3] = __uint_as_float(v.w);
        }
    } else {
        rows_singly(orow);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- The update is summed on the matrix cores into accumulators that start at zero while the old entries are on
    // their way, and added to them once per group: an entry takes one rounding per group at its own magnitude, and the
    // matrix comes out as if each group had been flushed by itself.  A group is a panel that shares the flush, or half
    // of a panel of 80.
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    floatx4 sum[8];
    // (Several groups of vectors, where the matrix cores are the tighter bound: the wave in the higher slot of a SIMD
    // goes first, so that the four do not all wait and all multiply together.  3072 x 768, 320 columns left, 2 x 40
    // vectors: 573 -> 548 us; 256 x 4608, 3816 left, 3 x 28: 4228 -> 4134.  One group of 48 or more: 1 % slower.)
    if constexpr (J > 1) {
        switch (__builtin_amdgcn_s_getreg(6148) & 3) {     // HW_ID, bits 0 .. 3: the wave's slot
        case 0: __builtin_amdgcn_s_setprio(0); break;
        case 1: __builtin_amdgcn_s_setprio(1); break;
        case 2: __builtin_amdgcn_s_setprio(2); break;
        default: __builtin_amdgcn_s_setprio(3); break;
        }
    }
#pragma unroll
    for (int ch = 0; ch < J; ++ch) {
        if (J > 1 && ch >= chunks) break;
#pragma unroll
        for (int q = 0; q < 8; ++q) sum[q] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int gg = ch * NG + g, b = gg % NB;
            const bool half = K % 8 && g == NG - 1;
            const float inv = ninv[ch][g / 4];
            const float s0 = g % 4 == 0 ? row16_bcast<0>(inv) : g % 4 == 1 ? row16_bcast<4>(inv) : g % 4 == 2 ? row16_bcast<8>(inv) : row16_bcast<12>(inv);
            const float s1 = g % 4 == 0 ? row16_bcast<1>(inv) : g % 4 == 1 ? row16_bcast<5>(inv) : g % 4 == 2 ? row16_bcast<9>(inv) : row16_bcast<13>(inv);
            const float s2 = g % 4 == 0 ? row16_bcast<2>(inv) : g % 4 == 1 ? row16_bcast<6>(inv) : g % 4 == 2 ? row16_bcast<10>(inv) : row16_bcast<14>(inv);
            const float s3 = g % 4 == 0 ? row16_bcast<3>(inv) : g % 4 == 1 ? row16_bcast<7>(inv) : g % 4 == 2 ? row16_bcast<11>(inv) : row16_bcast<15>(inv);
            const float fa[4] = {__fmul_rn(__uint_as_float(ua[b].x), s0), __fmul_rn(__uint_as_float(ua[b].y), s1),
                                 __fmul_rn(__uint_as_float(ua[b].z), s2), __fmul_rn(__uint_as_float(ua[b].w), s3)};
            // block q + 8 h of the first operand: rows 4 q .. of vector 4 h + i
#define OBC_MF(q, h) sum[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(fa[i], __uint_as_float(ub[b][h][i]), sum[q], 4, (q) + 8 * (h), 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                OBC_MF(0, 0) OBC_MF(1, 0) OBC_MF(2, 0) OBC_MF(3, 0) OBC_MF(4, 0) OBC_MF(5, 0) OBC_MF(6, 0) OBC_MF(7, 0)
            }
            if (!half) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    OBC_MF(0, 1) OBC_MF(1, 1) OBC_MF(2, 1) OBC_MF(3, 1) OBC_MF(4, 1) OBC_MF(5, 1) OBC_MF(6, 1) OBC_MF(7, 1)
                }
            }
#undef OBC_MF
            // (the products stay in front of the next loads, whose operands would otherwise all be in flight at once)
            asm volatile("" : "+v"(sum[0]), "+v"(sum[1]), "+v"(sum[2]), "+v"(sum[3]), "+v"(sum[4]), "+v"(sum[5]),
                         "+v"(sum[6]), "+v"(sum[7]));
            if (gg + NB < NG * J) fetch(gg + NB);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (QUADS && ch == 0) {
            // the tile's 32 rows to the front: over the first quad's earlier rows, then over the rows that were
            // eliminated behind row v
            if (o_first & 1) close_from<0, NX>(x);
            if (o_first & 2) {
#pragma unroll
                for (int v = 0; v + 2 < NX; ++v) x[v] = x[v + 2];
            }
            const int below = __builtin_amdgcn_update_dpp(0, orow, 0x130, 0xf, 0xf, false);   // wave_shl:1, of all lanes
            const int gap = below - orow - 1;
            unsigned long long gaps = fits ? __ballot(gap > 0 && lane + 1 < nr) : 0ull;
            while (gaps) {
                const int v = __builtin_ctzll(gaps);
                int n = __builtin_amdgcn_readlane(gap, v);
                do close_gap<0, 8>(x, v + 1); while (--n > 0);
                gaps &= gaps - 1;
            }
            if (!fits) {
                int om = orow;
                asm volatile("" : "+v"(om));              // (nothing of this is formed ahead)
                rows_singly(om);
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) x[4 * q + i] = __fadd_rn(x[4 * q + i], sum[q][i]);
    }

    // ---- store: four consecutive rows of a column = one 16-byte slot of the row-quad layout (slots wholly above the
    // diagonal are left out)
    __amdgpu_buffer_rsrc_t rnew = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(a.A_new + (size_t)row * a.new_row_stride), 0, ((mn + 3) >> 2) * ldn * 16, kBufWord3);
    const int coln = jcol < mn ? jcol * 16 : kFar;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int off = jcol > r0 + 4 * q + 3 ? kFar : coln, qo = (r0 / 4 + q) * ldn * 16;
        const uintx4 v = {__float_as_uint(x[4 * q]), __float_as_uint(x[4 * q + 1]), __float_as_uint(x[4 * q + 2]),
                          __float_as_uint(x[4 * q + 3])};
        if (a.keep) __builtin_amdgcn_raw_buffer_store_b128(v, rnew, off, qo, 0);
        else __builtin_amdgcn_raw_buffer_store_b128(v, rnew, off, qo, kMatStorePolicy);
    }
}

// The first flush of a call where there is enough of it (kStripEntries): all rows read the same plain H^-1, so that only the
// new matrices have to cross HBM and what tiles read from the caches weighs more -- with 48 vectors a 32 x 64 tile reads 2.2
// bytes of them per byte that it stores, and H^-1 past L2 once per row (256 x 2304: 2.8 GB, in strips of 16 rows at a time 0.65).
// So a workgroup of eight waves keeps them in LDS: it takes a strip of HALVES x 128 rows of one row's matrix, whose
// F = -u / a it holds throughout, and walks its column blocks of 128, whose vectors serve all its halves.  Wave (wm, wn)
// owns 64 x 32 entries of a 128 x 128 tile: two 32x32x2 accumulators, one sum per group of K vectors as in flush_kernel,
// the same bits.  The old entries come as whole lines (32 columns of a row per half wave), before the tile's products.
constexpr int FT = 128;        // tile edge
template <int K, int HALVES, int J>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4, 4))) void flush_first_kernel(FlushArgs a)
{
    constexpr int SR = HALVES * FT;            // rows per strip
    static_assert(K % 4 == 0 && K * J <= UCAP && (J == 1 || HALVES == 1), "a strip's vectors change within a tile");
    __shared__ __align__(16) float Fs[J * K][SR + 4];
    __shared__ __align__(16) float Us[K][FT + 4];
    __shared__ unsigned rowoff_s[SR];          // byte offset of each strip row in H^-1

    // All strips of one row on one XCD; there the rows go in groups of G, a group strip by strip, the longest first:
    // long strips start first, and workgroups that start together take equally long and read the same rows of H^-1.
    const int L = blockIdx.x;
    const int strips = (a.m + SR - 1) / SR;
    const int nx = gridDim.x / (8 * strips);              // rows per XCD
    constexpr int G = 16;
    const int grp = (L / 8) / (G * strips), within = (L / 8) - grp * G * strips;
    const int rig = nx - G * grp < G ? nx - G * grp : G;  // rows in this group
    const int strip = strips - 1 - within / rig;
    const int row = (G * grp + within % rig) * 8 + (L % 8);
    if (row >= a.R) return;
    const int chunks = J == 1 ? 1 : a.chunks;
    if (a.ws.nb[row] != K * chunks || a.ws.done[row] >= a.ws.total[row]) return;
    const int d = a.d, mn = a.m, i0 = strip * SR;
    const int *map = a.ws.map + (size_t)row * d;
    const int ldu = a.ws.ldu, ldn = a.ld_new;
    const float *U = a.ws.U + (size_t)row * UCAP * ldu;
    const float *invd = a.ws.invd + (size_t)row * UCAP;
    __amdgpu_buffer_rsrc_t rold = __builtin_amdgcn_make_buffer_rsrc((void *)a.A_old, 0, d * d * 4, kBufWord3);
    __amdgpu_buffer_rsrc_t rnew = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(a.A_new + (size_t)row * a.new_row_stride), 0, ((mn + 3) >> 2) * ldn * 16, kBufWord3);
    const int tid = threadIdx.x, lane = tid & 63, kl = lane >> 5, il = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (waves with the same wn share a SIMD and have the more work in a diagonal tile the smaller wn is;
    // odd strips number them the other way round, so that two workgroups on a CU even that out)
    const int wm = wave >> 2, wn = (strip & 1) ? 3 - (wave & 3) : wave & 3;
    const int jl = wn * 32 + il;

    for (int idx = tid; idx < K * chunks / 4 * SR; idx += 512) {
        const int k = idx / SR * 4, i = idx % SR;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (i0 + i < mn) v = *reinterpret_cast<const float4 *>(U + u_index(k, i0 + i, ldu));
        Fs[k][i] = __fmul_rn(v.x, -invd[k]);
        Fs[k + 1][i] = __fmul_rn(v.y, -invd[k + 1]);
        Fs[k + 2][i] = __fmul_rn(v.z, -invd[k + 2]);
        Fs[k + 3][i] = __fmul_rn(v.w, -invd[k + 3]);
    }
    for (int i = tid; i < SR; i += 512) rowoff_s[i] = (i0 + i < mn) ? (unsigned)(map[i0 + i] * d) * 4u : (unsigned)kFar;

    // a column block's vectors: four of a column (16 bytes) each, in registers until everyone is done with the last
    constexpr int UV = (K / 4 * FT + 511) / 512;
    float4 ureg[UV];
    auto fetch_u = [&](int j0, int chunk) {
#pragma unroll
        for (int h = 0; h < UV; ++h) {
            const int idx = tid + h * 512, k = idx / FT * 4, j = j0 + idx % FT;
            ureg[h] = (k < K && j < mn) ? *reinterpret_cast<const float4 *>(U + u_index(chunk * K + k, j, ldu))
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    auto stash_u = [&]() {
#pragma unroll
        for (int h = 0; h < UV; ++h) {
            const int idx = tid + h * 512, k = idx / FT * 4, j = idx % FT;
            if (k < K) {
                Us[k][j] = ureg[h].x;
                Us[k + 1][j] = ureg[h].y;
                Us[k + 2][j] = ureg[h].z;
                Us[k + 3][j] = ureg[h].w;
            }
        }
    };
    auto old_col = [&](int j) { return j < mn ? (unsigned)map[j] * 4u : (unsigned)kFar; };
    // halves of the strip that hold rows at all
    const int nh = (mn - i0 + FT - 1) / FT < HALVES ? (mn - i0 + FT - 1) / FT : HALVES;
    // the next tile: column blocks in order, and in each the halves whose rows reach down to it; false after the last
    auto advance = [&](int &j0, int &hf) {
        if (hf + 1 < nh) { hf += 1; return true; }
        j0 += FT;
        if (j0 >= mn) return false;
        hf = j0 <= i0 ? 0 : (j0 - i0) / FT;
        return hf < nh;
    };

    int j0 = 0, hf = 0;
    unsigned colo = old_col(jl);
    fetch_u(0, 0);
    stash_u();
    __syncthreads();                           // Us, Fs and rowoff_s visible
    for (;;) {
        const int rb = hf * FT + wm * 64;      // the wave's first strip row
        // a 32 x 32 piece that lies above the diagonal or beyond the matrix has nothing to add
        bool need[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
            need[mt] = j0 + wn * 32 < mn && i0 + rb + mt * 32 < mn && j0 + wn * 32 <= i0 + rb + mt * 32 + 31;
        // the old entries (those above the diagonal of a piece that it crosses only reach slots that nobody reads)
        floatx16 old[2], sum[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
            const unsigned co = need[mt] ? colo : (unsigned)kFar;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                old[mt][v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                    rold, (int)(rowoff_s[rb + mt * 32 + 8 * (v >> 2) + 4 * kl + (v & 3)] + co), 0, 0));
        }
        int j0n = j0, hfn = hf;
        const bool more = advance(j0n, hfn), new_col = more && j0n != j0;
        unsigned colon = colo;
        if (new_col) {
            if (J == 1) fetch_u(j0n, 0);
            colon = old_col(j0n + jl);
        }
        for (int ch = 0; ch < chunks; ++ch) {
            if (J > 1 && ch > 0) {
                __syncthreads();               // everyone is done reading Us
                stash_u();
                __syncthreads();
            }
            if (J > 1) {
                if (ch + 1 < chunks) fetch_u(j0, ch + 1);
                else if (new_col) fetch_u(j0n, 0);
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) { sum[0][v] = 0.f; sum[1][v] = 0.f; }
            auto mma = [&](auto both, int mt0) {
#pragma unroll
                for (int kk = 0; kk < K; kk += 2) {
                    const int kf = J == 1 ? kk + kl : ch * K + kk + kl;
                    const float b0 = Us[kk + kl][jl];
                    if constexpr (both) {
                        sum[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(Fs[kf][rb + il], b0, sum[0], 0, 0, 0);
                        sum[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(Fs[kf][rb + 32 + il], b0, sum[1], 0, 0, 0);
                    } else if (mt0) {
                        sum[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(Fs[kf][rb + 32 + il], b0, sum[1], 0, 0, 0);
                    } else {
                        sum[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(Fs[kf][rb + il], b0, sum[0], 0, 0, 0);
                    }
                }
            };
            if (need[0] && need[1]) mma(std::true_type{}, 0);
            else if (need[0]) mma(std::false_type{}, 0);
            else if (need[1]) mma(std::false_type{}, 1);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                old[0][v] = __fadd_rn(old[0][v], sum[0][v]);
                old[1][v] = __fadd_rn(old[1][v], sum[1][v]);
            }
        }
        // ---- store: registers 4q .. 4q+3 are four consecutive rows of the lane's column, one slot of the row-quad layout
        const int jcol = j0 + jl, colB = jcol < mn ? jcol * 16 : kFar;
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int qrow = i0 + rb + mt * 32 + 8 * q + 4 * kl;
                const int off = jcol > qrow + 3 ? kFar : (qrow >> 2) * ldn * 16 + colB;
                const uintx4 v = {__float_as_uint(old[mt][4 * q]), __float_as_uint(old[mt][4 * q + 1]),
                                  __float_as_uint(old[mt][4 * q + 2]), __float_as_uint(old[mt][4 * q + 3])};
                if (a.keep) __builtin_amdgcn_raw_buffer_store_b128(v, rnew, off, 0, 0);
                else __builtin_amdgcn_raw_buffer_store_b128(v, rnew, off, 0, kMatStorePolicy);
            }
        if (!more) break;
        if (new_col) {
            __syncthreads();                   // everyone is done reading Us
            stash_u();
            __syncthreads();                   // the new Us visible
        }
        j0 = j0n;
        hf = hfn;
        colo = colon;
    }
}

// ------------------------------------------------------------------------------------- host side
struct Variant {
    int cap;   // largest live size it handles (T * EPT)
    int B;     // steps per panel
    PanelLaunch *launch;
    PanelLaunch *launch_block;       // block pruning (null: never asked for)
    // panels that follow others of their outer block: one flush applies the eliminations of up to J
    int J;
    PanelLaunch *launch_old;
    PanelLaunch *launch_block_old;   // null: block pruning flushes after every panel
};

#define OBC_VARIANT(T, EPT, BR, BL)                                              \
    (T) * (EPT), (BR) + (BL), launch_panel_##T##_##EPT##_##BR##_##BL,            \
        launch_panel_block_##T##_##EPT##_##BR##_##BL

// (512 x 3: 24 vectors in LDS, 72 steps -- 203 x 1283 at 8 bit 5.10 -> 4.93 ms, 256 x 2304 at 4 bit 23.4 -> 23.1 against
// 16 and 64.  The number of steps fixes where the matrix's deferred fp32 sums are cut: with another one the results
// differ by their rounding, and candidates that are closer than that go in another order.)
constexpr Variant kVariants[] = {
    {OBC_VARIANT(256, 1, 64, 0)},
    {OBC_VARIANT(1024, 1, 64, 0)},
    {OBC_VARIANT(512, 3, 48, 24)},
    {OBC_VARIANT(512, 4, 40, 16)},
    {OBC_VARIANT(768, 3, 32, 16)},
    {OBC_VARIANT(512, 6, 28, 12), 2, launch_panel_old_512_6_28_12, nullptr},
    {OBC_VARIANT(512, 8, 20, 8), 3, launch_panel_512_8_20_8, launch_panel_block_512_8_20_8},
    {OBC_VARIANT(512, 9, 16, 8), 4, launch_panel_512_9_16_8, launch_panel_block_512_9_16_8},
};
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);

// Three of these fit on one CU (registers and LDS), two where a thread owns one index; with several times more
// rows than CUs that hides a row's latency behind the steps of two others.  So from past two full rounds of the wider ones
// on, pruning with less than three rows per CU only above 352 columns (below, one workgroup is done before three fill a
// CU).  In us, with 1024 x 1 and with these: 513 x 512 pruned 1304, 1263, at 4 bit 1399, 1246; 700 x 768 3853, 3543 and 3942,
// 3534; 3072 x 768 15453, 14537 and 16075, 14691; left out: 512 x 768 2775, 2825; 700 x 300 pruned 534, 550.  A last round of
// few rows loses: 1024 x 512 pruned 1928, 2133.
// With two owned indices the same registers and LDS hold 80 steps.
// Block pruning never takes them: its state does not fit beside them (83 registers in scratch memory at 256 x 3), and the
// steps of 1024 x 1, which are not a loop, are the faster ones at every width and row count: 768 x 260 497 against 531 us,
// 3072 x 400 3.86, 4.24 ms; 1536 x 512 2.92, 4.14; 768 x 768 3.99, 5.16; 3072 x 768 15.3, 18.9.
constexpr Variant kSharedCuVariants[] = {
    {512, 80, launch_panel_256_2_56_24, nullptr},
    {768, 48, launch_panel_256_3_32_16, nullptr},
};
constexpr int kSharedCuMinRows = 513;

// A flush applies K vectors at once, or several groups of K one after the other: as many as there is an instance for
// (0: none).
constexpr int flush_groups(int K)
{
    return K == 24 ? 4 : K == 28 ? 3 : K == 40 ? 2 : K == 48 || K == 56 || K == 64 || K == 72 ? 1 : 0;
}
// ... and panels of more than 72 vectors go as two groups
constexpr int flush_split(int B) { return B > 72 ? 2 : 1; }
// The least live size over a group's vectors at which a flush reads whole quads of the old matrix; below, too many tiles'
// rows lie in more than ten of them.  In us, single rows and quads, 64 vectors: 256 rows, 560 columns left 118, 111; 368 52.2,
// 52.6; 240 30.5, 31.2; 203 rows, 547 100, 92; 291 36, 39; 3072 rows, 176 201, 211; 2 x 40 vectors, 320 607, 573; 240 361, 342.
constexpr int kQuadsMinRatio = 6;

// Entries of all rows' new matrices from which the first flush goes by strips (flush_first_kernel); fewer do not give the
// CUs enough of its long workgroups.  Calls of one flush and one step after it, in us, by tiles and by strips: 256 x 2304 1254,
// 1109; 512 x 2304 2577, 2243; 256 x 2048 1113, 1030; 256 x 1536 790, 778; 3072 x 768 2172, 1991; 768 x 3072 12061, 10911; 256 x
// 4608 10278, 9431; blocks 256 x 3072 2097, 1778; at 510 .. 550 million entries 128 x 2048 652, 637; 1024 x 768 695, 667; below
// 64 x 2304 475, 492; 203 x 1283 514, 529; 32 x 4000 1809, 1821; 8 x 2304 264, 377 (but 64 x 2760 603, 591).
constexpr double kStripEntries = 5e8;

// what a flush reads has room in U and an instance of the kernel, whatever number of panels it serves
constexpr bool flush_serves(const Variant &v)
{
    const int panels = v.J > 1 ? v.J : 1, split = flush_split(v.B);
    return panels * v.B <= UCAP && v.B % split == 0 && panels * split <= flush_groups(v.B / split);
}
constexpr bool flush_serves_all()
{
    for (const Variant &v : kVariants)
        if (!flush_serves(v)) return false;
    for (const Variant &v : kSharedCuVariants)
        if (!flush_serves(v)) return false;
    return BMAX <= UCAP && flush_split(BMAX) == 1 && flush_groups(BMAX) >= 1;
}
static_assert(flush_serves_all(), "a panel's steps, or those of the panels that share a flush, without a flush kernel");

// Floats between two rows' matrices, and between two quads of a matrix with m live columns: multiples of 256 bytes, so that
// a wave's stores are whole lines at any live size.  In ms, with the live size as the distance and, where it was no
// multiple of 4, stores through the caches, and with this: 256 x 2303 at 4 bit 23.36, 21.91; 3071 x 765 at 4 bit 15.53, 14.81;
// 768 x 767 pruned 5.01, 4.78; 203 x 1283 at 8 bit 4.62, 4.51; 203 x 1999 pruned 17.08, 16.72; 40 x 4095 44.0, 43.0; 64 x 577
// 1.200, 1.187; aligned 256 x 2304 at 4 bit 21.84, 21.83.
constexpr size_t matrix_stride(int d) { return (size_t)d * d / 64 * 64; }
constexpr int quad_ld(int m) { return (m + 15) / 16 * 16; }

// The first flush leaves the largest matrix; the padded distances have to leave it within its row's share of what was
// laid out, d * d floats.
constexpr bool matrix_fits(int d, int steps)
{
    const int m = d - steps;
    return m <= 0 || (size_t)(m + 3) / 4 * 4 * quad_ld(m) <= matrix_stride(d);
}
constexpr bool matrices_fit()
{
    int fewest = BMAX;
    for (const Variant &v : kVariants) fewest = v.B < fewest ? v.B : fewest;
    for (const Variant &v : kSharedCuVariants) fewest = v.B < fewest ? v.B : fewest;
    for (int d = BMAX + 1; d <= kVariants[kNumVariants - 1].cap; ++d)
        if (!matrix_fits(d, fewest)) return false;
    return true;
}
static_assert(matrices_fit(), "a flush that eliminates too little for the padded matrix it leaves");

// Panels of 80 steps where they reach 256 live columns, from which on a thread owns one index, in fewer panels than
// those of 48 do; where both take as many (273..304 and 337..352 columns) the shorter ones leave more of the steps to
// the cheaper variant.  Up to 272 columns 80 steps save one of the panels below 256 instead.  In us, pruned, with 80 and
// with 48 steps: 1024 x 300 798, 727; 3072 x 288 1944, 1753; 1024 x 344 1111, 1030; 1536 x 344 1394, 1366; 3072 x 320 2126,
// 2371; 1536 x 416 1838, 2130; 768 x 264 499, 518; 1536 x 264 802, 864 (but 1024 x 264 653, 641).  Both in turn as the rule has
// it, against 80 throughout: 1536 x 384 1615, 1688; 3072 x 512 5553, 5642; 768 x 512 1582, 1574.
constexpr bool longer_panels(int m) { return m <= 272 || (m - 256 + 79) / 80 < (m - 256 + 47) / 48; }

// How many panels share a flush.  What the flushes save must exceed the re-reading of the earlier panels' vectors.  A
// flush takes the longer the more rows there are and the wider they are; the re-reading stands in each step's chain
// however few they are.  In us, a flush after each panel, after two, three and four:
//   40 a panel, 280 steps: 8 x 3072 1642, 2274; 64 x 3072 4050, 4202; 96 x 3072 5391, 5206; 128 x 2500 4715, 4681; 256 x 2650
//     9511, 8339 (below the best line 96 x 2500 3825, 3984); not with block pruning's larger state, 40 x 3000 18570, 19150
//   24 a panel, 288 steps: 2 x 4400 2850, 3020, 3427, 3884; 24 x 4608 6367, 4806, 4808, 5417; 64 x 4608 12938, 8271, 7918,
//     8292; 256 x 4608 43764, 25196, 22525, 21954; in blocks 4 x 4400 3327, 3606, 4187, 4883; 64 x 4608 13093, 8892, 8915, 9578
//   28 a panel, 336 steps: 192 x 3700 23505, 14943, 14254.  They share three at any row count -- the account of what three
//     such panels read is pinned at two rows -- though fewer are better with few rows: 48 x 3700 7734, 5737, 6338; 8 x 3700
//     3434, 3496, 3932
int shared_panels(const Variant &v, int m, int R)
{
    if (v.J == 2) return m >= 2416 && R >= 96 ? 2 : 1;
    if (v.J == 4) return R >= 96 ? 4 : R >= 64 ? 3 : R > 2 ? 2 : 1;
    return v.J;
}

// `left`: steps that the call has still to do (an upper bound over the rows).  Below 768 rows the shorter panels of three
// rows per CU are not taken where one panel of 64 steps ends the call and they would need a flush and a second one, in us,
// with them and without: 600 x 600, 56 steps 297, 261; 640 x 768, 60 419, 328; 767 x 768, 64 488, 359; 700 x 768, 100 (48 and
// 52) 875, 643.
const Variant *pick_variant(int m, int R, int mode, int left)
{
    const int least = R >= 3 * 256 || mode == MODE_QUANT ? 256 : 352;
    if (R >= kSharedCuMinRows && m > least && mode != MODE_BLOCK)
        for (const Variant &v : kSharedCuVariants)
            if (m <= v.cap && (v.B != 80 || longer_panels(m)) && !(R < 3 * 256 && left > v.B && left <= 64)) return &v;
    for (int i = 0; i < kNumVariants; ++i)
        if (m <= kVariants[i].cap) return &kVariants[i];
    return nullptr;
}

}  // namespace

namespace obc_rows {

int blocked_max_d() { return kVariants[kNumVariants - 1].cap; }

size_t blocked_workspace_bytes(int R, int d) { return carve(nullptr, nullptr, R, d); }

int potrf64_batched_launch(obc_ctx *ctx, double *M, double *T, int R);   // invert.hip

int blocked_launch(obc_ctx *ctx, int mode, const float *W, const float *Hinv, int R, int d, int k_steps,
                   int nm_n, int nm_m, const int32_t *stop_counts, const float *delta,
                   const float *offset, int maxq, const uint8_t *live, int flags, int32_t *order, float *loss,
                   int32_t *codes, float *W_out, float *trace, int out_ld, void *ws, size_t ws_bytes, int need_ws)
{
    if (d > blocked_max_d())
        return obc_fail(ctx, OBC_ERR_BAD_SHAPE, "row solver (blocked): d = %d exceeds the supported %d", d, blocked_max_d());
    BlockedWs bw;
    // One panel is the whole of such a row: no set-up launch, and no workspace (which only a caller who
    // names the strategy is still held to).
    const bool direct = d <= BMAX;
    size_t need = carve(&bw, ws, R, d);
    if ((!ws || ws_bytes < need) && !(direct && need_ws == 0))
        return obc_fail(ctx, OBC_ERR_WORKSPACE, "row solver: workspace of %zu bytes needed, %zu given", need, ws_bytes);
    hipStream_t st = ctx->stream;
    ctx->chain_fresh = false;   // the set-up kernels below are not timed: the first timed launch records its own start

    if (!direct) {
        InitArgs ia;
        ia.W = W; ia.Hinv = Hinv; ia.live_in = live; ia.stop_counts = stop_counts; ia.d = d;
        ia.k_steps = k_steps; ia.mode = mode; ia.ws = bw; ia.codes = codes; ia.W_out = W_out;
        blocked_init_kernel<<<R, 256, 0, st>>>(ia);
        OBC_LAUNCH_CHECK(ctx, "blocked_init_kernel");
    }
    if (trace && k_steps > 0) {
        size_t n = (size_t)R * out_ld * d;
        unsigned blocks = (unsigned)((n / 4 + 256 * 8 - 1) / (256 * 8));
        if (blocks > 65535) blocks = 65535;
        if (blocks == 0) blocks = 1;
        fill_f32_kernel<<<blocks, 256, 0, st>>>(trace, n, 0.f);
        OBC_LAUNCH_CHECK(ctx, "fill_f32_kernel");
    }

    PanelArgs pa;
    pa.d = d; pa.nm_n = nm_n; pa.nm_m = nm_m; pa.delta = delta; pa.offset = offset; pa.maxq = maxq;
    pa.ws = bw; pa.order = order; pa.loss = loss; pa.codes = codes; pa.W_out = W_out; pa.trace = trace;
    pa.out_ld = out_ld; pa.status = ctx->d_status; pa.outliers = (flags & OBC_QUANT_OUTLIERS) ? 1 : 0;
    pa.direct = direct ? 1 : 0; pa.W = W; pa.live_in = live; pa.stop_counts = stop_counts; pa.k_steps = k_steps;
    if (direct) {
        pa.A_cur = Hinv; pa.a_row_stride = 0; pa.ld = d; pa.swz = 0; pa.old = 0; pa.last = 1; pa.threads = BMAX;
        const Variant &v = kVariants[0];
        {
            obc_scope sc(ctx, OBC_KERNEL_PANEL, (double)R * d * 4.0 * d, (double)R * d * (double)d * d);
            if ((mode == MODE_BLOCK ? v.launch_block : v.launch)(mode, R, st, pa) != 0)
                return obc_fail(ctx, OBC_ERR_HIP, "panel kernel: cannot set its dynamic LDS size");
        }
        OBC_LAUNCH_CHECK(ctx, "panel_kernel");
        return OBC_OK;
    }
    FlushArgs fa;
    fa.d = d; fa.R = R; fa.ws = bw;

    int host_total = (mode == MODE_QUANT || live) ? d : k_steps;   // upper bound over the rows
    const size_t mat_stride = matrix_stride(d);
    int host_done = 0;
    int cur = -1;            // -1: the shared H^-1; otherwise index into Abuf
    int ld_cur = d;

    // where the rows' matrices are now, as the kernels take it
    auto cur_matrix = [&](const float **A, size_t *stride, int *swz) {
        *A = (cur < 0) ? Hinv : bw.Abuf[cur];
        *stride = (cur < 0) ? 0 : mat_stride;
        *swz = (cur < 0) ? 0 : 1;
    };
    // rank-K update and compaction of every row's matrix into the other buffer
    auto launch_flush = [&](int K, int chunks) -> int {
        chunks *= flush_split(K);
        K /= flush_split(K);
        const int m_next = d - host_done;
        const int nxt = (cur < 0) ? 0 : 1 - cur;
        int swz;
        cur_matrix(&fa.A_old, &fa.old_row_stride, &swz);
        fa.ld_old = ld_cur;
        fa.old_swz = swz;
        fa.A_new = bw.Abuf[nxt];
        fa.new_row_stride = mat_stride;
        fa.m = m_next;
        fa.ld_new = quad_ld(m_next);
        fa.chunks = chunks;
        fa.keep = (double)R * m_next * m_next * 2.0 <= kKeepBytes;
        fa.strips = (m_next + 127) / 128;
        const int rows8 = (R + 7) / 8 * 8;
        // whole quads of the old matrix where 32 rows nearly always come from ten of them
        const bool quads = swz && m_next >= kQuadsMinRatio * K;
        {
            // one triangle of the surviving m_next x m_next part of every row's inverse is read and
            // written once
            const double tri = 0.5 * (double)m_next * (m_next + 1.0);   // entries of one triangle
            obc_scope sc(ctx, OBC_KERNEL_FLUSH, (double)R * 8.0 * tri, (double)R * 2.0 * K * chunks * tri);
            const dim3 grid(fa.strips * (fa.strips + 1) * rows8);
            const bool strips = cur < 0 && (double)R * m_next * m_next >= kStripEntries;
            auto launch = [&](auto k) {
                constexpr int KK = decltype(k)::value, J = flush_groups(KK);
                constexpr int H = KK <= 48 ? 2 : 1;     // two workgroups' vectors in a CU's LDS
                if (strips && chunks == 1)
                    flush_first_kernel<KK, H, 1><<<(m_next + H * FT - 1) / (H * FT) * rows8, 512, 0, st>>>(fa);
                else if (strips)
                    flush_first_kernel<KK, 1, J><<<fa.strips * rows8, 512, 0, st>>>(fa);
                else if (quads) flush_kernel<KK, J, true><<<grid, 256, 0, st>>>(fa);
                else flush_kernel<KK, J, false><<<grid, 256, 0, st>>>(fa);
            };
            switch (K) {
            case 24: launch(std::integral_constant<int, 24>{}); break;
            case 28: launch(std::integral_constant<int, 28>{}); break;
            case 40: launch(std::integral_constant<int, 40>{}); break;
            case 48: launch(std::integral_constant<int, 48>{}); break;
            case 56: launch(std::integral_constant<int, 56>{}); break;
            case 64: launch(std::integral_constant<int, 64>{}); break;
            case 72: launch(std::integral_constant<int, 72>{}); break;
            default: return obc_fail(ctx, OBC_ERR_BAD_ARG, "row solver: no flush kernel for block size %d", K);
            }
        }
        OBC_LAUNCH_CHECK(ctx, "flush_kernel");
        cur = nxt;
        ld_cur = fa.ld_new;
        return OBC_OK;
    };

    // ---- already-pruned indices, BMAX at a time, as long as every row has that many left.  The
    // smallest count over the rows is read back once (the only wait in this call).
    // (Not at widths that a call without any wait has always served: there the panels do it all.)
    if (live && mode != MODE_BLOCK && d > kNoWaitMaxD) {
        int scal[2] = {0, 0};
        min_ndead_kernel<<<1, 256, 0, st>>>(bw.ndead, bw.total, R, bw.scal);
        OBC_LAUNCH_CHECK(ctx, "min_ndead_kernel");
        OBC_HIP(ctx, hipMemcpyAsync(scal, bw.scal, sizeof(scal), hipMemcpyDeviceToHost, st));
        OBC_HIP(ctx, hipStreamSynchronize(st));
        const int min_dead = scal[0];
        if (scal[1] < host_total) host_total = scal[1];    // no launches past the longest row's last step
        int nfast = min_dead / BMAX;
        if (d - nfast * BMAX < BMAX) nfast -= 1;            // keep a matrix for the flush to write
        DeadArgs da;
        da.d = d; da.ws = bw;
        for (int it = 0; it < nfast; ++it) {
            const int m_max = d - host_done;
            cur_matrix(&da.A_cur, &da.a_row_stride, &da.swz);
            da.ld = ld_cur;
            {
                obc_scope sc(ctx, OBC_KERNEL_PANEL, (double)R * BMAX * 4.0 * m_max,
                             (double)R * BMAX * (double)BMAX * m_max);
                dead_gather_kernel<<<R, 512, 0, st>>>(da);
                OBC_LAUNCH_CHECK(ctx, "dead_gather_kernel");
                int rc = potrf64_batched_launch(ctx, bw.Mb, bw.Tb, R);
                if (rc != OBC_OK) return rc;
                dead_apply_kernel<<<R, 512, 0, st>>>(da);
                OBC_LAUNCH_CHECK(ctx, "dead_apply_kernel");
            }
            host_done += BMAX;
            int rc = launch_flush(BMAX, 1);
            if (rc != OBC_OK) return rc;
        }
    }

    while (host_done < host_total) {
        const int m_max = d - host_done;
        const Variant *v = pick_variant(m_max, R, mode, host_total - host_done);
        int swz;
        cur_matrix(&pa.A_cur, &pa.a_row_stride, &swz);
        pa.ld = ld_cur;
        pa.swz = swz;
        // Panels that share a flush, as long as the live size keeps this variant.  Before the flush the
        // index space keeps its size, and a panel finds the earlier ones' vectors in memory.
        PanelLaunch *first = mode == MODE_BLOCK ? v->launch_block : v->launch;
        PanelLaunch *next = mode == MODE_BLOCK ? v->launch_block_old : v->launch_old;
        const int most = next ? shared_panels(*v, m_max, R) : 1;
        int panels = 1;
        for (int ahead = v->B; panels < most && host_done + ahead < host_total &&
                               pick_variant(m_max - ahead, R, mode, host_total - host_done - ahead) == v; ahead += v->B)
            ++panels;
        for (int j = 0; j < panels; ++j) {
            pa.old = j * v->B;
            pa.last = j == panels - 1;
            pa.threads = (m_max + 63) / 64 * 64;
            {
                // a panel reads one matrix row and the outer block's earlier vectors per step, 4 m bytes each,
                // and does ~B m flops on it
                const int steps = (host_total - host_done < v->B) ? host_total - host_done : v->B;
                obc_scope sc(ctx, OBC_KERNEL_PANEL, (double)R * steps * 4.0 * (1 + pa.old) * m_max,
                             (double)R * steps * (double)(steps + 2 * pa.old) * m_max);
                if ((j == 0 ? first : next)(mode, R, st, pa) != 0)
                    return obc_fail(ctx, OBC_ERR_HIP, "panel kernel: cannot set its dynamic LDS size");
            }
            OBC_LAUNCH_CHECK(ctx, "panel_kernel");
            host_done += v->B;
        }
        if (host_done >= host_total) break;
        int rc = launch_flush(v->B, panels);
        if (rc != OBC_OK) return rc;
    }
    return OBC_OK;
}

}  // namespace obc_rows

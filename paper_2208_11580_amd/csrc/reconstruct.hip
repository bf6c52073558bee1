// obc_reconstruct_rows: the weights of a given mask by the group-OBS closed form (Sec. 4 Step 2 of
// arxiv 2208.11580; the sign as in eq. (5)).  With P the pruned indices of a row,
//
//     w_hat = w - H^-1[:, P] ((H^-1)[P, P])^-1 w_P,        w_hat[P] = 0,
//
// from the ORIGINAL weights and inverse Hessian: no trace and no second run of the greedy loop.  The
// paper names it as the cheaper way to get a row's weights once the global step has fixed how many
// weights the row gives up.
//
// Everything in fp64 (the principal submatrix of H^-1 on half of the indices is as ill-conditioned as
// H^-1 itself, and its fp32 entries are exact inputs), all rows of the layer side by side:
//   1. per row: the list P of its pruned indices and w_P (recon_list_kernel), then G = (H^-1)[P, P]
//      (lower triangle, recon_gather_kernel: a workgroup per 64 of its rows)
//   2. G = L L^T for all rows at once, block column by block column of 64, two launches each (host loop
//      up to the caller's bound on the pruned count; a row that is through skips).  Left-looking: a
//      64 x 64 tile is formed once, from the block columns before it (64-deep slabs, the next one
//      requested while this one is multiplied, two workgroups per CU), so G is read and written once instead of once per block column.  The
//      diagonal tiles' workgroups factor them and invert the factor; the tiles below are multiplied by
//      that inverse before they are stored.
//   3. per row: L y = w_P and L^T z = y block by block with the inverted diagonal factors
//      (recon_solve_kernel), then w_hat = w - H^-1[:, P] z, pruned entries set to 0: for all rows in one
//      product Z H^-1 on the fp64 matrix core, z spread over the row's d columns (up to 640
//      pruned weights, along rows of H^-1 by the row's own workgroup instead: the same sums)
// Bound by the fp64 matrix core (c^3 / 3 flop per row): 768 x 3072 at 50 %, 0.93 TFLOP, in 28.5 ms for
// the factorisation (33 TFLOP/s of the 47 this unit sustains; 43.5 with a right-looking update of all
// of G per block column) and 33.8 ms in all (61.3); 256 x 4608 34 ms (72.5).
#include "dense64.h"

namespace {

using namespace obc_dense64;

struct ReconArgs {
    const float *W, *Hinv;
    const uint8_t *mask;
    int d, cmax, ldg;
    float *W_out;
    double *G;       // R x ldg x ldg
    double *Linv;    // R x (ldg / 64) x 64 x 64
    double *vec;     // R x ldg   (w_P, then z)
    double *Z;       // R x d     z spread over the columns (in G's place, which is through by then), or null
    int R;
    int *idx;        // R x ldg
    int *cnt;        // R     pruned weights of the row (0: nothing to do)
    int *status;
};

// ---- 1. pruned indices (ascending), their count and the right-hand side
__global__ __launch_bounds__(256) void recon_list_kernel(ReconArgs a)
{
    __shared__ int wcnt[4];
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int d = a.d, ldg = a.ldg;
    const float *w = a.W + (size_t)row * d;
    float *wo = a.W_out + (size_t)row * d;
    const uint8_t *mk_row = a.mask + (size_t)row * d;
    int *idx = a.idx + (size_t)row * ldg;
    double *v = a.vec + (size_t)row * ldg;

    int c = 0;                               // (every thread ends with the same count)
    for (int j0 = 0; j0 < d; j0 += 256) {
        const int j = j0 + tid;
        const bool pr = j < d && mk_row[j] != 0;
        const unsigned long long bal = __ballot(pr);
        if (lane == 0) wcnt[wave] = __popcll(bal);
        __syncthreads();
        int before = c, total = 0;
        for (int wv = 0; wv < 4; ++wv) {
            if (wv < wave) before += wcnt[wv];
            total += wcnt[wv];
        }
        const int rank = before + __popcll(bal & ((1ull << lane) - 1ull));
        if (pr && rank < a.cmax) idx[rank] = j;
        c += total;
        __syncthreads();
    }
    for (int j = tid; j < d; j += 256) wo[j] = w[j];
    if (c > a.cmax) {                        // more pruned weights than the workspace was sized for:
        if (tid == 0) {                      // the row stays a copy of W
            obc_latch(a.status, OBC_ERR_WORKSPACE);
            a.cnt[row] = 0;
        }
        return;
    }
    if (tid == 0) a.cnt[row] = c;
    if (c == 0) return;
    __threadfence_block();
    __syncthreads();
    for (int i = tid; i < c; i += 256) v[i] = (double)w[idx[i]];
}

// The tile of a workgroup: `nt` tiles per row, the rows dealt to the 8 XCDs, so that all tiles of a row
// -- they read the same block rows of L -- run on one XCD, one after the other.
__device__ __forceinline__ void recon_tile(int nt, int &row, int &tile)
{
    const int w = blockIdx.x / 8;
    row = w / nt * 8 + blockIdx.x % 8;
    tile = w % nt;
}

// 64 rows of G: each wave takes a row at a time, its lanes the row's entries
__global__ __launch_bounds__(256) void recon_gather_kernel(ReconArgs a, int nt)
{
    int row, tile;
    recon_tile(nt, row, tile);
    if (row >= a.R) return;
    const int c = a.cnt[row], ldg = a.ldg;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int *idx = a.idx + (size_t)row * ldg;
    double *G = a.G + (size_t)row * ldg * ldg;
    for (int i = tile * NB + wave; i < c && i < (tile + 1) * NB; i += 4) {
        const float *hrow = a.Hinv + (size_t)idx[i] * a.d;
#pragma unroll 4
        for (int j = lane; j <= i; j += 64) G[(size_t)i * ldg + j] = (double)hrow[idx[j]];
    }
}

// ---- 2. tile (i0, k0) of block column k0: C = G - sum_{k < k0} L_ik L_jk^T.  DIAG: the diagonal tile,
// which is then factored (the inverse of its factor goes to Linv; the factor itself is not needed
// again).  Else a tile below it: L = C Linv_kk^T.
template <bool DIAG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void recon_column_kernel(ReconArgs a, int k0, int nt)
{
    __shared__ double lds[DIAG ? POTRF_WG_LDS : 2 * NB * PL];
    double *As = lds, *Bs = lds + NB * PL;
    int row, tile = 0;
    if (DIAG) row = blockIdx.x;
    else recon_tile(nt, row, tile);
    if (row >= a.R) return;
    const int c = a.cnt[row], ldg = a.ldg;
    const int i0 = DIAG ? k0 : k0 + NB * (1 + tile);
    if (i0 >= c) return;
    const int Mi = (c - i0 < NB) ? c - i0 : NB, Nj = (c - k0 < NB) ? c - k0 : NB;
    double *G = a.G + (size_t)row * ldg * ldg;
    double *Lk = a.Linv + ((size_t)row * (ldg / NB) + k0 / NB) * NB * NB;
    const double *Li = G + (size_t)i0 * ldg, *Lj = G + (size_t)k0 * ldg;

    doublex4 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = doublex4{0.0, 0.0, 0.0, 0.0};
    double ra[16], rb[16];
    auto fetch = [&](int k) {
        tile_fetch(ra, Li + k, ldg, Mi, NB);
        if (!DIAG) tile_fetch(rb, Lj + k, ldg, Nj, NB);
    };
    if (k0 > 0) fetch(0);
    for (int k = 0; k < k0; k += NB) {
        tile_park<true>(As, ra);
        if (!DIAG) tile_park<true>(Bs, rb);
        __syncthreads();
        if (k + NB < k0) fetch(k + NB);
        tile_mma<true>(acc, As, DIAG ? As : Bs);
        __syncthreads();
    }
    double *C = G + (size_t)i0 * ldg + k0;
    doublex4 old[2][2];
    tile_fill(old, [&](int i, int j) { return (i < Mi && j < Nj && (!DIAG || j <= i)) ? C[(size_t)i * ldg + j] : 0.0; });
    if (DIAG) {
        // the factorisation's LDS layout: lower triangle, identity where the block is padded; the
        // inverse's area cleared
        tile_each2(acc, old, [&](int i, int j, double v, double o) {
            As[i * PL + j] = (i < Mi && j <= i) ? o - v : (i == j ? 1.0 : 0.0);
            Bs[i * PL + j] = 0.0;
        });
        __syncthreads();
        potrf_wg_core(Lk, Mi, a.status, OBC_ERR_NUMERIC, lds);
    } else {
        double rl[16];
        tile_fetch(rl, Lk, NB, NB, NB);
        tile_each2(acc, old, [&](int i, int j, double v, double o) { As[j * PL + i] = o - v; });   // a(i, k) = C[i][k]
        tile_park<true>(Bs, rl);                                                                   // b(k, j) = Linv[j][k]
        __syncthreads();
        tile_mma(acc, As, Bs);
        tile_each(acc, [&](int i, int j, double v) { if (i < Mi && j < Nj) C[(size_t)i * ldg + j] = v; });
    }
}

// ---- 3. L y = w_P, L^T z = y; w_P, y and z in turn in LDS, or in the workspace where they are longer than
// that (IN_LDS false).  Rows of L are read by eight lanes each (64 bytes a lane) on the way down, along
// their entries on the way up.
constexpr int kSolveLdsMax = (160 * 1024 - (NB + 8 * NB) * 8) / 8;   // doubles next to blk and red

template <bool IN_LDS>
__global__ __launch_bounds__(512) void recon_solve_kernel(ReconArgs a)
{
    extern __shared__ double v_lds[];        // ldg
    __shared__ double blk[NB], red[8][NB];
    const int row = blockIdx.x, tid = threadIdx.x;
    const int d = a.d, ldg = a.ldg;
    const int c = a.cnt[row];
    if (c == 0) return;
    const double *G = a.G + (size_t)row * ldg * ldg;
    const double *Li = a.Linv + (size_t)row * (ldg / NB) * NB * NB;
    double *gv = a.vec + (size_t)row * ldg;
    double *v = IN_LDS ? v_lds : gv;
    for (int i = tid; i < ldg; i += 512) v[i] = i < c ? gv[i] : 0.0;
    __syncthreads();
    const int nblk = (c + NB - 1) / NB;
    const int part = tid & 7, slot = tid >> 3;
    for (int kb = 0; kb < nblk; ++kb) {
        const int k0 = kb * NB;
        const double *Lk = Li + (size_t)kb * NB * NB;     // (zeros above the diagonal, identity beyond the row)
        double acc = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) acc = fma(Lk[slot * NB + part * 8 + q], v[k0 + part * 8 + q], acc);
        acc += __shfl_xor(acc, 1, 64);
        acc += __shfl_xor(acc, 2, 64);
        acc += __shfl_xor(acc, 4, 64);
        if (part == 0) blk[slot] = acc;
        __syncthreads();
        if (tid < NB) v[k0 + tid] = blk[tid];
        double b8[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) b8[q] = blk[part * 8 + q];
#pragma unroll 2
        for (int i = k0 + NB + slot; i < c; i += 64) {    // (all eight lanes of a row together)
            const double *gi = G + (size_t)i * ldg + k0 + part * 8;
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) s = fma(gi[q], b8[q], s);
            s += __shfl_xor(s, 1, 64);
            s += __shfl_xor(s, 2, 64);
            s += __shfl_xor(s, 4, 64);
            if (part == 0) v[i] -= s;
        }
        __syncthreads();
    }
    for (int kb = nblk - 1; kb >= 0; --kb) {
        const int k0 = kb * NB;
        const int bs = (c - k0 < NB) ? c - k0 : NB;
        const double *Lk = Li + (size_t)kb * NB * NB;
        const int col = tid & 63, grp = tid >> 6;
        double acc = 0.0;
#pragma unroll
        for (int q = 0; q < 8; ++q) acc = fma(Lk[(grp * 8 + q) * NB + col], v[k0 + grp * 8 + q], acc);
        red[grp][col] = acc;
        __syncthreads();
        if (tid < NB) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) s += red[q][tid];
            blk[tid] = tid < bs ? s : 0.0;
            v[k0 + tid] = blk[tid];
        }
        __syncthreads();
        for (int i = tid; i < k0; i += 512) {
            double s = 0.0;
            if (bs == NB) {
#pragma unroll 16
                for (int r = 0; r < NB; ++r) s = fma(G[(size_t)(k0 + r) * ldg + i], blk[r], s);
            } else {
                for (int r = 0; r < bs; ++r) s = fma(G[(size_t)(k0 + r) * ldg + i], blk[r], s);
            }
            v[i] -= s;
        }
        __syncthreads();
    }
    if (a.Z) {
        if (IN_LDS)
            for (int i = tid; i < c; i += 512) gv[i] = v[i];
        return;
    }
    // (row idx[t] of the symmetric H^-1 is its column idx[t])
    const float *w = a.W + (size_t)row * d;
    float *wo = a.W_out + (size_t)row * d;
    const int *idx = a.idx + (size_t)row * ldg;
    for (int j = tid; j < d; j += 512) {
        double acc = 0.0;
#pragma unroll 8
        for (int t = 0; t < c; ++t) acc = fma((double)a.Hinv[(size_t)idx[t] * d + j], v[t], acc);
        wo[j] = (float)((double)w[j] - acc);
    }
    __syncthreads();
    for (int t = tid; t < c; t += 512) wo[idx[t]] = 0.f;
}

__global__ __launch_bounds__(256) void recon_spread_kernel(ReconArgs a)
{
    const int row = blockIdx.x, c = a.cnt[row];
    double *z = a.Z + (size_t)row * a.d;
    for (int j = threadIdx.x; j < a.d; j += 256) z[j] = 0.0;
    __syncthreads();
    for (int t = threadIdx.x; t < c; t += 256) z[a.idx[(size_t)row * a.ldg + t]] = a.vec[(size_t)row * a.ldg + t];
}

// W_out = W - Z H^-1, pruned entries 0: a 64 x 64 tile per workgroup, slabs as above.  The product meets
// every row of H^-1, also those that a row of W does not use (times the zeros of Z): where it is not finite
// the entry is summed again over the row's own indices, so that an infinity or NaN in H^-1 reaches what it
// is a part of and nothing else.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void recon_product_kernel(ReconArgs a)
{
    __shared__ double lds[2 * NB * PL];
    double *As = lds, *Bs = lds + NB * PL;
    const int i0 = blockIdx.y * NB, j0 = blockIdx.x * NB, d = a.d;
    const int Mi = (a.R - i0 < NB) ? a.R - i0 : NB, Nj = (d - j0 < NB) ? d - j0 : NB;
    doublex4 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = doublex4{0.0, 0.0, 0.0, 0.0};
    double ra[16];
    float rb[16];
    auto fetch = [&](int k) {
        const int kr = (d - k < NB) ? d - k : NB;
        tile_fetch(ra, a.Z + (size_t)i0 * d + k, d, Mi, kr);          // (i, k)
#pragma unroll
        for (int h = 0; h < 16; ++h) {                                // (k, j)
            const int e = threadIdx.x + h * 256;
            rb[h] = ((e >> 6) < kr && (e & 63) < Nj) ? a.Hinv[(size_t)(k + (e >> 6)) * d + j0 + (e & 63)] : 0.f;
        }
    };
    fetch(0);
    for (int k = 0; k < d; k += NB) {
        tile_park<true>(As, ra);
#pragma unroll
        for (int h = 0; h < 16; ++h) {
            const int e = threadIdx.x + h * 256;
            Bs[(e >> 6) * PL + (e & 63)] = (double)rb[h];
        }
        __syncthreads();
        if (k + NB < d) fetch(k + NB);
        tile_mma<true>(acc, As, Bs);
        __syncthreads();
    }
    auto store = [&](int i, int j, double v) {
        const size_t e = (size_t)(i0 + i) * d + j0 + j;
        const bool off = a.mask[e] != 0 && a.cnt[i0 + i] > 0;
        a.W_out[e] = off ? 0.f : (float)((double)a.W[e] - v);
    };
    unsigned again = 0;                      // of the thread's 16 entries
    int n = 0;
    tile_each(acc, [&](int i, int j, double v) {
        if (i < Mi && j < Nj) {
            if (fabs(v) < __builtin_inf()) store(i, j, v);
            else again |= 1u << n;
        }
        ++n;
    });
#pragma unroll 1
    for (; again != 0; again &= again - 1) {
        int i = 0, j = 0, k = 0;
        const int want = __ffs(again) - 1;
        tile_each(acc, [&](int ii, int jj, double) {
            if (k++ == want) { i = ii; j = jj; }
        });
        const int *idx = a.idx + (size_t)(i0 + i) * a.ldg;
        const double *z = a.vec + (size_t)(i0 + i) * a.ldg;
        double v = 0.0;
#pragma unroll 1
        for (int t = 0; t < a.cnt[i0 + i]; ++t) v = fma((double)a.Hinv[(size_t)idx[t] * d + j0 + j], z[t], v);
        store(i, j, v);
    }
}

size_t recon_carve(ReconArgs *a, void *base, int R, int cmax)
{
    const size_t ldg = obc_align_up((size_t)(cmax > 0 ? cmax : 1), NB);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += obc_align_up(bytes, 256);
        return base ? (char *)base + o : (char *)nullptr;
    };
    char *pg = take((size_t)R * ldg * ldg * sizeof(double));
    char *pl = take((size_t)R * ldg * NB * sizeof(double));
    char *pv = take((size_t)R * ldg * sizeof(double));
    char *pi = take((size_t)R * ldg * sizeof(int));
    char *pc = take((size_t)R * sizeof(int));
    if (a) {
        a->G = (double *)pg; a->Linv = (double *)pl; a->vec = (double *)pv; a->idx = (int *)pi; a->cnt = (int *)pc;
        a->ldg = (int)ldg;
    }
    return off;
}

}  // namespace

extern "C" {

int obc_reconstruct_workspace_bytes(int R, int d, int max_pruned, size_t *bytes)
{
    if (!bytes || R < 0 || d <= 0 || max_pruned < 0 || max_pruned > d) return OBC_ERR_BAD_ARG;
    *bytes = recon_carve(nullptr, nullptr, R, max_pruned);
    return OBC_OK;
}

int obc_reconstruct_rows(obc_ctx *ctx, const float *W, const float *Hinv, const uint8_t *mask, int R, int d,
                         int max_pruned, float *W_out, void *ws, size_t ws_bytes)
{
    if (!ctx) return OBC_ERR_BAD_ARG;
    if (!W || !Hinv || !mask || !W_out) return obc_fail(ctx, OBC_ERR_BAD_ARG, "obc_reconstruct_rows: null argument");
    if (R < 0 || d <= 0 || max_pruned < 0 || max_pruned > d)
        return obc_fail(ctx, OBC_ERR_BAD_ARG, "obc_reconstruct_rows: bad size");
    ReconArgs a;
    const size_t need = recon_carve(&a, ws, R, max_pruned);
    if (!ws || ws_bytes < need)
        return obc_fail(ctx, OBC_ERR_WORKSPACE, "obc_reconstruct_rows: workspace of %zu bytes needed, %zu given", need, ws_bytes);
    if (R == 0) return OBC_OK;
    a.W = W; a.Hinv = Hinv; a.mask = mask; a.d = d; a.cmax = max_pruned; a.W_out = W_out; a.status = ctx->d_status;
    hipStream_t st = ctx->stream;
    a.R = R;
    // Z takes G's place.  The product over all d columns costs two launches and the columns that no row has;
    // the rows' own sums read H^-1 once per row.  In us, rows' own against product, half of each row pruned:
    // 300 x 64 41, 51; 256 x 576 394, 419; 768 x 576 895, 888; 256 x 1024 965, 987; 768 x 1024 2564, 2519;
    // 8 x 2304 2036, 1827; 256 x 2304 6385, 6229; a third: 256 x 2304 2494, 2418; a fifth: 984, 988; an eighth:
    // 482, 523.
    a.Z = (max_pruned >= 640 && (size_t)d <= (size_t)a.ldg * (a.ldg + NB)) ? a.G : nullptr;
    const unsigned rows8 = (unsigned)((R + 7) / 8 * 8);
    const int nt = (max_pruned + NB - 1) / NB;                    // 64-row tiles of the largest row
    recon_list_kernel<<<R, 256, 0, st>>>(a);
    if (nt > 0) recon_gather_kernel<<<rows8 * nt, 256, 0, st>>>(a, nt);
    OBC_LAUNCH_CHECK(ctx, "recon_gather_kernel");
    for (int k = 0; k < nt; ++k) {
        recon_column_kernel<true><<<R, 256, 0, st>>>(a, k * NB, 1);
        const int below = nt - 1 - k;
        if (below > 0) recon_column_kernel<false><<<rows8 * below, 256, 0, st>>>(a, k * NB, below);
    }
    if (a.ldg <= kSolveLdsMax) {
        const size_t lds = (size_t)a.ldg * sizeof(double);
        if (lds > 48 * 1024)
            OBC_HIP(ctx, hipFuncSetAttribute((const void *)recon_solve_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        recon_solve_kernel<true><<<R, 512, lds, st>>>(a);
    } else {
        recon_solve_kernel<false><<<R, 512, 0, st>>>(a);
    }
    if (a.Z) {
        recon_spread_kernel<<<R, 256, 0, st>>>(a);
        recon_product_kernel<<<dim3((d + NB - 1) / NB, (R + NB - 1) / NB), 256, 0, st>>>(a);
    }
    OBC_LAUNCH_CHECK(ctx, "closed-form recovery kernels");
    return OBC_OK;
}

}  // extern "C"

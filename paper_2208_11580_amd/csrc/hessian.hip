// obc_hessian: H = 2 X X^T (+ dampening), Sec. 4 of arxiv 2208.11580, and obc_cross: 2 Y X^T, the
// second moment that the sequential variant (appendix "Sequential Quantization with OBQ")
// accumulates beside it.
//
// A dense (symmetric) rank-N contraction of fp32 inputs.  An input of 2^-110 and more is the exact sum of
// three bf16 numbers, x = h + m + l (8 bits of the 24 each), so the contraction runs on the bf16 matrix
// cores as six of the nine products -- h h, h m, m h, m m, h l, l h; what is left out is below 2^-24 of
// x y -- at 16 times the fp32 rate each.  v_mfma_f32_32x32x16_bf16, square output tiles of 128 (four
// waves, two workgroups per CU) or 256 (eight waves), the split done in registers on the way into LDS, two
// LDS stages, one barrier per 16 samples.  A slab's products are summed from zero and added to the
// running sums once, so a sum takes N / 16 roundings (the fp32 MFMA's took N / 2): against fp64 the
// relative error is 0.6e-7 .. 1.2e-7 (fp32 MFMA: 1.0e-7 .. 4.3e-7) over d = 32 .. 3072, N = 256 ..
// 50 000.  A workgroup that meets what the split cannot hold -- a smaller value, an infinity, a product
// that overflows -- forms its piece again on the fp32 matrix instructions; to notice it costs 1 .. 2 % of a
// large call (576 x 20 001: 79 -> 80.5 us, 3072 x 20 001: 1034 -> 1043 us) and 0.5 .. 1 us of a small one.
//
// Only tiles on or above the block diagonal are computed; the contraction length N is cut into S
// slices so that small d still fills 256 CUs.  Slices go to a workspace and are summed in a fixed
// order by a second kernel, which also mirrors the upper tiles into the lower triangle (H comes out
// exactly symmetric) -- no float atomics, results are deterministic.
//
// Bound by the matrix cores: 2304 x 50 000 is 1.77e12 bf16 operations in the tiles that are formed, in 1.29 ms of
// kernel time 78 % of what a bare bf16 loop sustains (1.75 PFLOP/s of 2.5); the halves of the diagonal tiles that
// are not needed are 10 % of them.  The whole call takes 1.45 ms, 183 TFLOP/s of the d^2 N flop (fp32 MFMA: 2.37 ms,
// 112); 576 x 50 000 0.141 ms (0.326).
#include "common.h"

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));   // 16 bytes at any float's address
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));

constexpr int BK = 16;                // samples per slab: one MFMA deep
constexpr int kSplitFrom = 3;         // samples from which a sum goes through the split: see nt_partial_kernel
constexpr int kHalf = 32 * 16 + 32;   // bytes of 32 rows x 8 samples of a plane, plus 32: see stash
constexpr int kFrag = 2 * kHalf;      // bytes of 32 rows x 16 samples of a plane

__host__ __device__ inline int tiles_of(int d, int tile) { return (d + tile - 1) / tile; }

// The launch of a contraction: square output tiles of edge `tile`, S slices of `kchunk` samples
// (multiple of BK); the workspace holds `cap` >= S slices.
struct Plan {
    int tile, S, cap;
    int64_t kchunk;
};

// `ntiles(tile)` output tiles of that edge.  Time of a launch as measured, in microseconds: a slab
// takes 1.36 with two 128-tile workgroups on a CU and 0.75 with one (latency), 2.5 with one 256-tile
// workgroup; 3 to start a round of workgroups; and the partial results are written and read back at
// about 4 TB/s.  The large tile wins by 6 % where both fill the chip (d = 2304, 3072), the small one
// where they do not (576 x 50 000: 148 against 199 us).
//
// A workspace for N samples has to serve every smaller batch, but the best S goes up and down with N
// (whole slabs only).  The S that is best for fractions of slabs grows with N -- its cost is N g(S) + h(S)
// with h growing -- and S is bounded by a quarter more than that, which leaves the choice as it is without
// a bound (2500 random sizes); the workspace holds that many.
template <class Count>
inline Plan make_plan(Count ntiles, int64_t N)
{
    auto cost = [&](int tile, int64_t n, int64_t c, double slabs) {
        const int64_t w = n * c;
        double t;
        if (tile == 128) {
            const int64_t left = w % 512;
            t = (double)(w / 512) * (1.36 * slabs + 3.0)
                + (left > 256 ? 1.36 * slabs + 3.0 : left > 0 ? 0.75 * slabs + 3.0 : 0.0);
        } else {
            t = (double)((w + 255) / 256) * (2.5 * slabs + 3.0);
        }
        return t + (double)w * tile * tile * 8.0 / 4e6 + 0.1 * (double)c;
    };
    Plan best = {128, 1, 1, 0};
    double best_cost = 0.0;
    const int64_t smax = N / (2 * BK) < 1 ? 1 : N / (2 * BK) < 64 ? N / (2 * BK) : 64;
    // (a small call waits for this: one division per S)
    double slabs[65], whole[65];
    for (int64_t c = 1; c <= smax; ++c) {
        slabs[c] = (double)N / (double)(BK * c);
        whole[c] = (double)(int64_t)slabs[c];
        if (whole[c] < slabs[c]) whole[c] += 1.0;
    }
    for (int tile = 128; tile <= 256; tile += 128) {
        const int64_t n = ntiles(tile);
        int64_t bound = 1;
        double bound_cost = cost(tile, n, 1, slabs[1]);
        for (int64_t c = 2; c <= smax; ++c) {
            const double t = cost(tile, n, c, slabs[c]);
            if (t < bound_cost) {
                bound_cost = t;
                bound = c;
            }
        }
        bound = bound + bound / 4 + 1 < smax ? bound + bound / 4 + 1 : smax;
        if (bound > best.cap) best.cap = (int)bound;
        for (int64_t c = 1; c <= bound; ++c) {
            const double t = cost(tile, n, c, whole[c]);
            if (best_cost == 0.0 || t < best_cost) {
                best_cost = t;
                best.tile = tile;
                best.S = (int)c;
            }
        }
    }
    int64_t kc = (N + best.S - 1) / best.S;
    kc = (kc + BK - 1) / BK * BK;
    best.kchunk = kc;
    best.S = (int)((N + kc - 1) / kc);
    return best;
}

inline Plan hessian_plan(int d, int64_t N)
{
    return make_plan([&](int tile) { const int64_t nt = tiles_of(d, tile); return nt * (nt + 1) / 2; }, N);
}

inline Plan cross_plan(int d_row, int d_col, int64_t N)
{
    return make_plan([&](int tile) { return (int64_t)tiles_of(d_row, tile) * tiles_of(d_col, tile); }, N);
}

// One slice of P = Ya Xb^T over the samples [kbeg, kend): Ya is da x N (leading dimension lda),
// Xb is db x N (ldb).  SYM: Ya and Xb are the same matrix and only the tiles on or above the block
// diagonal are formed.  WR x WC waves, each MT x NT accumulators of 32 x 32.
template <bool SYM, int WR, int WC, int MT, int NT>
__global__ __launch_bounds__(WR *WC * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void nt_partial_kernel(const float *__restrict__ Ya, int da, int64_t lda, const float *__restrict__ Xb, int db,
                       int64_t ldb, int64_t N, int S, int64_t kchunk, float *__restrict__ partial)
{
    constexpr int TILE = WR * MT * 32, T = WR * WC * 64;
    static_assert(WC * NT * 32 == TILE && TILE * 4 == 2 * T, "square tiles, two quads per thread and operand");
    __shared__ __align__(16) uint8_t lds[2][2][3][TILE / 32][kFrag];   // stage, operand, plane, 32 rows
    __shared__ int redo_s;

    // Workgroups go round-robin to the 8 XCDs: each XCD takes a run of the (slice, tile) list, so
    // that the workgroups that share a slice of X run side by side and find it in their L2.
    const int ntri = SYM ? tiles_of(da, TILE) * (tiles_of(da, TILE) + 1) / 2 : tiles_of(da, TILE) * tiles_of(db, TILE);
    const int unit = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (unit >= ntri * S) return;
    const int tile_id = unit % ntri, slice = unit / ntri;
    int ti, tj;
    if (SYM) {
        // upper-triangular tile enumeration: tile_id -> (ti <= tj)
        int t = tile_id, rowlen = tiles_of(da, TILE);
        ti = 0;
        while (t >= rowlen) { t -= rowlen; ++ti; --rowlen; }
        tj = ti + t;
    } else {
        const int ntb = tiles_of(db, TILE);
        ti = tile_id / ntb;
        tj = tile_id % ntb;
    }

    const int64_t kbeg = (int64_t)slice * kchunk;
    const int64_t kend = (kbeg + kchunk < N) ? kbeg + kchunk : N;
    const int nslab = kend > kbeg ? (int)((kend - kbeg + BK - 1) / BK) : 0;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WC, wn = wave % WC;

    floatx16 acc[MT][NT];
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    // loader: four threads take the 64 bytes of a row's slab, 16 bytes each; a thread has two rows
    // of each operand.  Rows beyond the matrix re-read its last row: their products only reach
    // outputs that are never stored.
    const int q = tid & 3, r0 = tid >> 2;
    const float *src[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int ra = ti * TILE + r0 + h * (T / 4), rb = tj * TILE + r0 + h * (T / 4);
        src[0][h] = Ya + (int64_t)(ra < da ? ra : da - 1) * lda + kbeg + q * 4;
        src[1][h] = Xb + (int64_t)(rb < db ? rb : db - 1) * ldb + kbeg + q * 4;
    }
    floatx4u reg[2][2];
    auto fetch = [&](int op, int h, int slab) {
        reg[op][h] = *reinterpret_cast<const floatx4u *>(src[op][h] + (int64_t)slab * BK);
    };
    auto fetch_tail = [&](int op, int h, int slab) {
        const float *p = src[op][h] + (int64_t)slab * BK;
        const int64_t left = kend - kbeg - (int64_t)slab * BK - q * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) reg[op][h][i] = (i < left) ? p[i] : 0.f;
    };
    auto fetch_any = [&](int op, int h, int slab) {
        if ((int64_t)(slab + 1) * BK <= kend - kbeg) fetch(op, h, slab);
        else fetch_tail(op, h, slab);
    };
    // The least magnitude but zero that passes through the split, as 2 |bits| - 1 (zero wraps to the top):
    // below 2^-110 the third plane may fall under the smallest bf16.
    unsigned least = ~0u;
    // Split into three bf16 planes and store.  A plane's 32 rows x 16 samples lie as the MFMA
    // operand is read: lane l finds row l % 32, samples 8 (l / 32) .. + 7 in 16 bytes at
    // (l / 32) kHalf + (l % 32) 16.  The 32 bytes between the halves spread the four quads of a row
    // over different banks.
    auto stash = [&](int stage, int op, int h) {
        const int r = r0 + h * (T / 4);
        uint8_t *dst = &lds[stage][op][0][r >> 5][(q >> 1) * kHalf + (r & 31) * 16 + (q & 1) * 8];
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = reg[op][h][i];
            least = min(least, (__float_as_uint(v[i]) << 1) - 1u);
        }
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
            uintx2 w;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                typedef float floatx2 __attribute__((ext_vector_type(2)));
                const floatx2 f = {v[2 * i], v[2 * i + 1]};
                w[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
                v[2 * i] = __fsub_rn(v[2 * i], __uint_as_float(w[i] << 16));
                v[2 * i + 1] = __fsub_rn(v[2 * i + 1], __uint_as_float(w[i] & 0xffff0000u));
            }
            *reinterpret_cast<uintx2 *>(dst + pl * (TILE / 32) * kFrag) = w;
        }
    };
    const int loff = (lane >> 5) * kHalf + (lane & 31) * 16;
    auto frag = [&](int stage, int op, int pl, int g) {
        return *reinterpret_cast<const bf16x8 *>(&lds[stage][op][pl][g][loff]);
    };
    // One slab's six products, the smallest first, summed from zero on the matrix cores and added to
    // the running sums by the vector ALU.  (Fed straight into the running sums, the small products
    // would each be lost below their last bit: m m, always positive on the diagonal, left a bias of
    // -2e-6 there.)  One accumulator's six products are a chain; the vector instructions -- the additions of the
    // accumulator before it, and what `between(u)` does for the u-th -- are dealt between them, so that a wave keeps
    // both units busy by itself: the waves of a SIMD meet at every slab's barrier and would otherwise multiply
    // together and add together (2304 x 50 000 in four batches and its inverse 2.98 -> 2.91 ms; in one batch, with the
    // cross moment and the re-fit, 3.65 -> 3.56).
    constexpr int NU = MT * NT;
    auto mma = [&](int stage, auto between) {
        bf16x8 fa[3][MT], fb[3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll
            for (int a = 0; a < MT; ++a) fa[pl][a] = frag(stage, 0, pl, wm * MT + a);
        constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
        floatx16 t[2];
#pragma unroll
        for (int u = 0; u <= NU; ++u) {
            const int a = u % MT, b = u / MT;
            if (u < NU) {
                if (a == 0) {
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) fb[pl] = frag(stage, 1, pl, wn * NT + b);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) t[u & 1][v] = 0.f;
#pragma unroll
                for (int i = 0; i < 6; ++i)
                    t[u & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[pa[i]][a], fb[pb[i]], t[u & 1], 0, 0, 0);
                between(u);
            }
            if (u > 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    acc[(u - 1) % MT][(u - 1) / MT][v] = __fadd_rn(acc[(u - 1) % MT][(u - 1) / MT][v], t[(u - 1) & 1][v]);
            }
            if (u < NU) {
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // one matrix instruction,
                    if (u % (NU / 4) == 0) __builtin_amdgcn_sched_group_barrier(0x002, 9, 0);    // and its share of vector ones
                    else __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);   // (one accumulator at a time: registers)
            if (u == NU - 1) __syncthreads();
        }
    };

    // One or two products take fewer roundings as they are than through the split's six: largest error over
    // the sum of the magnitudes 0.6e-7 and 1.1e-7 against 1.4e-7 for both; from three on (1.5e-7 against
    // 1.1e-7) the split has the smaller one.  The time is the same.
    const int nsplit = N >= kSplitFrom ? nslab : 0;
    if (tid == 0) redo_s = 0;
    if (nsplit > 0) {
        for (int h = 0; h < 2; ++h) { fetch_any(0, h, 0); fetch_any(1, h, 0); }
        for (int h = 0; h < 2; ++h) { stash(0, 0, h); stash(0, 1, h); }
        if (nsplit > 1)
            for (int h = 0; h < 2; ++h) { fetch_any(0, h, 1); fetch_any(1, h, 1); }
    }
    __syncthreads();
    // Stage s % 2 holds slab s, the registers hold slab s + 1: it is split and stored into the other
    // stage, and slab s + 2 requested, among slab s's matrix instructions.  One barrier per slab, behind its last
    // read and store and ahead of its last additions.
    int s = 0;
    for (; (int64_t)(s + 3) * BK <= kend - kbeg; ++s) {
        const int cur = s & 1;
        mma(cur, [&](int u) {
            if (u % (NU / 4) == 0) {
                const int i = u / (NU / 4);
                stash(cur ^ 1, i >> 1, i & 1);
                fetch(i >> 1, i & 1, s + 2);
            }
        });
    }
    for (; s < nsplit; ++s) {
        const int cur = s & 1;
        if (s + 1 < nsplit)
            for (int h = 0; h < 2; ++h) { stash(cur ^ 1, 0, h); stash(cur ^ 1, 1, h); }
        if (s + 2 < nsplit)
            for (int h = 0; h < 2; ++h) { fetch_any(0, h, s + 2); fetch_any(1, h, s + 2); }
        mma(cur, [](int) {});
    }

    // The plain form of the piece: where an input was too small to split, or where a NaN came out -- an
    // infinity and a finite value that rounds to infinity in bf16 leave one, a product that overflows may --
    // it is formed again from the inputs themselves by fp32 matrix instructions.
    bool lost = nsplit < nslab || least < (17u << 24) - 1u;
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int v = 0; v < 16; v += 2) lost |= __builtin_isunordered(acc[a][b][v], acc[a][b][v + 1]);
    if (lost) redo_s = 1;
    __syncthreads();
    if (__builtin_expect(redo_s, 0)) {
        constexpr int LD = TILE + 4;
        static_assert(sizeof(lds) >= 2 * BK * LD * sizeof(float), "the plain form's stage");
        float *stage = reinterpret_cast<float *>(lds);       // operand, sample, row
#pragma unroll
        for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int b = 0; b < NT; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
        for (int h = 0; h < 2; ++h) { fetch_any(0, h, 0); fetch_any(1, h, 0); }
#pragma unroll 1
        for (s = 0; s < nslab; ++s) {
#pragma unroll
            for (int op = 0; op < 2; ++op)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) stage[(op * BK + q * 4 + i) * LD + r0 + h * (T / 4)] = reg[op][h][i];
            __syncthreads();
            if (s + 1 < nslab)
                for (int h = 0; h < 2; ++h) { fetch_any(0, h, s + 1); fetch_any(1, h, s + 1); }
#pragma unroll
            for (int kk = 0; kk < BK; kk += 2) {
                float fa[MT], fb[NT];
#pragma unroll
                for (int a = 0; a < MT; ++a) fa[a] = stage[(kk + (lane >> 5)) * LD + (wm * MT + a) * 32 + (lane & 31)];
#pragma unroll
                for (int b = 0; b < NT; ++b) fb[b] = stage[(BK + kk + (lane >> 5)) * LD + (wn * NT + b) * 32 + (lane & 31)];
#pragma unroll
                for (int a = 0; a < MT; ++a)
#pragma unroll
                    for (int b = 0; b < NT; ++b)
                        acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[a], fb[b], acc[a][b], 0, 0, 0);
            }
            __syncthreads();
        }
    }

    // accumulator layout of the 32x32 MFMA: lane holds column (lane % 32) and, for register v,
    // row 8 * (v / 4) + 4 * (lane / 32) + v % 4
    float *out = partial + (int64_t)slice * da * db;
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                int i = ti * TILE + (wm * MT + a) * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                int j = tj * TILE + (wn * NT + b) * 32 + (lane & 31);
                if (i < da && j < db) out[(int64_t)i * db + j] = acc[a][b][v];
            }
}

// H (+)= 2 * sum_s partial[s] on and above the diagonal, slices added in index order, and the mirror
// image below it.  One workgroup per 32 x 32 piece: the sums are read and written along rows, the
// mirrored piece goes through LDS so that it is written along rows too.  (Below the diagonal of a
// diagonal piece the mirror image is taken as well: the two halves of such a tile add their cross
// products in opposite order.)
// damp_rel >= 0, with one workgroup only (d <= 32): the dampening is done here, with the sum in dampen_kernel's order
// (whose 1024 terms are zeros but for the first d).
__global__ __launch_bounds__(256) void syrk_reduce_kernel(const float *__restrict__ partial, int S,
                                                          int d, int accumulate, float damp_rel, float *H)
{
    __shared__ float Tt[32][33];
    const int pi = blockIdx.y, pj = blockIdx.x;           // 32 x 32 piece (pi, pj)
    if (pi > pj) return;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = pi * 32 + ty + 8 * r, j = pj * 32 + tx;
        if (i > j || j >= d) continue;
        const int64_t e = (int64_t)i * d + j;
        float s = 0.f;
#pragma unroll 8
        for (int k = 0; k < S; ++k) s += partial[(int64_t)k * d * d + e];
        s *= 2.f;
        H[e] = accumulate ? H[e] + s : s;
        Tt[ty + 8 * r][tx] = s;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = pj * 32 + ty + 8 * r, j = pi * 32 + tx;   // (i, j) of the mirrored piece
        if (i <= j || i >= d) continue;
        const int64_t e = (int64_t)i * d + j;
        const float s = Tt[tx][ty + 8 * r];
        H[e] = accumulate ? H[e] + s : s;
    }
    if (damp_rel >= 0.f && gridDim.x == 1) {
        __shared__ double red[32];
        __syncthreads();                                  // (the workgroup's own stores, read back through its cache)
        const int j = threadIdx.x;
        float h = 0.f;
        if (j < 32) {
            h = j < d ? H[(int64_t)j * d + j] : 0.f;
            red[j] = (double)h;
        }
        __syncthreads();
        for (int w = 16; w > 0; w >>= 1) {
            if (j < w) red[j] += red[j + w];
            __syncthreads();
        }
        if (j < d) H[(int64_t)j * d + j] = h + (float)((double)damp_rel * red[0] / (double)d);
    }
}

// C[e] (+)= 2 * sum_s partial[s][e] over a dense da x db result, slices added in index order.
__global__ __launch_bounds__(256) void nt_reduce_kernel(const float *__restrict__ partial, int S,
                                                        int64_t n, int accumulate, float *__restrict__ C)
{
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    float s = 0.f;
#pragma unroll 8
    for (int k = 0; k < S; ++k) s += partial[(int64_t)k * n + e];
    s *= 2.f;
    C[e] = accumulate ? C[e] + s : s;
}

// diag(H) += damp_rel * mean(diag(H)); one workgroup, fixed-order tree sum in fp64.
__global__ __launch_bounds__(1024) void dampen_kernel(float *__restrict__ H, int d, float damp_rel)
{
    __shared__ double red[1024];
    double s = 0.0;
    for (int j = threadIdx.x; j < d; j += blockDim.x) s += (double)H[(int64_t)j * d + j];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    float lam = (float)((double)damp_rel * red[0] / (double)d);
    for (int j = threadIdx.x; j < d; j += blockDim.x) H[(int64_t)j * d + j] += lam;
}

// The slices of the contraction into partial (S x da x db).
template <bool SYM>
int launch_nt(obc_ctx *ctx, const Plan &p, const float *Ya, int da, int64_t lda, const float *Xb, int db, int64_t ldb,
              int64_t N, float *partial)
{
    const int64_t nt = tiles_of(da, p.tile);
    const int64_t n = SYM ? nt * (nt + 1) / 2 : nt * tiles_of(db, p.tile);
    const unsigned grid = (unsigned)((n * p.S + 7) / 8 * 8);
    if (p.tile == 256)
        nt_partial_kernel<SYM, 4, 2, 2, 4><<<grid, 512, 0, ctx->stream>>>(Ya, da, lda, Xb, db, ldb, N, p.S, p.kchunk, partial);
    else
        nt_partial_kernel<SYM, 2, 2, 2, 2><<<grid, 256, 0, ctx->stream>>>(Ya, da, lda, Xb, db, ldb, N, p.S, p.kchunk, partial);
    OBC_LAUNCH_CHECK(ctx, "nt_partial_kernel");
    return OBC_OK;
}

}  // namespace

extern "C" {

int obc_hessian_workspace_bytes(int d, int64_t N, size_t *bytes)
{
    if (!bytes || d <= 0 || N < 0) return OBC_ERR_BAD_ARG;
    const Plan p = hessian_plan(d, N > 0 ? N : 1);
    *bytes = obc_align_up((size_t)p.cap * d * d * sizeof(float), 256);
    return OBC_OK;
}

int obc_hessian(obc_ctx *ctx, const float *X, int d, int64_t N, int64_t ldx, float damp_rel,
                int accumulate, float *H, void *ws, size_t ws_bytes)
{
    if (!ctx) return OBC_ERR_BAD_ARG;
    if (!X || !H) return obc_fail(ctx, OBC_ERR_BAD_ARG, "obc_hessian: null X or H");
    if (d <= 0 || N <= 0) return obc_fail(ctx, OBC_ERR_BAD_ARG, "obc_hessian: d and N must be positive");
    if (ldx < N) return obc_fail(ctx, OBC_ERR_BAD_SHAPE, "obc_hessian: ldx (%lld) < N (%lld)", (long long)ldx, (long long)N);
    const Plan p = hessian_plan(d, N);
    const size_t need = obc_align_up((size_t)p.S * d * d * sizeof(float), 256);   // (what this N takes of the query's)
    if (!ws || ws_bytes < need)
        return obc_fail(ctx, OBC_ERR_WORKSPACE, "obc_hessian: workspace of %zu bytes needed, %zu given", need, ws_bytes);

    float *partial = (float *)ws;
    int rc = launch_nt<true>(ctx, p, X, d, ldx, X, d, ldx, N, partial);
    if (rc != OBC_OK) return rc;
    const unsigned np32 = (unsigned)((d + 31) / 32);
    syrk_reduce_kernel<<<dim3(np32, np32), 256, 0, ctx->stream>>>(partial, p.S, d, accumulate, damp_rel, H);
    OBC_LAUNCH_CHECK(ctx, "syrk_reduce_kernel");
    if (damp_rel >= 0.f && np32 > 1) {
        dampen_kernel<<<1, 1024, 0, ctx->stream>>>(H, d, damp_rel);
        OBC_LAUNCH_CHECK(ctx, "dampen_kernel");
    }
    return OBC_OK;
}

int obc_cross_workspace_bytes(int d_row, int d_col, int64_t N, size_t *bytes)
{
    if (!bytes || d_row <= 0 || d_col <= 0 || N < 0) return OBC_ERR_BAD_ARG;
    const Plan p = cross_plan(d_row, d_col, N > 0 ? N : 1);
    *bytes = obc_align_up((size_t)p.cap * d_row * d_col * sizeof(float), 256);
    return OBC_OK;
}

int obc_cross(obc_ctx *ctx, const float *X, const float *Y, int d_col, int d_row, int64_t N, int64_t ldx,
              int64_t ldy, int accumulate, float *C, void *ws, size_t ws_bytes)
{
    if (!ctx) return OBC_ERR_BAD_ARG;
    if (!X || !Y || !C) return obc_fail(ctx, OBC_ERR_BAD_ARG, "obc_cross: null X, Y or C");
    if (d_col <= 0 || d_row <= 0 || N <= 0)
        return obc_fail(ctx, OBC_ERR_BAD_ARG, "obc_cross: d_col, d_row and N must be positive");
    if (ldx < N || ldy < N)
        return obc_fail(ctx, OBC_ERR_BAD_SHAPE, "obc_cross: ldx (%lld) or ldy (%lld) < N (%lld)", (long long)ldx,
                        (long long)ldy, (long long)N);
    const Plan p = cross_plan(d_row, d_col, N);
    const size_t need = obc_align_up((size_t)p.S * d_row * d_col * sizeof(float), 256);
    if (!ws || ws_bytes < need)
        return obc_fail(ctx, OBC_ERR_WORKSPACE, "obc_cross: workspace of %zu bytes needed, %zu given", need, ws_bytes);

    float *partial = (float *)ws;
    int rc = launch_nt<false>(ctx, p, Y, d_row, ldy, X, d_col, ldx, N, partial);
    if (rc != OBC_OK) return rc;
    const int64_t n = (int64_t)d_row * d_col;
    nt_reduce_kernel<<<(unsigned)((n + 255) / 256), 256, 0, ctx->stream>>>(partial, p.S, n, accumulate, C);
    OBC_LAUNCH_CHECK(ctx, "nt_reduce_kernel");
    return OBC_OK;
}

}  // extern "C"

// Declarations shared by the blocked row solver's translation units: workspace layout, kernel
// argument blocks, and the per-variant panel launchers (one translation unit per variant so that
// they compile in parallel: a wide one takes over a minute).
#pragma once

#include "rows_common.h"

namespace obc_blocked {

using namespace obc_rows;

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int BMAX = 64;       // rank of a bulk elimination of pruned indices, and widest row that is one panel
constexpr int UCAP = 2 * BMAX; // vectors per row in U: an outer block's, or a bulk elimination's in and out
constexpr int kGone = (int)0x80000000;   // `orig` of an index eliminated since the last compaction
constexpr int kPanelDynLds = 160 * 1024 - 6144;   // what a panel's static LDS leaves of a CU's

// Layout of a row's private matrix after its first flush ("row-quad" layout): element (i, j) is at
// float index ((i / 4) * ld + j) * 4 + i % 4, i.e. four consecutive rows of a column sit together.
// It matches the MFMA accumulator layout (a lane holds four consecutive rows of one column: one
// 16-byte store) and it makes both ways the panel reads the symmetric matrix -- along a row and
// along a column -- cost the same 16-byte granularity instead of 4 bytes vs one cache line.
__host__ __device__ inline size_t quad_index(int i, int j, int ld)
{
    return ((size_t)(i >> 2) * ld + j) * 4 + (i & 3);
}

// Entry j of vector k of a row's U: four vectors of a column sit together, so that the panel writes and reads, and the
// flush reads, four of them at a time.
__host__ __device__ inline size_t u_index(int k, int j, int ldu)
{
    return ((size_t)(k >> 2) * ldu + j) * 4 + (k & 3);
}

struct BlockedWs {
    float *Abuf[2];     // R x d x d each
    float *U;           // R x UCAP x ldu (u_index)
    int ldu;            // leading dimension of U: d rounded up to a multiple of 4
    float *invd;        // R x UCAP   1 / a_r of U's vectors
    int *map;           // R x d     (new compact index -> old compact index)
    double *w;          // R x d     (compact)
    double *diag;       // R x d
    int *orig;          // R x d     compact -> original index; ~index for an already-pruned weight; kGone
    int *m;             // R   live size
    int *done;          // R   steps done (including up-front eliminations)
    int *total;         // R   steps to do
    int *ndead;         // R   up-front eliminations
    int *nb;            // R   steps done since the last flush
    uint8_t *blk;       // R x d  N:M counters (d / M used), between two panels
    // bulk elimination of already-pruned indices, BMAX at a time (rows_blocked.hip)
    // (the rows of the matrix at the block's pivots are parked in vectors BMAX .. of U, their
    // positions in the block's slots of invd until the vectors are formed)
    double *Mb;         // R x BMAX x BMAX the pivots' principal submatrix, then its Cholesky factor
    double *Tb;         // R x BMAX x BMAX inverse of that factor
    int *scal;          // [0] smallest number of up-front eliminations over the rows, [1] the most eliminations any row does
};


// Eliminations of a row with `survivors` live weights: the already-pruned indices and the greedy
// steps (block pruning: 4 per block step).
__device__ inline int panel_total(int mode, int d, int survivors, int k_steps, const int32_t *stop_counts, int row)
{
    int steps = (mode == MODE_QUANT) ? survivors : (k_steps < survivors ? k_steps : survivors);
    if (stop_counts) {
        int sc = stop_counts[row];
        sc = sc < 0 ? 0 : sc;
        if (mode == MODE_BLOCK) sc = sc > d / 4 ? d : sc * 4;
        steps = sc < steps ? sc : steps;
    }
    return d - survivors + steps;
}

struct PanelArgs {
    const float *A_cur;      // matrix buffer the rows are read from
    size_t a_row_stride;     // elements between two rows' matrices (0: all rows share H^-1)
    int ld;                  // leading dimension of A_cur
    int swz;                 // 0: A_cur is plain row-major (the shared H^-1); 1: row-quad layout
    int old;                 // vectors of this outer block already in U (every row still running has all of them)
    int threads;             // threads of the launch (variants with one owned index per thread)
    int last;                // the outer block's last panel: a flush follows
    int d;                   // original width (stride of the per-row state arrays)
    int nm_n, nm_m;
    const float *delta, *offset;
    int maxq;
    int outliers;            // OBQ: restrict the choice to outliers while there are any
    BlockedWs ws;
    int32_t *order;
    float *loss;
    int32_t *codes;
    float *W_out;
    float *trace;
    int out_ld;
    int *status;
    // rows that fit one panel (d <= BMAX) start from the caller's arrays and need no workspace
    int direct;
    const float *W;
    const uint8_t *live_in;
    const int32_t *stop_counts;
    int k_steps;
};

// launchers defined in panel_<T>x<EPT>x<BR>x<BL>.hip (pruning and OBQ) and
// panel_block_<T>x<EPT>x<BR>x<BL>.hip (block pruning, blocks of 4): T threads, EPT owned indices per thread,
// blocks of BR + BL steps (BR vectors in registers, BL in LDS).  Return 0 or -1 (HIP error).
typedef int PanelLaunch(int mode, int R, hipStream_t st, const PanelArgs &a);
#define OBC_DECLARE_PANEL(T, EPT, BR, BL) \
    PanelLaunch launch_panel_##T##_##EPT##_##BR##_##BL, launch_panel_block_##T##_##EPT##_##BR##_##BL
OBC_DECLARE_PANEL(256, 1, 64, 0);
OBC_DECLARE_PANEL(1024, 1, 64, 0);
OBC_DECLARE_PANEL(512, 3, 48, 24);
OBC_DECLARE_PANEL(512, 4, 40, 16);
OBC_DECLARE_PANEL(768, 3, 32, 16);
OBC_DECLARE_PANEL(512, 6, 28, 12);
OBC_DECLARE_PANEL(512, 8, 20, 8);
OBC_DECLARE_PANEL(512, 9, 16, 8);
PanelLaunch launch_panel_256_2_56_24, launch_panel_256_3_32_16, launch_panel_old_512_6_28_12;

}  // namespace obc_blocked

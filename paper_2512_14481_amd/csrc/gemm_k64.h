// Host-side interface of the 16x16x64 int8 GEMM kernels (static_linear_k64.hip, grouped_k64.hip), used by the entry
// points in static_linear.hip.
#pragma once

#include "gemm_tile.h"

namespace sasq {

struct GemmK64Args {
    const int8_t* xq;        // staged activation codes (1 KB blocks of 16 rows x 64 K-bytes)
    const uint8_t* wq;       // weights in the layout `wmode` names
    const float* s;          // activation factor (one, or one per row with `rows`)
    const float* s_w;
    const float* bias;
    uint16_t* y;
    int32_t* acc_out;
    int64_t M, N, K;
};

// wmode: 0 = int8 row-major, 2 = int8 pre-arranged, 3 = int4 pre-arranged (the values of the weight paths in static_linear.hip).
// tile: 0 = 256x256, 1 = 128x256, 2 = 128x128 (two workgroups per CU).  K must be a multiple of 64.
void launch_gemm_k64(const GemmK64Args& a, sasq_dtype dt, int wmode, int tile, bool rows, hipStream_t st);
// Grouped activation factors (a.s points at K / (64 group_tiles) factors, a.acc_out receives the fp32 sums):
// tile 1 = 128x256, 2 = 128x128.  group_tiles = 0: groups of 32 channels (two per K tile; 128x128 tiles).
void launch_gemm_k64_grouped(const GemmK64Args& a, sasq_dtype dt, int wmode, int tile, int group_tiles, hipStream_t st);
// Every other group size (grouped_valu.hip): row-major weights, row-major activation codes in a.xq, any
// group that divides K.
void launch_grouped_valu(const GemmK64Args& a, sasq_dtype dt, bool int4, int64_t group, hipStream_t st);
// Few output tiles (grouped_split.hip), K a multiple of 64: int8 weights, row-major or pre-arranged, row-major activation codes in a.xq.
// grouped_takes_split: the form to take, 0: the other kernels are better or the group is none of its own.
int grouped_takes_split(int64_t M, int64_t N, int64_t K, int64_t group, bool blocked);
void launch_grouped_split(const GemmK64Args& a, sasq_dtype dt, bool blocked, int64_t group, int form, hipStream_t st);
// K not a multiple of 64 (static_linear_anyk.hip): row-major activation codes in a.xq, row-major int8 or packed int4 weights.
// rows: one activation factor per row.
void launch_linear_anyk(const GemmK64Args& a, sasq_dtype dt, bool int4, bool rows, hipStream_t st);
// Rounds of 256x256 tiles (or of as much work) that a single call's GEMM takes with the tiles chosen for it (static_linear.hip).
double gemm_rounds(int64_t M, int64_t N);
// At most kSkinnyRows rows, or too few tiles for the GEMM (static_linear_skinny.hip; linear_takes_skinny says whether the
// sizes are such): the items of `b` (first_block and the tile counts are filled in here), weight layouts 0, 2 and 3.
// qx: quantize the activations in the kernel (where linear_quantizes_in_kernel allows it and no output overlaps an input, as
// workgroups read x while others write y); otherwise the items' xq hold the staged codes.
constexpr int kSkinnyRows = 64, kSkinnyQuantRows = 16;
bool linear_takes_skinny(const LinBatch& b, int wmode);
// More than kSkinnyRows rows: 32, small blocks; 64, 96 or 128, rows per workgroup of the row blocks; 0, the GEMM's tiles.
int linear_block_rows(const LinBatch& b, int wmode);
bool linear_quantizes_in_kernel(const LinBatch& b, int wmode, bool any_k);
bool linear_turns(const LinBatch& b, int wmode, bool qx);
bool linear_streams(const LinBatch& b, int wmode);
bool linear_long_rows(const LinBatch& b);
void launch_linear_skinny(LinBatch& b, sasq_dtype dt, int wmode, bool qx, int a_bits, int32_t* acc_out, hipStream_t st);
// The same for K that is not a multiple of 64, a single call with row-major int8 weights (row-major codes in xq).
bool linear_anyk_takes_skinny(int64_t M, int64_t N, int64_t K);
int linear_anyk_tile(int64_t M, int64_t N, int64_t K);
void launch_linear_anyk_skinny(LinBatch& b, sasq_dtype dt, bool qx, int a_bits, int32_t* acc_out, hipStream_t st);
// The choice of kernels in linear_bwd.hip: rows per workgroup without tiles, 0: tiles; the tile, 0: 256x256, 1: 128x256, 2: 128x128.
int bwd_rows(int64_t M, int64_t N, int64_t K);
int bwd_tile(int64_t M, int64_t N, int64_t K);
bool bwd_reads_lines(int64_t N, int tile_rows);
// The backward GEMM dX[M, K] = dY[M, N] . B^T over the prepared weight (linear_bwd.hip), for few rows or too few tiles; N a multiple
// of 32.  bwd_takes_skinny: rows per workgroup, 0: the tiles, which take tile_us, are better, or the contraction is too long.
// An estimate of a launch's time in us: its workgroups go in rounds of 256, one a CU; a round costs what a workgroup takes to start and end,
// and its K tiles, each the longer the more CUs are at work beside it (the clock comes down, the operands come later).
struct RoundTime {
    double call, round, k_tile, k_fill;
    double of(int64_t blocks, double k_tiles) const { return round + k_tiles * (k_tile + k_fill * (double)blocks / 256.0); }
    double launch(int64_t blocks, double k_tiles) const
    {
        const int64_t rest = blocks % 256;
        return call + (double)(blocks / 256) * of(256, k_tiles) + (rest ? of(rest, k_tiles) : 0.0);
    }
};
// Longest contraction of the kernels that reach a block's rows by 32-bit byte offsets (256 rows of dY, 2 GB; 64 columns' weight blocks).
constexpr int64_t kBwdOffsetCols = INT64_C(1) << 22;
int bwd_takes_skinny(int64_t M, int64_t N, int64_t K, double tile_us);
bool bwd_turns(int64_t M, int64_t N, int64_t K);
void launch_bwd_skinny(const void* dy, const void* wt, void* dx, float* acc_out, int64_t M, int64_t N, int64_t K, sasq_dtype dt, int rows, hipStream_t st);
// Batches of at least so many workgroup ids, and at most 128, go as half tiles throughout.
constexpr int kHalvesFrom = 32;
// split_tail: hand the tiles of a sparsely filled last round out as 128x256 halves (sets b.split_first / b.split_count)
void launch_gemm_k64_batch(LinBatch& b, int grid, sasq_dtype dt, int wmode, bool split_tail, hipStream_t st);

}  // namespace sasq

// Per-channel fake quantization: one learned factor per activation column (the granularity Sec. 4
// adopts for activations and weights; Sec. 2, Fig. 2(b): per-channel = the elements of a column
// share a factor).  Same element arithmetic as the per-tensor operator
// (Sec. 3, Eq. 1; Sec. 4.2, Eq. 4); the scale gradient becomes a column reduction:
//     ds[k] = sum_m dy[m,k] * (q[m,k] - m[m,k] * x[m,k]/s[k]).
//
// Traversal: a lane owns 8 consecutive columns (one 128-bit access) for the whole kernel, so its
// eight scales and reciprocals live in registers; a wave covers 512 consecutive columns of one
// row (1 KB, fully coalesced); the 4 waves of a block take rows r, r+1, r+2, r+3 of the block's
// row chunk.  Grid = column chunks x row chunks.
// x is loaded with the ordinary policy, as the layer's other operators and the backward read it again (up to 256 MB stay in the
// Infinity Cache); dy, y and dx go non-temporal.  One step's forward, backward and AdamW, us, x non-temporal | not: a 13B layer at 1777
// rows 149.5 | 126.7, 7B's at 500 43.7 | 39.5, 7B's MLP at 4000 148 | 136, 4096 rows of 13B 336 | 299.
#include "sasq_device.h"
#include <type_traits>
#include <cstring>

namespace sasq {

constexpr int kPcThreads = 256;
constexpr int kPcWaves = kPcThreads / kWave;
constexpr int kPcColsPerBlock = kWave * 8;        // 512
constexpr int kPcRowUnroll = 4;                   // rows in flight per wave
constexpr int kPcMaxRowChunks = 128;              // more row chunks than this lengthen the reduction tail (measured)
constexpr int kPcTargetBlocks = 2048;             // 8 blocks per CU
// Rows a block takes at least: it pays for its columns' factors (eight divisions a lane) and, backward, for its partial and
// ticket once, and from two groups of rows on it has loads in flight under its arithmetic.
// Forward, by the launch as a whole: 16 rows while that makes at most one block per CU, or nearly fills a second round of
// them.  Measured, us with 16 | 32 rows: 512 x 512 (32 blocks of 16) 3.8 | 4.3, 512 x 4096 (256) 4.4 | 5.0, two of 200 x 5120
// (260) 6.3 | 5.1, four of 300 x 2048 (304) 7.1 | 5.6, seven of 128 x 4096 (448) 5.9 | 6.1, 1024 x 4096 (512) 5.8 | 6.2,
// 2048 x 4096 (1024) 9.0 | 8.4, seven of 512 x 4096 (1792) 13.9 | 13.3, seven of 1777 x 5120 47.2 | 45.2.
constexpr int kPcMinRows = 32;
static int64_t pc_fwd_rows(int64_t blocks16)
{
    return blocks16 <= 256 || (blocks16 > 384 && blocks16 <= 512) ? 16 : kPcMinRows;
}
// Backward, where the rows per block decide how ds is rounded: they follow from the tensor alone, never from what shares its
// launch, so that a batch gives the bits of the single calls.  16 for a tensor of at most 64 such blocks, 64 for one that has
// more than 512 of those, of more than 256 if it is wide and has at least 704 rows (a wide tensor's rows are long enough to keep
// the memory busy from fewer blocks, and blocks of 32 rows compute its factors twice as often).  Measured, us with 16 | 32 | 64
// rows, one tensor, then seven in a launch: 512 x 512 (32 blocks of 16) 7.5 | 9.0 | 11.8, 10.8 | 10.2 | 13.3; 128 x 4096 (64) 7.7 |
// 9.1 | 11.6, 11.3 | 11.3 | 14.3; 300 x 2048 (76) 8.2 | 9.4 | -, 14.1 | 13.4 | -, four 12.1 | 11.2; 256 x 4096 (128) 8.6 | 9.4 | 12.0,
// 17.0 | 14.7 | 16.6; with 32 | 64 rows, one tensor, two, seven (28672: four): 1777 x 5120 (280 blocks of 64) 19.6 | 19.9, 28.5 |
// 29.4, 74.7 | 74.0, a layer of 13B 76 | 74; 2048 x 5120 (320) 19.6 | 20.2, 31.4 | 30.1, 84.5 | 83.1; 1024 x 13824 (432) 22.6 | 21.9,
// 38.5 | 39.8, 124 | 115; 400 x 28672 (392) 18.8 | 20.2, 31.5 | 31.7, 54.5 | 57.3; 2100 x 4096 (264) 20.6 | 20.3, 30.0 | 32.3, 70 | 75;
// 3000 x 4096 (376) 23.6 | 21.7, 36.6 | 35.8, 95 | 98; 4096 x 4096 (512) 29.1 | 30.5, 46 | 49, 139 | 147; 4096 x 5120 (640) 32.6 |
// 29.7, -, 169 | 164.
// (The long chunks' sums are no less exact: fp64 from four rows on; ds is off by 5.2e-8 of its norm, 5.9e-8 with fp32 chunks of
// 16 rows, 8.8e-8 with those of 32.)
constexpr int kPcMinRowsShort = 16, kPcMinRowsLong = 64;
constexpr int64_t kPcShortBlocks = 64, kPcLongBlocks = 512, kPcLongBlocksWide = 256, kPcWideCols = 4608, kPcWideRows = 704;

struct PcConst {
    float inv_s[8];
    float s[8];
    float lo, hi;
};

__device__ __forceinline__ PcConst load_pc(const float* __restrict__ s, int64_t col0, int64_t cols, int bits)
{
    PcConst c;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float v = s[col0 + e < cols ? col0 + e : cols - 1];
        c.s[e] = v;
        c.inv_s[e] = 1.0f / v;
    }
    c.lo = kMagic - (float)(1 << (bits - 1));
    c.hi = kMagic + (float)((1 << (bits - 1)) - 1);
    return c;
}

__device__ __forceinline__ QElem quantize_pc(float x, float inv_s, const PcConst& c)
{
    QElem e;
    e.f = __builtin_fmaf(x, inv_s, kMagic);
    e.c = __builtin_amdgcn_fmed3f(e.f, c.lo, c.hi);
    return e;
}

// The block (col_block, row_chunk) of one tensor's grid: the kernels below pass their block
// indices, or (batched) the position inside the tensor's run of blocks.
template <int DT, bool CODES>
__device__ __forceinline__ void fwd_pc_body(
    const uint16_t* __restrict__ x, const float* __restrict__ s, uint16_t* __restrict__ y,
    int8_t* __restrict__ codes, int64_t rows, int64_t cols, int64_t rows_per_chunk, int bits,
    int col_block, int row_chunk)
{
    using S = Store16<DT>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t col0 = (int64_t)col_block * kPcColsPerBlock + lane * 8;
    if (col0 >= cols) return;
    const int64_t r_begin = (int64_t)row_chunk * rows_per_chunk;
    const int64_t r_end = min(rows, r_begin + rows_per_chunk);
    // Groups of kPcRowUnroll rows per wave, double-buffered: the next group's loads are in flight
    // while the current one is computed, and the first group's loads are issued before the
    // column factors are fetched and inverted (few waves per CU: latency must be hidden in-wave).
    constexpr int64_t kStep = kPcWaves * kPcRowUnroll;
    auto full = [&](int64_t rr) { return rr + (kPcRowUnroll - 1) * kPcWaves < r_end; };
    auto load_group = [&](u32x4 (&buf)[kPcRowUnroll], int64_t rr) {
#pragma unroll
        for (int u = 0; u < kPcRowUnroll; ++u)
            buf[u] = *reinterpret_cast<const u32x4*>(x + (rr + u * kPcWaves) * cols + col0);
    };
    int64_t r = r_begin + wave;
    u32x4 bufa[kPcRowUnroll], bufb[kPcRowUnroll];
    bool have = full(r);
    if (have) load_group(bufa, r);
    const PcConst c = load_pc(s, col0, cols, bits);
    auto one_row = [&](const u32x4 in, int64_t rr) {
        u32x4 out;
        float cc[8];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            QElem a = quantize_pc(S::lo(in[w]), c.inv_s[2 * w], c);
            QElem b = quantize_pc(S::hi(in[w]), c.inv_s[2 * w + 1], c);
            out[w] = S::pack(codef_of(a) * c.s[2 * w], codef_of(b) * c.s[2 * w + 1]);
            cc[2 * w] = a.c;
            cc[2 * w + 1] = b.c;
        }
        __builtin_nontemporal_store(out, reinterpret_cast<u32x4*>(y + rr * cols + col0));
        if (CODES) {
            u32x2 cw = {pack_codes4(cc[0], cc[1], cc[2], cc[3]), pack_codes4(cc[4], cc[5], cc[6], cc[7])};
            *reinterpret_cast<u32x2*>(codes + rr * cols + col0) = cw;
        }
    };
    // full groups without per-row predication (a clamp or an early exit inside the unrolled loop
    // makes the compiler serialize the loads), then the leftover rows
    while (have) {
        bool more = full(r + kStep);
        if (more) load_group(bufb, r + kStep);
#pragma unroll
        for (int u = 0; u < kPcRowUnroll; ++u) one_row(bufa[u], r + u * kPcWaves);
        r += kStep;
        have = more;
        if (!have) break;
        more = full(r + kStep);
        if (more) load_group(bufa, r + kStep);
#pragma unroll
        for (int u = 0; u < kPcRowUnroll; ++u) one_row(bufb[u], r + u * kPcWaves);
        r += kStep;
        have = more;
    }
    for (; r < r_end; r += kPcWaves)
        one_row(*reinterpret_cast<const u32x4*>(x + r * cols + col0), r);
}

template <int DT, bool CODES>
__global__ __launch_bounds__(kPcThreads) void fakequant_fwd_pc_kernel(
    const uint16_t* __restrict__ x, const float* __restrict__ s, uint16_t* __restrict__ y,
    int8_t* __restrict__ codes, int64_t rows, int64_t cols, int64_t rows_per_chunk, int bits)
{
    fwd_pc_body<DT, CODES>(x, s, y, codes, rows, cols, rows_per_chunk, bits, (int)blockIdx.x, (int)blockIdx.y);
}

// SHORT: chunks of 16 rows, four a wave: a thread's sum is the fp32 sum of four rows and needs no fp64 before the waves meet, and
// there is no loop.  The same bits; 512 x 512 8.0 us in the general form, 7.5 in this, 64 x 4096 7.8 and 7.3.  A kernel has one form:
// with both the bf16 batch needs 173 registers, which leaves two waves a SIMD instead of three.
template <int DT, bool WRITE_DX, bool SHORT>
__device__ __forceinline__ void bwd_pc_body(
    const uint16_t* __restrict__ x, const uint16_t* dy, const float* __restrict__ s,
    uint16_t* dx, float* __restrict__ ds, uint32_t* __restrict__ tickets, float* __restrict__ partials,
    int64_t rows, int64_t cols, int64_t rows_per_chunk, int bits,
    int col_block, int row_chunk, int nchunks, double (&red)[kPcWaves][kPcColsPerBlock], bool& is_last)
{
    using S = Store16<DT>;
    static_assert(kPcWaves * kPcRowUnroll == 16, "a chunk of 16 rows is one group");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t cbase = (int64_t)col_block * kPcColsPerBlock;
    const int64_t col0 = cbase + lane * 8;
    const bool active = col0 < cols;
    // four rows are summed in fp32, everything above that in fp64 up to the block's partial
    using Sum = std::conditional_t<SHORT, float, double>;
    Sum sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (active) {
        const int64_t r_begin = (int64_t)row_chunk * rows_per_chunk;
        const int64_t r_end = min(rows, r_begin + rows_per_chunk);
        // same double-buffered traversal as the forward kernel, two input streams
        constexpr int64_t kStep = kPcWaves * kPcRowUnroll;
        auto full = [&](int64_t rr) { return rr + (kPcRowUnroll - 1) * kPcWaves < r_end; };
        auto load_group = [&](u32x4 (&bx)[kPcRowUnroll], u32x4 (&bg)[kPcRowUnroll], int64_t rr) {
#pragma unroll
            for (int u = 0; u < kPcRowUnroll; ++u) {
                bx[u] = *reinterpret_cast<const u32x4*>(x + (rr + u * kPcWaves) * cols + col0);
                bg[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(dy + (rr + u * kPcWaves) * cols + col0));
            }
        };
        int64_t r = r_begin + wave;
        u32x4 xa_[kPcRowUnroll], ga_[kPcRowUnroll], xb_[kPcRowUnroll], gb_[kPcRowUnroll];
        bool have = full(r);
        if (have) load_group(xa_, ga_, r);
        const PcConst c = load_pc(s, col0, cols, bits);
        float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        auto add_group = [&]() {
#pragma unroll
            for (int e = 0; e < 8; ++e) { sum[e] = SHORT ? (Sum)acc[e] : sum[e] + (Sum)acc[e]; if (!SHORT) acc[e] = 0.0f; }
        };
        auto one_row = [&](const u32x4 xin, const u32x4 gin, int64_t rr) {
            u32x4 out;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float xa = S::lo(xin[w]), xb = S::hi(xin[w]);
                QElem a = quantize_pc(xa, c.inv_s[2 * w], c);
                QElem b = quantize_pc(xb, c.inv_s[2 * w + 1], c);
                const bool ka = unclipped(a), kb = unclipped(b);
                const float qa = codef_of(a), qb = codef_of(b);
                const float ua = __builtin_fmaf(-xa, c.inv_s[2 * w], qa), ub = __builtin_fmaf(-xb, c.inv_s[2 * w + 1], qb);
                acc[2 * w] += S::lo(gin[w]) * (ka ? ua : qa);
                acc[2 * w + 1] += S::hi(gin[w]) * (kb ? ub : qb);
                out[w] = gin[w] & ((ka ? 0x0000FFFFu : 0u) | (kb ? 0xFFFF0000u : 0u));
            }
            if (WRITE_DX) __builtin_nontemporal_store(out, reinterpret_cast<u32x4*>(dx + rr * cols + col0));
        };
        // full groups, then the leftover rows (same row order per wave either way)
        if (SHORT && have) {
#pragma unroll
            for (int u = 0; u < kPcRowUnroll; ++u) one_row(xa_[u], ga_[u], r + u * kPcWaves);
            r = r_end;
        }
        while (!SHORT && have) {
            bool more = full(r + kStep);
            if (more) load_group(xb_, gb_, r + kStep);
#pragma unroll
            for (int u = 0; u < kPcRowUnroll; ++u) one_row(xa_[u], ga_[u], r + u * kPcWaves);
            add_group();
            r += kStep;
            have = more;
            if (!have) break;
            more = full(r + kStep);
            if (more) load_group(xa_, ga_, r + kStep);
#pragma unroll
            for (int u = 0; u < kPcRowUnroll; ++u) one_row(xb_[u], gb_[u], r + u * kPcWaves);
            add_group();
            r += kStep;
            have = more;
        }
        for (; r < r_end; r += kPcWaves)
            one_row(*reinterpret_cast<const u32x4*>(x + r * cols + col0),
                    __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(dy + r * cols + col0)), r);
        add_group();
    }
    // block partial per column: waves in fixed order
    Sum* part = reinterpret_cast<Sum*>(&red[0][0]);
#pragma unroll
    for (int e = 0; e < 8; ++e) part[wave * kPcColsPerBlock + lane * 8 + e] = sum[e];
    __syncthreads();
    // One 128-bit store per 4 columns, with the agent-scope cache policy the compiler gives its own
    // agent-scope atomic stores (sc1): 4-byte stores of the same data are four times as many
    // write-through transactions, and every block waits for their acknowledgement below.
    if (threadIdx.x < kPcColsPerBlock / 4) {
        const int c4 = threadIdx.x * 4;
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double a = 0.0;
#pragma unroll
            for (int w = 0; w < kPcWaves; ++w) a += (double)part[w * kPcColsPerBlock + c4 + e];
            v[e] = (float)a;
        }
        if (cbase + c4 < cols) {        // cols is a multiple of 8: a group of 4 is all in or all out
            float* dst = &partials[(int64_t)row_chunk * cols + cbase + c4];
            asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(dst), "v"(v) : "memory");
        }
    }
    // the stores above are agent-scope (sc1: written through to the level all XCDs share) and
    // acknowledged before the ticket is taken: see publish_then_ticket in sasq_device.h
    wait_stores_acknowledged();
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t ticket = __hip_atomic_fetch_add(&tickets[col_block], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        is_last = (ticket == (uint32_t)nchunks - 1);
        if (ticket >= (uint32_t)nchunks) ds[cbase < cols ? cbase : 0] = __uint_as_float(0x7FC00000u);   // uninitialised workspace
    }
    __syncthreads();
    if (!is_last) return;
    // last block of this column chunk: row chunks summed in ascending order, in fp64.  The
    // acquire fence makes the other blocks' write-through partials visible to ordinary loads.  A
    // thread takes four adjacent columns (one 128-bit load per row chunk) of one half of the row
    // chunks and keeps 32 loads in flight (loading them a few at a time leaves the whole grid's
    // tail waiting on a chain of memory latencies); the halves meet in LDS, lower half first.
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    {
        constexpr int kBatch = 32;
        const int half = threadIdx.x >> 7;                               // 0: first half of the chunks, 1: second
        const int c4 = (threadIdx.x & 127) * 4;
        const bool ok = cbase + c4 < cols;                               // cols is a multiple of 8
        const uint32_t colv = ok ? (uint32_t)c4 : 0u;
        const int split = (nchunks + 1) >> 1;
        const int rc_begin = half ? split : 0, rc_end = half ? nchunks : split;
        double t[4] = {0.0, 0.0, 0.0, 0.0};
        for (int rc0 = rc_begin; rc0 < rc_end; rc0 += kBatch) {
            f32x4 pv[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int rc = rc0 + j < rc_end ? rc0 + j : nchunks - 1;
                const float* rowp = partials + (int64_t)rc * cols + cbase;  // uniform: scalar base, lane offset
                pv[j] = *reinterpret_cast<const f32x4*>(rowp + colv);
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j)
                if (rc0 + j < rc_end) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[e] += (double)pv[j][e];
                }
        }
        double* meet = &red[0][0];
        __syncthreads();                                                 // red's earlier contents are consumed
        if (half) {
#pragma unroll
            for (int e = 0; e < 4; ++e) meet[c4 + e] = t[e];
        }
        __syncthreads();
        if (!half && ok) {
            f32x4 out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (float)(t[e] + meet[c4 + e]);
            *reinterpret_cast<f32x4*>(&ds[cbase + c4]) = out;
        }
    }
    if (threadIdx.x == 0) __hip_atomic_store(&tickets[col_block], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int DT, bool WRITE_DX, bool SHORT>
__global__ __launch_bounds__(kPcThreads) void fakequant_bwd_pc_kernel(
    const uint16_t* __restrict__ x, const uint16_t* dy, const float* __restrict__ s,
    uint16_t* dx, float* __restrict__ ds, uint32_t* __restrict__ tickets, float* __restrict__ partials,
    int64_t rows, int64_t cols, int64_t rows_per_chunk, int bits)
{
    __shared__ double red[kPcWaves][kPcColsPerBlock];
    __shared__ bool is_last;
    bwd_pc_body<DT, WRITE_DX, SHORT>(x, dy, s, dx, ds, tickets, partials, rows, cols, rows_per_chunk, bits,
                                     (int)blockIdx.x, (int)blockIdx.y, (int)gridDim.y, red, is_last);
}

// ---- several tensors in one launch -------------------------------------------------------------
// Each tensor owns a run of consecutive block ids, column block fastest (the order a 2-D grid
// dispatches in); one launch for the fake-quant operators of a layer pays one ramp and one drain.
struct PcItem {
    const uint16_t* x;
    const uint16_t* dy;
    const float* s;
    uint16_t* out;        // y (forward) or dx (backward, may be null)
    float* ds;
    uint32_t* tickets;
    float* partials;
    int64_t rows, cols, rpc;
    int col_blocks, chunks;
};
struct PcBatch {
    PcItem it[SASQ_MAX_BATCH];
    int first_block[SASQ_MAX_BATCH + 1];
    int count;
};

__device__ __forceinline__ int pc_item_of(const PcBatch& b, int bid)
{
    int k = 0;
#pragma unroll
    for (int i = 1; i < SASQ_MAX_BATCH; ++i)
        if (i < b.count && bid >= b.first_block[i]) k = i;
    return k;
}

template <int DT>
__global__ __launch_bounds__(kPcThreads) void fakequant_fwd_pc_batch_kernel(const PcBatch b, int bits)
{
    const int k = pc_item_of(b, (int)blockIdx.x);
    const PcItem& it = b.it[k];
    const int lb = (int)blockIdx.x - b.first_block[k];
    fwd_pc_body<DT, false>(it.x, it.s, it.out, nullptr, it.rows, it.cols, it.rpc, bits, lb % it.col_blocks, lb / it.col_blocks);
}

template <int DT, bool SHORT>
__global__ __launch_bounds__(kPcThreads) void fakequant_bwd_pc_batch_kernel(const PcBatch b, int bits)
{
    __shared__ double red[kPcWaves][kPcColsPerBlock];
    __shared__ bool is_last;
    const int k = pc_item_of(b, (int)blockIdx.x);
    const PcItem& it = b.it[k];
    const int lb = (int)blockIdx.x - b.first_block[k];
    const int cb = lb % it.col_blocks, rc = lb / it.col_blocks;
    if (it.out) bwd_pc_body<DT, true, SHORT>(it.x, it.dy, it.s, it.out, it.ds, it.tickets, it.partials, it.rows, it.cols, it.rpc, bits,
                                             cb, rc, it.chunks, red, is_last);
    else        bwd_pc_body<DT, false, SHORT>(it.x, it.dy, it.s, nullptr, it.ds, it.tickets, it.partials, it.rows, it.cols, it.rpc, bits,
                                              cb, rc, it.chunks, red, is_last);
}

// cols not a multiple of 8: one thread per column walks the rows (rarely used, kept simple)
template <int DT>
__global__ void fakequant_pc_scalar_kernel(const uint16_t* __restrict__ x, const uint16_t* dy, const float* __restrict__ s,
                                           uint16_t* y, int8_t* codes, uint16_t* dx, float* ds,
                                           int64_t rows, int64_t cols, int bits, int backward)
{
    using S = Store16<DT>;
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= cols) return;
    const QConst c = make_qconst(s[k], bits);
    double acc = 0.0;
    for (int64_t r = 0; r < rows; ++r) {
        const int64_t i = r * cols + k;
        const float xv = S::one(x[i]);
        const QElem e = quantize(xv, c);
        if (!backward) {
            y[i] = S::enc(codef_of(e) * c.s);
            if (codes) codes[i] = (int8_t)code_of(e);
        } else {
            const bool keep = unclipped(e);
            const float q = codef_of(e);
            const uint16_t g = dy[i];
            acc += (double)(S::one(g) * (keep ? __builtin_fmaf(-xv, c.inv_s, q) : q));
            if (dx) dx[i] = keep ? g : (uint16_t)0;
        }
    }
    if (backward) ds[k] = (float)acc;
}

// Row chunks of a tensor, `rows_min` rows each at least: enough blocks to fill the chip, at most kPcMaxRowChunks (the
// workspace has room for that many partials), whole unpredicated groups of 16 rows in every chunk but the last.
static void pc_geometry(int64_t rows, int64_t cols, int64_t rows_min, int64_t& col_blocks, int64_t& rpc, int& chunks)
{
    col_blocks = (cols + kPcColsPerBlock - 1) / kPcColsPerBlock;
    int64_t want = (kPcTargetBlocks + col_blocks - 1) / col_blocks;
    const int64_t by_rows = (rows + rows_min - 1) / rows_min;
    if (want > by_rows) want = by_rows;
    if (want > kPcMaxRowChunks) want = kPcMaxRowChunks;
    rpc = ((rows + want - 1) / want + 15) / 16 * 16;
    chunks = (int)((rows + rpc - 1) / rpc);
}

static int64_t pc_blocks16(int64_t rows, int64_t cols)
{
    return (cols + kPcColsPerBlock - 1) / kPcColsPerBlock * ((rows + 15) / 16);
}

// The backward's row chunks (rule and figures at kPcMinRowsShort)
static void pc_geometry_bwd(int64_t rows, int64_t cols, int64_t& col_blocks, int64_t& rpc, int& chunks)
{
    auto blocks = [&](int64_t n) { return (cols + kPcColsPerBlock - 1) / kPcColsPerBlock * ((rows + n - 1) / n); };
    const int64_t rows_min = blocks(kPcMinRowsShort) <= kPcShortBlocks ? kPcMinRowsShort
                           : blocks(kPcMinRowsLong) > (cols > kPcWideCols && rows >= kPcWideRows ? kPcLongBlocksWide : kPcLongBlocks) ? kPcMinRowsLong
                           : kPcMinRows;
    pc_geometry(rows, cols, rows_min, col_blocks, rpc, chunks);
}

static int check_pc(int64_t rows, int64_t cols, int bits, int dt)
{
    if (rows <= 0 || cols <= 0) return SASQ_ERR_SHAPE;
    if (rows > (INT64_C(1) << 40) / cols) return SASQ_ERR_SHAPE;
    if ((cols + kPcColsPerBlock - 1) / kPcColsPerBlock > (int64_t)(kWsHeaderBytes / 4)) return SASQ_ERR_SHAPE;
    if (bits < 2 || bits > 8) return SASQ_ERR_UNSUPPORTED;
    if (dt != SASQ_F16 && dt != SASQ_BF16) return SASQ_ERR_UNSUPPORTED;
    return SASQ_OK;
}

}  // namespace sasq

using namespace sasq;

extern "C" int sasq_fakequant_fwd_pc(const void* x, const float* s, void* y, int8_t* codes,
                                     int64_t rows, int64_t cols, int bits, sasq_dtype dt, void* stream)
{
    if (!x || !s || !y) return SASQ_ERR_NULL;
    int rc = check_pc(rows, cols, bits, (int)dt);
    if (rc) return rc;
    if (!aligned16(x) || !aligned16(y) || (codes && (reinterpret_cast<uintptr_t>(codes) & 7u))) return SASQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);
    auto X = static_cast<const uint16_t*>(x);
    auto Y = static_cast<uint16_t*>(y);
    if (cols % 8 != 0) {
        const int blocks = (int)((cols + 255) / 256);
        if (dt == SASQ_F16) fakequant_pc_scalar_kernel<SASQ_F16><<<blocks, 256, 0, st>>>(X, nullptr, s, Y, codes, nullptr, nullptr, rows, cols, bits, 0);
        else                fakequant_pc_scalar_kernel<SASQ_BF16><<<blocks, 256, 0, st>>>(X, nullptr, s, Y, codes, nullptr, nullptr, rows, cols, bits, 0);
        return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
    }
    int64_t col_blocks, rpc;
    int chunks;
    pc_geometry(rows, cols, pc_fwd_rows(pc_blocks16(rows, cols)), col_blocks, rpc, chunks);
    dim3 grid((unsigned)col_blocks, (unsigned)chunks);
    if (dt == SASQ_F16) {
        if (codes) fakequant_fwd_pc_kernel<SASQ_F16, true><<<grid, kPcThreads, 0, st>>>(X, s, Y, codes, rows, cols, rpc, bits);
        else       fakequant_fwd_pc_kernel<SASQ_F16, false><<<grid, kPcThreads, 0, st>>>(X, s, Y, codes, rows, cols, rpc, bits);
    } else {
        if (codes) fakequant_fwd_pc_kernel<SASQ_BF16, true><<<grid, kPcThreads, 0, st>>>(X, s, Y, codes, rows, cols, rpc, bits);
        else       fakequant_fwd_pc_kernel<SASQ_BF16, false><<<grid, kPcThreads, 0, st>>>(X, s, Y, codes, rows, cols, rpc, bits);
    }
    return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
}

extern "C" size_t sasq_fakequant_bwd_pc_workspace(int64_t rows, int64_t cols)
{
    (void)rows;
    if (cols <= 0) return kWsHeaderBytes;
    return kWsHeaderBytes + sizeof(float) * (size_t)kPcMaxRowChunks * (size_t)cols;
}

extern "C" int sasq_fakequant_bwd_pc(const void* x, const void* dy, const float* s, void* dx, float* ds,
                                     int64_t rows, int64_t cols, int bits, sasq_dtype dt,
                                     void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !dy || !s || !ds) return SASQ_ERR_NULL;
    int rc = check_pc(rows, cols, bits, (int)dt);
    if (rc) return rc;
    if (!aligned16(x) || !aligned16(dy) || (dx && !aligned16(dx))) return SASQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);
    auto X = static_cast<const uint16_t*>(x);
    auto G = static_cast<const uint16_t*>(dy);
    auto DX = static_cast<uint16_t*>(dx);
    if (cols % 8 != 0) {
        const int blocks = (int)((cols + 255) / 256);
        if (dt == SASQ_F16) fakequant_pc_scalar_kernel<SASQ_F16><<<blocks, 256, 0, st>>>(X, G, s, nullptr, nullptr, DX, ds, rows, cols, bits, 1);
        else                fakequant_pc_scalar_kernel<SASQ_BF16><<<blocks, 256, 0, st>>>(X, G, s, nullptr, nullptr, DX, ds, rows, cols, bits, 1);
        return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
    }
    if (!workspace || workspace_bytes < sasq_fakequant_bwd_pc_workspace(rows, cols)) return SASQ_ERR_WORKSPACE;
    if (!aligned16(workspace)) return SASQ_ERR_ALIGN;
    int64_t col_blocks, rpc;
    int chunks;
    pc_geometry_bwd(rows, cols, col_blocks, rpc, chunks);
    dim3 grid((unsigned)col_blocks, (unsigned)chunks);
    auto tickets = static_cast<uint32_t*>(workspace);
    auto parts = reinterpret_cast<float*>(static_cast<char*>(workspace) + kWsHeaderBytes);
    auto launch = [&](auto dt_tag, auto dx_tag, auto short_tag) {
        fakequant_bwd_pc_kernel<decltype(dt_tag)::value, decltype(dx_tag)::value, decltype(short_tag)::value><<<grid, kPcThreads, 0, st>>>(
            X, G, s, DX, ds, tickets, parts, rows, cols, rpc, bits);
    };
    auto by_chunk = [&](auto dt_tag, auto dx_tag) {
        if (rpc <= 16) launch(dt_tag, dx_tag, std::true_type{});
        else           launch(dt_tag, dx_tag, std::false_type{});
    };
    auto by_dx = [&](auto dt_tag) {
        if (dx) by_chunk(dt_tag, std::true_type{});
        else    by_chunk(dt_tag, std::false_type{});
    };
    if (dt == SASQ_F16) by_dx(std::integral_constant<int, SASQ_F16>{});
    else                by_dx(std::integral_constant<int, SASQ_BF16>{});
    return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
}

// ---- batched entry points ----------------------------------------------------------------------
namespace sasq {

constexpr size_t kPcBatchLaunchBytes = (size_t)192 << 20;   // bytes of x per launch: more concurrent streams run slower

static int check_pc_items(const sasq_fq_item* items, int count, int bits, sasq_dtype dt, bool backward)
{
    if (!items) return SASQ_ERR_NULL;
    if (count < 1 || count > SASQ_MAX_BATCH) return SASQ_ERR_SHAPE;
    for (int i = 0; i < count; ++i) {
        const sasq_fq_item& it = items[i];
        if (!it.x || !it.s || (backward ? (!it.dy || !it.ds) : !it.out)) return SASQ_ERR_NULL;
        int rc = check_pc(it.rows, it.cols, bits, (int)dt);
        if (rc) return rc;
        if (it.cols % 8) return SASQ_ERR_SHAPE;              // such tensors take the single-tensor call
        if (!aligned16(it.x) || (it.out && !aligned16(it.out)) || (backward && !aligned16(it.dy))) return SASQ_ERR_ALIGN;
    }
    return SASQ_OK;
}

// Workspace of a batch: the 1 KB header holds the tickets of all items back to back (one word per
// column block; sasq_workspace_init clears exactly that header), each item's partials follow.
struct PcBatchLayout {
    size_t ticket_word[SASQ_MAX_BATCH];
    size_t partials_off[SASQ_MAX_BATCH];
    size_t total;
    bool fits;
};

static PcBatchLayout pc_batch_layout(const sasq_fq_item* items, int count)
{
    PcBatchLayout L;
    size_t words = 0, off = kWsHeaderBytes;
    for (int i = 0; i < count; ++i) {
        L.ticket_word[i] = words;
        L.partials_off[i] = off;
        const int64_t cols = items[i].cols > 0 ? items[i].cols : 0;
        words += (size_t)((cols + kPcColsPerBlock - 1) / kPcColsPerBlock);
        off += sizeof(float) * (size_t)kPcMaxRowChunks * (size_t)cols;
    }
    L.total = off;
    L.fits = words <= kWsHeaderBytes / 4;
    return L;
}

// Launches items [i0, i1) as one grid.
template <bool BACKWARD>
static int launch_pc_batch(const sasq_fq_item* items, int i0, int i1, int bits, sasq_dtype dt, char* ws,
                           const PcBatchLayout* L, hipStream_t st)
{
    PcBatch b;
    memset(&b, 0, sizeof(b));
    int64_t blocks = 0, blocks16 = 0, longest = 0;
    for (int i = i0; i < i1; ++i) blocks16 += pc_blocks16(items[i].rows, items[i].cols);
    for (int i = i0; i < i1; ++i) {
        const sasq_fq_item& src = items[i];
        PcItem& it = b.it[i - i0];
        int64_t col_blocks;
        if (BACKWARD) pc_geometry_bwd(src.rows, src.cols, col_blocks, it.rpc, it.chunks);
        else          pc_geometry(src.rows, src.cols, pc_fwd_rows(blocks16), col_blocks, it.rpc, it.chunks);
        longest = it.rpc > longest ? it.rpc : longest;
        it.col_blocks = (int)col_blocks;
        it.x = static_cast<const uint16_t*>(src.x);
        it.dy = static_cast<const uint16_t*>(src.dy);
        it.s = src.s;
        it.out = static_cast<uint16_t*>(src.out);
        it.ds = src.ds;
        it.rows = src.rows;
        it.cols = src.cols;
        if (BACKWARD) {
            it.tickets = reinterpret_cast<uint32_t*>(ws) + L->ticket_word[i];
            it.partials = reinterpret_cast<float*>(ws + L->partials_off[i]);
        }
        b.first_block[i - i0] = (int)blocks;
        blocks += col_blocks * it.chunks;
        if (blocks > 0x7FFFFFFF) return SASQ_ERR_SHAPE;
    }
    b.count = i1 - i0;
    b.first_block[b.count] = (int)blocks;
    if (BACKWARD) {
        auto launch = [&](auto dt_tag) {                     // chunks of 16 rows beside longer ones take the general form
            constexpr int DT = decltype(dt_tag)::value;
            if (longest <= 16) fakequant_bwd_pc_batch_kernel<DT, true><<<(int)blocks, kPcThreads, 0, st>>>(b, bits);
            else               fakequant_bwd_pc_batch_kernel<DT, false><<<(int)blocks, kPcThreads, 0, st>>>(b, bits);
        };
        if (dt == SASQ_F16) launch(std::integral_constant<int, SASQ_F16>{});
        else                launch(std::integral_constant<int, SASQ_BF16>{});
    } else {
        if (dt == SASQ_F16) fakequant_fwd_pc_batch_kernel<SASQ_F16><<<(int)blocks, kPcThreads, 0, st>>>(b, bits);
        else                fakequant_fwd_pc_batch_kernel<SASQ_BF16><<<(int)blocks, kPcThreads, 0, st>>>(b, bits);
    }
    return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
}

template <bool BACKWARD>
static int run_pc_batch(const sasq_fq_item* items, int count, int bits, sasq_dtype dt, char* ws, const PcBatchLayout* L,
                        hipStream_t st)
{
    // consecutive items share a launch while their input stays under the per-launch cap
    int i0 = 0;
    while (i0 < count) {
        size_t bytes = 0;
        int i1 = i0;
        while (i1 < count) {
            const size_t add = (size_t)items[i1].rows * (size_t)items[i1].cols * 2;      // bytes of x, as the per-tensor batch counts
            if (i1 > i0 && bytes + add > kPcBatchLaunchBytes) break;
            bytes += add;
            ++i1;
        }
        int rc = launch_pc_batch<BACKWARD>(items, i0, i1, bits, dt, ws, L, st);
        if (rc) return rc;
        i0 = i1;
    }
    return SASQ_OK;
}

}  // namespace sasq

extern "C" int sasq_fakequant_fwd_pc_batch(const sasq_fq_item* items, int count, int bits, sasq_dtype dt, void* stream)
{
    int rc = check_pc_items(items, count, bits, dt, false);
    if (rc) return rc;
    return run_pc_batch<false>(items, count, bits, dt, nullptr, nullptr, as_stream(stream));
}

extern "C" size_t sasq_fakequant_bwd_pc_batch_workspace(const sasq_fq_item* items, int count)
{
    if (!items || count < 1 || count > SASQ_MAX_BATCH) return 0;
    const PcBatchLayout L = pc_batch_layout(items, count);
    return L.fits ? L.total : 0;
}

extern "C" int sasq_fakequant_bwd_pc_batch(const sasq_fq_item* items, int count, int bits, sasq_dtype dt,
                                           void* workspace, size_t workspace_bytes, void* stream)
{
    int rc = check_pc_items(items, count, bits, dt, true);
    if (rc) return rc;
    const PcBatchLayout L = pc_batch_layout(items, count);
    if (!L.fits) return SASQ_ERR_SHAPE;                      // more than 256 column blocks in all
    if (!workspace || workspace_bytes < L.total) return SASQ_ERR_WORKSPACE;
    if (!aligned16(workspace)) return SASQ_ERR_ALIGN;
    return run_pc_batch<true>(items, count, bits, dt, static_cast<char*>(workspace), &L, as_stream(stream));
}

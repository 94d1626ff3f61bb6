// int8 linear for few rows (token generation): Y = X . W^T where M is a handful of rows and the weights are what is read;
// and for some hundred rows where the GEMM's tiles are too few to fill the chip (a chunk of a prefill), in row blocks.
//
// What bounds it: the weight bytes (a 7B layer's seven projections at 8 rows, int8: 202 MB in 36 us = 5.6 TB/s, the GEMM's
// tiles took 93; a 13B layer's at one row, int4: 159 MB in 30 us, from 128; row-major int8, whose rows are gathered in
// 64-byte pieces: 51 us).  The tiled GEMM hands out 256 (or 128) weight rows per workgroup, which at small M is
// a few dozen workgroups with a K loop that nothing overlaps.  Here a workgroup owns 16 NT weight rows and its NW waves
// share out K: a wave streams its part of the weights straight from memory into MFMA operand registers (a pre-arranged
// 1 KB block IS one operand read of a wave), D K tiles ahead, with no LDS and no barrier until the waves' int32 sums are
// added up at the end, so that some thousand waves each keep several KB in flight.  Integer sums make the split exact.
// QX: the activations are quantized on the way into the operand registers, 16 elements per lane and K tile, which takes
// the pre-pass's launch out of the call; each workgroup repeats that work, so it is for at most 16 rows.  Otherwise the
// codes come from the pre-pass in their staging blocks.
// Row blocks (more than 64 rows): what bounds them is the operands' delivery from L2, (BM + 64) K bytes per workgroup for
// BM x 64 outputs; 333 x 4096 x 4096 takes 18.7 us with its pre-pass, 27.1 on 96 GEMM tiles of 128 x 128
// (weights that the caches hold; other ones each call: 21.6).
#include "sasq_device.h"
#include "gemm_tile.h"
#include "gemm_k64.h"
#include <type_traits>

namespace sasq {

template <int DT, int WMODE, int MT, int NT, int NW, int D, bool QX>
__device__ __forceinline__
void skinny_body(const LinItem& it, int mblk, int nblk, int a_bits, int32_t* __restrict__ acc_out, char* lds)
{
    using S = Store16<DT>;
    constexpr bool I4 = WMODE == 3, ROWMAJOR = WMODE == 0;
    static_assert(!I4 || NT % 2 == 0, "int4 blocks hold 32 weight rows");
    constexpr int WL = I4 ? NT / 2 : NT;               // 128-bit weight loads per lane and K tile
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int frow = lane & 15, fq = lane >> 4;
    const int M = it.M, N = it.N, K = it.K, KT = K >> 6;
    const int m0 = mblk * 16 * MT, n0 = nblk * 16 * NT;

    // This wave's K tiles: an equal run of consecutive ones.
    const int per = (KT + NW - 1) / NW;
    const int t0 = min(wave * per, KT), count = min(per, KT - t0);

    // Scalar base + 32-bit lane offset for every stream; a base advances 1 KB (or 64 bytes of a row) per K tile.
    const char* wbase[WL];
    uint32_t woff;
    if (I4) {
        // Lane l takes 16 bytes: the K tile's codes 16 (l/16) .. + 15 of the weight rows 2 (l%16) and 2 (l%16) + 1.
        woff = 256 * fq + 16 * frow;
    } else if (ROWMAJOR) {
        woff = (uint32_t)(16 * fq);                     // + the row, below
    } else {
        woff = (4 * frow + (fq ^ swz64(frow))) * 16;
    }
#pragma unroll
    for (int j = 0; j < WL; ++j) {
        const char* w = reinterpret_cast<const char*>(it.wq);
        if (I4)            wbase[j] = w + ((int64_t)min((n0 >> 5) + j, (N - 1) >> 5) * KT + t0) * 1024;
        else if (ROWMAJOR) wbase[j] = w + (int64_t)min(n0 + 16 * j, ((N - 1) >> 4) << 4) * K + (int64_t)t0 * 64;
        else               wbase[j] = w + ((int64_t)min((n0 >> 4) + j, (N - 1) >> 4) * KT + t0) * 1024;
    }
    uint32_t wrow[ROWMAJOR ? NT : 1];                   // row-major: this lane's row inside each 16-row tile, clamped to N - 1
    if (ROWMAJOR) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int first = min(n0 + 16 * j, ((N - 1) >> 4) << 4);
            wrow[j] = (uint32_t)min(frow, N - 1 - first) * (uint32_t)K + woff;
        }
    }
    constexpr int kWStep = ROWMAJOR ? 64 : 1024;
    const char* xbase[MT];
    uint32_t xoff[MT];
#pragma unroll
    for (int b = 0; b < MT; ++b) {
        const int first = min(m0 + 16 * b, ((M - 1) >> 4) << 4);
        if (QX) {
            xbase[b] = reinterpret_cast<const char*>(it.x) + ((int64_t)first * K + (int64_t)t0 * 64) * 2;
            xoff[b] = (uint32_t)min(frow, M - 1 - first) * (uint32_t)K * 2 + fq * 32;
        } else {
            xbase[b] = reinterpret_cast<const char*>(it.xq) + ((int64_t)(first >> 4) * KT + t0) * 1024;
            xoff[b] = (4 * frow + (fq ^ swz64(frow))) * 16;
        }
    }
    constexpr int kXStep = QX ? 128 : 1024;
    const QConst qk = make_qconst(*it.s, a_bits);

    struct Frag {
        u32x4 w[WL];
        u32x4 x[MT][QX ? 2 : 1];
    };
    auto load = [&](Frag& f, int t) {
#pragma unroll
        for (int j = 0; j < WL; ++j) {
            const u32x4* p = reinterpret_cast<const u32x4*>(wbase[j] + (int64_t)t * kWStep + (ROWMAJOR ? wrow[ROWMAJOR ? j : 0] : woff));
            // Row-major: a K tile is half a 128-byte line of each row, the other half is the next K tile's; it has to stay cached
            // until then (non-temporal: 54 us for the 7B layer below, cached: 51).
            f.w[j] = ROWMAJOR ? *p : __builtin_nontemporal_load(p);
        }
#pragma unroll
        for (int b = 0; b < MT; ++b)
#pragma unroll
            for (int h = 0; h < (QX ? 2 : 1); ++h)
                f.x[b][h] = *reinterpret_cast<const u32x4*>(xbase[b] + (int64_t)t * kXStep + xoff[b] + 16 * h);
    };
    i32x4 acc[NT][MT];
#pragma unroll
    for (int g = 0; g < NT; ++g)
#pragma unroll
        for (int b = 0; b < MT; ++b) acc[g][b] = i32x4{0, 0, 0, 0};
    auto multiply = [&](const Frag& f) {
        i32x4 xv[MT];
#pragma unroll
        for (int b = 0; b < MT; ++b) {
            if constexpr (QX) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float c[8];
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        c[2 * w] = quantize(S::lo(f.x[b][h][w]), qk).c;
                        c[2 * w + 1] = quantize(S::hi(f.x[b][h][w]), qk).c;
                    }
                    xv[b][2 * h] = (int)pack_codes4(c[0], c[1], c[2], c[3]);
                    xv[b][2 * h + 1] = (int)pack_codes4(c[4], c[5], c[6], c[7]);
                }
            } else {
                xv[b] = __builtin_bit_cast(i32x4, f.x[b][0]);
            }
        }
#pragma unroll
        for (int g = 0; g < NT; ++g) {
            i32x4 wv;
            if constexpr (I4) {
                const uint32_t p0 = f.w[g / 2][2 * (g & 1)], p1 = f.w[g / 2][2 * (g & 1) + 1];   // 16 x the code in every byte
                wv = i32x4{(int)((p0 << 4) & 0xF0F0F0F0u), (int)(p0 & 0xF0F0F0F0u), (int)((p1 << 4) & 0xF0F0F0F0u), (int)(p1 & 0xF0F0F0F0u)};
            } else {
                wv = __builtin_bit_cast(i32x4, f.w[g]);
            }
#pragma unroll
            for (int b = 0; b < MT; ++b) acc[g][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wv, xv[b], acc[g][b], 0, 0, 0);
        }
    };

    Frag ring[D];
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (j < count) load(ring[j], j);
    int i = 0;
#pragma unroll 1
    for (; i + 2 * D <= count; i += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            multiply(ring[j]);
            load(ring[j], i + j + D);
        }
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (i + j < count) {
            multiply(ring[j]);
            if (i + j + D < count) load(ring[j], i + j + D);
        }
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (i + D + j < count) multiply(ring[j]);

    // The waves' sums meet in LDS; wave w finishes the output tiles w, w + NW, ...
    constexpr int kTiles = (I4 ? NT / 2 : NT) * MT, kRegs = I4 ? 2 : 1;      // int4: two tiles interleave into 32 columns
    i32x4* part = reinterpret_cast<i32x4*>(lds);
#pragma unroll
    for (int g = 0; g < NT; ++g)
#pragma unroll
        for (int b = 0; b < MT; ++b) part[((wave * NT + g) * MT + b) * 64 + lane] = acc[g][b];
    __syncthreads();
    const float s = qk.s;
#pragma unroll
    for (int t = wave; t < kTiles; t += NW) {
        const int b = t % MT, g0 = t / MT * kRegs;
        int v[4 * kRegs];
#pragma unroll
        for (int r = 0; r < kRegs; ++r) {
            i32x4 sum = {0, 0, 0, 0};
#pragma unroll
            for (int w = 0; w < NW; ++w) sum += part[((w * NT + g0 + r) * MT + b) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[kRegs * e + r] = I4 ? sum[e] >> 4 : sum[e];
        }
        const int m = m0 + 16 * b + frow, n = n0 + 16 * g0 + 4 * kRegs * fq;      // 4 (8) consecutive columns of one row
        if (m >= M || n >= N) continue;
        uint16_t* dst = it.y + (int64_t)m * N + n;
        float yv[4 * kRegs];
#pragma unroll
        for (int e = 0; e < 4 * kRegs; ++e) {
            const int ne = min(n + e, N - 1);
            float f = (float)v[e] * (s * it.s_w[ne]);
            if (it.bias) f = f + it.bias[ne];
            yv[e] = f;
        }
        if ((N & 7) == 0) {                                                  // then every full run is aligned to its own size
#pragma unroll
            for (int h = 0; h < kRegs; ++h)
                *reinterpret_cast<u32x2*>(dst + 4 * h) = u32x2{S::pack(yv[4 * h], yv[4 * h + 1]), S::pack(yv[4 * h + 2], yv[4 * h + 3])};
        } else {
#pragma unroll
            for (int e = 0; e < 4 * kRegs; ++e)
                if (n + e < N) dst[e] = S::enc(yv[e]);
        }
        if (acc_out) {
#pragma unroll
            for (int e = 0; e < 4 * kRegs; ++e)
                if (n + e < N) acc_out[(int64_t)m * N + n + e] = v[e];
        }
    }
}

template <int DT, int WMODE, int MT, int NT, int NW, int D, bool QX>
__global__ __launch_bounds__(64 * NW)
void skinny_kernel(const LinBatch b, int a_bits, int32_t* __restrict__ acc_out)
{
    __shared__ __attribute__((aligned(1024))) char lds[NW * NT * MT * 1024];
    const int k = lin_item_of(b, (int)blockIdx.x);
    // Eight neighbours in the id go to the eight XCDs: the row blocks of one run of weight rows stay on one, 8 ids apart.
    const int id = (int)blockIdx.x - b.first_block[k], octet = id >> 3, tiles_m = b.it[k].tiles_m;
    const int mblk = octet % tiles_m, nblk = octet / tiles_m * 8 + (id & 7);
    if (nblk >= b.it[k].tiles_n) return;
    skinny_body<DT, WMODE, MT, NT, NW, D, QX>(b.it[k], mblk, nblk, a_bits, acc_out, lds);
}


template <int DT, int WMODE, int MT, int NT, int NW, int D, bool QX>
static void launch_one(LinBatch& b, int a_bits, int32_t* acc_out, hipStream_t st)
{
    b.first_block[0] = 0;
    for (int i = 0; i < kMaxLinearBatch; ++i) {
        int blocks = 0;
        if (i < b.count) {
            LinItem& it = b.it[i];
            it.tiles_m = (int)(((int64_t)it.M + 16 * MT - 1) / (16 * MT));
            it.tiles_n = (int)(((int64_t)it.N + 16 * NT - 1) / (16 * NT));
            blocks = (it.tiles_n + 7) / 8 * 8 * it.tiles_m;
        }
        b.first_block[i + 1] = b.first_block[i] + blocks;
    }
    skinny_kernel<DT, WMODE, MT, NT, NW, D, QX><<<b.first_block[b.count], 64 * NW, 0, st>>>(b, a_bits, acc_out);
}

// Wide or narrow workgroups: the narrow form (16 weight rows, K over eight waves) gives four times the waves for the same
// weights, the wide one reads the activations half or a quarter as often.  Measured at 8 rows, int8, wide | narrow:
// 4096 x 4096 (256 tiles of 16 rows) 8.3 | 6.5 us, 4096 x 11008 17.3 | 12.8, 11008 x 4096 (688 tiles) 12.3 | 13.4, the 7B
// layer (2656 tiles) 36 | 51; the line lies at two workgroups of the wide form per CU.
template <int DT, int WMODE, int MT, bool QX>
static void launch_mt(LinBatch& b, int64_t tiles16, int a_bits, int32_t* acc_out, hipStream_t st)
{
    const bool wide = tiles16 >= 512;
    if constexpr (WMODE == 3) {                        // int4: half the bytes per tile, a block is two tiles
        if (!wide)             launch_one<DT, WMODE, MT, 2, 8, 2, QX>(b, a_bits, acc_out, st);
        else if constexpr (QX) launch_one<DT, WMODE, MT, 4, 8, 2, QX>(b, a_bits, acc_out, st);
        else                   launch_one<DT, WMODE, MT, 4, 4, 2, QX>(b, a_bits, acc_out, st);
    } else {
        if (!wide)               launch_one<DT, WMODE, MT, 1, 8, 4, QX>(b, a_bits, acc_out, st);
        else if constexpr (MT > 2) launch_one<DT, WMODE, MT, 4, 4, 2, QX>(b, a_bits, acc_out, st);
        else                     launch_one<DT, WMODE, MT, 2, 4, 4, QX>(b, a_bits, acc_out, st);
    }
}

// Rows per workgroup (64 weight rows each, K over four waves) for more than kSkinnyRows rows, 0: the GEMM's tiles are better.
// Such a call is a few dozen tiles of 128 x 128 with a long K loop; cut finer, without LDS in the loop, every CU has
// operands in flight, until the operands' L2 reads (the smaller the block, the more of them) cost more than that.  A round is
// 256 workgroups, one per CU.  Measured with the pre-pass, int8, us, one call repeated on the same weights, GEMM tiles | 64 | 96 |
// 128 rows:
//   4096 x 4096:  128 rows 25.9 | 15.2 | 17.5 | 20.9; 256 rows 26.6 | 15.1 (one round) | 17.3 | 20.0;
//                 333 rows 27.1 | 21.0 | 18.7 (one round) | 21.3; 512 rows 27.5 | 24.2 (two) | 32.7; 768 rows 28.8 | 40.6 (three)
//   11008 x 4096: 256 rows 56.0 | 34.6 | 40.2 | 45.7; 333 rows 57.4 | 54.6 | 42.6 | 47.4; 512 rows 57.4 | 57.0 | 71.3 | 49.0
//   7B layer:     96 rows 93.6 | 83.3 | 66.1 | 69.7; 128 rows 94.3 | 80.2 | 103.6 | 75.0 (int4 100 | 60 | 83 | 61); 192 rows
//                 95.1 | 107 | 106 | 121
// So: one round of small blocks first; then blocks that take all rows at once and read the weights once, while the GEMM's tiles
// leave enough of the chip idle (tiles_are_better; one projection: half of it with 128 x 128 tiles); then
// a round and a half (5056 x 5504, 227 rows: 39 | 28), with int4's shorter loads two (8192 x 1024, 2048 rows: 54.2 | 41.6; int8
// 28672 x 8192, 256 rows, is better on the tiles: 135 | 154).  Fewer than eight runs of weight rows would leave XCDs without work.
// All rows at once in blocks of 96 comes up in batches only: one projection of at most 96 rows with more than 256 such blocks has
// more than 128 tiles.

// Share of the CUs' time that the GEMM's 256 x 256 tiles use, longest K first.
static double tile_fill(const LinBatch& b, int64_t& tiles, int& k_max)
{
    double work = 0.0;
    tiles = 0;
    k_max = 0;
    for (int i = 0; i < b.count; ++i) {
        const int64_t t = ((int64_t)b.it[i].M + 255) / 256 * (((int64_t)b.it[i].N + 255) / 256);
        tiles += t;
        work += (double)t * b.it[i].K;
        k_max = b.it[i].K > k_max ? b.it[i].K : k_max;
    }
    const double span = (double)((tiles + 255) / 256) * work / (double)tiles;
    return work / (256.0 * (span > k_max ? span : (double)k_max));
}

// Whether the GEMM's tiles take at most 128 rows faster than the kernels here: they read the weights at a better rate once
// enough of them run at a time, and an XCD's tiles share the activations.  Measured, us, GEMM | here, on weights that the
// caches have not seen, a projection (or two of half the size) K -> N, with the tiles' fill:
//   single, int8, K = 4096, 64 rows:  N = 32768 (0.50) 38 | 33, 36864 (0.56) 39 | 43, 49152 (0.75) 45 | 54, 65536 (1.0) 56 | 61,
//     69632 (two rounds, 0.53) 79 | 72, 81920 (0.63) 79 | 79, 131072 (1.0) 100 | 114; int4 98304 (0.75) 61 | 60; 48 rows: 49152
//     (0.75) 45 | 44, 57344 (0.88) 50 | 57, int4 131072 (1.0) 76 | 69; 32 rows: never behind by more than 5 %
//   batch of two, int8, K = 4096, 96 rows:  (0.50) 46 | 41, (0.56) 48 | 54, two rounds (0.53) 101 | 90, (0.63) 96 | 93, (0.75) 97 |
//     112; 128 rows: (0.38) 45 | 44, (0.50) 46 | 46, (0.56) 48 | 63, (0.53) 101 | 101; K = 1024, 128 rows: (0.25) 22 | 16, (0.31)
//     22 | 24; int4, 96 rows: (0.75) 49 | 47, (0.88) 53 | 59; 128 rows: (0.50) 46 | 38, (0.56) 47 | 53
//     70B gate and up, 8192 -> 28672 (0.88), int8: 96 rows 104 | 141, 128 rows 107 | 156; int4: 87 | 95, 87 | 119
//   row-major int8 (64-byte pieces of rows), part of the GEMM's time:  single, K = 8192, 8 rows 0.98 at most, 16 rows (0.44)
//     0.93, (0.75) 1.07, (0.88) 1.28, 32 rows (0.75) 1.04, (0.88) 1.15, (1.0) 1.19; two, 64 rows: (0.50) 0.78, (0.63) 1.05, (0.75) 1.08
// The layers of 7B, 13B and 70B (their long down projections leave most CUs to the rest: 0.28, 0.35 and 0.46) are better here.
static bool tiles_are_better(const LinBatch& b, int rows, int wmode)
{
    const bool int4 = wmode == 3, row_major = wmode == 0, single = b.count == 1;
    int64_t tiles;
    int k_max;
    const double fill = tile_fill(b, tiles, k_max);
    const bool one_round = tiles <= 256;
    if (rows <= 12) return false;
    if (rows <= 32) return row_major && k_max >= 4096 && (rows <= 16 ? fill > 0.7 : single && fill > 0.8);
    if (rows <= 48) return single && fill > 0.8 && (one_round || !int4);
    if (rows <= 64) return single ? fill > (one_round ? 0.5 : int4 ? 0.8 : 0.7) : row_major && fill > (one_round ? 0.5 : 0.8);
    if (rows <= 96) return fill > (k_max < 2048 ? 0.5 : !one_round ? 0.7 : int4 ? 0.8 : 0.5);
    return fill > 0.5 || (!int4 && k_max < 2048 && tiles > 64);
}

static int block_rows(const LinBatch& b, int wmode)
{
    int64_t blocks64 = 0, blocks96 = 0, tiles128 = 0;
    int rows = 0;
    for (int i = 0; i < b.count; ++i) {
        const int64_t m = b.it[i].M, cols = ((int64_t)b.it[i].N + 63) / 64;
        if (cols < 8) return 0;
        blocks64 += (m + 63) / 64 * cols;
        blocks96 += (m + 95) / 96 * cols;
        tiles128 += (m + 127) / 128 * ((cols + 1) / 2);
        rows = b.it[i].M > rows ? b.it[i].M : rows;
    }
    if (blocks64 <= 256) return 64;
    if (blocks96 <= 256) return 96;
    if (rows <= 128 && (b.count > 1 ? !tiles_are_better(b, rows, wmode) : tiles128 <= 128)) return rows <= 96 ? 96 : 128;
    return blocks64 <= (wmode == 3 ? 512 : 384) ? 64 : 0;
}

bool linear_takes_skinny(const LinBatch& b, int wmode)
{
    int rows = 0;
    int64_t cols = 0;
    for (int i = 0; i < b.count; ++i) {
        rows = b.it[i].M > rows ? b.it[i].M : rows;
        cols += b.it[i].N;
    }
    if (cols > INT64_C(1) << 28) return false;         // up to 8 work items a column, and a launch holds fewer than 2^32
    return rows <= kSkinnyRows ? !tiles_are_better(b, rows, wmode) : block_rows(b, wmode) != 0;
}

template <int DT, int WMODE>
static void launch_wmode(LinBatch& b, bool qx, int a_bits, int32_t* acc_out, hipStream_t st)
{
    int64_t tiles16 = 0;
    int rows = 0;
    for (int i = 0; i < b.count; ++i) {
        tiles16 += (b.it[i].N + 15) / 16;
        rows = b.it[i].M > rows ? b.it[i].M : rows;
    }
    if (rows > kSkinnyRows) {
        switch (block_rows(b, WMODE)) {
        case 64:  launch_one<DT, WMODE, 4, 4, 4, 2, false>(b, a_bits, acc_out, st); break;
        case 96:  launch_one<DT, WMODE, 6, 4, 4, 3, false>(b, a_bits, acc_out, st); break;
        default:  launch_one<DT, WMODE, 8, 4, 4, 3, false>(b, a_bits, acc_out, st); break;
        }
    } else if (qx)       launch_mt<DT, WMODE, 1, true>(b, tiles16, a_bits, acc_out, st);
    else if (rows <= 32) launch_mt<DT, WMODE, 2, false>(b, tiles16, a_bits, acc_out, st);
    else if (rows <= 48) launch_mt<DT, WMODE, 3, false>(b, tiles16, a_bits, acc_out, st);
    else                 launch_mt<DT, WMODE, 4, false>(b, tiles16, a_bits, acc_out, st);
}

void launch_linear_skinny(LinBatch& b, sasq_dtype dt, int wmode, bool qx, int a_bits, int32_t* acc_out, hipStream_t st)
{
    auto by_wmode = [&](auto dt_tag) {
        constexpr int DT = decltype(dt_tag)::value;
        if (wmode == 0)      launch_wmode<DT, 0>(b, qx, a_bits, acc_out, st);
        else if (wmode == 2) launch_wmode<DT, 2>(b, qx, a_bits, acc_out, st);
        else                 launch_wmode<DT, 3>(b, qx, a_bits, acc_out, st);
    };
    if (dt == SASQ_F16) by_wmode(std::integral_constant<int, SASQ_F16>{});
    else                by_wmode(std::integral_constant<int, SASQ_BF16>{});
}

}  // namespace sasq

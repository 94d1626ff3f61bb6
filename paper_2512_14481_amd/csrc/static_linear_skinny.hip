// int8 linear for few rows (token generation): Y = X . W^T where M is a handful of rows and the weights are what is read;
// and for some hundred rows where the GEMM's tiles are too few to fill the chip (a chunk of a prefill), in row blocks.
//
// What bounds it: the weight bytes (a 7B layer's seven projections at 8 rows, int8: 202 MB in 34.8 us = 5.8 TB/s, the GEMM's
// tiles took 93; a 13B layer's at one row, int4: 159 MB in 25.8 us, from 128; row-major int8, eight rows of a line each a load: 36 us).
// The tiled GEMM hands out 256 (or 128) weight rows per workgroup, which at small M is a few dozen workgroups with a K loop that nothing
// overlaps.  Here a workgroup owns 16 NT weight rows and its NW waves share out K: a wave streams its part of the weights straight from
// memory into MFMA operand registers (a pre-arranged 1 KB block IS one operand read of a wave), D K tiles ahead, with no barrier, and LDS
// only as each wave's own (operands that lie in rows turn there, below), until the waves' int32 sums are added up at the end, so that some
// thousand waves each keep several KB in flight.  Integer sums make the split exact.
// QX: the activations are quantized on the way into the operand registers, 16 elements per lane and K tile, which takes
// the pre-pass's launch out of the call; each workgroup repeats that work, so it is for at most 16 rows, or for few codes
// (linear_quantizes_in_kernel).  Otherwise the codes come from the pre-pass in their staging blocks.
// Row blocks (more than 64 rows): what bounds them is the operands' delivery from L2, (BM + 64) K bytes per workgroup for
// BM x 64 outputs, and the few us in which a workgroup starts and ends; 333 x 4096 x 4096 takes 16.0 us with its pre-pass (27.1 on
// 96 GEMM tiles of 128 x 128).  Of 333 x 4096 x 4096's 11 us in the kernel, 1.3 are arguments and addresses, 8 the K loop (19 TB/s
// out of the L2s), 1.6 the sums' meeting and the stores; it was 15 (row blocks 21.6) while the factors were fetched at the end (3 us),
// the weights, which four row blocks read, went past the L2s (2), and the loop waited for a round's last load before its first
// product.  K over eight waves, two a SIMD, instead of four: 256 rows 14.7 | 13.6.
#include "sasq_device.h"
#include "gemm_tile.h"
#include "gemm_k64.h"
#include "gemm_k64_body.h"
#include <cmath>
#include <type_traits>

namespace sasq {

// An operand from `base` on as a buffer: a load is then a lane offset + a scalar offset, with no 64-bit address to form, and one
// that is not wanted (an empty buffer) returns zeros without a memory access and without a branch.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand_rsrc(const void* base, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

// Row tiles whose sums meet in LDS at a time (128 KB at most).
template <int MT, int NT, int NW> constexpr int skinny_rows_per_phase() { return NW * NT * MT <= 128 ? MT : MT / 2; }
// A wave's own LDS in the K loop, where its operands turn from the order of memory into that of the MFMA.
template <int WMODE, int MT, int NT, bool QX, bool EVEN, bool FLT, bool TURN> constexpr int skinny_turn_bytes()
{
    constexpr bool w = TURN && WMODE == 0, x = TURN && (FLT || QX);
    return (w && !EVEN ? 2 : 1) * ((w ? NT : 0) + (x ? MT : 0)) * 1024;
}
template <int WMODE, int MT, int NT, int NW, bool QX, bool EVEN, bool FLT, bool TURN> constexpr int skinny_lds_bytes()
{
    constexpr int sums = NW * NT * skinny_rows_per_phase<MT, NT, NW>() * 1024, turn = NW * skinny_turn_bytes<WMODE, MT, NT, QX, EVEN, FLT, TURN>();
    return sums > turn ? sums : turn;
}

// FLT: the backward GEMM of the frozen linear.  x is dY, 16-bit and row-major, K the contraction's bytes per row, the weight blocks
// hold 16 rows x 32 numbers, the sums are fp32 (the waves' parts added in their order) and go out rounded, without factors.
// ANYK: K not a multiple of 64, few rows of row-major int8; the activation codes are row-major too.  Rows then start at any byte, and
// the last wave multiplies the rest of the row, with zeros behind, after its whole K tiles.
// TURN: operands that lie in rows are loaded in memory's order and turned in LDS (below).
template <int DT, int WMODE, int MT, int NT, int NW, int D, bool QX, bool ONCE, bool EVEN, bool TURN, bool FLT = false, bool ANYK = false>
__device__ __forceinline__
void skinny_body(const LinItem& it, int mblk, int nblk, int a_bits, int32_t* __restrict__ acc_out, char* lds)
{
    using S = Store16<DT>;
    constexpr bool I4 = WMODE == 3, ROWMAJOR = WMODE == 0;
    static_assert(!I4 || NT % 2 == 0, "int4 blocks hold 32 weight rows");
    static_assert(!FLT || (WMODE == 2 && !QX), "float contraction: weight blocks, no codes");
    static_assert(!ANYK || (ROWMAJOR && !EVEN && !TURN), "rows at any byte: plain loads");
    using AccT = std::conditional_t<FLT, f32x4, i32x4>;
    constexpr int WL = I4 ? NT / 2 : NT;               // 128-bit weight loads per lane and K tile
    constexpr bool WTURN = TURN && ROWMAJOR, XTURN = TURN && QX, FTURN = TURN && FLT;
    constexpr bool LINES = WTURN && !EVEN;
    constexpr int TS = LINES ? 2 : 1;                  // K tiles per step
    constexpr int DS = (D + TS - 1) / TS;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int frow = lane & 15, fq = lane >> 4;
    const int M = it.M, N = it.N, K = it.K, KT = K >> 6;
    const int m0 = mblk * 16 * MT, n0 = nblk * 16 * NT;

    // This wave's steps: an equal run of consecutive ones.  KT odd: the last step of two K tiles has one.
    const int steps = (KT + TS - 1) / TS, per = (steps + NW - 1) / NW;
    const int s0 = min(wave * per, steps), count = min(per, steps - s0), t0 = s0 * TS;
    const int half_step = LINES && (KT & 1) && s0 + count == steps ? count - 1 : -1;

    // One scalar base per operand, advanced 1 KB (or 64 bytes of a row) per K tile, + a 32-bit lane offset per stream: the products of 96
    // rows leave no registers for 64-bit lane addresses.  At K <= 131071 the codes are at most 8 row blocks of 2 MB; FLT's 96 rows stay
    // under 0.8 GB and its four weight blocks under 0.4 GB as no contraction here is longer than kBwdOffsetCols.  Blocks and rows past the
    // matrix repeat its last one.
    const int wblk = I4 ? n0 >> 5 : n0 >> 4, wlast = I4 ? (N - 1) >> 5 : (N - 1) >> 4;
    const char* wbase = reinterpret_cast<const char*>(it.wq) +
                        (ROWMAJOR ? (int64_t)n0 * K + (int64_t)t0 * 64 : ((int64_t)wblk * KT + t0) * 1024);
    // a load takes 8 rows x 128 bytes or 16 rows x 64 bytes in the order of memory (see the turn below)
    const int lrow = lane >> 3, lchunk = lane & 7, prow = lane >> 2, pchunk = lane & 3;
    uint32_t woff[TS * WL];
#pragma unroll
    for (int j = 0; j < TS * WL; ++j) {
        if (LINES)      woff[j] = (uint32_t)min(8 * j + lrow, N - 1 - n0) * (uint32_t)K + 16 * lchunk;
        else if (WTURN) woff[j] = (uint32_t)min(16 * j + prow, N - 1 - n0) * (uint32_t)K + 16 * pchunk;
        else if (ROWMAJOR) {
            woff[j] = (uint32_t)min(16 * j + frow, N - 1 - n0) * (uint32_t)K + 16 * fq;
        } else {
            // int4: lane l takes 16 bytes: the K tile's codes 16 (l/16) .. + 15 of the weight rows 2 (l%16) and 2 (l%16) + 1.
            const uint32_t in_block = I4 ? 256 * fq + 16 * frow : (4 * frow + (fq ^ swz64(frow))) * 16;
            woff[j] = (uint32_t)min(j, wlast - wblk) * (uint32_t)KT * 1024 + in_block;
        }
    }
    constexpr int kWStep = ROWMAJOR ? 64 * TS : 1024;
    const char* xbase = FLT ? reinterpret_cast<const char*>(it.x) + (int64_t)m0 * K + (int64_t)t0 * 64
                      : QX ? reinterpret_cast<const char*>(it.x) + ((int64_t)m0 * K + (int64_t)t0 * 64) * 2
                      : ANYK ? reinterpret_cast<const char*>(it.xq) + (int64_t)m0 * K + (int64_t)t0 * 64
                           : reinterpret_cast<const char*>(it.xq) + ((int64_t)(m0 >> 4) * KT + t0) * 1024;
    uint32_t xoff[XTURN ? 2 * MT : MT];
#pragma unroll
    for (int b = 0; b < (XTURN ? 2 * MT : MT); ++b) {
        if (XTURN)             xoff[b] = (uint32_t)min(8 * b + lrow, M - 1 - m0) * (uint32_t)K * 2 + 16 * lchunk;
        else if (FTURN)        xoff[b] = (uint32_t)min(16 * b + prow, M - 1 - m0) * (uint32_t)K + 16 * pchunk;
        else if (FLT || (ANYK && !QX)) xoff[b] = (uint32_t)min(16 * b + frow, M - 1 - m0) * (uint32_t)K + 16 * fq;
        else if (QX) xoff[b] = (uint32_t)min(16 * b + frow, M - 1 - m0) * (uint32_t)K * 2 + fq * 32;
        else         xoff[b] = (uint32_t)min(b, ((M - 1) >> 4) - (m0 >> 4)) * (uint32_t)KT * 1024 + (4 * frow + (fq ^ swz64(frow))) * 16;
    }
    constexpr int kXStep = FLT || (ANYK && !QX) ? 64 : (QX ? 128 : 1024) * TS;
    const QConst qk = FLT ? QConst{} : make_qconst(*it.s, a_bits);

    constexpr int WN = TS * WL, XN = (QX ? 2 : 1) * TS;                // loads per step
    struct Frag {
        u32x4 w[WN];
        u32x4 x[MT][XN];
    };
    const bool few = XTURN && MT == 1 && M <= 8;        // then a K tile's second load would be of rows past the last
    auto load = [&](Frag& f, int t) {
        int bytes = -1;                                 // in so many words: from a select the compiler builds the buffers in vector registers
        if (EVEN) asm("s_cmp_lt_i32 %1, %2\n\ts_cselect_b32 %0, -1, 0" : "=s"(bytes) : "s"(t), "s"(count) : "scc");
        const __amdgpu_buffer_rsrc_t wrsrc = operand_rsrc(wbase, bytes), xrsrc = operand_rsrc(xbase, bytes);
        // ONCE: no other workgroup reads these weights.  Where row blocks share them they have to stay in L2 (333 x 4096 x 4096
        // 18.8 us non-temporal, 16.8 cached).
        constexpr int kNonTemporal = 2;
        // Row-major in the MFMA's order: plain loads (7B layer, 8 rows 50.6 us through buffers, 49.8 so; 12 x 2368 x 28544's MLP 72.9, 70.0).
        constexpr bool kPlain = ROWMAJOR && !ANYK && !EVEN && !TURN;
        // a step of one K tile takes that one twice: nothing behind a row's end is read
        const bool half = LINES && t == half_step;
        const uint32_t back = half && lchunk >= 4 ? 64 : 0;
#pragma unroll
        for (int j = 0; j < WN; ++j)
            if constexpr (ANYK)       f.w[j] = load_piece<u32x4>(reinterpret_cast<const uint8_t*>(wbase) + (int64_t)t * kWStep + woff[j]);
            else if constexpr (kPlain) f.w[j] = *reinterpret_cast<const u32x4*>(wbase + (int64_t)t * kWStep + woff[j]);
            else if constexpr (LINES) f.w[j] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, woff[j] - back, t * kWStep, ONCE ? kNonTemporal : 0);
            else                  f.w[j] = __builtin_amdgcn_raw_buffer_load_b128(wrsrc, woff[j], t * kWStep, ONCE && !ROWMAJOR ? kNonTemporal : 0);
#pragma unroll
        for (int b = 0; b < MT; ++b)
#pragma unroll
            for (int h = 0; h < XN; ++h) {
                constexpr int kTile = QX ? 2 : 1;                       // loads of a K tile
                const int step = t * kXStep + (half ? 0 : h / kTile * (QX ? 128 : 1024));
                if constexpr (kPlain) f.x[b][h] = *reinterpret_cast<const u32x4*>(xbase + (int64_t)t * kXStep + xoff[b] + 16 * h);
                else if constexpr (ANYK) f.x[b][h] = load_piece<u32x4>(reinterpret_cast<const uint8_t*>(xbase) + (int64_t)t * kXStep + xoff[b] + 16 * h);
                else if constexpr (XTURN) {
                    if (h % 2 == 0 || !few) f.x[b][h] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, xoff[2 * b + h % 2], step, 0);
                } else f.x[b][h] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, xoff[b] + (QX ? 16 * h : 0), step, 0);
            }
    };
    AccT acc[NT][MT];
#pragma unroll
    for (int g = 0; g < NT; ++g)
#pragma unroll
        for (int b = 0; b < MT; ++b) acc[g][b] = AccT{0, 0, 0, 0};
    // The turn: operands that memory holds in rows are loaded in memory's order and go through the wave's own LDS into the MFMA's (a
    // wave's LDS accesses are served in order: no wait, no barrier).  Loaded in the MFMA's order, sixteen rows side by side, the four
    // lanes that the L1 cache looks at together want the same banks of four lines and get them one by one: 9.6 TB/s out of the L2s where
    // rows are whole lines apart, 28 to 30 in memory's order.  Few rows of row-major weights also take whole lines: memory delivers the
    // halves one by one.  us, MFMA's order | memory's: weights, 7B layer, row-major, 8 rows 50 | 36, 16 rows 60 | 41, 40 rows 64 | 48, 8 x
    // 4096 -> 11008 16.3 | 13.1; dY, the 7B layer's training step of 200 rows 405 | 350, attention, hidden 2048, of 130 rows 58 | 53; the
    // activations quantized here, 7B layer, pre-arranged, 16 rows 43.4 | 38.6, 13B int4, 16 rows 36.8 | 33.4, one row 28.0 | 26.6.
    constexpr int kTurn = skinny_turn_bytes<WMODE, MT, NT, QX, EVEN, FLT, TURN>();
    char* wturn = lds + wave * kTurn;
    char* xturn = wturn + (WTURN ? NT * TS * 1024 : 0);
    const int line_put = lrow * 128 + ((lchunk ^ lrow) << 4), line_get = frow * 128 + ((fq ^ (frow & 7)) << 4);
    const int piece_put = prow * 64 + ((pchunk ^ swz64(prow)) << 4), piece_get = frow * 64 + ((fq ^ swz64(frow)) << 4);
    auto quantize8 = [&](const u32x4& v) -> u32x2 {
        float c[8];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            c[2 * w] = quantize(S::lo(v[w]), qk).c;
            c[2 * w + 1] = quantize(S::hi(v[w]), qk).c;
        }
        return u32x2{pack_codes4(c[0], c[1], c[2], c[3]), pack_codes4(c[4], c[5], c[6], c[7])};
    };
    auto multiply = [&](const Frag& f, int t) {
        if constexpr (WTURN) {
#pragma unroll
            for (int j = 0; j < WN; ++j) *reinterpret_cast<u32x4*>(wturn + j * 1024 + (LINES ? line_put : piece_put)) = f.w[j];
        }
        if constexpr (FTURN) {
#pragma unroll
            for (int b = 0; b < MT; ++b) *reinterpret_cast<u32x4*>(xturn + b * 1024 + piece_put) = f.x[b][0];
        }
        if constexpr (XTURN) {
#pragma unroll
            for (int b = 0; b < MT; ++b)
#pragma unroll
                for (int h = 0; h < XN; ++h)
                    if (h % 2 == 0 || !few) {
                        const int r = 8 * (h % 2) + lrow;
                        *reinterpret_cast<u32x2*>(xturn + (h / 2 * MT + b) * 1024 + r * 64 + (((lchunk >> 1) ^ swz64(r)) << 4) + 8 * (lchunk & 1)) = quantize8(f.x[b][h]);
                    }
        }
#pragma unroll
        for (int p = 0; p < TS; ++p) {
            if (p == 1 && t == half_step) break;
            i32x4 xv[MT];
#pragma unroll
            for (int b = 0; b < MT; ++b) {
                if constexpr (FTURN || XTURN) {
                    xv[b] = *reinterpret_cast<const i32x4*>(xturn + (p * MT + b) * 1024 + piece_get);
                } else if constexpr (QX) {
                    const u32x2 lo = quantize8(f.x[b][0]), hi = quantize8(f.x[b][1]);
                    xv[b] = i32x4{(int)lo[0], (int)lo[1], (int)hi[0], (int)hi[1]};
                } else {
                    xv[b] = __builtin_bit_cast(i32x4, f.x[b][p]);
                }
            }
#pragma unroll
            for (int g = 0; g < NT; ++g) {
                i32x4 wv;
                if constexpr (I4) {
                    const uint32_t p0 = f.w[g / 2][2 * (g & 1)], p1 = f.w[g / 2][2 * (g & 1) + 1];   // 16 x the code in every byte
                    wv = i32x4{(int)((p0 << 4) & 0xF0F0F0F0u), (int)(p0 & 0xF0F0F0F0u), (int)((p1 << 4) & 0xF0F0F0F0u), (int)(p1 & 0xF0F0F0F0u)};
                } else if constexpr (WTURN) {
                    wv = *reinterpret_cast<const i32x4*>(wturn + (LINES ? g * 2048 + (line_get ^ (64 * p)) : g * 1024 + piece_get));
                } else {
                    wv = __builtin_bit_cast(i32x4, f.w[g]);
                }
#pragma unroll
                for (int b = 0; b < MT; ++b) {
                    if constexpr (FLT) acc[g][b] = Mfma16x16<DT>::mma(wv, xv[b], acc[g][b]);
                    else               acc[g][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wv, xv[b], acc[g][b], 0, 0, 0);
                }
            }
        }
    };

    // At the end a wave finishes output tiles of one run of 16 (int4: 32) columns; their factors are requested behind the first
    // operands instead of being waited for there.
    constexpr int kRegs = I4 ? 2 : 1, kCols = 4 * kRegs, kRuns = NT / kRegs;         // int4: two tiles interleave into 32 columns
    static_assert(NW % kRuns == 0, "a wave stays in one run of columns");
    const int g0 = wave % kRuns * kRegs, n = n0 + 16 * g0 + kCols * fq;
    float sw[kCols], bv[kCols];
    auto load_factors = [&]() {
        if (FLT) return;
#pragma unroll
        for (int e = 0; e < kCols; ++e) {
            const int ne = min(n + e, N - 1);
            sw[e] = it.s_w[ne];
            bv[e] = (it.bias ? it.bias : it.s_w)[ne];                                // without a bias: not used
        }
    };

    Frag rest;                                          // ANYK: the channels behind the last whole K tile
    const bool has_rest = ANYK && wave == NW - 1;
    if constexpr (ANYK) {
        if (has_rest) {
            const uint8_t* w = reinterpret_cast<const uint8_t*>(it.wq);
            const uint8_t* x = QX ? static_cast<const uint8_t*>(it.x) : reinterpret_cast<const uint8_t*>(it.xq);
            constexpr int kBytes = QX ? 2 : 1;
#pragma unroll
            for (int j = 0; j < WL; ++j) rest.w[j] = load_piece_edge<u32x4>(w + (int64_t)min(n0 + 16 * j + frow, N - 1) * K, KT * 64 + 16 * fq, K);
#pragma unroll
            for (int b = 0; b < MT; ++b)
#pragma unroll
                for (int h = 0; h < kBytes; ++h)
                    rest.x[b][h] = load_piece_edge<u32x4>(x + (int64_t)min(m0 + 16 * b + frow, M - 1) * K * kBytes, (KT * 64 + 16 * fq) * kBytes + 16 * h, K * kBytes);
        }
    }
    Frag ring[DS];
    if constexpr (EVEN) {
        // DS steps in flight.  Loads and products carry no conditions (tiles past the last are zeros), so that the wait in front of
        // a product counts exactly the loads behind its own; the barriers keep the scheduler from moving all products of a round in
        // front of all its loads, which exposed the whole latency once a round.
#pragma unroll
        for (int j = 0; j < DS; ++j) {
            load(ring[j], j);
            __builtin_amdgcn_sched_barrier(0);
        }
        load_factors();
        asm volatile("" ::: "memory");                  // here, not behind the loop
#pragma unroll 1
        for (int i = 0; i < count; i += DS) {
#pragma unroll
            for (int j = 0; j < DS; ++j) {
                multiply(ring[j], i + j);
                load(ring[j], i + j + DS);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < DS; ++j)
            if (j < count) load(ring[j], j);
        load_factors();
        asm volatile("" ::: "memory");
        int i = 0;
#pragma unroll 1
        for (; i + 2 * DS <= count; i += DS) {
#pragma unroll
            for (int j = 0; j < DS; ++j) {
                multiply(ring[j], i + j);
                load(ring[j], i + j + DS);
            }
        }
#pragma unroll
        for (int j = 0; j < DS; ++j)
            if (i + j < count) {
                multiply(ring[j], i + j);
                if (i + j + DS < count) load(ring[j], i + j + DS);
            }
#pragma unroll
        for (int j = 0; j < DS; ++j)
            if (i + DS + j < count) multiply(ring[j], i + DS + j);
    }
    if constexpr (ANYK) {
        if (has_rest) multiply(rest, 0);
    }

    // The waves' sums meet in LDS, as many row tiles at a time as fit; wave w finishes the output tiles w, w + NW, ...
    constexpr int kRows = skinny_rows_per_phase<MT, NT, NW>(), kTiles = kRuns * kRows;
    AccT* part = reinterpret_cast<AccT*>(lds);
    const float s = qk.s;
#pragma unroll
    for (int b0 = 0; b0 < MT; b0 += kRows) {
        if (b0 > 0 || kTurn > 0) __syncthreads();
#pragma unroll
        for (int g = 0; g < NT; ++g)
#pragma unroll
            for (int b = 0; b < kRows; ++b) part[((wave * NT + g) * kRows + b) * 64 + lane] = acc[g][b0 + b];
        __syncthreads();
#pragma unroll
        for (int t = wave; t < kTiles; t += NW) {
            const int b = t / kRuns;
            std::conditional_t<FLT, float, int> v[kCols];
#pragma unroll
            for (int r = 0; r < kRegs; ++r) {
                AccT sum = {0, 0, 0, 0};
#pragma unroll
                for (int w = 0; w < NW; ++w) sum += part[((w * NT + g0 + r) * kRows + b) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (I4) v[kRegs * e + r] = sum[e] >> 4;
                    else              v[kRegs * e + r] = sum[e];
                }
            }
            const int m = m0 + 16 * (b0 + b) + frow;                         // 4 (8) consecutive columns of one row
            if (m >= M || n >= N) continue;
            uint16_t* dst = it.y + (int64_t)m * N + n;
            float yv[kCols];
#pragma unroll
            for (int e = 0; e < kCols; ++e) {
                float f = (float)v[e];
                if (!FLT) f = f * (s * sw[e]);
                if (!FLT && it.bias) f = f + bv[e];
                yv[e] = f;
            }
            if ((N & 7) == 0) {                                              // then every full run is aligned to its own size
#pragma unroll
                for (int h = 0; h < kRegs; ++h)
                    *reinterpret_cast<u32x2*>(dst + 4 * h) = u32x2{S::pack(yv[4 * h], yv[4 * h + 1]), S::pack(yv[4 * h + 2], yv[4 * h + 3])};
            } else {
#pragma unroll
                for (int e = 0; e < kCols; ++e)
                    if (n + e < N) dst[e] = S::enc(yv[e]);
            }
            if (acc_out) {
#pragma unroll
                for (int e = 0; e < kCols; ++e)
                    if (n + e < N) acc_out[(int64_t)m * N + n + e] = __builtin_bit_cast(int32_t, v[e]);
            }
        }
    }
}

template <int DT, int WMODE, int MT, int NT, int NW, int D, bool QX, bool ONCE, bool EVEN, bool TURN, bool ANYK>
__global__ __launch_bounds__(64 * NW)
void skinny_kernel(const LinBatch b, int a_bits, int32_t* __restrict__ acc_out)
{
    __shared__ __attribute__((aligned(1024))) char lds[skinny_lds_bytes<WMODE, MT, NT, NW, QX, EVEN, false, TURN>()];
    const int k = lin_item_of(b, (int)blockIdx.x);
    // Eight neighbours in the id go to the eight XCDs: the row blocks of one run of weight rows stay on one, 8 ids apart.
    const int id = (int)blockIdx.x - b.first_block[k], octet = id >> 3, tiles_m = b.it[k].tiles_m;
    const int mblk = octet % tiles_m, nblk = octet / tiles_m * 8 + (id & 7);
    if (nblk >= b.it[k].tiles_n) return;
    skinny_body<DT, WMODE, MT, NT, NW, D, QX, ONCE, EVEN, TURN, false, ANYK>(b.it[k], mblk, nblk, a_bits, acc_out, lds);
}

template <int DT, int WMODE, int MT, int NT, int NW, int D, bool QX, bool ONCE, bool EVEN, bool TURN, bool ANYK = false>
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
    skinny_kernel<DT, WMODE, MT, NT, NW, D, QX, ONCE, EVEN, TURN, ANYK><<<b.first_block[b.count], 64 * NW, 0, st>>>(b, a_bits, acc_out);
}

static int longest(const LinBatch& b)
{
    int k = 0;
    for (int i = 0; i < b.count; ++i) k = b.it[i].K > k ? b.it[i].K : k;
    return k;
}
static int64_t weight_bytes(const LinBatch& b)
{
    int64_t n = 0;
    for (int i = 0; i < b.count; ++i) n += (int64_t)b.it[i].N * b.it[i].K;
    return n;
}

// Whether the weights' rows are 8192 and more codes long, on average over the columns.
bool linear_long_rows(const LinBatch& b)
{
    int64_t columns = 0;
    for (int i = 0; i < b.count; ++i) columns += b.it[i].N;
    return weight_bytes(b) >= 8192 * columns;
}

// Whether a call's weights go past the caches (ONCE), where nothing else is said.  Row-major weights up to half of the 256 MB Infinity Cache keep the ordinary policy, as
// they may be found there by the next call.  us, ordinary | non-temporal, found there: 8 x 4096 -> 11008 10.1 | 12.2, attention, hidden 4096, of
// 20 rows 15.9 | 18.4; not found: 13.1 | 12.4 and 20.0 | 18.7; the 7B layer, 202 MB, 8 rows 40 | 36.  Over 460 calls of up to 16 rows, 128 to
// 256 MB, ordinary in parts of non-temporal: not in the caches 1.08 to 1.10, in them 0.86 to 0.89.  Rows off whole 128-byte lines (K / 64 odd)
// keep it at any size: neighbouring pieces then share a line, which the first read would give up; 260 such calls 0.92 to 0.95 and 0.72 to 0.74.
constexpr int64_t kCachedWeights = INT64_C(128) << 20;
bool linear_streams(const LinBatch& b, int wmode)
{
    if (wmode != 0) return true;
    for (int i = 0; i < b.count; ++i)
        if (b.it[i].K % 128) return false;
    return weight_bytes(b) > kCachedWeights;
}

// Wide or narrow workgroups: the narrow form (16 weight rows, K over eight waves) gives more workgroups for the same weights, the
// wide one reads the activations half or a quarter as often.  Measured at 8 rows, int8, wide (then K over four waves) | narrow:
// 4096 x 4096 (256 tiles of 16 rows) 8.3 | 6.5 us, 4096 x 11008 17.3 | 12.8, 11008 x 4096 (688 tiles) 12.3 | 13.4, the 7B
// layer (2656 tiles) 36 | 51; the line lies at 512 tiles.
// Waves of the wide form and K tiles each has in flight, quantizing in the kernel, us, eight with three | eight with two | four with four |
// four with six: the 7B layer at 8 rows 37.3 | 35.9 | 34.9 | 35.9, at 16 44.2 | 40.4 | 38.7 | 40.3, hidden 2048 at 12 15.3 | 14.4 | 12.8 |
// 13.9, 8 x 8192 -> 16384 28.8 | 28.1 | 31.4 | 28.5, 8192 -> 28672 (512 and 896 workgroups, rows of 128 K tiles) - | 44.9 | 47.1 | 44.8:
// six where the rows are 8192 and more codes long.  With codes from the pre-pass eight with three: MLP of 30 rows 32.5 | - | 36.0 | 32.1,
// hidden 2048 at 24 17.1 | - | 18.9 | 19.1.  int4, blocks twice as wide, the 13B layer at 16 rows, eight with two | four with two, three,
// four: 35.2 | 45.7, 35.2, 33.4, at one row 26.9 | 31.9, 27.3, 26.6.  Row-major, in steps of two K tiles, layer at 1, 8, 16 rows, four waves with
// four | four with two | eight with two: 39.9, 39.3, 42.5 | 34.7, 36.2, 41.0 | 33.6, 36.4, 42.2; row tiles of 32, MLP of 30 rows 34.1 | 36.9 | 33.7,
// of 20 rows, hidden 2048, 12.7 | 13.4 | 13.1; narrow, 30 and 40 x 4096 -> 4096, eight with four | two: 9.4, 10.1 | 8.7, 9.5.
// Without the turn, the forms that were the best before it: int8 eight waves with three, int4 with two, row-major four with four; of up to four K
// tiles four waves, as half of eight have none (0.93 to 1.05 of eight's time).  Narrow int8 with the turn takes 133 registers with four K tiles
// in flight, so that one workgroup fits a CU, 109 with three: from 257 workgroups on four took 1.2 to 1.4 of the time without the turn.
template <int DT, int WMODE, int MT, bool QX, bool TURN, bool ANYK = false, bool ONCE = true>
static void launch_mt(LinBatch& b, int64_t tiles16, int a_bits, int32_t* acc_out, hipStream_t st)
{
    if constexpr (WMODE == 0 && TURN && ONCE) {
        if (!linear_streams(b, WMODE)) return launch_mt<DT, WMODE, MT, QX, TURN, ANYK, false>(b, tiles16, a_bits, acc_out, st);
    }
    const bool wide = tiles16 >= 512, long_rows = linear_long_rows(b);
    if constexpr (WMODE == 0 && !TURN) {               // K not a multiple of 64 too (ANYK)
        if (!wide)                 launch_one<DT, WMODE, MT, 1, 8, 4, QX, false, false, false, ANYK>(b, a_bits, acc_out, st);
        else if constexpr (MT > 2) launch_one<DT, WMODE, MT, 4, 4, 2, QX, false, false, false, ANYK>(b, a_bits, acc_out, st);
        else                       launch_one<DT, WMODE, MT, 2, 4, 4, QX, false, false, false, ANYK>(b, a_bits, acc_out, st);
    } else if constexpr (WMODE == 0) {
        if (!wide)                 launch_one<DT, WMODE, MT, 1, 8, 2, QX, ONCE, false, true>(b, a_bits, acc_out, st);
        else if constexpr (MT > 2) launch_one<DT, WMODE, MT, 4, 4, 2, QX, ONCE, false, true>(b, a_bits, acc_out, st);
        else                       launch_one<DT, WMODE, MT, 2, 4, MT == 1 ? 2 : 4, QX, ONCE, false, true>(b, a_bits, acc_out, st);
    } else if constexpr (WMODE == 3) {                 // int4: half the bytes per tile, a block is two tiles
        if (!wide)                     launch_one<DT, WMODE, MT, 2, 8, 2, QX, true, false, TURN>(b, a_bits, acc_out, st);
        else if constexpr (QX && TURN) launch_one<DT, WMODE, MT, 4, 4, 4, QX, true, false, TURN>(b, a_bits, acc_out, st);
        else if constexpr (QX) {
            if (longest(b) <= 256) launch_one<DT, WMODE, MT, 4, 4, 4, QX, true, false, TURN>(b, a_bits, acc_out, st);
            else                   launch_one<DT, WMODE, MT, 4, 8, 2, QX, true, false, TURN>(b, a_bits, acc_out, st);
        }
        else                           launch_one<DT, WMODE, MT, 4, 4, 2, QX, true, false, TURN>(b, a_bits, acc_out, st);
    } else {
        if (!wide) {
            if constexpr (TURN) {
                if (tiles16 > 256) return launch_one<DT, WMODE, MT, 1, 8, 3, QX, true, false, TURN>(b, a_bits, acc_out, st);
            }
            launch_one<DT, WMODE, MT, 1, 8, 4, QX, true, false, TURN>(b, a_bits, acc_out, st);
        }
        else if constexpr (MT > 2) launch_one<DT, WMODE, MT, 4, 4, 2, QX, true, false, TURN>(b, a_bits, acc_out, st);
        else if constexpr (!QX)    launch_one<DT, WMODE, MT, 2, 8, 3, QX, true, false, TURN>(b, a_bits, acc_out, st);
        else if constexpr (!TURN) {
            if (longest(b) <= 256) launch_one<DT, WMODE, MT, 2, 4, 4, QX, true, false, TURN>(b, a_bits, acc_out, st);
            else                   launch_one<DT, WMODE, MT, 2, 8, 3, QX, true, false, TURN>(b, a_bits, acc_out, st);
        }
        else if (long_rows)        launch_one<DT, WMODE, MT, 2, 4, 6, QX, true, false, TURN>(b, a_bits, acc_out, st);
        else                       launch_one<DT, WMODE, MT, 2, 4, 4, QX, true, false, TURN>(b, a_bits, acc_out, st);
    }
}

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

// Whether the GEMM's tiles take at most 64 rows faster than the kernels here: they read the weights at a better rate once
// enough of them run at a time, and an XCD's tiles share the activations.  Measured, us, GEMM | here, on weights that the
// caches have not seen, a projection (or two of half the size) K -> N, with the tiles' fill:
//   single, int8, K = 4096, 64 rows:  N = 32768 (0.50) 38 | 33, 36864 (0.56) 39 | 43, 49152 (0.75) 45 | 54, 65536 (1.0) 56 | 61,
//     69632 (two rounds, 0.53) 79 | 72, 81920 (0.63) 79 | 79, 131072 (1.0) 100 | 114; int4 98304 (0.75) 61 | 60; 48 rows: 49152
//     (0.75) 45 | 44, 57344 (0.88) 50 | 57, int4 131072 (1.0) 76 | 69; 32 rows: never behind by more than 5 %
//   row-major int8 in the MFMA's order, part of the GEMM's time:  single, K = 8192, 8 rows 0.98 at most, 16 rows (0.44) 0.93, (0.75)
//     1.07, (0.88) 1.28, 32 rows (0.75) 1.04, (0.88) 1.15, (1.0) 1.19; two, 64 rows: (0.50) 0.78, (0.63) 1.05, (0.75) 1.08
//   The lines are of then.  With the turn, single row-major projections, 3700 calls: 13 to 16 rows 0.86 to 0.90 up to (0.9); 17 to 32 rows (0.7)
//     0.83 to 0.94, (0.8) 0.90 to 1.02; 33 to 48 (0.7) 0.85 to 1.00, (0.8) 0.92 to 1.06; 49 to 64 (0.5) 0.89 to 0.98, (0.6) 0.87 to 0.98, (0.7) 0.95
//     to 1.03, (0.8) 1.00 to 1.07: what goes to the tiles below that takes up to 1.17 of its time here, 0.8 % over all of the calls
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
    return single ? fill > (one_round ? 0.5 : int4 ? 0.8 : 0.7) : row_major && fill > (one_round ? 0.5 : 0.8);
}

// They take the loop that loads only K tiles there are: a wave has few of them, and the loop without conditions (EVEN) requests tiles past
// the last and multiplies their zeros.  Parts of that loop's time, weights not in the caches | in them: forward 16 x 16 0.94 | 0.93, 32 x 16
// 0.96 | 0.95, 32 x 32 0.92 | 0.91, 32 x 64 0.94 | 0.92, row-major 0.85 to 0.91, backward 0.94 | 0.92, 0.91 | 0.88, 0.87 | 0.85, 0.90 | 0.87.
// The weights keep the ordinary cache policy: non-temporal, another 0.95 | 1.13.
// Small blocks, for more than 16 rows: the smallest of 16 x 16 outputs (int4 16 x 32), 32 x 16 (32 x 32), 32 x 32 and 32 x 64 that
// the call has no more than a round of, one a CU.  All run at once, so the call takes as long as one of them, and the smallest are the
// shortest; from a second round on the larger ones of the other rules read less.  The runs of columns go round the eight XCDs, so a
// round is 32 blocks on the XCD with the most of them.  Measured, us, before | 16 x 16 | 32 x 16: pre-arranged 64 x 4096 -> 512 10.2 |
// 7.0 | 7.6, 20 x 4096 -> 2048 9.2 | 7.4 | 8.3, row-major 64 x 1024 -> 256 7.2 | 4.8 | 6.5, backward 64 x 4096 -> 1024 19.8 | 7.3 |
// 10.7, 64 x 1024 -> 2048 6.2 | 5.2 (two rounds) | 4.7, 32 x 4096 -> 512 11.2 | 6.9 | 10.2; | 32 x 32 | 32 x 64: pre-arranged 80 x 1024 x
// 1024 8.6 | 7.2 | 7.8, 143 x 2816 x 2816 11.0 | 11.8 | 9.5, 1000 x 11008 -> 250 66.8 | 23.7, row-major 96 x 11008 -> 1024 31.2 | 18.9;
// backward 143 x 1280 x 1280 9.4 | 6.4 | 6.8, 143 x 2816 x 2816 16.5 | 16.4 | 11.3, 128 x 5248 -> 2048 26.8 | 15.4, 224 x 5248 -> 1792
// 26.9 | - | 17.7.  Beyond a round: backward 171 x 1344 -> 1344 (36 blocks of 32 x 32 on one XCD) 9.4 | 10.4, 224 x 2240 -> 2240 (35 of
// 32 x 64) 14.2 | - | 16.2, 64 x 4096 x 1024 (128 of 16 x 16) 7.0 | 8.4 | 7.5.
// Row-major int8 leaves its few-row kernel for blocks of 16 columns only, and of those for at least two row blocks: in the MFMA's order,
// 40 x 2048 -> 3000 7.4 | 9.0 as 32 x 32, 50 x 8192 -> 3500 14.3 | 15.9, 24 x 2048 -> 3000 6.8 | 7.8 as 32 x 16.  In the orders that both take
// now, over 1160 calls, 32 x 16 at 17 to 32 rows 1.00 to 1.02 of the few-row kernel's time, but 32 x 32 at 33 to 64 rows 0.89 to 1.00 and 32 x 64
// 0.75 to 0.95, the shorter the contraction the less.
struct SmallBlock { int mt, nt; };                                       // in units of 16; 0: none
static SmallBlock small_block(const LinItem* items, int count, int wmode)
{
    const bool int4 = wmode == 3, row_major = wmode == 0;
    int rows = 0;
    for (int i = 0; i < count; ++i) {
        rows = items[i].M > rows ? items[i].M : rows;
        if (count > 1 && items[i].N <= 448) return {0, 0};           // as block_rows: the other items' blocks share the XCDs unevenly
    }
    if (rows <= 16) return {0, 0};
    static const SmallBlock forms[] = {{1, 1}, {1, 2}, {2, 1}, {2, 2}, {2, 4}};
    for (const SmallBlock& f : forms) {
        if (int4 ? f.nt == 1 : f.mt == 1 && f.nt == 2) continue;     // int4 blocks hold 32 weight rows
        if (rows <= 32 && (f.nt == 4 || (f.nt == 2 && !int4))) continue;
        if (row_major && rows <= kSkinnyRows && (f.nt > 1 || (f.mt == 2 && rows <= 32))) continue;
        int64_t blocks = 0;
        for (int i = 0; i < count; ++i)
            blocks += ((int64_t)items[i].M + 16 * f.mt - 1) / (16 * f.mt) * (((int64_t)items[i].N + 128 * f.nt - 1) / (128 * f.nt) * 8);
        if (blocks <= 256) return f;
    }
    return {0, 0};
}

// Rows per workgroup (64 weight rows each, K over eight waves or four) for more than kSkinnyRows rows, 0: the GEMM's tiles are better.
// A call of few tiles leaves CUs idle or waiting for one long K loop; cut finer every CU has operands in flight, until the operands'
// L2 reads (the smaller the block, the more of them) cost more than that.  Neither side's time follows from one size, so both are
// estimated, in us, from what they do: workgroups go in rounds (of 256; row blocks one workgroup a CU), a round costs what a
// workgroup takes to start and end, and the operands of its K tiles.  The constants are least squares over 550 calls of 65 to 1200
// rows, K and N from 1024 to 28672, single projections and layers, of times from 8 to 500 us: rms error 7 to 11 %.  Over those calls
// the choice costs 0.8 % against the best of the four each time, and the calls take 0.87 of what they took with lines drawn by hand.
// The constants of row-major int8 are of its loads in the MFMA's order: over 1900 such calls as they are now the choice costs 3.7 % against the best
// of the four, 0.5 to 4 % where blocks are taken and 11 to 14 % where tiles are.
// Row blocks are taken from 10 % less time on: the estimates are no better than that.  Blocks of 64 rows take four waves instead of eight from
// a second round on: their sums then meet in 64 KB of LDS and two of them share a CU, 0.91 of the time at 257 to 768 blocks, 0.87 to 1536, 0.84
// beyond, weights in the caches or not (eight waves are 1.00 to 1.04 of four in a single round).  us, GEMM tiles | 64 | 96 | 128 rows:
//   4096 x 4096: 128 rows 26.2 | 12.9 | 14.8 | 20.4, 256 rows 26.4 | 13.7 | 15.5 | 17.3, 333 rows 26.7 | 20.3 | 16.0 | 17.3, 512 rows
//   27.1 | 21.3 | 24.3 | 18.9, 768 rows 27.9 | 29.7 | 27.1 | 30.4, 1000 rows 28.8 | 40.5 | 39.1 | 34.6; 8192 x 8192, 200 rows 56.5 |
//   37.1 | 42.8 | 33.5; 7B layer, 96 rows 98.6 | 68.3 | 60.4 | 61.8, 192 rows 113 | 104 | 92.7 | 94.3, 333 rows tiles
struct BlockTime { double call, round, k_tile; };
static const BlockTime kBlockTime[3][3] = {                          // row-major int8, pre-arranged int8, pre-arranged int4; 64, 96, 128 rows
    {{4.8, 2.4, 0.167}, {4.7, 3.7, 0.195}, {4.6, 4.6, 0.213}},
    {{4.6, 2.9, 0.107}, {5.1, 3.9, 0.137}, {5.3, 4.7, 0.161}},
    {{4.6, 2.8, 0.076}, {4.8, 4.1, 0.100}, {4.9, 4.9, 0.121}}};
static const BlockTime kTileTime[3] = {{1.0, 12.0, 0.72}, {1.0, 13.0, 0.54}, {1.0, 16.0, 0.49}};

// Row blocks of r rows, the runs of columns filled up to the eight XCDs.
static int64_t blocks_of(const LinBatch& b, int r)
{
    int64_t blocks = 0;
    for (int i = 0; i < b.count; ++i) blocks += ((int64_t)b.it[i].M + r - 1) / r * (((int64_t)b.it[i].N + 511) / 512 * 8);
    return blocks;
}

static int block_rows(const LinBatch& b, int wmode)
{
    const int format = wmode == 0 ? 0 : wmode == 2 ? 1 : 2;
    double work = 0.0, k_max = 0.0;                                  // GEMM tiles x K tiles
    int64_t tiles = 0, ids = 0;
    for (int i = 0; i < b.count; ++i) {
        if (b.it[i].N <= 448) return 0;                              // fewer than eight runs of weight rows leave XCDs without work
        const double kt = b.it[i].K / 64;
        const int64_t t = ((int64_t)b.it[i].M + 255) / 256 * (((int64_t)b.it[i].N + 255) / 256);
        tiles += t;
        ids += (t + 7) / 8 * 8;
        work += (double)t * kt;
        k_max = kt > k_max ? kt : k_max;
    }
    // A single call has its choice of tiles, and rounds in units of whole ones.  The tiles of a batch fill each other's last round
    // in part: between whole rounds and none; where they go as halves throughout (launch_gemm_k64_batch), a round is 0.7 of one.
    const BlockTime& tt = kTileTime[format];
    double best;
    if (b.count == 1) {
        best = tt.call + gemm_rounds(b.it[0].M, b.it[0].N) * (tt.round + tt.k_tile * k_max);
    } else {
        const double rounds = (double)((tiles + 255) / 256), span = work / 256.0 * std::sqrt(rounds * 256.0 / (double)tiles);
        best = tt.call + (ids >= kHalvesFrom && ids <= 128 ? 0.7 : 1.0) * (rounds * tt.round + tt.k_tile * (span > k_max ? span : k_max));
    }
    best *= 0.9;
    int rows = 0;
    for (int f = 0; f < 3; ++f) {
        const int r = f == 0 ? 64 : f == 1 ? 96 : 128;
        const int64_t blocks = blocks_of(b, r);
        double block_work = 0.0;
        for (int i = 0; i < b.count; ++i)
            block_work += (double)(((int64_t)b.it[i].M + r - 1) / r * (((int64_t)b.it[i].N + 511) / 512 * 8)) * (b.it[i].K / 64);
        if (blocks >= INT64_C(1) << 22) continue;                    // a launch holds fewer than 2^32 work items
        const double rounds = (double)((blocks + 255) / 256), span = block_work / (double)blocks * rounds;
        const BlockTime& bt = kBlockTime[format][f];
        const double us = bt.call + (r == 64 && blocks > 256 ? 0.87 : 1.0) * (rounds * bt.round + bt.k_tile * (span > k_max ? span : k_max));
        if (us < best) { best = us; rows = r; }
    }
    return rows;
}

int linear_block_rows(const LinBatch& b, int wmode) { return small_block(b.it, b.count, wmode).mt ? 32 : block_rows(b, wmode); }

bool linear_takes_skinny(const LinBatch& b, int wmode)
{
    int rows = 0;
    int64_t cols = 0;
    for (int i = 0; i < b.count; ++i) {
        rows = b.it[i].M > rows ? b.it[i].M : rows;
        cols += b.it[i].N;
    }
    if (cols > INT64_C(1) << 27) return false;         // up to 16 work items a column, and a launch holds fewer than 2^32
    return rows <= kSkinnyRows ? !tiles_are_better(b, rows, wmode) : linear_block_rows(b, wmode) != 0;
}

// Whether such a call quantizes in the kernel: at most 16 rows, or so few codes in a workgroup's rows (of row tiles of 32 or 64, or of a
// small block) that repeating them costs it less than a launch.  Measured in the MFMA's order, us, pre-pass | in the kernel: 32 rows, K = 256
// 4.8 | 3.3, 1024 5.4 | 4.9, 2048 6.8 | 7.0, 4096 8.5 | 10.6; 64 rows, K = 256 5.1 | 3.7, 512 5.3 | 4.7, 1024 6.0 | 7.1; small blocks of 16
// rows, K = 1024 6.8 | 4.8, 4096 7.8 | 8.2.  In the orders taken now, of 6800 calls of 17 to 64 rows, K to 3072, in all three layouts, the
// pre-pass would be ahead by more than 5 % in 19.  any_k: K not a multiple of 64, where there are no small blocks.
bool linear_quantizes_in_kernel(const LinBatch& b, int wmode, bool any_k)
{
    int rows = 0, k_max = 0;
    int64_t tiles16 = 0;
    for (int i = 0; i < b.count; ++i) {
        rows = b.it[i].M > rows ? b.it[i].M : rows;
        k_max = b.it[i].K > k_max ? b.it[i].K : k_max;
        tiles16 += (b.it[i].N + 15) / 16;
    }
    if (rows <= kSkinnyQuantRows) return true;
    if (const int mt = any_k ? 0 : small_block(b.it, b.count, wmode).mt) return k_max <= (mt == 1 ? 3072 : 1024);
    return rows <= kSkinnyRows && (int64_t)(rows <= 32 ? 32 : 64) * k_max <= 32768 && tiles16 < 512;
}

// Whether operands that lie in rows go through LDS (TURN).  It saves accesses of the L1 cache with every K tile, most of them where rows are
// whole 128-byte lines apart (an even number of K tiles of row-major weights), and costs each wave the way through LDS once and registers:
// a wave with one or two K tiles is done sooner in the MFMA's order.  Time with the turn by time without it over 35 000 calls of 1 to 600
// rows, half of them on cached weights, by K tiles:
//   row-major, quantized here, at most 16 rows: 1 to 4 1.05 to 1.10; even 6 1.01 to 1.03 (wide 0.92 to 0.95), 8 1.00 (0.89), 16 0.91, 64 0.80; odd
//     7 1.00 to 1.04, 9 1.01 to 1.04, 11 0.97 to 1.01, 33 and more 0.85 to 0.91, but 1.02 to 1.07 on 64 K tiles and more, 1500 to 4096
//     columns, that are not in the caches;  small blocks, 17 to 32 rows: even 6 1.01 to 1.05, 8 0.96 to 1.00, 14 0.87 to 0.92; odd 7 1.03
//     to 1.11, 9 1.00 to 1.06, 11 0.97 to 1.01
//   row-major, codes from the pre-pass: even 6 1.03 to 1.10, 8 0.99 to 1.01, 10 0.96 to 1.02, 16 0.85 to 0.98; odd 9 1.04 to 1.11, 17 and more rows
//     than 32 0.98 to 1.02, others 1.02 to 1.07 up to 27, 0.95 to 1.02 from 33 on
//   pre-arranged weights, of which the activations turn: small blocks of 16 rows 1 to 5 1.04 to 1.07, 8 0.99 to 1.01, 16 0.94 to 0.96; of 32 rows 1 to 6
//     1.03 to 1.11, 12 0.97 to 1.01; 17 to 32 rows 6 1.02, 8 0.96; at most 8 rows, narrow, int8 8 1.05, 16 0.99, 64 0.86, int4 8 1.01, 10 0.98, 64 0.86;
//     9 to 16 rows int8 16 1.03, 32 0.99, 64 0.92, int4 64 and more 1.15 to 1.23 (0.95 to 1.10 on cached weights of 16 to 63); wide 5 to 31 K
//     tiles 0.97 to 1.13, 32 and more 0.92 to 0.98
// More than 32 rows quantized here have at most 8 K tiles: 1.39 (one) to 1.05 (eight).
bool linear_turns(const LinBatch& b, int wmode, bool qx)
{
    int rows = 0, k_max = 0;
    int64_t tiles16 = 0;
    for (int i = 0; i < b.count; ++i) {
        rows = b.it[i].M > rows ? b.it[i].M : rows;
        k_max = b.it[i].K > k_max ? b.it[i].K : k_max;
        tiles16 += (b.it[i].N + 15) / 16;
    }
    const int kt = k_max / 64;
    const bool lines = kt % 2 == 0, wide = tiles16 >= 512;
    const SmallBlock small = small_block(b.it, b.count, wmode);
    if (qx && !small.mt && rows > 32) return false;
    if (wmode == 0 && qx) return kt >= (!lines ? 11 : rows <= kSkinnyQuantRows && wide ? 6 : 8);
    if (wmode == 0) return kt >= (lines ? 12 : small.mt || rows <= 32 ? 28 : 17);
    if (!qx) return false;
    if (small.mt) return kt >= (small.mt == 1 ? 8 : 12);
    if (rows > kSkinnyQuantRows) return kt >= 8;
    if (wide) return kt >= 32;
    return wmode == 2 ? kt >= (rows <= 8 ? 16 : 32) : rows <= 8 && kt >= 9;
}

template <int DT, int WMODE, bool QX, bool TURN>
static void launch_small(LinBatch& b, SmallBlock f, int a_bits, int32_t* acc_out, hipStream_t st)
{
    if (f.nt == 4)                launch_one<DT, WMODE, 2, 4, 8, 2, QX, false, false, TURN>(b, a_bits, acc_out, st);
    else if (f.mt == 2 && f.nt == 2) launch_one<DT, WMODE, 2, 2, 8, 3, QX, false, false, TURN>(b, a_bits, acc_out, st);
    else if constexpr (WMODE == 3)   launch_one<DT, WMODE, 1, 2, 8, 3, QX, false, false, TURN>(b, a_bits, acc_out, st);
    else if (f.mt == 2)              launch_one<DT, WMODE, 2, 1, 8, 3, QX, false, false, TURN>(b, a_bits, acc_out, st);
    else                             launch_one<DT, WMODE, 1, 1, 8, 3, QX, false, false, TURN || (WMODE == 0 && !QX)>(b, a_bits, acc_out, st);
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
    const SmallBlock small = small_block(b.it, b.count, WMODE);
    const bool turn = linear_turns(b, WMODE, qx);
    constexpr bool kTurnPre = WMODE == 0;                               // codes from the pre-pass: only row-major weights lie in rows
    if (small.mt) {
        if (qx && turn)       launch_small<DT, WMODE, true, true>(b, small, a_bits, acc_out, st);
        else if (qx)          launch_small<DT, WMODE, true, false>(b, small, a_bits, acc_out, st);
        else if (turn)        launch_small<DT, WMODE, false, kTurnPre>(b, small, a_bits, acc_out, st);
        else                  launch_small<DT, WMODE, false, false>(b, small, a_bits, acc_out, st);
    } else if (rows > kSkinnyRows) {
        const int block = block_rows(b, WMODE);
        if (block == 64 && blocks_of(b, 64) > 256) launch_one<DT, WMODE, 4, 4, 4, 2, false, false, true, kTurnPre>(b, a_bits, acc_out, st);
        else if (block == 64)                launch_one<DT, WMODE, 4, 4, 8, 2, false, false, true, kTurnPre>(b, a_bits, acc_out, st);
        else if (block == 96 && rows > 96)   launch_one<DT, WMODE, 6, 4, 8, 2, false, false, true, kTurnPre>(b, a_bits, acc_out, st);
        else if (block == 96)                launch_one<DT, WMODE, 6, 4, 8, 2, false, true, true, kTurnPre>(b, a_bits, acc_out, st);
        else if (rows > 128)                 launch_one<DT, WMODE, 8, 4, 8, 2, false, false, true, kTurnPre>(b, a_bits, acc_out, st);
        else                                 launch_one<DT, WMODE, 8, 4, 8, 2, false, true, true, kTurnPre>(b, a_bits, acc_out, st);
    } else if (qx && rows > 32)              launch_one<DT, WMODE, 4, WMODE == 3 ? 2 : 1, 8, 2, true, true, false, false>(b, a_bits, acc_out, st);
    else if (qx && rows > kSkinnyQuantRows) {
        if (turn) launch_one<DT, WMODE, 2, WMODE == 3 ? 2 : 1, 8, 2, true, true, false, true>(b, a_bits, acc_out, st);
        else      launch_one<DT, WMODE, 2, WMODE == 3 ? 2 : 1, 8, 2, true, true, false, false>(b, a_bits, acc_out, st);
    } else if (qx) {
        if (turn) launch_mt<DT, WMODE, 1, true, true>(b, tiles16, a_bits, acc_out, st);
        else      launch_mt<DT, WMODE, 1, true, false>(b, tiles16, a_bits, acc_out, st);
    } else {
        auto by_rows = [&](auto turn_tag) {
            constexpr bool TURN = decltype(turn_tag)::value;
            if (rows <= 32)      launch_mt<DT, WMODE, 2, false, TURN>(b, tiles16, a_bits, acc_out, st);
            else if (rows <= 48) launch_mt<DT, WMODE, 3, false, TURN>(b, tiles16, a_bits, acc_out, st);
            else                 launch_mt<DT, WMODE, 4, false, TURN>(b, tiles16, a_bits, acc_out, st);
        };
        if (turn) by_rows(std::integral_constant<bool, kTurnPre>{});
        else      by_rows(std::false_type{});
    }
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

// K not a multiple of 64, at most kSkinnyRows rows of a single call; row-major codes in it.xq unless qx.  Rows that do not start on a
// whole dword cost each load several accesses, and every workgroup reads all activation rows: more than 32 of those stay with the
// tiles.  Measured, us, tiles (static_linear_anyk.hip) | here: 8 x 3000, K = 1000 8.1 | 4.1, 16 x 4096, 2500 11.8 | 6.5, 1 x 1000, 4000
// 14.6 | 5.5, 32 x 4096, 1376 9.1 | 7.1, 64 x 4096, 1376 9.2 | 8.4, 64 x 1000, 4000 15.9 | 12.2; odd K: 1 x 4000, 3001 14.3 | 7.4, 16
// rows 15.0 | 13.7, 32 rows 14.9 | 15.0, 40 rows 15.0 | 17.4, 64 rows 15.1 | 21.5; 32 x 900, 777 8.3 | 7.6, 64 rows 8.5 | 9.7.
// Rows a few bytes longer or shorter than whole 128-byte lines begin at about the same place of a line, so that the sixteen rows of a load
// contend for the same part of the L1 cache: at most 3 bytes and K over 600 the tiles are ahead from 17 rows on, 32 x 540, K = 2561 13.9 |
// 18.8, 30 x 1732, 1026 8.6 | 10.5 (1024 + 2), 32 x 540, 2569 13.9 | 11.9; 3 bytes from 25 rows, one byte and long rows from 14, 16 x 975, 3841
// 18.4 | 22.0; 4 bytes from 49, 62 x 3224, 516 6.9 | 7.5.
bool linear_anyk_takes_skinny(int64_t M, int64_t N, int64_t K)
{
    const int64_t over = K % 128, off = over < 64 ? over : 128 - over;
    int64_t most = K % 4 == 0 ? kSkinnyRows : 32;
    if (K % 4 == 0 && off == 4 && K < 1200) most = 48;
    if (off <= 3 && K > 600) most = off == 3 ? 24 : off == 1 && K > 1600 ? 13 : 16;
    return M <= most && K > 64 && N <= INT64_C(1) << 27;
}

template <int DT>
static void launch_anyk_dt(LinBatch& b, bool qx, int a_bits, int32_t* acc_out, hipStream_t st)
{
    const int rows = b.it[0].M;
    const int64_t tiles16 = ((int64_t)b.it[0].N + 15) / 16;
    if (qx && rows > 32)                    launch_one<DT, 0, 4, 1, 8, 2, true, false, false, false, true>(b, a_bits, acc_out, st);
    else if (qx && rows > kSkinnyQuantRows) launch_one<DT, 0, 2, 1, 8, 2, true, false, false, false, true>(b, a_bits, acc_out, st);
    else if (qx)         launch_mt<DT, 0, 1, true, false, true, false>(b, tiles16, a_bits, acc_out, st);
    else if (rows <= 32) launch_mt<DT, 0, 2, false, false, true, false>(b, tiles16, a_bits, acc_out, st);
    else if (rows <= 48) launch_mt<DT, 0, 3, false, false, true, false>(b, tiles16, a_bits, acc_out, st);
    else                 launch_mt<DT, 0, 4, false, false, true, false>(b, tiles16, a_bits, acc_out, st);
}

void launch_linear_anyk_skinny(LinBatch& b, sasq_dtype dt, bool qx, int a_bits, int32_t* acc_out, hipStream_t st)
{
    if (dt == SASQ_F16) launch_anyk_dt<SASQ_F16>(b, qx, a_bits, acc_out, st);
    else                launch_anyk_dt<SASQ_BF16>(b, qx, a_bits, acc_out, st);
}

// ---- the backward GEMM ----------------------------------------------------------------------
template <int DT, int MT, int NT, int NW, int D, bool ONCE, bool EVEN, bool TURN>
__global__ __launch_bounds__(64 * NW)
void bwd_skinny_kernel(const LinItem it, float* __restrict__ acc_out)
{
    __shared__ __attribute__((aligned(1024))) char lds[skinny_lds_bytes<2, MT, NT, NW, false, EVEN, true, TURN>()];
    const int id = (int)blockIdx.x, octet = id >> 3;                 // as in skinny_kernel
    const int mblk = octet % it.tiles_m, nblk = octet / it.tiles_m * 8 + (id & 7);
    if (nblk >= it.tiles_n) return;
    skinny_body<DT, 2, MT, NT, NW, D, false, ONCE, EVEN, TURN, true>(it, mblk, nblk, 8, reinterpret_cast<int32_t*>(acc_out), lds);
}

template <int DT, int MT, int NT, int NW, int D, bool ONCE, bool EVEN, bool TURN>
static void launch_bwd_one(LinItem& it, float* acc_out, hipStream_t st)
{
    it.tiles_m = (it.M + 16 * MT - 1) / (16 * MT);
    it.tiles_n = (it.N + 16 * NT - 1) / (16 * NT);
    bwd_skinny_kernel<DT, MT, NT, NW, D, ONCE, EVEN, TURN><<<(it.tiles_n + 7) / 8 * 8 * it.tiles_m, 64 * NW, 0, st>>>(it, acc_out);
}

static LinItem bwd_item(const void* dy, const void* wt, void* dx, int64_t M, int64_t N, int64_t K)
{
    LinItem it{};
    it.x = dy;
    it.wq = static_cast<const uint8_t*>(wt);
    it.y = static_cast<uint16_t*>(dx);
    it.M = (int)M;
    it.N = (int)K;                                                   // the body's columns and contraction bytes
    it.K = (int)(2 * N);
    return it;
}

// Rows per workgroup: 32, small blocks, where small_block has some; at most 64 rows 64 (in row tiles of 16, 32 or 64); more rows 64 or
// 96 by 64 columns (128 never pay).  At most 16 rows are never behind the tiles, which read the weight as often: of 540 calls 15 x 1696 ->
// 20160 is the worst, 14.3 us on the tiles | 15.4 here.  More rows read dY once in 32 or 64 columns, so that with many columns they end up
// waiting for it, while one round of 128x128 tiles holds them all: weights that the caches hold, us, 30 x 4480 -> 24768 33.5 | 57.6, 28 x
// 2400 -> 25216 20.2 | 31.3; that they have not seen, 40 x 4224 -> 17792 42.9 | 50.1, 51 x 960 -> 24960 11.7 | 17.7, but 17 x 9696 -> 9728 79 |
// 49, 25 x 13248 -> 8896 107 | 77.  And 64 x 256 x 256 4.8 | 3.4, 131 x 2816 x 1344 23.4 | 17.3, 334 x 11072 x 1536 76.2 | 52.5.
// So both sides are estimated, here from the same 3900 calls as the tiles, on weights that the caches have not seen (rms error 8 to 9 %), and
// the tiles left from 10 % less time on: the calls then take 0.71 of what the tiles alone take, 2 % more than the best form of each.  That is with
// dY in the MFMA's order here and in half lines there; as both are now, over 4250 calls of 17 to 1500 rows, it is 2.1 %: up to 0.5 where these kernels
// are taken, 4 to 9 on tiles of 128x128.
int bwd_takes_skinny(int64_t M, int64_t N, int64_t K, double tile_us)
{
    if (N > kBwdOffsetCols) return 0;                                // the body's lane offsets are 32-bit
    const LinItem it = bwd_item(nullptr, nullptr, nullptr, M, N, K);
    const SmallBlock small = small_block(&it, 1, 2);
    // blocks of 32 x 64 leave most of their eight waves idle under four contraction tiles: 198 x 64 -> 1984 3.6 | 4.1, 65 x 96 -> 4928 4.1 | 4.3
    if (small.mt && (small.nt < 4 || N >= 128)) return 32;
    if (M <= 16) return K <= INT64_C(1) << 26 ? 64 : 0;              // up to 32 work items a column
    if (M > 32 && K <= 448) return 0;                                // fewer than eight runs of weight rows leave XCDs without work
    struct Form { int rows, block_rows, block_cols; RoundTime time; };
    static const Form forms[] = {{64, 32, 32, {2.5, 0.05, 0.065, 0.039}}, {64, 64, 64, {1.3, 1.8, 0.131, 0.094}},
                                 {64, 64, 64, {1.5, 2.5, 0.120, 0.032}}, {96, 96, 64, {1.5, 3.7, 0.160, 0.046}}};
    const int first = M <= 32 ? 0 : M <= 64 ? 1 : 2, last = M <= 64 ? first : 3;
    double best = 0.9 * tile_us;
    int rows = 0;
    for (int i = first; i <= last; ++i) {
        const Form& f = forms[i];
        const int64_t blocks = (M + f.block_rows - 1) / f.block_rows * ((K + 8 * f.block_cols - 1) / (8 * f.block_cols) * 8);
        if (blocks >= INT64_C(1) << 22) continue;                    // a launch holds fewer than 2^32 work items
        const double us = f.time.launch(blocks, (double)(N / 32));
        if (us < best) { best = us; rows = f.rows; }
    }
    return rows;
}

// At most 16 rows: narrow workgroups (16 columns) while they make one round of at most 256, wide ones from then on.
template <int DT, bool TURN>
static void launch_bwd_dt(LinItem& it, float* acc_out, int rows, hipStream_t st)
{
    if (rows == 32) {
        const SmallBlock f = small_block(&it, 1, 2);
        if (f.nt == 4)      launch_bwd_one<DT, 2, 4, 8, 2, false, false, TURN>(it, acc_out, st);
        else if (f.nt == 2) launch_bwd_one<DT, 2, 2, 8, 3, false, false, TURN>(it, acc_out, st);
        else if (f.mt == 2) launch_bwd_one<DT, 2, 1, 8, 3, false, false, TURN>(it, acc_out, st);
        else                launch_bwd_one<DT, 1, 1, 8, 3, false, false, TURN>(it, acc_out, st);
    } else if (it.M > 64) {
        if (rows == 64) launch_bwd_one<DT, 4, 4, 8, 2, false, true, TURN>(it, acc_out, st);
        else            launch_bwd_one<DT, 6, 4, 8, 2, false, true, TURN>(it, acc_out, st);
    } else if (it.M <= 16) {
        if (it.N > 4096) launch_bwd_one<DT, 1, 2, 8, 3, true, false, TURN>(it, acc_out, st);
        else             launch_bwd_one<DT, 1, 1, 8, 4, true, false, TURN>(it, acc_out, st);
    } else if (it.M <= 32) {
        launch_bwd_one<DT, 2, 2, 8, 3, true, false, TURN>(it, acc_out, st);
    } else {
        launch_bwd_one<DT, 4, 4, 8, 2, true, false, TURN>(it, acc_out, st);
    }
}

// Whether dY turns in LDS (linear_turns; its rows are whole lines apart where the contraction has an even number of tiles of 32).  Time with the
// turn by time without it over 23 000 calls, half of them on cached weights, by contraction tiles:
//   at most 8 rows, of which a load brings as many that are none: 1.02 to 1.06 at any length (wide 1.00 to 1.04);  9 to 16 rows: even 8
//     1.00, 12 0.98, 64 0.95, wide 32 1.00, 64 0.98; odd 33 1.01, 65 0.98
//   small blocks: even 2 1.02 to 1.05, 6 0.98 to 1.00, 8 0.95 to 0.97, 32 0.80 to 0.86; odd 9 to 27 1.00 to 1.06, 33 0.96 to 0.98, 65 0.84 to 0.92; of
//     32 x 64: even 8 to 10 1.00 to 1.03, 14 0.99, 64 0.84; odd 9 to 27 1.04 to 1.09, 33 1.00, 65 0.95
//   17 to 32 rows: even 8 1.01, 16 0.98; odd 1.01 to 1.07 at any length;  33 to 64 rows: even 20 1.05, 32 0.99, 64 0.94; odd 33 1.02, 65 0.96
//   row blocks: even 0.80 to 0.87; odd 25 to 31 1.05, 33 0.97
bool bwd_turns(int64_t M, int64_t N, int64_t K)
{
    const int64_t kt = N / 32;
    const bool lines = kt % 2 == 0;
    const LinItem it = bwd_item(nullptr, nullptr, nullptr, M, N, K);
    const SmallBlock small = small_block(&it, 1, 2);
    if (small.mt) return kt >= (small.nt == 4 ? (lines ? 14 : 64) : (lines ? 8 : 32));
    if (M <= 8) return false;
    if (M <= 16) return kt >= (lines && K <= 4096 ? 10 : 64);
    if (M <= 32) return lines && kt >= 16;
    if (M <= 64) return kt >= (lines ? 32 : 64);
    return lines || kt >= 32;
}

void launch_bwd_skinny(const void* dy, const void* wt, void* dx, float* acc_out, int64_t M, int64_t N, int64_t K, sasq_dtype dt, int rows, hipStream_t st)
{
    LinItem it = bwd_item(dy, wt, dx, M, N, K);
    auto by_dt = [&](auto turn_tag) {
        constexpr bool TURN = decltype(turn_tag)::value;
        if (dt == SASQ_F16) launch_bwd_dt<SASQ_F16, TURN>(it, acc_out, rows, st);
        else                launch_bwd_dt<SASQ_BF16, TURN>(it, acc_out, rows, st);
    };
    if (bwd_turns(M, N, K)) by_dt(std::true_type{});
    else                    by_dt(std::false_type{});
}

}  // namespace sasq

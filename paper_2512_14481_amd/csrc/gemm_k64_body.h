// The tile body shared by the GEMM kernels on the 16-row MFMA shapes (v_mfma_i32_16x16x64_i8 for the static linear,
// v_mfma_f32_16x16x32_{f16,bf16} for the backward of the frozen linear): K pipeline, fragment reads, epilogue.
// Included by static_linear_k64.hip, grouped_k64.hip and linear_bwd.hip; the description of the machine shape is at the top of the former.
#pragma once

#include "sasq_device.h"
#include "gemm_tile.h"
#include <type_traits>

namespace sasq {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

template <int DT> struct Mfma16x16;
template <> struct Mfma16x16<SASQ_F16> {
    static __device__ __forceinline__ f32x4 mma(const i32x4& a, const i32x4& b, const f32x4& c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};
template <> struct Mfma16x16<SASQ_BF16> {
    static __device__ __forceinline__ f32x4 mma(const i32x4& a, const i32x4& b, const f32x4& c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};

// Weight paths (values shared with static_linear.hip): int8 row-major, int8 pre-arranged in 1 KB blocks, int4
// pre-arranged (it stays packed through L2 -> LDS and is unpacked between the fragment read and the MFMA: a nibble
// moved to the high half of a byte is the int8 value 16 w, so two mask/shift operations per dword turn 8 nibbles into
// 8 bytes; the accumulators are then exactly 16 acc and are shifted back in the epilogue).
enum { KW_I8 = 0, KW_I8B = 2, KW_I4B = 3 };

// Groups of channels with a factor each (GROUPED below): none; 32 channels, half a K tile; one K tile; two; a multiple of four; another even
// number; another odd one.
enum { GR_NONE = 0, GR_HALF, GR_ONE, GR_TWO, GR_FOURS, GR_EVEN, GR_ODD };

constexpr int kFacBytes = 1024;      // per wave: the epilogue's per-column factors (BN/2 floats, loaded twice over)
template <int BM, int BN> constexpr int lds_bytes_k64() { return Tile<BM, BN>::kLds + 4 * kFacBytes; }
// OP 2 (below): three slots of two K tiles of X, four stages of the weights, no factors.
template <int BM, int BN> constexpr int lds_bytes_lines()
{
    using T = Tile<BM, BN>;
    constexpr int ring = 3 * 2 * T::kXBytes + kStages * T::kWBytes, epi = 4 * T::kEpiBytes;
    return ring > epi ? ring : epi;
}

// One direct 128-bit-per-lane load from global memory into LDS: lane i deposits its 16 bytes at
// LDS address lds_addr + 16 i.  The memory address is a scalar base plus a 32-bit per-lane offset,
// so that the instruction needs no vector address arithmetic.  The compiler does not see the LDS
// write: the callers order it against their LDS reads with s_waitcnt vmcnt and barriers.
__device__ __forceinline__ void lds_load16(uint32_t lds_addr, const void* base, uint32_t lane_off)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(lane_off), "s"(base) : "memory");
}
// The same with the LDS address given as a sum of two scalars (a slot's fixed address + the stage's offset): the
// addition writes M0 itself, one scalar instruction less in front of every load of the K loop.
__device__ __forceinline__ void lds_load16(uint32_t lds_a, uint32_t lds_b, const void* base, uint32_t lane_off)
{
    asm volatile("s_add_i32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3"
                 :: "s"(lds_a), "s"(lds_b), "v"(lane_off), "s"(base) : "memory", "scc");
}

// Measurement hook: a translation unit that wants cycle and wall-clock stamps at five points of every tile (body start,
// pipeline filled, K loop done, stages drained, epilogue done) defines SASQ_TILE_TS(k) before including this file (the
// benchmark's instrumented build of static_linear_k64.hip does); everywhere else it expands to nothing.
#ifndef SASQ_TILE_TS
#define SASQ_TILE_TS(k)
#endif

// GROUPED (Sec. 3, Eq. 3): one activation factor per group of `group_tiles` K tiles; s_ptr then
// points at the factors.  The int32 accumulators cover one group at a time (a group's first K tile
// multiplies into a zero accumulator operand) and are folded into fp32 sums at its end,
// f = fma(fl32(acc), s_g, f) in ascending group order; the epilogue applies s_w and the bias to f,
// and acc_out receives f (as float bits).  Tiles of 128 rows only (f doubles the accumulator registers);
// with 128x128 tiles two waves share a SIMD and one wave's fold runs under the other's MFMAs.
// GR_HALF: groups of 32 channels, two per K tile.  One MFMA contracts the whole 64-byte stage, so every K tile
// is multiplied twice, once with the activation fragments of channels 32..63 zeroed and once with those of 0..31
// zeroed (lanes 32..63 resp. 0..31 of a fragment), each pass into zero accumulators and folded with its own factor:
// twice the matrix work and a fold per 32 channels, and faster than sums on the VALUs all the same.
// OP 1: the same machine on v_mfma_f32_16x16x32_{f16,bf16} (DT picks the type): both operands hold 16-bit floats, 32
// per 64-byte stage row; the "activation" operand xq is then read ROW-MAJOR (rows of K bytes, the 16-byte chunks of a
// row gathered per lane as for row-major weights), the weight operand from 1 KB blocks; K is the contraction length in
// BYTES; the accumulators are fp32, written out rounded to 16 bits without any factor (s_ptr, s_w, bias unused), and
// acc_out receives the fp32 sums.  This is the backward GEMM of the frozen linear (linear_bwd.hip).
// OP 2: OP 1 with X read in whole cache lines, an even number of K tiles: a load takes 8 rows x 128 bytes, two K tiles, instead of 16
// rows x 64 bytes, which are half a line each: L2 then answers two requests for a line, and memory delivers it in halves, two K tiles
// apart.  X has a ring of its own, three slots of two K tiles, that fills the LDS to its 160 KB (256x256) and is requested four to five
// K tiles ahead.  us, halves | lines, operands from memory: f16 4096 x 11008 -> 4096 254 | 231, 4096 x 4096 -> 11008 273 | 258, bf16 255 | 231
// and 268 | 258, 4096 x 4096 -> 4096 101 | 94, 1024 x 5120 -> 5120 79 | 66, 777 x 4096 -> 4096 36 | 36; weights in the caches, f16 241 | 234, 259 |
// 258, bf16 235 | 227, 258 | 257, 95 | 93, 71 | 62, 32 | 29.
template <int DT, int WMODE, int BM, int BN, bool ROWS, int GROUPED = GR_NONE, int OP = 0>
__device__ __forceinline__
void gemm_k64_body(const int8_t* __restrict__ xq, const uint8_t* __restrict__ wq,
                   const float* __restrict__ s_ptr, const float* __restrict__ s_w,
                   const float* __restrict__ bias, uint16_t* __restrict__ y,
                   int32_t* __restrict__ acc_out, int M, int N, int K,
                   int tm, int tn, char* lds, int group_tiles = 0)
{
    static_assert(!GROUPED || (BM == 128 && !ROWS), "grouped factors: 128-row tiles");
    static_assert(OP == 0 || (WMODE == KW_I8B && !ROWS && !GROUPED), "float contraction: pre-arranged weight blocks, no factors");
    constexpr bool FLT = OP != 0, XL = OP == 2;
    constexpr bool WHOLE = GROUPED && GROUPED != GR_HALF && GROUPED != GR_ONE;       // groups of whole K tiles
    using AccT = std::conditional_t<FLT, f32x4, i32x4>;
    using S = Store16<DT>;
    using T = Tile<BM, BN>;
    constexpr int MF = BM / 32, NF = BN / 32;          // 16x16 tiles per wave along m, n
    constexpr int XS = T::XS, WS = T::WS;              // 1 KB slabs per wave per stage
    constexpr bool I4 = WMODE == KW_I4B;
    constexpr int WSL = I4 ? WS / 2 : WS;              // weight loads per wave per K tile (packed int4: half the bytes)
    constexpr int kLoads = XS + WSL;                   // direct loads per wave per K tile
    constexpr int kAccShift = I4 ? 4 : 0;
    // LDS: four stages of X and weights; XL: three slots of two K tiles of X, then four stages of weights
    constexpr int kXSlot = 2 * T::kXBytes, kXSlots = 3;
    constexpr int kWArea = XL ? kXSlots * kXSlot : T::kXBytes, kWStep = XL ? T::kWBytes : T::kStageBytes;
    auto x_stage = [&](int st) -> char* { return &lds[st * T::kStageBytes]; };
    auto w_stage = [&](int st) -> char* { return &lds[kWArea + st * kWStep]; };

    const int m0 = tm * BM, n0 = tn * BN;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // uniform: LDS addresses of the loads stay scalar
    const int wm = wave & 1, wn = wave >> 1;
    const int KT = K / kBK;

    // ---- direct L2 -> LDS loads: load j of wave w fills rows (4j + w)*16 .. +16 of a stage ----
    // Address of a load = scalar base of the operand panel at the K tile (advanced once per K tile)
    // + a per-lane 32-bit offset fixed for the whole tile: the load itself then costs the wave two
    // scalar instructions and the load (anything more does not fit behind a 16-cycle MFMA).
    const int lrow = lane >> 2;
    const int lchunk = (lane & 3) ^ (((lane >> 3) & 3) ^ ((lane >> 5) & 1));
    const int last_rb = (M - 1) >> 4;
    const int8_t* xpanel = FLT ? xq + (int64_t)m0 * K : xq + (int64_t)(m0 >> 4) * KT * 1024;
    constexpr int kXTileStep = FLT ? kBK : 1024;
    const int8_t* wpanel = reinterpret_cast<const int8_t*>(wq) + (WMODE == KW_I8B ? (int64_t)(n0 >> 4) * KT * 1024
                                                                  : I4 ? (int64_t)(n0 >> 5) * KT * 1024 : (int64_t)n0 * K);
    constexpr int XO = XL ? 2 * XS : XS;
    uint32_t xoff[XO], woff[WSL];
#pragma unroll
    for (int j = 0; j < XO; ++j)
        xoff[j] = XL  ? (uint32_t)(min((4 * j + wave) * 8 + (lane >> 3), M - 1 - m0) * K + (((lane & 7) ^ (lane >> 3)) << 4))
                : FLT ? (uint32_t)(min((4 * j + wave) * 16 + lrow, M - 1 - m0) * K + lchunk * 16)
                      : (uint32_t)(min(4 * j + wave, last_rb - (m0 >> 4)) * KT * 1024 + lane * 16);
#pragma unroll
    for (int j = 0; j < WSL; ++j) {
        if (I4) woff[j] = (uint32_t)(min(4 * j + wave, ((N - 1) >> 5) - (n0 >> 5)) * KT * 1024 + lane * 16);   // blocks of 32 rows
        else if (WMODE == KW_I8B) woff[j] = (uint32_t)(min(4 * j + wave, ((N - 1) >> 4) - (n0 >> 4)) * KT * 1024 + lane * 16);
        else                 woff[j] = (uint32_t)(min((4 * j + wave) * 16 + lrow, N - 1 - n0) * K + lchunk * 16);
    }
    constexpr int kWTileStep = (WMODE == KW_I8B || I4) ? 1024 : kBK;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_ptr_t)&lds[0] + (uint32_t)wave * 1024u;
    // loads 0..XS-1: activations, XS..: weights.  XL: the activations are half `xh` (rows 0..BM/2 or BM/2..BM) of the pair of K tiles at
    // xtile, into the slot at xslot.
    auto dma_at = [&](const int8_t* xtile, const int8_t* wtile, int j, int st, int xh, uint32_t xslot) {
        if (j >= XS)  lds_load16(lds_base + kWArea + (j - XS) * 4096, (uint32_t)(st * kWStep), wtile, woff[j - XS < WSL ? j - XS : 0]);
        else if (XL)  lds_load16(lds_base + (xh * XS + j) * 4096, xslot, xtile, xoff[XL ? xh * XS + j : 0]);
        else          lds_load16(lds_base + j * 4096, (uint32_t)st * T::kStageBytes, xtile, xoff[j < XS ? j : 0]);
    };
    // K tile Tk into stage st = Tk & 3.  XL: with an odd tile go the first halves of the pair that begins with the tile after it, with an
    // even one the second halves of its own pair; past the last pair it is fetched again, into a slot that is free, to keep the counts.
    auto dma = [&](int Tk, int j, int st) {
        const int pair = (Tk + 1) >> 1;
        dma_at(XL ? xpanel + (int64_t)min(pair, KT / 2 - 1) * (2 * kBK) : xpanel + (int64_t)Tk * kXTileStep, wpanel + (int64_t)Tk * kWTileStep, j, st,
               1 - (Tk & 1), (uint32_t)(pair % kXSlots * kXSlot));
    };
    // The steady loop keeps the operands' addresses at its current group of four K tiles here: a load of
    // tile i + 4 then adds a constant to them.
    const int8_t* xrun = xpanel;
    const int8_t* wrun = wpanel;

    // ---- LDS -> MFMA fragments: lane l reads chunk l/16 of row l%16 of a 16-row tile ----
    const int frow = lane & 15, fq = lane >> 4;
    const int foff = frow * kBK + ((fq ^ swz64(frow)) << 4);
    const int xbase = wm * (BM / 2) * kBK, wbase = wn * (BN / 2) * kBK;
    // Packed int4: a 1 KB block holds 32 rows x 64 k; the 16 codes k = 16 G .. + 15 of row r are the 8 bytes at
    // 256 G + 8 r (G = 2 kk + g in the layout's own terms), so lane l fetches 8 bytes at 256 (l/16) + 8 (16 h + l%16),
    // h = the 16-row half of the block its tile is.
    using WFrag = std::conditional_t<I4, u32x2, i32x4>;
    i32x4 fx[2][MF];
    WFrag fw[2][NF];
    // XL: row r of a slot holds 128 bytes, chunk c at position c ^ (r & 7); the second K tile's chunks are 4 .. 7
    const int xl_off = (wm * (BM / 2) + frow) * 2 * kBK + ((fq ^ (frow & 7)) << 4);
    auto read_frag = [&](int set, int st, int idx, uint32_t xslot, int odd) {   // the MF activation fragments first, then the NF weight ones
        if (idx < MF) {
            fx[set][idx] = *reinterpret_cast<const i32x4*>(XL ? &lds[xslot + (xl_off ^ (odd * kBK)) + idx * 32 * kBK]
                                                              : x_stage(st) + xbase + idx * 16 * kBK + foff);
        } else if constexpr (I4) {
            const int g = idx - MF;
            fw[set][g] = *reinterpret_cast<const u32x2*>(w_stage(st) + (wn * (BN / 64) + (g >> 1)) * 1024 + 256 * fq + 8 * (16 * (g & 1) + frow));
        } else {
            fw[set][idx - MF] = *reinterpret_cast<const i32x4*>(w_stage(st) + wbase + (idx - MF) * 16 * kBK + foff);
        }
    };
    auto wfrag_piece = [&](const WFrag& f, int j) -> int {   // output dword j of the unpacked operand
        if constexpr (I4) {
            const uint32_t p = f[j >> 1];
            return (int)(((j & 1) ? p : (p << 4)) & 0xF0F0F0F0u);
        } else {
            return f[j];
        }
    };
    i32x4 wv_ahead = {0, 0, 0, 0}, wv_next = {0, 0, 0, 0};   // packed int4: the weight operand of the row to come
    auto wfrag = [&](const WFrag& f) -> i32x4 {         // the MFMA's weight operand: as read, or unpacked here
        if constexpr (I4) {
            const uint32_t p0 = f[0], p1 = f[1];
            return i32x4{(int)((p0 << 4) & 0xF0F0F0F0u), (int)(p0 & 0xF0F0F0F0u), (int)((p1 << 4) & 0xF0F0F0F0u), (int)(p1 & 0xF0F0F0F0u)};
        } else {
            return f;
        }
    };

    AccT acc[NF][MF];
    f32x4 fsum[GROUPED ? NF : 1][GROUPED ? MF : 1];           // fp32 sums over groups
#pragma unroll
    for (int g = 0; g < (GROUPED ? NF : 1); ++g)
#pragma unroll
        for (int b = 0; b < (GROUPED ? MF : 1); ++b) fsum[g][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    // ---- K pipeline ----
    // Iteration i multiplies K tile i from fragment set i&1 while it reads the fragments of tile
    // i+1 into the other set and issues the loads of tile i+4 into the stage tile i has just left.
    // At its top: this wave's fragment reads of tile i are complete and its own loads of tile i+1
    // have landed (loads return in issue order, so that is one s_waitcnt vmcnt with the loads of
    // the later tiles still allowed in flight); after the barrier the same holds for every wave,
    // so tile i+1 may be read and stage i&3 refilled.
    // Side work is dealt out behind the MFMAs (one wave per SIMD: nothing else hides a clump of
    // issue): the fragment reads first, every `kFragStep` MFMAs, then the loads.
    // The last four or five iterations (TAIL) request a tile only if there is one left and wait for
    // what is still due.
    constexpr int NM = MF * NF, NFR = MF + NF;
    constexpr int kFragStep = NM / 2 / NFR >= 1 ? NM / 2 / NFR : 1;
    constexpr int kLoadStep = (NM - kFragStep * NFR) / kLoads;
    static_assert(kLoadStep >= 1, "side work does not fit behind the MFMAs");
    // The constant address space keeps a group's factor a scalar load; as a vector load it would stand behind the stages' loads and wait
    // for all of them.
    const auto factors = (const __attribute__((address_space(4))) float*)s_ptr;
    auto fold = [&](float sg) {                                // f = fma(fl32(acc), s_g, f) for every accumulator
#pragma unroll
        for (int g = 0; g < NF; ++g)
#pragma unroll
            for (int b = 0; b < MF; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    fsum[GROUPED ? g : 0][GROUPED ? b : 0][e] =
                        __builtin_fmaf((float)((int)acc[g][b][e] >> kAccShift), sg, fsum[GROUPED ? g : 0][GROUPED ? b : 0][e]);
    };
    // XL: the slots of the steady trip's first three pairs; the fourth and fifth take the first two's
    uint32_t slot0 = 0, slot1 = kXSlot, slot2 = 2 * kXSlot;
    auto iteration = [&](int i, auto cur_tag, auto stage_tag, auto first_tag, auto tail_tag) {
        constexpr int CUR = decltype(cur_tag)::value;
        constexpr int STG = decltype(stage_tag)::value;        // i & 3 where the copy of the body knows it, else -1
        constexpr bool FIRST = decltype(first_tag)::value;
        constexpr bool TAIL = decltype(tail_tag)::value;
        if (!TAIL) {
            __builtin_amdgcn_s_waitcnt(kWaitLgkm0 & waitcnt_vm(2 * kLoads));
        } else {
            const int later = min(i + 3, KT - 1) - (i + 1);    // tiles after i+1 already requested
            if (later >= 2)      __builtin_amdgcn_s_waitcnt(kWaitLgkm0 & waitcnt_vm(2 * kLoads));
            else if (later == 1) __builtin_amdgcn_s_waitcnt(kWaitLgkm0 & waitcnt_vm(kLoads));
            else                 __builtin_amdgcn_s_waitcnt(kWaitLgkm0 & waitcnt_vm(0));
        }
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int stn = STG >= 0 ? (STG + 1) & 3 : (i + 1) & 3;
        const bool more = !TAIL || i + 1 < KT;                 // a next tile to read fragments of
        const int rodd = STG >= 0 ? (STG + 1) & 1 : (i + 1) & 1;
        const uint32_t rslot = !XL ? 0 : STG >= 0 ? (STG == 0 ? slot0 : STG == 3 ? slot2 : slot1) : (uint32_t)(((i + 1) >> 1) % kXSlots * kXSlot);
        i32x4 xhalf[GROUPED == GR_HALF ? MF : 1];                    // groups of 32: the fragments with one half of the channels zeroed
        if constexpr (GROUPED == GR_HALF) {
#pragma unroll
            for (int b = 0; b < MF; ++b) xhalf[b] = fq < 2 ? fx[CUR][b] : i32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int g = 0; g < NF; ++g) {
            // Packed int4: the operand of this row was unpacked while the previous row multiplied (wv_ahead), and the next
            // row's -- at the end of the tile, row 0 of the next tile -- is unpacked one output dword behind each of this
            // row's first four MFMAs: done at the top of a row, the six VALU operations and their latency stand in front of
            // the row's first MFMA (195 of 1405 cycles per K tile on the 13B layer).
            const i32x4 wv = I4 ? wv_ahead : wfrag(fw[CUR][g]);
            const bool ahead_in_tile = g + 1 < NF;
            // Rows go back and forth, so that every MFMA keeps one operand of the one before it: fewer bits toggle, and with data the
            // clock is what the power leaves.  A register-only loop sustains 0.6 to 1 % more (f16 1957 -> 1973 TFLOP/s, int8 on the
            // workload's codes 4606 -> 4648 TOP/s, on random bytes 4175 -> 4217), the GEMMs 0.2 to 0.9 % (8192 x 8192 x 8192 int8 401 -> 398 us).
            const WFrag& fnext = ahead_in_tile ? fw[CUR][g + 1 < NF ? g + 1 : 0] : fw[1 - CUR][0];
#pragma unroll
            for (int bi = 0; bi < MF; ++bi) {
                const int b = (g & 1) ? MF - 1 - bi : bi;
                // K tile 0 multiplies into a zero accumulator operand instead of clearing the accumulators
                if constexpr (FLT) {
                    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                    acc[g][b] = Mfma16x16<DT>::mma(wv, fx[CUR][b], FIRST ? zero : acc[g][b]);
                } else {
                    const i32x4 zero = {0, 0, 0, 0};
                    acc[g][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wv, GROUPED == GR_HALF ? xhalf[GROUPED == GR_HALF ? b : 0] : fx[CUR][b],
                                                                      FIRST ? zero : acc[g][b], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                const int t = g * MF + bi;
                if (t < kFragStep * NFR) {
                    if (t % kFragStep == 0 && more) read_frag(1 - CUR, stn, t / kFragStep, rslot, rodd);
                } else if (!TAIL || i + 4 < KT) {
                    const int u = t - kFragStep * NFR;
                    if (u % kLoadStep == 0 && u / kLoadStep < kLoads) {
                        if constexpr (WHOLE) dma(min(i + 4, KT - 1), u / kLoadStep, STG >= 0 ? STG : i & 3);
                        else if constexpr (STG >= 0) dma_at(xrun + (XL ? (STG + 5) / 2 * 2 : STG + 4) * kXTileStep, wrun + (STG + 4) * kWTileStep, u / kLoadStep, STG,
                                                       1 - (STG & 1), STG == 0 ? slot2 : STG == 3 ? slot1 : slot0);
                        else                    dma(i + 4, u / kLoadStep, i & 3);
                    }
                }
                if constexpr (I4) {
                    if (bi < 4 && (ahead_in_tile || more)) wv_next[bi] = wfrag_piece(fnext, bi);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (I4) wv_ahead = wv_next;
        }
        if constexpr (GROUPED == GR_HALF) {
            // channels 0..31 of this K tile are in acc: fold them, then the same tile with channels 32..63
            fold(factors[2 * i]);
#pragma unroll
            for (int b = 0; b < MF; ++b) xhalf[b] = fq < 2 ? i32x4{0, 0, 0, 0} : fx[CUR][b];
#pragma unroll
            for (int g = 0; g < NF; ++g) {
                const i32x4 wv = wfrag(fw[CUR][g]);
#pragma unroll
                for (int b = 0; b < MF; ++b)
                    acc[g][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wv, xhalf[GROUPED == GR_HALF ? b : 0], i32x4{0, 0, 0, 0}, 0, 0, 0);
            }
            fold(factors[2 * i + 1]);
        }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    using S2 = std::integral_constant<int, 2>;
    using S3 = std::integral_constant<int, 3>;
    using SR = std::integral_constant<int, -1>;               // stage known only at run time
    using Yes = std::true_type;
    using No = std::false_type;
    auto step = [&](int i, auto cur_tag, auto stage_tag, auto first_tag, auto tail_tag) {
        if constexpr (GROUPED == GR_HALF) {
            iteration(i, cur_tag, stage_tag, Yes{}, tail_tag);     // both folds of the tile happen inside
        } else if constexpr (GROUPED == GR_ONE) {
            iteration(i, cur_tag, stage_tag, Yes{}, tail_tag);
            fold(factors[i]);
        } else {
            iteration(i, cur_tag, stage_tag, first_tag, tail_tag);
        }
    };
    SASQ_TILE_TS(0);
    // fill: the first four tiles requested, tile 0 landed for everyone, its fragments read
    const int nfill = WHOLE ? 4 : min(KT, 4);
    if constexpr (XL) {
#pragma unroll
        for (int j = 0; j < XS; ++j) dma(-1, j, 3);            // the first pair's first halves
    }
    for (int t = 0; t < nfill; ++t)
#pragma unroll
        for (int j = 0; j < kLoads; ++j) dma(WHOLE ? min(t, KT - 1) : t, j, t);
    if (nfill == 4)      __builtin_amdgcn_s_waitcnt(waitcnt_vm(3 * kLoads));
    else if (nfill == 3) __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * kLoads));
    else if (nfill == 2) __builtin_amdgcn_s_waitcnt(waitcnt_vm(kLoads));
    else                 __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < NFR; ++k) read_frag(0, 0, k, 0, 0);
    if constexpr (I4) wv_ahead = wfrag(fw[0][0]);
    SASQ_TILE_TS(1);
    // A multiple of four steady iterations (they always have a tile i+4 to request), then the tail.
    // The steady loop is written out four iterations at a time: every copy of the body then knows
    // its fragment set and its LDS stages at compile time, and the addresses of its fragment reads
    // and loads are constants instead of a chain of scalar arithmetic in front of the first read.
    // XL: its last steady iteration requests the first halves of a pair that is there.
    const int steady = XL ? (KT >= 10 ? ((KT - 6) & ~3) : 0) : WHOLE ? 0 : KT >= 8 ? ((KT - 4) & ~3) : 0;
    if (!WHOLE && steady > 0) {
        step(0, C0{}, S0{}, Yes{}, No{});
        step(1, C1{}, S1{}, No{}, No{});
        step(2, C0{}, S2{}, No{}, No{});
        step(3, C1{}, S3{}, No{}, No{});
#pragma unroll 1
        for (int it = 4; it < steady; it += 4) {
            xrun += 4 * kXTileStep;
            wrun += 4 * kWTileStep;
            if constexpr (XL) {                                // the pairs 2 it + 4 .. of this trip
                const uint32_t first = slot2;
                slot2 = slot1;
                slot1 = slot0;
                slot0 = first;
            }
            step(it, C0{}, S0{}, No{}, No{});
            step(it + 1, C1{}, S1{}, No{}, No{});
            step(it + 2, C0{}, S2{}, No{}, No{});
            step(it + 3, C1{}, S3{}, No{}, No{});
        }
    } else if (!GROUPED) {
#pragma unroll
        for (int g = 0; g < NF; ++g)
#pragma unroll
            for (int b = 0; b < MF; ++b) acc[g][b] = AccT{0, 0, 0, 0};
    }
    // The per-column factors of the epilogue are requested here, a few K tiles before they are
    // needed (fetched inside the epilogue they cost eight memory latencies in a row): one direct
    // load per wave parks the BN/2 factors of its block in LDS, behind the stages.  (An extra load
    // in the in-order queue only makes the counted waits of the tail wait for more, never less.)
    const int wn0 = n0 + wn * (BN / 2), wm0 = m0 + wm * (BM / 2);
    const bool cols_inside = !FLT && wn0 + BN / 2 <= N && (reinterpret_cast<uintptr_t>(s_w) & 15u) == 0 &&
                             (bias == nullptr || (reinterpret_cast<uintptr_t>(bias) & 15u) == 0);
    char* fac = &lds[T::kLds + wave * kFacBytes];
    if (cols_inside)
        lds_load16(lds_base - (uint32_t)wave * 1024u + T::kLds + (uint32_t)wave * kFacBytes, s_w + wn0,
                   (uint32_t)(lane & (BN / 8 - 1)) * 16u);   // lanes past BN/8 fetch the same factors again: no lane reads past the block
    if constexpr (WHOLE) {
        // Groups in straight lines: a branch that decides between the first K tile's body and the others' costs a copy of each in the loop and
        // registers (254 and 256, int8 20 of them spilled around the loops; 192 to 226 so).  Requests are unconditional: past the end the
        // last tile comes again and a stage's old fragments are read, which nothing uses.  us, branches and a separate tail | straight lines,
        // weights in the caches, groups of 64, 128, 256, 512: int8 2048 x 4096 -> 11008 137, 116, 110, 102 | 132, 107, 99, 93; 2048 x 4096 ->
        // 4096 54, 48, 45, 43 | 52, 44, 42, 40; 700 x 8192 -> 5000 69, 57, 47, 43 | 60, 47, 41, 38; int4 157, 128, 109, 100 | 155, 120, 102,
        // 93 and 62, 51, 45, 44 | 63, 49, 43, 41.  One K tile a group takes the loop of the plain GEMM; int4 is slower so where some CUs hold two
        // workgroups and the rest one, or the last of several rounds does (257 to 511, 768 to 1023 tiles), by 1.03 to 1.09 at 16 to 31 K tiles
        // and 1.00 to 1.03 beyond, 0.94 to 1.00 elsewhere.  Not kept for it: straight lines (1.02 to 1.06 there, 0.98 to 1.02 beyond),
        // two K tiles a trip with run-time stages (1.07 to 1.20).  Nor the fold tile by tile between the next group's first MFMAs (128, 256,
        // 512: 148, 124, 116 against 139, 123, 120, one series).
        auto first = [&](int i, auto cur_tag, auto stage_tag) { iteration(i, cur_tag, stage_tag, Yes{}, No{}); };
        auto rest = [&](int i, auto cur_tag, auto stage_tag) { iteration(i, cur_tag, stage_tag, No{}, No{}); };
        auto rest_of_group = [&](int& i, int tiles, auto cur_tag) {      // an even number of tiles
            using CUR = decltype(cur_tag);
#pragma unroll 1
            for (; tiles > 0; tiles -= 2, i += 2) {
                rest(i, CUR{}, SR{});
                rest(i + 1, std::integral_constant<int, 1 - CUR::value>{}, SR{});
            }
        };
        // A group's factor is requested when the one before it is folded: it then lands under the K tiles between.
        const int groups = KT / group_tiles;
        int group_idx = 0;
        float sg = factors[0];
        auto fold_group = [&] {
            fold(sg);
            group_idx = min(group_idx + 1, groups - 1);
            sg = factors[group_idx];
        };
        int i = 0;
        if constexpr (GROUPED == GR_TWO) {                          // two K tiles each, stages known in every copy of the body
            auto group = [&](auto stage_tag) {
                constexpr int S = decltype(stage_tag)::value;
                first(i + S, C0{}, stage_tag);
                rest(i + S + 1, C1{}, std::integral_constant<int, S + 1>{});
                fold_group();
            };
#pragma unroll 1
            for (; i + 4 <= KT; i += 4) {
                group(S0{});
                group(S2{});
            }
            if (i < KT) group(S0{});
        } else if constexpr (GROUPED == GR_FOURS) {                   // multiples of four
#pragma unroll 1
            do {
                first(i, C0{}, S0{});
                rest(i + 1, C1{}, S1{});
                rest(i + 2, C0{}, S2{});
                rest(i + 3, C1{}, S3{});
                i += 4;
#pragma unroll 1
                for (int tiles = group_tiles - 4; tiles > 0; tiles -= 4, i += 4) {
                    rest(i, C0{}, S0{});
                    rest(i + 1, C1{}, S1{});
                    rest(i + 2, C0{}, S2{});
                    rest(i + 3, C1{}, S3{});
                }
                fold_group();
            } while (i < KT);
        } else if constexpr (GROUPED == GR_EVEN) {                   // other even numbers
#pragma unroll 1
            do {
                first(i, C0{}, SR{});
                rest(i + 1, C1{}, SR{});
                i += 2;
                rest_of_group(i, group_tiles - 2, C0{});
                fold_group();
            } while (i < KT);
        } else {                                               // an odd number: the next group's fragments move back to set 0
#pragma unroll 1
            do {
                first(i++, C0{}, SR{});
                rest_of_group(i, group_tiles - 1, C1{});
                fold_group();
#pragma unroll
                for (int b = 0; b < MF; ++b) fx[0][b] = fx[1][b];
#pragma unroll
                for (int g = 0; g < NF; ++g) fw[0][g] = fw[1][g];
            } while (i < KT);
        }
    } else {
#pragma unroll 1
        for (int i = steady; i < KT; i += 2) {                  // KT - steady is 1 .. 8, steady is even
            step(i, C0{}, SR{}, No{}, Yes{});
            if (i + 1 < KT) step(i + 1, C1{}, SR{}, No{}, Yes{});
        }
    }
    SASQ_TILE_TS(2);
    // the last fragment reads (none pending) and loads (none in flight) are complete; LDS is reused
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0 & waitcnt_vm(0));
    SASQ_TILE_TS(3);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // ---- epilogue: Y = fl32(fl32(acc) * fl32(s * s_w[n])) (+ bias), staged through LDS in [m][n]
    // order as 16-bit values, written with 128-bit stores, BN contiguous bytes per row ----
    const float s = (ROWS || GROUPED || FLT) ? 1.0f : *s_ptr;
    const bool has_bias = !FLT && bias != nullptr;
    char* epi = &lds[wave * T::kEpiBytes];
    float srow[MF];                                            // ROWS: the factor of each row this lane holds
#pragma unroll
    for (int b = 0; b < MF; ++b) srow[b] = ROWS ? s_ptr[min(wm0 + b * 16 + frow, M - 1)] : 1.0f;
    // Common case (block inside the matrix): the block goes out in chunks of 16 rows through a small
    // staging buffer, software-pipelined: while chunk b is dequantized, the LDS reads of chunk b-1 are
    // in flight; then chunk b-1 is stored, chunk b written to the buffer and read back.  LDS serves a
    // wave's requests in order, so one buffer is enough.  (Staging the whole block first and storing
    // it afterwards left the wave waiting for LDS and for the store queue in turn: 11 k cycles per
    // 256x256 tile against 5 k.)
    const bool vec_ok = (N & 7) == 0;
    constexpr int kChunksPerRow = BN / 16;                      // 16-byte chunks in a wave-block row
    constexpr int kRowsPerPass = 64 / kChunksPerRow;
    const int crow = lane / kChunksPerRow, cchunk = lane % kChunksPerRow;
    auto write_tile_chunked = [&](auto bias_tag) {
        constexpr bool BIAS = decltype(bias_tag)::value;
        constexpr int kPasses = 16 / kRowsPerPass;             // read-back passes per 16-row chunk
        float cs[NF][4], bs[NF][4];
#pragma unroll
        for (int g = 0; g < NF; ++g) {
            const int nl = g * 16 + 4 * fq;
            f32x4 sv = {1.0f, 1.0f, 1.0f, 1.0f}, bv = {0.0f, 0.0f, 0.0f, 0.0f};
            if (FLT) {
            } else if (cols_inside) {
                sv = *reinterpret_cast<const f32x4*>(fac + nl * 4);
                if (BIAS) bv = *reinterpret_cast<const f32x4*>(bias + wn0 + nl);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) { sv[e] = s_w[wn0 + nl + e]; if (BIAS) bv[e] = bias[wn0 + nl + e]; }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) { cs[g][e] = (ROWS || GROUPED) ? sv[e] : s * sv[e]; bs[g][e] = bv[e]; }
        }
        char* wr = epi + frow * T::kEpiStride + 4 * fq * 2;
        const char* rd = epi + crow * T::kEpiStride + cchunk * 16;
        char* dst = reinterpret_cast<char*>(y + (int64_t)(wm0 + crow) * N + wn0 + cchunk * 8);
        const int64_t row_step = (int64_t)kRowsPerPass * N * 2, chunk_step = (int64_t)16 * N * 2;
        u32x4 back[kPasses];
#pragma unroll
        for (int b = 0; b <= MF; ++b) {
            u32x2 pk[NF];
            if (b < MF) {
#pragma unroll
                for (int g = 0; g < NF; ++g) {
                    float yv[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float cc = ROWS ? srow[b < MF ? b : 0] * cs[g][e] : cs[g][e];
                        float v;
                        if constexpr (FLT)          v = acc[g][b < MF ? b : 0][e];
                        else if constexpr (GROUPED) v = fsum[GROUPED ? g : 0][GROUPED ? (b < MF ? b : 0) : 0][e] * cc;   // Y = fl32(f * s_w[n])
                        else                        v = (float)((int)acc[g][b < MF ? b : 0][e] >> kAccShift) * cc;
                        if (BIAS) v = v + bs[g][e];
                        yv[e] = v;
                    }
                    pk[g] = u32x2{S::pack(yv[0], yv[1]), S::pack(yv[2], yv[3])};
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (b > 0) {
#pragma unroll
                for (int p = 0; p < kPasses; ++p) *reinterpret_cast<u32x4*>(dst + (b - 1) * chunk_step + p * row_step) = back[p];
            }
            if (b < MF) {
#pragma unroll
                for (int g = 0; g < NF; ++g) *reinterpret_cast<u32x2*>(wr + g * 32) = pk[g];
#pragma unroll
                for (int p = 0; p < kPasses; ++p) back[p] = *reinterpret_cast<const u32x4*>(rd + p * kRowsPerPass * T::kEpiStride);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (vec_ok && wm0 + BM / 2 <= M && wn0 + BN / 2 <= N) {
        if (has_bias) write_tile_chunked(std::true_type{});
        else          write_tile_chunked(std::false_type{});
    } else {
    auto write_tile = [&](auto bias_tag) {
        constexpr bool BIAS = decltype(bias_tag)::value;
        f32x4 svs[NF];                                         // all parked factors requested together: one LDS latency
#pragma unroll
        for (int g = 0; g < NF; ++g) svs[g] = *reinterpret_cast<const f32x4*>(fac + (g * 16 + 4 * fq) * 4);
#pragma unroll
        for (int g = 0; g < NF; ++g) {
            const int nl = g * 16 + 4 * fq;                    // column within the wave's block
            float cs[4], bs[4];
            if (FLT) {
#pragma unroll
                for (int e = 0; e < 4; ++e) { cs[e] = 1.0f; bs[e] = 0.0f; }
            } else if (cols_inside) {
                const f32x4 sv = svs[g];
                f32x4 bv = {0.0f, 0.0f, 0.0f, 0.0f};
                if (BIAS) bv = *reinterpret_cast<const f32x4*>(bias + wn0 + nl);
#pragma unroll
                for (int e = 0; e < 4; ++e) { cs[e] = (ROWS || GROUPED) ? sv[e] : s * sv[e]; bs[e] = bv[e]; }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int ne = min(wn0 + nl + e, N - 1);
                    cs[e] = (ROWS || GROUPED) ? s_w[ne] : s * s_w[ne];
                    bs[e] = BIAS ? bias[ne] : 0.0f;
                }
            }
#pragma unroll
            for (int b = 0; b < MF; ++b) {
                const int ml = b * 16 + frow;
                float yv[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float cc = ROWS ? srow[b] * cs[e] : cs[e];
                    float v;
                    if constexpr (FLT)          v = acc[g][b][e];
                    else if constexpr (GROUPED) v = fsum[GROUPED ? g : 0][GROUPED ? b : 0][e] * cc;      // Y = fl32(f * s_w[n])
                    else                        v = (float)((int)acc[g][b][e] >> kAccShift) * cc;
                    if (BIAS) v = v + bs[e];
                    yv[e] = v;
                }
                u32x2 pk = {S::pack(yv[0], yv[1]), S::pack(yv[2], yv[3])};
                *reinterpret_cast<u32x2*>(epi + ml * T::kEpiStride + nl * 2) = pk;
            }
        }
    };
    if (has_bias) write_tile(std::true_type{});
    else          write_tile(std::false_type{});
    // each wave reads back only what it wrote itself: no workgroup barrier needed
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
#pragma unroll 4
    for (int p = 0; p < (BM / 2) / kRowsPerPass; ++p) {
        const int ml = p * kRowsPerPass + crow;
        const int m = wm0 + ml, n = wn0 + cchunk * 8;
        if (m >= M || n >= N) continue;
        const u32x4 v = *reinterpret_cast<const u32x4*>(epi + ml * T::kEpiStride + cchunk * 16);
        uint16_t* dst = y + (int64_t)m * N + n;
        if (vec_ok && n + 7 < N) {
            *reinterpret_cast<u32x4*>(dst) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (n + e < N) dst[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        }
    }
    }   // block at an edge of the matrix
    // inspection output (int32 accumulators): straight from the registers, apart from the common path
    if (acc_out) {
#pragma unroll
        for (int g = 0; g < NF; ++g)
#pragma unroll
            for (int b = 0; b < MF; ++b) {
                const int m = wm0 + b * 16 + frow, n = wn0 + g * 16 + 4 * fq;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (m < M && n + e < N)
                        acc_out[(int64_t)m * N + n + e] = GROUPED ? __float_as_int(fsum[GROUPED ? g : 0][GROUPED ? b : 0][e])
                                                                  : FLT ? __float_as_int((float)acc[g][b][e]) : ((int)acc[g][b][e] >> kAccShift);
            }
    }
    SASQ_TILE_TS(4);
}

}  // namespace sasq

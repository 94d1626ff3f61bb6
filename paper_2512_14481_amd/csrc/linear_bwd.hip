// Backward of the frozen quantized linear with respect to its input (Sec. 4.2: during scale
// training the gradient reaches each quantization factor through the frozen layers):
//     dX[m,k] = sum_n dY[m,n] * Wq[n,k],   Wq[n,k] = round16(fl32(W_int[n,k]) * s_w[n])   (Eq. 2's W_int * S_w)
// as a 16-bit MFMA GEMM with fp32 accumulation for gfx950.  The dequantized weight is prepared
// once (it is frozen) in the GEMM's operand blocks, transposed so that the contraction index n
// runs along operand rows.
#include "sasq_device.h"
#include "gemm_tile.h"
#include "gemm_k64.h"
#include "gemm_k64_body.h"
#include <cstdlib>
#include <cstring>
#include <type_traits>

namespace sasq {

constexpr int kBwdCols = kBK / 2;                  // contraction elements per stage row (16-bit)

// Prepared weight layout: the matrix B[k][n] = Wq[n][k] (K rows, N 16-bit columns; rows padded
// to a multiple of 16 and columns to a multiple of 32 with zeros) cut into 1 KB blocks of 16 rows
// x 32 columns, block (kb, nb) at (kb * Npad/32 + nb) * 1024, the 16-byte chunk c (8 columns) of
// row r at 16 * (4r + (c ^ swz64(r))): what one wave's direct load deposits in an LDS stage.
__device__ __forceinline__ int64_t bwd_weight_offset(int64_t k, int64_t n, int64_t Npad)
{
    const int r = (int)(k & 15), c = (int)((n >> 3) & 3);
    return ((k >> 4) * (Npad / kBwdCols) + (n >> 5)) * 1024 + ((4 * r + (c ^ swz64(r))) << 4) + ((n & 7) << 1);
}

// The transpose goes through LDS: a workgroup takes 32 rows of W (one block column) x WK codes, 128-byte pieces of the rows
// in, whole 1 KB blocks out, lane l of a wave writing the block's 16-byte chunk l from eight byte reads.  Bound by its bytes,
// one in and two out per weight: 11008 x 4096 and 4096 x 11008 22.7 us, 6.0 TB/s (a thread per chunk that read its eight codes
// from memory one by one: 63 on average, 47 to 97).
// WK: 512, or 128 where workgroups of 512 would leave CUs without work or be mostly past the row's end.  Measured, us, a thread per
// chunk | 512 | 128 codes: 16 x 64 2.6 | 2.8 | 2.4, 256 x 256 3.3 | 3.6 | 2.7, 100 x 1000 3.3 | 4.3 | 2.7, 1024 x 2048 6.0 | 4.3 | 3.7,
// 16384 x 64 3.7 | 3.8 | 3.2.
template <int DT, bool INT4, int WK>
__global__ __launch_bounds__(256) void prepare_bwd_weight_kernel(
    const uint8_t* __restrict__ wq, const float* __restrict__ s_w, uint8_t* __restrict__ out,
    int64_t N, int64_t K, int64_t Npad, int64_t Kpad, uint32_t ktiles, uint32_t first)
{
    using S = Store16<DT>;
    using Piece = std::conditional_t<INT4, u32x2, u32x4>;
    constexpr int kPiece = (int)sizeof(Piece), kPieces = WK / 16 / 8;
    __shared__ __attribute__((aligned(16))) int8_t tile[kBwdCols][WK + 16];
    const uint32_t id = first + blockIdx.x;
    const int64_t k0 = (int64_t)(id % ktiles) * WK, n0 = (int64_t)(id / ktiles) * kBwdCols;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane >> 2, c = (lane & 3) ^ swz64(r);
    float sw[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {                      // requested with the codes, not behind the barrier
        const float f = s_w[min(n0 + 8 * c + e, N - 1)];
        sw[e] = n0 + 8 * c + e < N ? f : 0.0f;
    }
    {
        const int64_t row = n0 + (threadIdx.x >> 3), len = INT4 ? K / 2 : K;
        const uint8_t* src = wq + min(row, N - 1) * len;
        const int64_t at = (k0 >> 4) * kPiece + (threadIdx.x & 7) * kPiece;
        Piece v[kPieces];
        if (k0 + WK <= K) {
#pragma unroll
            for (int j = 0; j < kPieces; ++j) v[j] = load_piece<Piece>(src + at + j * 8 * kPiece);
        } else {
#pragma unroll
            for (int j = 0; j < kPieces; ++j) v[j] = load_piece_edge<Piece>(src, at + j * 8 * kPiece, len);
        }
#pragma unroll
        for (int j = 0; j < kPieces; ++j) {
            u32x4 codes;
            if constexpr (INT4) codes = widen_int4(v[j]);
            else                codes = v[j];
            if (row >= N) codes = u32x4{0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4*>(&tile[threadIdx.x >> 3][((threadIdx.x & 7) + 8 * j) * 16]) = codes;
        }
    }
    __syncthreads();
#pragma unroll 2
    for (int b = wave; b < WK / 16; b += 4) {
        const int64_t k = k0 + 16 * b + r;
        if (k0 + 16 * b >= Kpad) break;
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            o[e] = S::pack((float)tile[8 * c + 2 * e][16 * b + r] * sw[2 * e], (float)tile[8 * c + 2 * e + 1][16 * b + r] * sw[2 * e + 1]);
        if (k >= K) o = u32x4{0u, 0u, 0u, 0u};
        __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(out + ((k0 >> 4) + b) * (Npad / kBwdCols) * 1024 + (n0 >> 5) * 1024 + lane * 16));
    }
}

// Any-shape fallback (contraction length not a multiple of 32, or unaligned rows): one thread per
// output, fp32 accumulation in ascending n.
template <int DT>
__global__ __launch_bounds__(256) void linear_bwd_scalar_kernel(
    const uint16_t* __restrict__ dy, const uint8_t* __restrict__ wt, uint16_t* __restrict__ dx,
    float* __restrict__ acc_out, int64_t M, int64_t N, int64_t K, int64_t Npad)
{
    using S = Store16<DT>;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= M * K) return;
    const int64_t m = idx / K, k = idx - m * K;
    float acc = 0.0f;
    for (int64_t n = 0; n < N; ++n) {
        const float w = S::one(*reinterpret_cast<const uint16_t*>(wt + bwd_weight_offset(k, n, Npad)));
        acc = acc + S::one(dy[m * N + n]) * w;
    }
    if (acc_out) acc_out[idx] = acc;
    dx[idx] = S::enc(acc);
}

template <int DT> struct Mfma16;
template <> struct Mfma16<SASQ_F16> {
    static __device__ __forceinline__ f32x16 mma(const i32x4& a, const i32x4& b, const f32x16& c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};
template <> struct Mfma16<SASQ_BF16> {
    static __device__ __forceinline__ f32x16 mma(const i32x4& a, const i32x4& b, const f32x16& c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};

// ---------------------------------------------------------------------------------------------
// 16-bit MFMA GEMM, dX[M,K] = dY[M,N] . B^T with B the prepared weight.
//
// Same machine shape as the int8 forward GEMM: workgroup tile BM (m) x BN (k), 4 waves 2x2, each
// wave (BM/2) x (BN/2) as 32x32 tiles of v_mfma_f32_32x32x16_{f16,bf16}; a ring of 4 LDS stages
// of 64 contraction bytes (32 elements) per operand row, filled three stages ahead with direct
// 128-bit L2 -> LDS loads dealt out one per MFMA group; fragments of the next contraction substep
// are read from LDS behind the MFMAs of the current one; one workgroup barrier per stage.
// dY is read row-major (16 rows x 64 bytes per wave load), the weight block-wise (1 KB per load).
// The weight tile is the MFMA's A operand, the dY tile its B operand: D[i][j], i <-> k, j <-> m,
// so a lane holds 4 consecutive k per accumulator quad; lane group g of an operand holds
// contraction elements 8g..8g+7 of the 16-element substep, the natural order of a 16-byte chunk.
// The accumulation order inside the matrix unit is the hardware's; results are compared within
// the fp32 accumulation bound, not bit for bit.
// ---------------------------------------------------------------------------------------------
template <int DT, int BM, int BN>
__global__ __launch_bounds__(kGemmThreads)
__attribute__((amdgpu_waves_per_eu(Tile<BM, BN>::kWavesPerSimd, Tile<BM, BN>::kWavesPerSimd)))
void linear_bwd_mfma_kernel(const uint8_t* __restrict__ dy, const uint8_t* __restrict__ wt,
                            uint16_t* __restrict__ dx, float* __restrict__ acc_out,
                            int M, int N, int K, int tiles_m, int tiles_n)
{
    using S = Store16<DT>;
    using T = Tile<BM, BN>;
    constexpr int MF = T::MF, NF = T::NF, XS = T::XS, WS = T::WS;
    __shared__ __attribute__((aligned(1024))) char lds[T::kLds];
    auto stage_ptr = [&](int st, int operand) -> char* { return &lds[st * T::kStageBytes + operand * T::kXBytes]; };

    int tm, tn;
    if (!tile_of_block((int)blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    const int m0 = tm * BM, k0 = tn * BN;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave & 1, wn = wave >> 1;
    const int KT = N / kBwdCols;                                   // contraction tiles
    auto eff_tile = [&](int Tk) { return min(max(Tk, 0), KT - 1); };
    auto stage_of = [&](int Tk) { return (Tk < 0 ? 0 : Tk) & 3; };

    // direct loads: load j of wave w fills rows (4j + w)*16 .. +16 of a stage; lane i writes LDS
    // slot i of that 1 KB (row i/4, position i%4) and so fetches logical chunk (i%4) ^ swz64(row)
    const int lrow = lane >> 2;
    const int lchunk = (lane & 3) ^ (((lane >> 3) & 3) ^ ((lane >> 5) & 1));
    const uint8_t* gx[XS];
    const uint8_t* gw[WS];
    const int64_t row_bytes = (int64_t)N * 2;
#pragma unroll
    for (int j = 0; j < XS; ++j)
        gx[j] = dy + (int64_t)min(m0 + (4 * j + wave) * 16 + lrow, M - 1) * row_bytes + lchunk * 16;
#pragma unroll
    for (int j = 0; j < WS; ++j)
        gw[j] = wt + (int64_t)min((k0 >> 4) + 4 * j + wave, (K - 1) >> 4) * KT * 1024 + lane * 16;
    auto dma_x = [&](int Tk, int j) {
        __builtin_amdgcn_global_load_lds((glb_ptr_t)(gx[j] + (int64_t)eff_tile(Tk) * kBK),
                                         (lds_ptr_t)(stage_ptr(stage_of(Tk), 0) + (4 * j + wave) * 1024), 16, 0, 0);
    };
    auto dma_w = [&](int Tk, int j) {
        __builtin_amdgcn_global_load_lds((glb_ptr_t)(gw[j] + (int64_t)eff_tile(Tk) * 1024),
                                         (lds_ptr_t)(stage_ptr(stage_of(Tk), 1) + (4 * j + wave) * 1024), 16, 0, 0);
    };

    // LDS -> MFMA fragments
    const int frow = lane & 31, fgrp = lane >> 5;
    int foff[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) foff[kk] = frow * kBK + (((kk * 2 + fgrp) ^ swz64(frow)) << 4);
    const int xbase = wm * (BM / 2) * kBK, wbase = wn * (BN / 2) * kBK;
    i32x4 fx[2][MF], fw[2][NF];
    auto read_frag = [&](int set, int st, int kk, int idx) {
        if (idx < MF) fx[set][idx] = *reinterpret_cast<const i32x4*>(stage_ptr(st, 0) + xbase + idx * 32 * kBK + foff[kk]);
        else          fw[set][idx - MF] = *reinterpret_cast<const i32x4*>(stage_ptr(st, 1) + wbase + (idx - MF) * 32 * kBK + foff[kk]);
    };

    f32x16 acc[NF][MF];   // [k tile][m tile]; first written by the MFMAs of contraction tile 0

    constexpr int kFrags = MF + NF;
    // group g of substep `set`: MF MFMAs with the group's side items dealt out behind them
    auto group = [&](int set, int g, auto mode_tag, int nitems, auto&& item) {
        constexpr int MODE = decltype(mode_tag)::value;     // 0: pipeline fill, 1: math, 2: math into zero
        if (MODE == 0) {
            for (int k = 0; k < nitems; ++k) item(k);
            __builtin_amdgcn_sched_barrier(0);
            return;
        }
#pragma unroll
        for (int b = 0; b < MF; ++b) {
            if (MODE == 2 && set == 0) {
                const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                acc[g][b] = Mfma16<DT>::mma(fw[set][g], fx[set][b], zero);
            } else {
                acc[g][b] = Mfma16<DT>::mma(fw[set][g], fx[set][b], acc[g][b]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (b < MF - 1) {
                if (b < nitems) item(b);
            } else {
                for (int k = MF - 1; k < nitems; ++k) item(k);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // Iteration i consumes contraction tile i in two substeps; phase 0 issues the weight loads of
    // tile i+3, phase 1 the dY loads of tile i+4; loads return in issue order, so "tile i+1 has
    // landed" is one vmcnt wait with the number of loads issued after it.
    auto iteration = [&](int i, auto mode_tag) {
        constexpr bool MATH = decltype(mode_tag)::value != 0;
        const int st = i & 3;
#pragma unroll
        for (int g = 0; g < NF; ++g) {
            const int r0 = g * kFrags / NF, nr = MATH ? (g + 1) * kFrags / NF - r0 : 0;
            group(0, g, mode_tag, nr + 1, [&](int k) {
                if (k < nr) { read_frag(1, st, 1, r0 + k); return; }
                if (g < WS) dma_w(i + 3, g);
            });
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0 & waitcnt_vm(2 * XS + 2 * WS));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int g = 0; g < NF; ++g) {
            const int r0 = g * kFrags / NF, nr = (i + 1 >= 0) ? (g + 1) * kFrags / NF - r0 : 0;
            group(1, g, mode_tag, nr + 1, [&](int k) {
                if (k < nr) { read_frag(0, (i + 1) & 3, 0, r0 + k); return; }
                if (g < XS) dma_x(i + 4, g);
            });
        }
    };
    using Fill = std::integral_constant<int, 0>;
    using Math = std::integral_constant<int, 1>;
    using Open = std::integral_constant<int, 2>;
    iteration(-4, Fill{});
    iteration(-3, Fill{});
    iteration(-2, Fill{});
    iteration(-1, Fill{});
    iteration(0, Open{});
#pragma unroll 1
    for (int it = 1; it < KT; ++it) iteration(it, Math{});
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0 & waitcnt_vm(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // epilogue: D[i][j], i = 8*(v/4) + 4*(lane/32) + v%4 -> k, j = lane%32 -> m.  Each wave rounds
    // its block to 16 bits, stages it through its own LDS region in [m][k] order and writes dX
    // with 128-bit stores.
    char* epi = &lds[wave * T::kEpiBytes];
    const int wk0 = k0 + wn * (BN / 2), wm0 = m0 + wm * (BM / 2);
#pragma unroll
    for (int a = 0; a < NF; ++a)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int kl = a * 32 + 8 * g + 4 * fgrp;
#pragma unroll
            for (int b = 0; b < MF; ++b) {
                const int ml = b * 32 + frow;
                u32x2 pk = {S::pack(acc[a][b][4 * g], acc[a][b][4 * g + 1]), S::pack(acc[a][b][4 * g + 2], acc[a][b][4 * g + 3])};
                *reinterpret_cast<u32x2*>(epi + ml * T::kEpiStride + kl * 2) = pk;
            }
        }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    const bool vec_ok = (K & 7) == 0;
    constexpr int kChunksPerRow = BN / 16;
    constexpr int kRowsPerPass = 64 / kChunksPerRow;
    const int crow = lane / kChunksPerRow, cchunk = lane % kChunksPerRow;
#pragma unroll 4
    for (int p = 0; p < (BM / 2) / kRowsPerPass; ++p) {
        const int ml = p * kRowsPerPass + crow;
        const int m = wm0 + ml, k = wk0 + cchunk * 8;
        if (m >= M || k >= K) continue;
        const u32x4 v = *reinterpret_cast<const u32x4*>(epi + ml * T::kEpiStride + cchunk * 16);
        uint16_t* dst = dx + (int64_t)m * K + k;
        if (vec_ok && k + 7 < K) {
            *reinterpret_cast<u32x4*>(dst) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (k + e < K) dst[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
        }
    }
    // inspection output: the fp32 sums before the 16-bit rounding, straight from the registers
    if (acc_out) {
#pragma unroll
        for (int a = 0; a < NF; ++a)
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int b = 0; b < MF; ++b) {
                    const int m = wm0 + b * 32 + frow, k = wk0 + a * 32 + 8 * g + 4 * fgrp;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (m < M && k + e < K) acc_out[(int64_t)m * K + k + e] = acc[a][b][4 * g + e];
                }
    }
}

template <int DT, int BM, int BN>
static void launch_bwd(const void* dy, const void* wt, void* dx, float* acc_out, int64_t M, int64_t N, int64_t K, hipStream_t st)
{
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (int)((K + BN - 1) / BN);
    const int grid = ((tiles_m * tiles_n + 7) / 8) * 8;
    linear_bwd_mfma_kernel<DT, BM, BN><<<grid, kGemmThreads, 0, st>>>(
        static_cast<const uint8_t*>(dy), static_cast<const uint8_t*>(wt), static_cast<uint16_t*>(dx), acc_out,
        (int)M, (int)N, (int)K, tiles_m, tiles_n);
}

// The same GEMM on v_mfma_f32_16x16x32_{f16,bf16} through the tile body shared with the int8 forward GEMM
// (gemm_k64_body.h): 16x16 tiles, one MFMA per 64-byte stage row, scalar-addressed direct loads, chunked epilogue.
// The default: a register-only loop of the 16x16x32 form sustains about 18 % more than 32x32x16 on this
// power-limited part (1.97 against 1.67 PFLOP/s for f16).  dY is the body's row-major operand, the prepared
// weight its block operand; K of the body is the contraction length in bytes.  LINES: dY in whole cache lines (bwd_reads_lines).
template <int DT, int BM, int BN, bool LINES>
__global__ __launch_bounds__(kGemmThreads)
__attribute__((amdgpu_waves_per_eu(Tile<BM, BN>::kWavesPerSimd, Tile<BM, BN>::kWavesPerSimd)))
void linear_bwd_k32_kernel(const uint8_t* __restrict__ dy, const uint8_t* __restrict__ wt,
                           uint16_t* __restrict__ dx, float* __restrict__ acc_out,
                           int M, int N, int K, int tiles_m, int tiles_n)
{
    __shared__ __attribute__((aligned(1024))) char lds[LINES ? lds_bytes_lines<BM, BN>() : lds_bytes_k64<BM, BN>()];
    int tm, tn;
    if (!tile_of_block((int)blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    gemm_k64_body<DT, KW_I8B, BM, BN, false, false, LINES ? 2 : 1>(reinterpret_cast<const int8_t*>(dy), wt, nullptr, nullptr, nullptr, dx,
                                                        reinterpret_cast<int32_t*>(acc_out), M, K, N * 2, tm, tn, lds);
}

// Whether a tile of so many rows reads dY in whole cache lines (the body's OP 2): rows of whole 128-byte pieces, and enough of them that what
// the ring's longer fill and tail cost is made up.  Whole lines in parts of halves over 2000 calls, half of them on cached weights, by contraction
// tiles of 32: tiles of 128 rows 2 to 6 1.02, 8 1.10, 12 1.08, 16 1.04, 24 1.00, 32 to 63 0.97, 64 0.92, 128 0.89; of 256 rows 8 to 24
// 1.02 to 1.06, 32 to 63 1.01, 64 0.99, 128 0.96, 256 0.93.
bool bwd_reads_lines(int64_t N, int tile_rows) { return N % (2 * kBwdCols) == 0 && N >= (tile_rows == 256 ? 64 : 32) * kBwdCols; }

template <int DT, int BM, int BN>
static void launch_bwd_k32(const void* dy, const void* wt, void* dx, float* acc_out, int64_t M, int64_t N, int64_t K, hipStream_t st)
{
    const int tiles_m = (int)((M + BM - 1) / BM), tiles_n = (int)((K + BN - 1) / BN);
    const int grid = ((tiles_m * tiles_n + 7) / 8) * 8;
    auto launch = [&](auto lines_tag) {
        linear_bwd_k32_kernel<DT, BM, BN, decltype(lines_tag)::value><<<grid, kGemmThreads, 0, st>>>(
            static_cast<const uint8_t*>(dy), static_cast<const uint8_t*>(wt), static_cast<uint16_t*>(dx), acc_out,
            (int)M, (int)N, (int)K, tiles_m, tiles_n);
    };
    if (bwd_reads_lines(N, BM)) launch(std::true_type{});
    else                        launch(std::false_type{});
}

// The 32x32x16 kernel: 256x256 tiles unless they would leave most of the 256 CUs idle for a round; then 128x128
// (two workgroups per CU).  sasq_set_tuning(SASQ_TUNE_BWD_TILE, 1 | 2) forces one of them.
static double rounds256(int64_t M, int64_t K) { return (double)((((M + 255) / 256) * ((K + 255) / 256) + 255) / 256); }
static double rounds128(int64_t M, int64_t K) { return (double)((((M + 127) / 128) * ((K + 127) / 128) + 511) / 512) * 0.5 * 1.42; }
static bool bwd_small_tiles(int64_t M, int64_t K)
{
    if (tuning(SASQ_TUNE_BWD_TILE) == 1) return false;
    if (tuning(SASQ_TUNE_BWD_TILE) == 2) return true;
    return rounds128(M, K) < rounds256(M, K);
}
// The tile of the 16x16x32 kernel: 0: 256x256, 1: 128x256, 2: 128x128, by the rounds of a 256x256 tile's time that a launch takes (all figures
// here with dY in half lines).  A
// 128x256 tile alone on its CU takes 0.65 of it (several rounds of them 0.68 each), a 128x128 tile 0.44, two of them on a CU 0.8: of 257
// to 512 tiles of 128x128 some CUs hold two, and as 128x256 they all run at once.  But the one wave a SIMD of a 128x256 tile has nothing
// beside it while it fills its pipeline, stores, or waits for weights that the caches have not seen, as those of a training step: it pays from
// about 390 tiles of 128x128 and 32 contraction tiles on.  128x256 | 128x128, on such weights and on ones that the caches hold, part of the
// other's time: 257 to 350 tiles 0.95 to 1.04 and 0.82 to 1.02, 350 to 512 0.87 to 0.97 and 0.81 to 0.94, under 32 contraction tiles 0.97 to
// 1.04 and 1.01.  us, M x N -> K, 256x256 | 128x256 | 128x128, weights not in the caches: 409 x 8576 -> 15808 (496 tiles of 128x128) 189 |
// 129 | 184, 674 x 6016 -> 10560 (498) 138 | 91 | 131, 2176 x 4000 -> 3136 (425) 92 | 78 | 74, 1144 x 1568 -> 4928 (351) 43 | 34 | 30; a
// layer's four in a training step, 128x256 | 128x128, 1023 x 4416 -> 4416 (280) 320 | 280, 1400 rows (385) 1.11 of the time, 1500 rows (420) 1.02, 2000
// x 3904 (496) 0.86, 3500 x 1920 (420) 0.81, 1100 x 5120 (360) 0.95.  In the caches: 900 x 5504 -> 4992 (312) 92 | 63 | 85, 2048 x
// 4096 -> 2304 (288) 48 | 35 | 40, 1000 x 2304 -> 2816 (176) 42.5 | 27.3 | 19.8, 3000 x 2304 -> 3328 (624) 45.4 | 57.9 | 52.1; several rounds: 4096 x
// 2304 -> 5120 95.7 | 92.0 | 94.7, 2920 x 3904 -> 8448 175 | 204 | 216; short: 537 x 128 -> 6720 10.7 | 7.4 | 6.1, 1647 x 96 -> 19008 28.5 | 24.5 | 19.3.
int bwd_tile(int64_t M, int64_t N, int64_t K)
{
    if (const int t = tuning(SASQ_TUNE_BWD_TILE)) return t == 1 ? 0 : 2;
    const double c0 = rounds256(M, K);
    if (N < 32 * kBwdCols) return rounds128(M, K) < c0 ? 2 : 0;
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((K + bn - 1) / bn); };
    const int64_t t128 = tiles(128, 128), rest = t128 % 512, r1 = (tiles(128, 256) + 255) / 256;
    const double c2 = 0.8 * (double)(t128 / 512) + (rest == 0 ? 0.0 : rest <= 256 ? 0.44 : 0.8);
    const double c1 = r1 > 1 ? 0.68 * (double)r1 : t128 >= 390 ? 0.65 : c2;
    return c0 <= c1 && c0 <= c2 ? 0 : c1 < c2 ? 1 : 2;
}
// The time of those tiles, us, for the choice between them and the few-row and row-block kernels: least squares over 3900 calls of 1 to 4000
// rows, contractions of 64 to 14000 and outputs of 128 to 28000, each tile timed in all of them (rms error 7 %, 8 % and 10 %), with dY in half
// lines; an even number of 32 and more contraction tiles now takes 0.87 to 1.01 of that (bwd_reads_lines).  Of 128x128 tiles a CU holds two in
// rounds of more than 256.
static double bwd_tile_us(int64_t M, int64_t N, int64_t K)
{
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((K + bn - 1) / bn); };
    const double kt = (double)(N / kBwdCols);
    const int tile = bwd_tile(M, N, K);
    if (tile == 0) return RoundTime{0.0, 7.8, 0.466, 0.311}.launch(tiles(256, 256), kt);
    if (tile == 1) return RoundTime{0.65, 4.4, 0.284, 0.207}.launch(tiles(128, 256), kt);
    const RoundTime one{2.0, 1.5, 0.163, 0.175}, two{2.0, 2.9, 0.354, 0.088};
    const int64_t t = tiles(128, 128), rest = t % 512;
    return two.call + (double)(t / 512) * two.of(512, kt) + (rest == 0 ? 0.0 : rest <= 256 ? one.of(rest, kt) : two.of(rest, kt));
}

// Rows per workgroup of the kernels without tiles, 0: tiles.
int bwd_rows(int64_t M, int64_t N, int64_t K) { return N % kBwdCols ? 0 : bwd_takes_skinny(M, N, K, bwd_tile_us(M, N, K)); }

static int64_t bwd_kpad(int64_t K) { return (K + 15) / 16 * 16; }
static int64_t bwd_npad(int64_t N) { return (N + kBwdCols - 1) / kBwdCols * kBwdCols; }
constexpr int64_t kBwdMaxProduct = INT64_C(1) << 40;    // elements of any operand or of the output

}  // namespace sasq

using namespace sasq;

extern "C" size_t sasq_bwd_weight_bytes(int64_t N, int64_t K)
{
    if (N <= 0 || K <= 0 || N > 0x3FFFFFFF || K > 0x7FFFFFFF || N > kBwdMaxProduct / K) return 0;
    return (size_t)bwd_kpad(K) * (size_t)bwd_npad(N) * 2;
}

extern "C" int sasq_prepare_bwd_weight(const void* wq, const float* s_w, void* wt, int64_t N, int64_t K,
                                       sasq_wfmt wf, sasq_dtype dt, void* stream)
{
    if (!wq || !s_w || !wt) return SASQ_ERR_NULL;
    if (N <= 0 || K <= 0 || N > 0x3FFFFFFF || K > 0x7FFFFFFF || N > kBwdMaxProduct / K) return SASQ_ERR_SHAPE;
    if (wf != SASQ_W_INT8 && wf != SASQ_W_INT4_PACKED) return SASQ_ERR_UNSUPPORTED;
    if (wf == SASQ_W_INT4_PACKED && (K & 1)) return SASQ_ERR_SHAPE;
    if (dt != SASQ_F16 && dt != SASQ_BF16) return SASQ_ERR_UNSUPPORTED;
    if (!aligned16(wt)) return SASQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);
    const int64_t Kpad = bwd_kpad(K), Npad = bwd_npad(N);
    auto tiles = [&](int64_t wk) { return (Kpad + wk - 1) / wk; };
    const bool narrow = Kpad <= 256 || tiles(512) * (Npad / kBwdCols) < 256;
    const int64_t ktiles = tiles(narrow ? 128 : 512), grid = ktiles * (Npad / kBwdCols);
    if (grid > 0x7FFFFFFF) return SASQ_ERR_SHAPE;
    auto launch = [&](auto dt_tag, auto i4_tag, auto wk_tag) {
        launch_in_parts(grid, 256, [&](unsigned blocks, int first) {
            prepare_bwd_weight_kernel<decltype(dt_tag)::value, decltype(i4_tag)::value, decltype(wk_tag)::value><<<blocks, 256, 0, st>>>(
                static_cast<const uint8_t*>(wq), s_w, static_cast<uint8_t*>(wt), N, K, Npad, Kpad, (uint32_t)ktiles, (uint32_t)first);
        });
    };
    auto by_width = [&](auto dt_tag, auto i4_tag) {
        if (narrow) launch(dt_tag, i4_tag, std::integral_constant<int, 128>{});
        else        launch(dt_tag, i4_tag, std::integral_constant<int, 512>{});
    };
    auto by_format = [&](auto dt_tag) {
        if (wf == SASQ_W_INT4_PACKED) by_width(dt_tag, std::true_type{});
        else                          by_width(dt_tag, std::false_type{});
    };
    if (dt == SASQ_F16) by_format(std::integral_constant<int, SASQ_F16>{});
    else                by_format(std::integral_constant<int, SASQ_BF16>{});
    return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
}

extern "C" int sasq_linear_bwd_input(const void* dy, const void* wt, void* dx, float* acc_out,
                                     int64_t M, int64_t N, int64_t K, sasq_dtype dt, void* stream)
{
    if (!dy || !wt || !dx) return SASQ_ERR_NULL;
    if (M <= 0 || N <= 0 || K <= 0) return SASQ_ERR_SHAPE;
    if (M > 0x7FFFFFFF || N > 0x3FFFFFFF || K > 0x7FFFFFFF) return SASQ_ERR_SHAPE;
    if (M > kBwdMaxProduct / N || M > kBwdMaxProduct / K || N > kBwdMaxProduct / K) return SASQ_ERR_SHAPE;
    if (dt != SASQ_F16 && dt != SASQ_BF16) return SASQ_ERR_UNSUPPORTED;
    if (!aligned16(dy) || !aligned16(wt) || !aligned16(dx)) return SASQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);
    if (N % kBwdCols) {
        // rows of dY are not whole 64-byte stage rows: scalar kernel
        const int64_t grid = (M * K + 255) / 256;
        if (grid > 0x7FFFFFFF) return SASQ_ERR_SHAPE;
        auto* DY = static_cast<const uint16_t*>(dy);
        auto* WT = static_cast<const uint8_t*>(wt);
        auto* DX = static_cast<uint16_t*>(dx);
        if (dt == SASQ_F16) linear_bwd_scalar_kernel<SASQ_F16><<<(int)grid, 256, 0, st>>>(DY, WT, DX, acc_out, M, N, K, bwd_npad(N));
        else                linear_bwd_scalar_kernel<SASQ_BF16><<<(int)grid, 256, 0, st>>>(DY, WT, DX, acc_out, M, N, K, bwd_npad(N));
        return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
    }
    if (tuning(SASQ_TUNE_LINEAR_MFMA) == 0 && tuning(SASQ_TUNE_BWD_TILE) == 0)
        if (const int rows = bwd_rows(M, N, K)) {
            launch_bwd_skinny(dy, wt, dx, acc_out, M, N, K, dt, rows, st);
            return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
        }
    const bool small = bwd_small_tiles(M, K);
    // the 16x16x32 kernel addresses dY rows with 32-bit byte offsets inside a 256-row tile
    if (tuning(SASQ_TUNE_LINEAR_MFMA) != 1 && N <= kBwdOffsetCols) {
        auto by_tile = [&](auto dt_tag) {
            constexpr int DT = decltype(dt_tag)::value;
            switch (bwd_tile(M, N, K)) {
                case 0:  launch_bwd_k32<DT, 256, 256>(dy, wt, dx, acc_out, M, N, K, st); break;
                case 1:  launch_bwd_k32<DT, 128, 256>(dy, wt, dx, acc_out, M, N, K, st); break;
                default: launch_bwd_k32<DT, 128, 128>(dy, wt, dx, acc_out, M, N, K, st); break;
            }
        };
        if (dt == SASQ_F16) by_tile(std::integral_constant<int, SASQ_F16>{});
        else                by_tile(std::integral_constant<int, SASQ_BF16>{});
        return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
    }
    if (dt == SASQ_F16) {
        if (small) launch_bwd<SASQ_F16, 128, 128>(dy, wt, dx, acc_out, M, N, K, st);
        else       launch_bwd<SASQ_F16, 256, 256>(dy, wt, dx, acc_out, M, N, K, st);
    } else {
        if (small) launch_bwd<SASQ_BF16, 128, 128>(dy, wt, dx, acc_out, M, N, K, st);
        else       launch_bwd<SASQ_BF16, 256, 256>(dy, wt, dx, acc_out, M, N, K, st);
    }
    return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
}

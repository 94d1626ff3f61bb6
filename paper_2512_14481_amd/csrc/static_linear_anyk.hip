// int8 linear for contraction lengths that are not whole 64-channel tiles (a projection sharded over GPUs: 11008 / 8 =
// 1376), row-major weights with any row alignment, over row-major activation codes.  (Few rows of int8: static_linear_skinny.hip.)
//
// What bounds it: at 1000 x 4096 x 1376 the 17 MB of operands and output take 3 us and the 11.3 G operations as much; the
// rest is the latency of a short K loop and the operands out of the L2s.  One thread per output walking its row and column byte by byte took
// 10.65 ms there, this kernel with its pre-pass 18.1 us on 64x128 tiles of four waves, 16.5 on 128x128 tiles of eight (0.68 POP/s).
// The pre-arranged formats and the direct memory -> LDS loads of the other GEMMs need rows of whole 16-byte pieces.  Here a
// row starts at any byte, so 16 codes travel through registers: an unaligned 128-bit load (the memory pipeline splits it
// where it has to), requested D stages ahead, then an aligned LDS write.  A stage is 128 channels, so that a row's piece is
// a whole cache line.  The last stage of a row loads its last 16 codes and shifts them into place, zeros behind: nothing
// outside a row is read.  Integer sums, so the order is free.
#include "sasq_device.h"
#include "gemm_tile.h"
#include "gemm_k64.h"
#include <type_traits>

namespace sasq {

constexpr int kAnyStage = 128;                     // channels per LDS stage

// WM x 2 waves, each (BM/WM) x (BN/2) of the tile as 16x16 tiles of v_mfma_i32_16x16x64_i8; two LDS buffers, D stages
// in flight in registers.  LDS rows are 128 bytes, 16-byte chunk c of row r at position c ^ (r & 7).
template <int DT, bool INT4, bool ROWS, int BM, int BN, int D, int WM = 2>
__global__ __launch_bounds__(128 * WM, 2) void linear_anyk_kernel(
    const uint8_t* __restrict__ xq, const uint8_t* __restrict__ wq, const float* __restrict__ s_ptr,
    const float* __restrict__ s_w, const float* __restrict__ bias, uint16_t* __restrict__ y,
    int32_t* __restrict__ acc_out, int M, int N, int K, int tiles_m, int tiles_n, int first)
{
    using S = Store16<DT>;
    using WPiece = std::conditional_t<INT4, u32x2, u32x4>;
    constexpr int kRows = 16 * WM;                                 // rows that a load of every thread takes
    constexpr int MF = BM / (16 * WM), NF = BN / 32, XL = BM / kRows, WL = BN / kRows;
    constexpr int kXBytes = BM * kAnyStage, kBufBytes = (BM + BN) * kAnyStage;
    static_assert(D % 2 == 0, "the unrolled loop knows its LDS buffer at compile time");
    __shared__ __attribute__((aligned(128))) char lds[2 * kBufBytes];

    int tm, tn;
    if (!tile_of_block(first + (int)blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int stages = (K + kAnyStage - 1) / kAnyStage;
    const int wlen = INT4 ? K / 2 : K;                             // bytes of a weight row

    // thread t moves chunk t%8 of rows t/8 + kRows j; rows past the edge repeat the last one
    const int lrow = tid >> 3, lch = tid & 7;
    const uint8_t* xb = xq + (int64_t)m0 * K;
    const uint8_t* wb = wq + (int64_t)n0 * wlen;
    uint32_t xo[XL], wo[WL];                                       // at most 256 rows of 131071 bytes
#pragma unroll
    for (int j = 0; j < XL; ++j) xo[j] = (uint32_t)min(lrow + kRows * j, M - 1 - m0) * (uint32_t)K;
#pragma unroll
    for (int j = 0; j < WL; ++j) wo[j] = (uint32_t)min(lrow + kRows * j, N - 1 - n0) * (uint32_t)wlen;
    struct Regs { u32x4 x[XL]; WPiece w[WL]; };
    Regs ring[D];
    constexpr int kWPiece = (int)sizeof(WPiece);
    auto fetch = [&](Regs& r, int st) {
        if ((st + 1) * kAnyStage <= K) {
#pragma unroll
            for (int j = 0; j < XL; ++j) r.x[j] = load_piece<u32x4>(xb + st * kAnyStage + (xo[j] + lch * 16));
#pragma unroll
            for (int j = 0; j < WL; ++j) r.w[j] = load_piece<WPiece>(wb + st * 8 * kWPiece + (wo[j] + lch * kWPiece));
        } else {
#pragma unroll
            for (int j = 0; j < XL; ++j) r.x[j] = load_piece_edge<u32x4>(xb + xo[j], st * kAnyStage + lch * 16, K);
#pragma unroll
            for (int j = 0; j < WL; ++j) r.w[j] = load_piece_edge<WPiece>(wb + wo[j], (st * 8 + lch) * kWPiece, wlen);
        }
    };
    const int slot = lrow * kAnyStage + ((lch ^ (lrow & 7)) << 4);
    auto put = [&](const Regs& r, int buf) {
        char* base = &lds[buf * kBufBytes];
#pragma unroll
        for (int j = 0; j < XL; ++j) *reinterpret_cast<u32x4*>(base + slot + j * kRows * kAnyStage) = r.x[j];
#pragma unroll
        for (int j = 0; j < WL; ++j) {
            u32x4 v;
            if constexpr (INT4) v = widen_int4(r.w[j]);
            else                v = r.w[j];
            *reinterpret_cast<u32x4*>(base + kXBytes + slot + j * kRows * kAnyStage) = v;
        }
    };
    // this wave's LDS traffic is done, then everyone's
    auto sync = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    const int frow = lane & 15, fq = lane >> 4;
    const int xbase = wave % WM * (BM / WM) * kAnyStage, wbase = kXBytes + wave / WM * (BN / 2) * kAnyStage;
    i32x4 acc[NF][MF];
#pragma unroll
    for (int g = 0; g < NF; ++g)
#pragma unroll
        for (int b = 0; b < MF; ++b) acc[g][b] = i32x4{0, 0, 0, 0};
    auto multiply = [&](int buf) {
        const char* base = &lds[buf * kBufBytes];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int off = frow * kAnyStage + (((4 * h + fq) ^ (frow & 7)) << 4);
            i32x4 fx[MF], fw[NF];
#pragma unroll
            for (int b = 0; b < MF; ++b) fx[b] = *reinterpret_cast<const i32x4*>(base + xbase + b * 16 * kAnyStage + off);
#pragma unroll
            for (int g = 0; g < NF; ++g) fw[g] = *reinterpret_cast<const i32x4*>(base + wbase + g * 16 * kAnyStage + off);
#pragma unroll
            for (int g = 0; g < NF; ++g)
#pragma unroll
                for (int b = 0; b < MF; ++b) acc[g][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fw[g], fx[b], acc[g][b], 0, 0, 0);
        }
    };

    const int wn0 = n0 + wave / WM * (BN / 2), wm0 = m0 + wave % WM * (BM / WM);
    float srow[MF], sw[NF][4], bv[NF][4];
    auto load_factors = [&]() {
#pragma unroll
        for (int b = 0; b < MF; ++b) srow[b] = s_ptr[ROWS ? min(wm0 + b * 16 + frow, M - 1) : 0];
#pragma unroll
        for (int g = 0; g < NF; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int ne = min(wn0 + g * 16 + 4 * fq + e, N - 1);
                sw[g][e] = s_w[ne];
                bv[g][e] = bias ? bias[ne] : 0.0f;
            }
    };
    // The small tiles, whose calls are short, request the factors ahead of the operands instead of waiting for them at the end;
    // the large ones need the registers.
    constexpr bool kAhead = BN == 64;
    if (kAhead) load_factors();

#pragma unroll
    for (int j = 0; j < D; ++j)
        if (j < stages) fetch(ring[j], j);
    put(ring[0], 0);
    if (D < stages) fetch(ring[0], D);
    sync();
    // Stage i is in LDS buffer i & 1.  Its products are issued, stage i + 1 goes into the other buffer (whose readers passed
    // the last barrier), and its registers take stage i + 1 + D.
    for (int i = 0; i < stages; i += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            if (i + j < stages) {
                multiply(j & 1);
                if (i + j + 1 < stages) {
                    put(ring[(j + 1) % D], (j + 1) & 1);
                    if (i + j + 1 + D < stages) fetch(ring[(j + 1) % D], i + j + 1 + D);
                    sync();
                }
            }
        }
    }

    // D[i][j]: i <-> n, j <-> m; a lane holds four consecutive columns of one row per 16x16 tile
    if (!kAhead) load_factors();
    const bool vec = (N & 3) == 0;
#pragma unroll
    for (int g = 0; g < NF; ++g) {
        const int n = wn0 + g * 16 + 4 * fq;
#pragma unroll
        for (int b = 0; b < MF; ++b) {
            const int m = wm0 + b * 16 + frow;
            if (m >= M || n >= N) continue;
            float yv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                yv[e] = (float)acc[g][b][e] * (srow[b] * sw[g][e]);
                if (bias) yv[e] = yv[e] + bv[g][e];
            }
            const int64_t o = (int64_t)m * N + n;
            if (vec) {
                *reinterpret_cast<u32x2*>(y + o) = u32x2{S::pack(yv[0], yv[1]), S::pack(yv[2], yv[3])};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) y[o + e] = S::enc(yv[e]);
            }
            if (acc_out) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) acc_out[o + e] = acc[g][b][e];
            }
        }
    }
}

// Rows of a few codes, few outputs: one thread per output.  There is next to no work, and the kernel above is as long as its
// instructions take to arrive.  Measured, us with the pre-pass, this | the tiles: int8, 1 x 20000 outputs, K = 1, 8, 20, 32 3.8 |
// 5.4, 4.1 | 5.1, 4.9 | 5.4, 7.3 | 5.5; 64 x 1000, K = 20, 24 5.1 | 5.2, 5.3 | 5.1; 512 x 512, K = 4, 8, 12 4.5 | 5.2, 5.2 | 5.1, 5.7 |
// 5.3; 2000 x 2000, K = 1 10.1 | 8.5; int4, whose rows are half as long: 64 x 1000, K = 32, 48 5.1 | 5.3, 5.8 | 5.5; 512 x 512,
// K = 12, 20 5.1 | 5.6, 5.7 | 5.7.
constexpr int64_t kShortRow = 20, kShortRows = 3 << 19;        // bytes of a weight row; the same times the outputs

template <int DT, bool INT4, bool ROWS>
__global__ __launch_bounds__(256) void linear_short_row_kernel(
    const int8_t* __restrict__ xq, const uint8_t* __restrict__ wq, const float* __restrict__ s_ptr,
    const float* __restrict__ s_w, const float* __restrict__ bias, uint16_t* __restrict__ y,
    int32_t* __restrict__ acc_out, int outputs, int N, int K)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i >= outputs) return;
    const int m = i / N, n = i - m * N;
    const int8_t* xr = xq + m * K;
    int acc = 0;
    if (INT4) {
        const uint8_t* wr = wq + (int64_t)n * (K / 2);
        for (int j = 0; j < K / 2; ++j) {
            const int b = wr[j];
            acc += (int)xr[2 * j] * (((b & 15) ^ 8) - 8) + (int)xr[2 * j + 1] * (((b >> 4) ^ 8) - 8);
        }
    } else {
        const int8_t* wr = reinterpret_cast<const int8_t*>(wq) + (int64_t)n * K;
        for (int k = 0; k < K; ++k) acc += (int)xr[k] * (int)wr[k];
    }
    float yv = (float)acc * (s_ptr[ROWS ? m : 0] * s_w[n]);
    if (bias) yv = yv + bias[n];
    y[i] = Store16<DT>::enc(yv);
    if (acc_out) acc_out[i] = acc;
}

template <int DT, bool INT4, bool ROWS, int BM, int BN, int D, int WM = 2>
static void launch_anyk_one(const GemmK64Args& a, hipStream_t st)
{
    const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (int)((a.N + BN - 1) / BN);
    launch_in_parts((tiles_m * tiles_n + 7) / 8 * 8, 128 * WM, [&](unsigned blocks, int first) {
        linear_anyk_kernel<DT, INT4, ROWS, BM, BN, D, WM><<<blocks, 128 * WM, 0, st>>>(
            reinterpret_cast<const uint8_t*>(a.xq), a.wq, a.s, a.s_w, a.bias, a.y, a.acc_out, (int)a.M, (int)a.N, (int)a.K, tiles_m, tiles_n, first);
    });
}

// Big tiles read the operands less often, small ones put more CUs to work.  Eight waves a workgroup from 64x128 tiles on: the loads in
// flight that it takes to keep the L2s busy then fit a tile of twice the outputs, which asks for two thirds
// (64x128 -> 128x128) or three quarters (128x128 -> 256x128) of the operands (rows that begin inside cache lines cost two lines for most of their
// pieces).  Measured, us with the pre-pass, the earlier choice of 128x128, 64x128
// (from 256 tiles) and smaller tiles of four waves | 64x128 | 128x128 | 256x128 of eight, by number of 128x128 tiles:
//   96: 333 x 4000, K = 1376 int8 12.4 | 12.3 | 15.2 | 21.6, K = 1801 19.1 | 16.6 | 20.8 | 30.5, int4 15.2 | 14.7 | 17.6 | 23.2
//   128: 1000 x 2048, K = 1376 15.2 | 13.8 | 16.6 | 23.2, K = 3976 30.0 | 28.4 | 32.9 | 47.5, int4 39.6 | 34.3 | 38.7 | 52.2
//   160: 1000 x 2560, K = 1376 18.8 | 18.4 | 17.2 | 23.9, K = 1801 28.2 | 28.0 | 23.1 | 33.5, int4 23.6 | 22.0 | 19.2 | 25.5
//   256: 1000 x 4096, K = 1376 20.5 | 19.6 | 18.7 | 24.6, K = 3976 42.1 | 42.8 | 35.7 | 49.2, int4 55.8 | 56.1 | 42.1 | 55.1
//   320: 1000 x 5000, K = 1376 25.9 | 24.8 | 24.3 | 24.6, K = 3976 57.1 | 54.9 | 51.0 | 49.0, int4 69.0 | 72.5 | 59.8 | 55.2
//   448: 1000 x 7168, K = 1376 33.2 | 32.1 | 27.4 | 27.3, K = 3976 79.2 | 82.8 | 57.2 | 55.2, int4 93.1 | 94.4 | 68.1 | 59.8
//   768 (384 of 256x128, a round and a half): 2000 x 6144, K = 1376 44.3 | 46.9 | 40.0 | 49.3, K = 3976 97.2 | 120 | 95.3 | 101
//   1024 (512, two rounds): 4096 x 4096, K = 1376 56.3 | 64.7 | 53.5 | 53.3, K = 3976 126 | 160 | 124 | 115, int4 148 | 188 | 133 | 128
// Beyond, four waves: 8192 x 16384 (8192), K = 1040 293 | - | - | 393, int4 327 | - | - | 374 (128x128 of eight, not taken there: 0.95 to 0.98 over
// 880 calls of 1025 to 8192 tiles); and where the larger tile has many rows past the end: 300 x 16385, K = 200 17.7 | - | 19.1 | -, K = 1040 25.8 | - | 27.2 | -.
// Fewer tiles, four waves, 128x128 / 64x128 / 64x64 / 32x64: 512 x 1024 x 3000 (64 of 64x128, 256 of 32x64) 28.2 / 21.5 / 16.3 / 14.9, 64 x
// 4096 x 3976 (128 of 32x64) 31.3 / 24.8 / 19.4 / 16.7.
// 257 to 511 tiles of 128x128 that are at most 768 of 64x128: the latter, of four waves, run three a CU, all at once, in parts of the larger
// tiles' time, by K up to 255, 511, 1023, 2047 and beyond, 0.90 to 0.96, 0.90 to 0.95, 0.93 to 1.01, 0.97 to 1.10, 1.03 to 1.14; up to 512 of them,
// two a CU, 0.78 to 0.83 at any K.  Two rounds of 256x128 tiles, K under 1024: 128x128 0.94 to 0.99 of their time.  192 to 255 tiles of 64x128, K
// under 256: 64x64 0.95 to 0.99 of the time of eight waves.
// 0: 256x128, eight waves; 1: 128x128, eight; 2: 128x128, four; 3: 64x128, eight; 4: 64x128, four; 5: 64x64; 6: 32x64.
int linear_anyk_tile(int64_t M, int64_t N, int64_t K)
{
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    const int64_t t256 = tiles(256, 128), t128 = tiles(128, 128), t64 = tiles(64, 128);
    const bool mid = t128 <= 1024 && t128 * 20 <= t64 * 11;          // and at most a tenth of the rows past the matrix's end
    // rounds of 256x128 tiles, one a CU, that are nearly full
    const bool rounds_fill = (t256 <= 256 || t256 * 10 >= (t256 + 255) / 256 * 2304) && t256 * 20 <= t128 * 11;
    if (t128 > 256 && t128 < 512 && t64 <= (K < 1024 ? 768 : 512)) return 4;
    if (mid && t128 > 256 && rounds_fill && (t128 <= 512 || K >= 1024)) return 0;
    if (mid && t64 > 256)          return 1;
    if (t128 >= 512)               return 2;
    if (t64 > 256)                 return 4;
    if (t64 == 256 || (t64 >= 192 && K >= 256)) return 3;
    return tiles(64, 64) >= 256 ? 5 : 6;
}

template <int DT, bool INT4, bool ROWS>
static void launch_anyk_w(const GemmK64Args& a, hipStream_t st)
{
    const int64_t wlen = INT4 ? a.K / 2 : a.K;
    if (wlen <= kShortRow && a.M * a.N * wlen <= kShortRows) {
        linear_short_row_kernel<DT, INT4, ROWS><<<(unsigned)((a.M * a.N + 255) / 256), 256, 0, st>>>(
            a.xq, a.wq, a.s, a.s_w, a.bias, a.y, a.acc_out, (int)(a.M * a.N), (int)a.N, (int)a.K);
        return;
    }
    switch (linear_anyk_tile(a.M, a.N, a.K)) {
        case 0: launch_anyk_one<DT, INT4, ROWS, 256, 128, 2, 4>(a, st); break;
        case 1: launch_anyk_one<DT, INT4, ROWS, 128, 128, 2, 4>(a, st); break;
        case 2: launch_anyk_one<DT, INT4, ROWS, 128, 128, 2>(a, st); break;
        case 3: launch_anyk_one<DT, INT4, ROWS, 64, 128, 2, 4>(a, st); break;
        case 4: launch_anyk_one<DT, INT4, ROWS, 64, 128, 2>(a, st); break;
        case 5: launch_anyk_one<DT, INT4, ROWS, 64, 64, 4>(a, st); break;
        default: launch_anyk_one<DT, INT4, ROWS, 32, 64, 4>(a, st); break;
    }
}

void launch_linear_anyk(const GemmK64Args& a, sasq_dtype dt, bool int4, bool rows, hipStream_t st)
{
    auto by_dt = [&](auto dt_tag) {
        constexpr int DT = decltype(dt_tag)::value;
        if (int4) { if (rows) launch_anyk_w<DT, true, true>(a, st);  else launch_anyk_w<DT, true, false>(a, st); }
        else      { if (rows) launch_anyk_w<DT, false, true>(a, st); else launch_anyk_w<DT, false, false>(a, st); }
    };
    if (dt == SASQ_F16) by_dt(std::integral_constant<int, SASQ_F16>{});
    else                by_dt(std::integral_constant<int, SASQ_BF16>{});
}

}  // namespace sasq

// Grouped-factor linear (Sec. 3, Eq. 3) for the group sizes the matrix units cannot take: groups of one channel (the
// strict per-channel factors that Sec. 4 trains), and every other group that is not whole 32- or 64-channel pieces.
//
//     acc_i = sum over the k of group i of xq[m,k] * Wq[n,k]   (exact)      f = fma(fl32(acc_i), s_g[i], f)
//
// The chain of fused multiply-adds is part of the contract, so the work is fp32 VALU work: with one channel per group
// two operations per multiply-add, the exact product of two codes and the fused multiply-add with the factor.  What the
// kernels have to do is keep the VALU issuing: codes are widened once, on their way into LDS (each then serves 64 or 128
// outputs) or out of it; a thread owns a block of outputs, so that a step of k reads TM + TN values for 2 TM TN
// operations; the factors come from LDS with the codes (read as scalars they cost a memory latency every few k, because
// scalar loads share their counter with LDS); products are formed before the adds that depend on them; the next slab is
// fetched into registers while the current one is multiplied.
// Measured, group 1: 512 x 4096 x 4096 414 us (42 T operations/s of the 79 that the VALUs issue at full rate; one thread
// per output reading global memory took 32.2 ms), 2048 x 4096 x 11008 3.31 ms (56 T), 64 x 4096 x 4096 122 us.
#include "sasq_device.h"
#include "gemm_k64.h"
#include <type_traits>

namespace sasq {

constexpr int kSlab = 32;                          // k per LDS slab
constexpr int64_t kOneMinTiles = 768;              // group 1: tiles a launch needs for a tile shape to be chosen (three per CU)

// How a group is summed.  ONE: one channel, codes in LDS as floats.  DOT4: a multiple of four channels, codes stay
// packed and v_dot4 sums four products exactly.  ANY: codes as 32-bit integers, one multiply-add each.
enum { GV_ONE = 0, GV_DOT4 = 1, GV_ANY = 2 };

// 16 consecutive codes of a row from k0 on, as bytes; zeros past K or outside the matrix
template <bool INT4>
__device__ __forceinline__ u32x4 load_codes16(const uint8_t* __restrict__ base, int64_t row, bool row_ok, int k0, int K, bool vec)
{
    u32x4 v = {0u, 0u, 0u, 0u};
    if (!row_ok || k0 >= K) return v;
    if constexpr (INT4) {
        const uint8_t* p = base + row * (K / 2) + k0 / 2;
        uint32_t q[2] = {0u, 0u};
        if (vec) {
            const u32x2 t = *reinterpret_cast<const u32x2*>(p);
            q[0] = t[0]; q[1] = t[1];
        } else {
            for (int b = 0; b < 8; ++b)
                if (k0 + 2 * b < K) q[b >> 2] |= (uint32_t)p[b] << (8 * (b & 3));
        }
        // nibble j -> byte j, sign-extended: move it to the top of its byte, then (n ^ 8) - 8 per byte
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const uint32_t h = q[d >> 1] >> (16 * (d & 1));
            const uint32_t n4 = (h & 0xFu) | ((h & 0xF0u) << 4) | ((h & 0xF00u) << 8) | ((h & 0xF000u) << 12);
            v[d] = (n4 | ((n4 & 0x08080808u) * 0x1Eu));      // 8 * 0x1E = 0xF0: the sign bit repeated in the upper nibble
        }
    } else {
        const uint8_t* p = base + row * K + k0;
        if (vec) {
            v = *reinterpret_cast<const u32x4*>(p);
        } else {
            for (int b = 0; b < 16; ++b)
                if (k0 + b < K) v[b >> 2] |= (uint32_t)p[b] << (8 * (b & 3));
        }
    }
    return v;
}

__device__ __forceinline__ int sext_byte(uint32_t w, int e) { return (int)(w << (24 - 8 * e)) >> 24; }

template <int DT, bool INT4, int MODE, int BM, int BN>
__global__ __launch_bounds__(256) void linear_grouped_valu_kernel(
    const int8_t* __restrict__ xq, const uint8_t* __restrict__ wq, const float* __restrict__ s_g,
    const float* __restrict__ s_w, const float* __restrict__ bias, uint16_t* __restrict__ y,
    float* __restrict__ f_out, int M, int N, int K, int group, int tiles_m)
{
    using S = Store16<DT>;
    using Elem = std::conditional_t<MODE == GV_ONE, float, int>;
    constexpr int TM = BM / 16, TN = BN / 16, TNV = TN / 4;
    constexpr int kSteps = MODE == GV_DOT4 ? kSlab / 4 : kSlab;          // LDS rows per slab
    __shared__ __attribute__((aligned(16))) Elem lx[2][kSteps][BM];
    __shared__ __attribute__((aligned(16))) Elem lw[2][kSteps][BN];
    __shared__ __attribute__((aligned(16))) float ls[2][kSlab];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int tm = (int)blockIdx.x % tiles_m, tn = (int)blockIdx.x / tiles_m;
    const int m0 = tm * BM, n0 = tn * BN;
    const bool vec = (K & 15) == 0;

    // staging: item (row, half) = 16 codes.  W: BN x 2 items from thread 0 on; X: BM x 2 items on the last threads.
    constexpr int kWItems = 2 * BN, kXItems = 2 * BM;
    static_assert(kWItems <= 256 && kXItems <= 256, "one item per thread and operand");
    const bool has_w = tid < kWItems, has_x = tid >= 256 - kXItems;
    const int wrow = tid % BN, whalf = tid / BN;
    const int xi = tid - (256 - kXItems), xrow = has_x ? xi % BM : 0, xhalf = has_x ? xi / BM : 0;
    u32x4 rw, rx;
    float rs = 0.0f;
    auto fetch = [&](int k0) {
        if (MODE == GV_ONE) rs = s_g[min(k0 + (tid & (kSlab - 1)), K - 1)];
        if (has_w) rw = load_codes16<INT4>(wq, n0 + wrow, n0 + wrow < N, k0 + 16 * whalf, K, vec);
        if (has_x) rx = load_codes16<false>(reinterpret_cast<const uint8_t*>(xq), m0 + xrow, m0 + xrow < M, k0 + 16 * xhalf, K, vec);
    };
    auto put = [&](int buf) {
        if (MODE == GV_ONE && tid < kSlab) ls[buf][tid] = rs;
        if constexpr (MODE == GV_DOT4) {
            if (has_w) {
#pragma unroll
                for (int d = 0; d < 4; ++d) lw[buf][4 * whalf + d][wrow] = (int)rw[d];
            }
            if (has_x) {
#pragma unroll
                for (int d = 0; d < 4; ++d) lx[buf][4 * xhalf + d][xrow] = (int)rx[d];
            }
        } else {
            if (has_w) {
#pragma unroll
                for (int e = 0; e < 16; ++e) lw[buf][16 * whalf + e][wrow] = (Elem)sext_byte(rw[e >> 2], e & 3);
            }
            if (has_x) {
#pragma unroll
                for (int e = 0; e < 16; ++e) lx[buf][16 * xhalf + e][xrow] = (Elem)sext_byte(rx[e >> 2], e & 3);
            }
        }
    };

    float f[TM][TN];
    int acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) { f[i][j] = 0.0f; acc[i][j] = 0; }
    int in_group = 0, gi = 0;
    auto fold = [&]() {
        const float sg = s_g[gi];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) { f[i][j] = __builtin_fmaf((float)acc[i][j], sg, f[i][j]); acc[i][j] = 0; }
        ++gi;
        in_group = 0;
    };

    fetch(0);
    put(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < K; k0 += kSlab, buf ^= 1) {
        const bool more = k0 + kSlab < K;
        if (more) fetch(k0 + kSlab);
        auto step = [&](int st, float sk) {
            Elem a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = lx[buf][st][ty * TM + i];
#pragma unroll
            for (int v = 0; v < TNV; ++v)
#pragma unroll
                for (int j = 0; j < 4; ++j) b[4 * v + j] = lw[buf][st][64 * v + tx * 4 + j];
            if constexpr (MODE == GV_ONE) {
                float p[TM][TN];
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) p[i][j] = a[i] * b[j];
                __builtin_amdgcn_sched_barrier(0x0100);                    // only LDS reads may move across
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) f[i][j] = __builtin_fmaf(p[i][j], sk, f[i][j]);
                __builtin_amdgcn_sched_barrier(0x0100);
            } else
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if constexpr (MODE == GV_DOT4) {
                        acc[i][j] = __builtin_amdgcn_sdot4(a[i], b[j], acc[i][j], false);
                    } else {
                        acc[i][j] += __mul24(a[i], b[j]);
                    }
                }
        };
        if constexpr (MODE == GV_ONE) {
            if (more || K - k0 == kSlab) {
#pragma unroll 2
                for (int s4 = 0; s4 < kSteps / 4; ++s4) {
                    const f32x4 sv = *reinterpret_cast<const f32x4*>(&ls[buf][4 * s4]);
#pragma unroll
                    for (int q = 0; q < 4; ++q) step(4 * s4 + q, sv[q]);
                }
            } else {
                for (int st = 0; st < K - k0; ++st) step(st, ls[buf][st]);
            }
        } else {
            constexpr int kPer = MODE == GV_DOT4 ? 4 : 1;
            const int steps = more ? kSteps : (K - k0) / kPer;
#pragma unroll 4
            for (int st = 0; st < steps; ++st) {
                step(st, 0.0f);
                in_group += kPer;
                if (in_group == group) fold();
            }
        }
        if (more) {
            put(buf ^ 1);              // the other buffer: its readers passed the barrier of the previous slab
            __syncthreads();
        }
    }

    const bool vec_out = (N & 3) == 0;
#pragma unroll
    for (int v = 0; v < TNV; ++v) {
        const int n = n0 + 64 * v + tx * 4;
        float sw[4], bv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sw[j] = n + j < N ? s_w[n + j] : 0.0f;
            bv[j] = bias && n + j < N ? bias[n + j] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = m0 + ty * TM + i;
            if (m >= M || n >= N) continue;
            uint16_t h[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float yv = f[i][4 * v + j] * sw[j];
                if (bias) yv = yv + bv[j];
                h[j] = S::enc(yv);
            }
            const int64_t o = (int64_t)m * N + n;
            if (vec_out) {
                *reinterpret_cast<u32x2*>(y + o) = u32x2{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16)};
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (n + j < N) y[o + j] = h[j];
            }
            if (f_out) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (n + j < N) f_out[o + j] = f[i][4 * v + j];
            }
        }
    }
}

// Groups of one channel.  A wave owns TM rows x 64 columns of the output: lane = column, and the codes of the TM rows sit
// in the lanes of one register, from where the multiply takes row i with a lane broadcast inside its own operand fetch
// (DPP row_newbcast) -- no LDS read per row and k, which is what bounded the tiled form above (3 x 128-bit reads for 64
// operations) when there are too few rows for many waves.  LDS holds the codes as bytes, 64 k per slab, rows padded to 80 bytes so that 128-bit reads of consecutive
// rows use all banks; a lane reads 16 codes at once and widens them as it goes (2 operations per 2 TM of useful work).
constexpr int kOneSlab = 64;
constexpr int kOneStride = kOneSlab + 16;

template <int LANE>
__device__ __forceinline__ float row_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + LANE, 0xF, 0xF, true));
}

// One k: all TM products first, then the TM fused multiply-adds (left to itself the compiler pairs each product with its
// add through one register: a dependent pair and a wait state per output).
template <int TM, int I = 0>
__device__ __forceinline__ void products(float (&p)[TM], float a, float b)
{
    if constexpr (I < TM) {
        p[I] = row_bcast<I>(a) * b;                                      // exact: |p| <= 2^14
        products<TM, I + 1>(p, a, b);
    }
}

template <int TM>
__device__ __forceinline__ void one_step(float (&f)[TM], float a, float b, float s)
{
    float p[TM];
    products<TM>(p, a, b);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < TM; ++i) f[i] = __builtin_fmaf(p[i], s, f[i]);
    __builtin_amdgcn_sched_barrier(0);
}

template <int DT, bool INT4, int TM>
__global__ __launch_bounds__(256) void linear_per_channel_kernel(
    const int8_t* __restrict__ xq, const uint8_t* __restrict__ wq, const float* __restrict__ s_g,
    const float* __restrict__ s_w, const float* __restrict__ bias, uint16_t* __restrict__ y,
    float* __restrict__ f_out, int M, int N, int K, int tiles_m)
{
    using S = Store16<DT>;
    constexpr int BM = 4 * TM, BN = 64;
    __shared__ __attribute__((aligned(16))) uint8_t lx[2][BM * kOneStride];
    __shared__ __attribute__((aligned(16))) uint8_t lw[2][BN * kOneStride];
    __shared__ __attribute__((aligned(16))) float ls[2][kOneSlab];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = ((int)blockIdx.x % tiles_m) * BM, n0 = ((int)blockIdx.x / tiles_m) * BN;
    const bool vec = (K & 15) == 0;
    const int srow = tid >> 2, sch = tid & 3;           // staging: 16 codes of row srow per thread and operand
    const bool has_x = srow < BM;
    u32x4 rw, rx;
    float rs;
    auto fetch = [&](int k0) {
        rs = s_g[min(k0 + (tid & (kOneSlab - 1)), K - 1)];
        rw = load_codes16<INT4>(wq, n0 + srow, n0 + srow < N, k0 + 16 * sch, K, vec);
        if (has_x) rx = load_codes16<false>(reinterpret_cast<const uint8_t*>(xq), m0 + srow, m0 + srow < M, k0 + 16 * sch, K, vec);
    };
    auto put = [&](int buf) {
        *reinterpret_cast<u32x4*>(&lw[buf][srow * kOneStride + 16 * sch]) = rw;
        if (tid < kOneSlab) ls[buf][tid] = rs;
        if (has_x) *reinterpret_cast<u32x4*>(&lx[buf][srow * kOneStride + 16 * sch]) = rx;
    };
    float f[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) f[i] = 0.0f;
    fetch(0);
    put(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < K; k0 += kOneSlab, buf ^= 1) {
        const bool more = k0 + kOneSlab < K;
        if (more) fetch(k0 + kOneSlab);
        const uint8_t* pa = &lx[buf][(wave * TM + (lane & (TM - 1))) * kOneStride];
        const uint8_t* pb = &lw[buf][lane * kOneStride];
        if (K - k0 >= kOneSlab) {
#pragma unroll 2
            for (int c = 0; c < 4; ++c) {
                const u32x4 av = *reinterpret_cast<const u32x4*>(pa + 16 * c), bv = *reinterpret_cast<const u32x4*>(pb + 16 * c);
                f32x4 sv[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) sv[q] = *reinterpret_cast<const f32x4*>(&ls[buf][16 * c + 4 * q]);
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    one_step<TM>(f, (float)sext_byte(av[e >> 2], e & 3), (float)sext_byte(bv[e >> 2], e & 3), sv[e >> 2][e & 3]);
            }
        } else {
            for (int k = 0; k < K - k0; ++k) one_step<TM>(f, (float)(int8_t)pa[k], (float)(int8_t)pb[k], ls[buf][k]);
        }
        if (more) {
            put(buf ^ 1);              // the other buffer: its readers passed the barrier of the previous slab
            __syncthreads();
        }
    }
    const int n = n0 + lane;
    if (n >= N) return;
    const float sw = s_w[n], bv = bias ? bias[n] : 0.0f;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wave * TM + i;
        if (m >= M) continue;
        float yv = f[i] * sw;
        if (bias) yv = yv + bv;
        const int64_t o = (int64_t)m * N + n;
        y[o] = S::enc(yv);
        if (f_out) f_out[o] = f[i];
    }
}

template <int DT, bool INT4, int TM>
static void launch_per_channel(const GemmK64Args& a, hipStream_t st)
{
    const int64_t tm = (a.M + 4 * TM - 1) / (4 * TM), tn = (a.N + 63) / 64;
    linear_per_channel_kernel<DT, INT4, TM><<<(unsigned)(tm * tn), 256, 0, st>>>(
        a.xq, a.wq, a.s, a.s_w, a.bias, a.y, reinterpret_cast<float*>(a.acc_out), (int)a.M, (int)a.N, (int)a.K, (int)tm);
}

template <int DT, bool INT4, int MODE, int BM, int BN>
static void launch_gv(const GemmK64Args& a, int64_t group, hipStream_t st)
{
    const int64_t tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN;
    linear_grouped_valu_kernel<DT, INT4, MODE, BM, BN><<<(unsigned)(tm * tn), 256, 0, st>>>(
        a.xq, a.wq, a.s, a.s_w, a.bias, a.y, reinterpret_cast<float*>(a.acc_out), (int)a.M, (int)a.N, (int)a.K, (int)group, (int)tm);
}

template <int DT, bool INT4, int MODE>
static void launch_gv_mode(const GemmK64Args& a, int64_t group, hipStream_t st)
{
    auto tiles = [&](int bm, int bn) { return ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); };
    // The larger the thread's block, the fewer LDS reads per operation; the more workgroups, the more waves to issue from
    // (one wave per SIMD issues a VALU operation every 6 cycles, three every 2.8).  Group 1: 2048 x 4096 x 11008 takes
    // 3307 / 3391 / 3557 us on 64x128 / 64x64 / 32x64 tiles, 512 x 4096 x 4096 (256 / 512 / 1024 tiles) 630 / 429 / 414.
    if constexpr (MODE == GV_ONE) {
        if (tiles(64, 128) >= kOneMinTiles)     launch_gv<DT, INT4, MODE, 64, 128>(a, group, st);
        else if (tiles(64, 64) >= kOneMinTiles) launch_gv<DT, INT4, MODE, 64, 64>(a, group, st);
        else                                    launch_gv<DT, INT4, MODE, 32, 64>(a, group, st);
    } else {
        if (tiles(64, 128) >= 512)     launch_gv<DT, INT4, MODE, 64, 128>(a, group, st);
        else if (tiles(64, 64) >= 256) launch_gv<DT, INT4, MODE, 64, 64>(a, group, st);
        else if (tiles(32, 64) >= 256) launch_gv<DT, INT4, MODE, 32, 64>(a, group, st);
        else                           launch_gv<DT, INT4, MODE, 16, 64>(a, group, st);
    }
}

template <int DT, bool INT4>
static void launch_gv_w(const GemmK64Args& a, int64_t group, hipStream_t st)
{
    // One channel per group: above two 32x64 tiles per CU the LDS-tiled kernel, below that the lane-broadcast one (its
    // multiply with a broadcast operand runs at half rate, but it needs few waves to get there).  At K = N = 4096, tiled
    // against broadcast: M = 512 414 us and 528, M = 300 340 and 407, M = 250 302 and 288, M = 128 333 and 175, M = 64 331
    // and 122.  The latter with eight rows per wave while that gives 1.5 workgroups per CU (M = 250: 288 us, four rows
    // 308), else with four (M = 128: 175, eight 183).
    auto tiles = [&](int bm) { return ((a.M + bm - 1) / bm) * ((a.N + 63) / 64); };
    if (group == 1 && tiles(32) > 512)           launch_gv_mode<DT, INT4, GV_ONE>(a, group, st);
    else if (group == 1 && tiles(32) >= 384)     launch_per_channel<DT, INT4, 8>(a, st);
    else if (group == 1)                         launch_per_channel<DT, INT4, 4>(a, st);
    else if (group % 4 == 0) launch_gv_mode<DT, INT4, GV_DOT4>(a, group, st);
    else                     launch_gv_mode<DT, INT4, GV_ANY>(a, group, st);
}

void launch_grouped_valu(const GemmK64Args& a, sasq_dtype dt, bool int4, int64_t group, hipStream_t st)
{
    if (dt == SASQ_F16) { if (int4) launch_gv_w<SASQ_F16, true>(a, group, st);  else launch_gv_w<SASQ_F16, false>(a, group, st); }
    else                { if (int4) launch_gv_w<SASQ_BF16, true>(a, group, st); else launch_gv_w<SASQ_BF16, false>(a, group, st); }
}

}  // namespace sasq

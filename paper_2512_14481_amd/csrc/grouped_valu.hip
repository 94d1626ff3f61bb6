// Grouped-factor linear (Sec. 3, Eq. 3) for the group sizes the int8 GEMM cannot take: groups of one channel (the strict
// per-channel factors that Sec. 4 trains), and every other group that is not whole 32- or 64-channel pieces.
//
//     acc_i = sum over the k of group i of xq[m,k] * Wq[n,k]   (exact)      f = fma(fl32(acc_i), s_g[i], f)
//
// The chain of fused multiply-adds is part of the contract, so at least one fp32 VALU operation per output and group is due;
// the kernels differ in who makes the group sums.  Groups of 1, 2, 4, 8, 16: the matrix units (linear_small_group_kernel;
// single channels with few rows: the VALUs, with a lane broadcast, linear_per_channel_kernel).  Other sizes: the VALUs, from
// codes in LDS, a thread owning a block of outputs, so that a step of k reads TM + TN values for TM TN operations; the next
// slab is fetched into registers while the current one is multiplied.
// Measured, us, group 1: 512 x 4096 x 4096 282 (sums made by VALU multiplies, two operations per multiply-add: 414; one thread
// per output reading global memory: 32.2 ms), 2048 x 4096 x 11008 2590 (3310), 64 x 4096 x 4096 122; 512 x 4096 x 4096, group 2
// 170 (739), group 4 103 (301), group 8 83 (218), group 16 74 (182).
#include "sasq_device.h"
#include "gemm_k64.h"
#include <type_traits>

namespace sasq {

constexpr int kSlab = 32;                          // k per LDS slab

// How a group is summed.  DOT4: a multiple of four channels, codes stay packed and v_dot4 sums four products exactly.  ANY: codes as 32-bit integers, one multiply-add each.
enum { GV_DOT4 = 1, GV_ANY = 2 };

// 16 consecutive codes of a row from k0 on, a multiple of 16, as bytes; zeros past K or outside the matrix.  One unaligned load,
// at the row's end shifted into place (byte by byte the loads were most of a call: 64 x 1000 codes by 200 rows in groups of 20
// 79 us, with this 28).  WHOLE: rows of whole pieces, where no piece has an end to look for.
template <bool INT4, bool WHOLE = false>
__device__ __forceinline__ u32x4 load_codes16(const uint8_t* __restrict__ base, int64_t row, bool row_ok, int k0, int K)
{
    if (!row_ok || k0 >= K) return u32x4{0u, 0u, 0u, 0u};
    const bool full = WHOLE || k0 + 16 <= K;
    const int len = INT4 ? K / 2 : K;
    const uint8_t* p = base + row * len;
    if constexpr (INT4) return widen_int4(full ? load_piece<u32x2>(p + k0 / 2) : load_piece_edge<u32x2>(p, k0 / 2, len));
    else                return full ? load_piece<u32x4>(p + k0) : load_piece_edge<u32x4>(p, k0, len);
}

__device__ __forceinline__ int sext_byte(uint32_t w, int e) { return (int)(w << (24 - 8 * e)) >> 24; }

template <int DT, bool INT4, int MODE, int BM, int BN, bool WHOLE>
__global__ __launch_bounds__(256) void linear_grouped_valu_kernel(
    const int8_t* __restrict__ xq, const uint8_t* __restrict__ wq, const float* __restrict__ s_g,
    const float* __restrict__ s_w, const float* __restrict__ bias, uint16_t* __restrict__ y,
    float* __restrict__ f_out, int M, int N, int K, int group, int tiles_m, int first)
{
    using S = Store16<DT>;
    constexpr int TM = BM / 16, TN = BN / 16, TNV = TN / 4;
    constexpr int kSteps = MODE == GV_DOT4 ? kSlab / 4 : kSlab;          // LDS rows per slab
    __shared__ __attribute__((aligned(16))) int lx[2][kSteps][BM];
    __shared__ __attribute__((aligned(16))) int lw[2][kSteps][BN];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int tile = first + (int)blockIdx.x, tm = tile % tiles_m, tn = tile / tiles_m;
    const int m0 = tm * BM, n0 = tn * BN;

    // staging: item (row, half) = 16 codes.  W: BN x 2 items from thread 0 on; X: BM x 2 items on the last threads.
    constexpr int kWItems = 2 * BN, kXItems = 2 * BM;
    static_assert(kWItems <= 256 && kXItems <= 256, "one item per thread and operand");
    const bool has_w = tid < kWItems, has_x = tid >= 256 - kXItems;
    const int wrow = tid % BN, whalf = tid / BN;
    const int xi = tid - (256 - kXItems), xrow = has_x ? xi % BM : 0, xhalf = has_x ? xi / BM : 0;
    u32x4 rw, rx;
    auto fetch = [&](int k0) {
        if (has_w) rw = load_codes16<INT4, WHOLE>(wq, n0 + wrow, n0 + wrow < N, k0 + 16 * whalf, K);
        if (has_x) rx = load_codes16<false, WHOLE>(reinterpret_cast<const uint8_t*>(xq), m0 + xrow, m0 + xrow < M, k0 + 16 * xhalf, K);
    };
    auto put = [&](int buf) {
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
                for (int e = 0; e < 16; ++e) lw[buf][16 * whalf + e][wrow] = sext_byte(rw[e >> 2], e & 3);
            }
            if (has_x) {
#pragma unroll
                for (int e = 0; e < 16; ++e) lx[buf][16 * xhalf + e][xrow] = sext_byte(rx[e >> 2], e & 3);
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
        auto step = [&](int st) {
            int a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = lx[buf][st][ty * TM + i];
#pragma unroll
            for (int v = 0; v < TNV; ++v)
#pragma unroll
                for (int j = 0; j < 4; ++j) b[4 * v + j] = lw[buf][st][64 * v + tx * 4 + j];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    if constexpr (MODE == GV_DOT4) acc[i][j] = __builtin_amdgcn_sdot4(a[i], b[j], acc[i][j], false);
                    else                           acc[i][j] += __mul24(a[i], b[j]);
                }
        };
        constexpr int kPer = MODE == GV_DOT4 ? 4 : 1;
        const int steps = more ? kSteps : (K - k0) / kPer;
#pragma unroll 4
        for (int st = 0; st < steps; ++st) {
            step(st);
            in_group += kPer;
            if (in_group == group) fold();
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
// (DPP row_newbcast), with no LDS read per row and k.  For few rows: one wave per SIMD issues an operation every 6 cycles
// whatever it is, and this form needs the fewest.  LDS holds the codes as bytes, 64 k per slab, rows padded to 80 bytes so
// that 128-bit reads of consecutive rows use all banks; a lane reads 16 codes at once and widens them as it goes (2 operations per 2 TM of useful work).
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

// One or two rows: a row's products and adds are a chain, so the products of several k are made ahead of their adds.
template <int TM, int KS>
__device__ __forceinline__ void few_row_steps(float (&f)[TM], const float (&a)[KS], const float (&b)[KS], const float (&s)[KS])
{
    float p[KS][TM];
#pragma unroll
    for (int k = 0; k < KS; ++k) products<TM>(p[k], a[k], b[k]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
        for (int i = 0; i < TM; ++i) f[i] = __builtin_fmaf(p[k][i], s[k], f[i]);
    __builtin_amdgcn_sched_barrier(0);
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
    float* __restrict__ f_out, int M, int N, int K, int tiles_m, int first)
{
    using S = Store16<DT>;
    constexpr int BM = 4 * TM, BN = 64;
    __shared__ __attribute__((aligned(16))) uint8_t lx[2][BM * kOneStride];
    __shared__ __attribute__((aligned(16))) uint8_t lw[2][BN * kOneStride];
    __shared__ __attribute__((aligned(16))) float ls[2][kOneSlab];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tile = first + (int)blockIdx.x, m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
    const int srow = tid >> 2, sch = tid & 3;           // staging: 16 codes of row srow per thread and operand
    const bool has_x = srow < BM;
    u32x4 rw, rx;
    float rs;
    auto fetch = [&](int k0) {
        rs = s_g[min(k0 + (tid & (kOneSlab - 1)), K - 1)];
        rw = load_codes16<INT4>(wq, n0 + srow, n0 + srow < N, k0 + 16 * sch, K);
        if (has_x) rx = load_codes16<false>(reinterpret_cast<const uint8_t*>(xq), m0 + srow, m0 + srow < M, k0 + 16 * sch, K);
    };
    auto put = [&](int buf) {
        *reinterpret_cast<u32x4*>(&lw[buf][srow * kOneStride + 16 * sch]) = rw;
        if (tid < kOneSlab) ls[buf][tid] = rs;
        if (has_x) *reinterpret_cast<u32x4*>(&lx[buf][srow * kOneStride + 16 * sch]) = rx;
    };
    float f[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) f[i] = 0.0f;
    const int n = n0 + lane;
    const float sw = s_w[min(n, N - 1)], bv = bias ? bias[min(n, N - 1)] : 0.0f;      // requested ahead: a short K has little to hide them
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
                if constexpr (TM <= 2) {
                    float a[16], b[16], s[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        a[e] = (float)sext_byte(av[e >> 2], e & 3);
                        b[e] = (float)sext_byte(bv[e >> 2], e & 3);
                        s[e] = sv[e >> 2][e & 3];
                    }
                    few_row_steps<TM, 16>(f, a, b, s);
                } else {
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        one_step<TM>(f, (float)sext_byte(av[e >> 2], e & 3), (float)sext_byte(bv[e >> 2], e & 3), sv[e >> 2][e & 3]);
                }
            }
        } else {
            for (int k = 0; k < K - k0; ++k) one_step<TM>(f, (float)(int8_t)pa[k], (float)(int8_t)pb[k], ls[buf][k]);
        }
        if (more) {
            put(buf ^ 1);              // the other buffer: its readers passed the barrier of the previous slab
            __syncthreads();
        }
    }
    if (n >= N) return;
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

// Groups of 1, 2, 4, 8 or 16 channels: the matrix units form the group sums while the VALUs run the chain of fused
// multiply-adds, one operation per output and group instead of two or more.  v_mfma_f32_{16x16x4, 4x4x4}_f16 with a zero
// accumulator operand: 16 or 4 rows, the activations' block broadcast to all column blocks, by 64 columns, four
// channels; codes are exact in f16, their products and sums (below 2^19) in fp32.  Smaller groups zero the other channels'
// halves of the activation operand, larger ones chain.  Both forms deliver 32 outputs a cycle and SIMD.
// Measured on register loops, cycles per 16 x 64 products and adds, four | two waves per SIMD: multiply and multiply-add 72 | 85,
// this 60 | 65 (the same with the fp32 outer product v_mfma_f32_16x16x1 70 | 73; a factor in a scalar register takes the
// multiply-add from 2.4 cycles to 4.6, so the factors come from LDS into vector registers).
// A wave owns F rows x 64 columns; LDS holds the codes as halves, 64 channels per slab, rows padded to 144 bytes so that the
// 128-bit reads of 16 consecutive rows use all banks.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
template <int F> struct Outer;
template <> struct Outer<16> {
    typedef float Vec __attribute__((ext_vector_type(16)));
    static __device__ __forceinline__ Vec mma(const f16x4& a, const f16x4& b, const Vec& c) { return __builtin_amdgcn_mfma_f32_16x16x4f16(a, b, c, 2, 0, 0); }
    static __device__ __forceinline__ int row(int r, int lane) { return 4 * (lane >> 4) + (r & 3); }
    static __device__ __forceinline__ int col(int r, int lane) { return 16 * (r >> 2) + (lane & 15); }
};
template <> struct Outer<4> {
    typedef float Vec __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ Vec mma(const f16x4& a, const f16x4& b, const Vec& c) { return __builtin_amdgcn_mfma_f32_4x4x4f16(a, b, c, 4, 0, 0); }
    static __device__ __forceinline__ int row(int r, int lane) { return r; }
    static __device__ __forceinline__ int col(int r, int lane) { return lane; }
};

constexpr int kSgSlab = 64;
constexpr int kSgStride = 2 * kSgSlab + 16;        // bytes

// four codes -> four halves: byte u = code + 128 under the exponent of 1024 is 1024 + u
__device__ __forceinline__ u32x2 halves4(uint32_t codes)
{
    const uint32_t u = codes ^ 0x80808080u;
    const f16x2 bias = {(_Float16)-1152.0f, (_Float16)-1152.0f};
    const f16x2 lo = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0x64646464u, u, 0x04010400u)) + bias;
    const f16x2 hi = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0x64646464u, u, 0x04030402u)) + bias;
    return u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
}

template <int DT, bool INT4, int G, int F, bool WHOLE>
__global__ __launch_bounds__(256, F == 16 || G == 2 ? 3 : 4) void linear_small_group_kernel(
    const int8_t* __restrict__ xq, const uint8_t* __restrict__ wq, const float* __restrict__ s_g,
    const float* __restrict__ s_w, const float* __restrict__ bias, uint16_t* __restrict__ y,
    float* __restrict__ f_out, int M, int N, int K, int tiles_m, int first)
{
    using S = Store16<DT>;
    using O = Outer<F>;
    constexpr int BM = 4 * F, BN = 64, kFactors = kSgSlab / G;
    constexpr int U = 16 / F < kFactors ? 16 / F : kFactors;              // groups per batch: 16 sums per lane, two batches in turn
    __shared__ __attribute__((aligned(16))) char lx[2][BM * kSgStride];
    __shared__ __attribute__((aligned(16))) char lw[2][BN * kSgStride];
    __shared__ __attribute__((aligned(16))) float ls[2][kSgSlab];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tile = first + (int)blockIdx.x, m0 = (tile % tiles_m) * BM, n0 = (tile / tiles_m) * BN;
    // staging: 16 codes of weight row tid/4 per thread and, on the first 4 BM threads, of activation row tid/4; two slabs ahead
    // in registers (one ahead left 64 x 4096 x 4096 waiting for memory in every slab: 133 us)
    const int irow = tid >> 2, ich = tid & 3;
    const bool has_x = tid < 4 * BM;
    struct Slab { u32x4 w, x; float s; };
    Slab ring[2];
    auto fetch = [&](Slab& r, int k0) {
        const int gi = k0 / G + tid;
        if (tid < kFactors) r.s = gi < K / G ? s_g[gi] : 0.0f;            // past the end: 0 * 0 leaves every sum as it is
        r.w = load_codes16<INT4, WHOLE>(wq, n0 + irow, n0 + irow < N, k0 + 16 * ich, K);
        if (has_x) r.x = load_codes16<false, WHOLE>(reinterpret_cast<const uint8_t*>(xq), m0 + irow, m0 + irow < M, k0 + 16 * ich, K);
    };
    auto widen = [&](char* dst, const u32x4& v) {
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const u32x2 p = halves4(v[2 * d]), q = halves4(v[2 * d + 1]);
            *reinterpret_cast<u32x4*>(dst + 16 * d) = u32x4{p[0], p[1], q[0], q[1]};
        }
    };
    auto put = [&](const Slab& r, int buf) {
        if (tid < kFactors) ls[buf][tid] = r.s;
        widen(&lw[buf][irow * kSgStride + 32 * ich], r.w);
        if (has_x) widen(&lx[buf][irow * kSgStride + 32 * ich], r.x);
    };
    float f[F];
#pragma unroll
    for (int r = 0; r < F; ++r) f[r] = 0.0f;
    const int slabs = (K + kSgSlab - 1) / kSgSlab;
    auto multiply = [&](int buf) {
        const char* pa = &lx[buf][(wave * F + lane % F) * kSgStride];
        const char* pb = &lw[buf][lane * kSgStride];
        constexpr int kPieces = kSgSlab / 8;                              // eight channels of codes per LDS read
        u32x4 av[kPieces], bv[kPieces];
        f32x4 sv[2];
        auto read_s = [&](int q) { sv[q & 1] = *reinterpret_cast<const f32x4*>(&ls[buf][4 * q]); };
        read_s(0);
#pragma unroll
        for (int p = 0; p < kPieces; ++p) {
            av[p] = *reinterpret_cast<const u32x4*>(pa + 16 * p);
            bv[p] = *reinterpret_cast<const u32x4*>(pb + 16 * p);
        }
        typename O::Vec sum[2][U];
        auto form = [&](int batch) {                                       // the sums of U groups of this slab
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int c = 0; c < (G + 3) / 4; ++c) {
                    const typename O::Vec zero = {0.0f};
                    const int k = (batch * U + u) * G + 4 * c, h = (k >> 2) & 1;
                    uint32_t a0 = av[k >> 3][2 * h], a1 = av[k >> 3][2 * h + 1];
                    if (G == 1) {
                        a0 = (k & 3) == 0 ? a0 & 0xFFFFu : (k & 3) == 1 ? a0 & 0xFFFF0000u : 0u;
                        a1 = (k & 3) == 2 ? a1 & 0xFFFFu : (k & 3) == 3 ? a1 & 0xFFFF0000u : 0u;
                    } else if (G == 2) {
                        if (k & 2) a0 = 0u; else a1 = 0u;
                    }
                    // keeps the batches apart: left alone the compiler forms all sums of the slab first, in accumulator registers
                    asm volatile("" : "+v"(a0), "+v"(a1));
                    const f16x4 a = __builtin_bit_cast(f16x4, u32x2{a0, a1});
                    const f16x4 b = __builtin_bit_cast(f16x4, u32x2{bv[k >> 3][2 * h], bv[k >> 3][2 * h + 1]});
                    sum[batch & 1][u] = O::mma(a, b, c == 0 ? zero : sum[batch & 1][u]);
                }
        };
        form(0);
        // the sums of batch i + 1 are formed while those of batch i are added up
#pragma unroll
        for (int i = 0; i < kFactors / U; ++i) {
            if (i + 1 < kFactors / U) form(i + 1);
            __builtin_amdgcn_sched_barrier(0x0100);                        // only LDS reads may move across
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int g = i * U + u;
                if ((g & 3) == 0 && g + 4 < kFactors) read_s((g >> 2) + 1);
                const float sg = sv[(g >> 2) & 1][g & 3];
#pragma unroll
                for (int r = 0; r < F; ++r) f[r] = __builtin_fmaf(sum[i & 1][u][r], sg, f[r]);
            }
#pragma unroll
            for (int r = 0; r < F; ++r) asm volatile("" : "+v"(f[r]));
            __builtin_amdgcn_sched_barrier(0x0100);
        }
    };
    // Four rows: the one column's factors are requested ahead, as a short K has little to hide them behind.
    float sw = 0.0f, bv = 0.0f;
    if constexpr (F == 4) {
        const int n = min(n0 + lane, N - 1);
        sw = s_w[n];
        bv = bias ? bias[n] : 0.0f;
    }
    fetch(ring[0], 0);
    if (slabs > 1) fetch(ring[1], kSgSlab);
    put(ring[0], 0);
    if (slabs > 2) fetch(ring[0], 2 * kSgSlab);
    __syncthreads();
    for (int i = 0; i < slabs; i += 2) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (i + j >= slabs) break;
            multiply(j);
            if (i + j + 1 < slabs) {
                put(ring[1 - j], 1 - j);           // the other buffer: its readers passed the barrier of the previous slab
                if (i + j + 3 < slabs) fetch(ring[1 - j], (i + j + 3) * kSgSlab);
                __syncthreads();
            }
        }
    }
#pragma unroll
    for (int r = 0; r < F; ++r) {
        const int m = m0 + wave * F + O::row(r, lane), n = n0 + O::col(r, lane);
        if (m >= M || n >= N) continue;
        float yv = f[r] * (F == 4 ? sw : s_w[n]);
        if (bias) yv = yv + (F == 4 ? bv : bias[n]);
        const int64_t o = (int64_t)m * N + n;
        y[o] = S::enc(yv);
        if (f_out) f_out[o] = f[r];
    }
}

// Rows of a few codes, few outputs: one thread per output, as the kernels above take longer to start than there is work.
// Measured, us with the pre-pass, this | those: 64 x 1000 outputs, K = 2, 4, 8, 12 in groups of two 4.1 | 5.3, 4.4 | 5.4, 5.2 | 5.5,
// 5.8 | 5.7, one group of 8 4.5 | 4.9; 512 x 512, K = 4, 8 in groups of two 5.1 | 5.7, 5.9 | 5.8.
constexpr int64_t kShortRow = 12, kShortRows = 1 << 20;        // channels; channels times outputs

template <int DT, bool INT4>
__global__ __launch_bounds__(256) void linear_grouped_short_row_kernel(
    const int8_t* __restrict__ xq, const uint8_t* __restrict__ wq, const float* __restrict__ s_g,
    const float* __restrict__ s_w, const float* __restrict__ bias, uint16_t* __restrict__ y,
    float* __restrict__ f_out, int outputs, int N, int K, int group)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i >= outputs) return;
    const int m = i / N, n = i - m * N;
    const int8_t* xr = xq + m * K;
    const uint8_t* wr = wq + (int64_t)n * (INT4 ? K / 2 : K);
    float f = 0.0f;
    for (int k = 0, g = 0; k < K; ++g) {
        int acc = 0;
        for (const int end = k + group; k < end; ++k) {
            const int b = wr[INT4 ? k / 2 : k];
            const int w = INT4 ? (((k & 1 ? b >> 4 : b & 15) ^ 8) - 8) : (int)(int8_t)b;
            acc += (int)xr[k] * w;
        }
        f = __builtin_fmaf((float)acc, s_g[g], f);
    }
    if (f_out) f_out[i] = f;
    float yv = f * s_w[n];
    if (bias) yv = yv + bias[n];
    y[i] = Store16<DT>::enc(yv);
}

template <int DT, bool INT4, int TM>
static void launch_per_channel(const GemmK64Args& a, hipStream_t st)
{
    const int64_t tm = (a.M + 4 * TM - 1) / (4 * TM), tn = (a.N + 63) / 64;
    launch_in_parts(tm * tn, 256, [&](unsigned blocks, int first) {
        linear_per_channel_kernel<DT, INT4, TM><<<blocks, 256, 0, st>>>(
            a.xq, a.wq, a.s, a.s_w, a.bias, a.y, reinterpret_cast<float*>(a.acc_out), (int)a.M, (int)a.N, (int)a.K, (int)tm, first);
    });
}

template <int DT, bool INT4, int G, int F>
static void launch_small_group(const GemmK64Args& a, hipStream_t st)
{
    const int64_t tm = (a.M + 4 * F - 1) / (4 * F), tn = (a.N + 63) / 64;
    auto launch = [&](auto whole) {
        launch_in_parts(tm * tn, 256, [&](unsigned blocks, int first) {
            linear_small_group_kernel<DT, INT4, G, F, decltype(whole)::value><<<blocks, 256, 0, st>>>(
                a.xq, a.wq, a.s, a.s_w, a.bias, a.y, reinterpret_cast<float*>(a.acc_out), (int)a.M, (int)a.N, (int)a.K, (int)tm, first);
        });
    };
    if (a.K % 16 == 0) launch(std::true_type{});
    else               launch(std::false_type{});
}

template <int DT, bool INT4, int MODE, int BM, int BN>
static void launch_gv(const GemmK64Args& a, int64_t group, hipStream_t st)
{
    const int64_t tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN;
    auto launch = [&](auto whole) {
        launch_in_parts(tm * tn, 256, [&](unsigned blocks, int first) {
            linear_grouped_valu_kernel<DT, INT4, MODE, BM, BN, decltype(whole)::value><<<blocks, 256, 0, st>>>(
                a.xq, a.wq, a.s, a.s_w, a.bias, a.y, reinterpret_cast<float*>(a.acc_out), (int)a.M, (int)a.N, (int)a.K, (int)group, (int)tm, first);
        });
    };
    if (a.K % 16 == 0) launch(std::true_type{});
    else               launch(std::false_type{});
}

template <int DT, bool INT4, int MODE>
static void launch_gv_mode(const GemmK64Args& a, int64_t group, hipStream_t st)
{
    // The larger the thread's block, the fewer LDS reads per operation; the more workgroups, the more waves to issue from
    // (one wave per SIMD issues a VALU operation every 6 cycles, three every 2.8).
    auto tiles = [&](int bm, int bn) { return ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); };
    if (a.M <= 16)                 launch_gv<DT, INT4, MODE, 16, 64>(a, group, st);
    else if (tiles(64, 128) >= 512) launch_gv<DT, INT4, MODE, 64, 128>(a, group, st);
    else if (tiles(64, 64) >= 256) launch_gv<DT, INT4, MODE, 64, 64>(a, group, st);
    else if (tiles(32, 64) >= 256) launch_gv<DT, INT4, MODE, 32, 64>(a, group, st);
    else                           launch_gv<DT, INT4, MODE, 16, 64>(a, group, st);
}

// Sixteen rows per wave while that makes enough 64x64 tiles, below that four rows per wave or, for single channels, the
// lane-broadcast kernel.  K = N = 4096 (64 tiles per 64 rows), sixteen rows against the other: group 1, M = 64 190 us and 122,
// M = 128 190 and 175, M = 192 191 and 288; group 4, M = 64 76 and 52, M = 192 77 and 73, M = 256 78 and 87; group 16, M = 64
// 60 and 47, M = 192 62 and 63, M = 256 62 and 73.
template <int DT, bool INT4, int G>
static void launch_small_group_rows(const GemmK64Args& a, hipStream_t st)
{
    const int64_t tiles = ((a.M + 63) / 64) * ((a.N + 63) / 64);
    if (a.M > 16 && tiles > (G == 1 ? 128 : 192)) launch_small_group<DT, INT4, G, 16>(a, st);
    else if constexpr (G == 1) {
        // Rows of a wave: fewer give more waves, and a wave alone on its SIMD takes as long as it has operations.  Measured, us, four |
        // one | two: 16 x 1024 x 1024 (256 rows of 64 outputs) 33.6 | 20.5 | 26.3, 16 x 2048 x 4096 (1024) 63.4 | 37.5 | 48.5, 72 x 1024 x 1024 (1152) - | 25.7 | 23.2, 200 x
        // 1024 x 1024 (3200) 34.0 | 41.6 | 32.5, 64 x 2048 x 4096 (4096) 63.6 | 78 | 61, 200 x 4096 x 1500 (4800) 175 | 183 | 159,
        // 512 x 1024 x 1024 (8192) 48 | 71 | 54.
        const int64_t rows64 = a.M * ((a.N + 63) / 64);              // rows of 64 outputs: waves of the one-row form
        if (rows64 <= 1024)      launch_per_channel<DT, INT4, 1>(a, st);
        else if (rows64 <= 4800) launch_per_channel<DT, INT4, 2>(a, st);
        else                     launch_per_channel<DT, INT4, 4>(a, st);
    }
    else                              launch_small_group<DT, INT4, G, 4>(a, st);
}

template <int DT, bool INT4>
static void launch_gv_w(const GemmK64Args& a, int64_t group, hipStream_t st)
{
    if (a.K <= kShortRow && a.M * a.N * a.K <= kShortRows) {
        linear_grouped_short_row_kernel<DT, INT4><<<(unsigned)((a.M * a.N + 255) / 256), 256, 0, st>>>(
            a.xq, a.wq, a.s, a.s_w, a.bias, a.y, reinterpret_cast<float*>(a.acc_out), (int)(a.M * a.N), (int)a.N, (int)a.K, (int)group);
        return;
    }
    switch (group) {
        case 1: launch_small_group_rows<DT, INT4, 1>(a, st); break;
        case 2: launch_small_group_rows<DT, INT4, 2>(a, st); break;
        case 4: launch_small_group_rows<DT, INT4, 4>(a, st); break;
        case 8: launch_small_group_rows<DT, INT4, 8>(a, st); break;
        case 16: launch_small_group_rows<DT, INT4, 16>(a, st); break;
        default:
            if (group % 4 == 0) launch_gv_mode<DT, INT4, GV_DOT4>(a, group, st);
            else                launch_gv_mode<DT, INT4, GV_ANY>(a, group, st);
    }
}

void launch_grouped_valu(const GemmK64Args& a, sasq_dtype dt, bool int4, int64_t group, hipStream_t st)
{
    if (dt == SASQ_F16) { if (int4) launch_gv_w<SASQ_F16, true>(a, group, st);  else launch_gv_w<SASQ_F16, false>(a, group, st); }
    else                { if (int4) launch_gv_w<SASQ_BF16, true>(a, group, st); else launch_gv_w<SASQ_BF16, false>(a, group, st); }
}

}  // namespace sasq

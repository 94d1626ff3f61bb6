// Set-up operations: workspace initialisation, frozen-weight quantization and re-arrangement,
// absmax initial scale.
#include "sasq_device.h"
#include <type_traits>

namespace sasq {

constexpr int kPrepThreads = 256;
constexpr int kMaxAbsmaxBlocks = 2048;       // partials the workspace has room for
constexpr int kAbsmaxBlocks = 256;           // one per CU: every block ends with a ticket on one address
constexpr int kAbsmaxThreads = 512, kAbsmaxUnroll = 4;   // 128-bit loads in flight per thread
constexpr int kAbsmaxThreadsOnce = 256, kAbsmaxBlocksOnce = 128;

__global__ void fill_zero_kernel(uint32_t* p, int64_t nwords)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nwords) p[i] = 0u;
}

template <int THREADS>
__device__ __forceinline__ float block_max(float v, float* sh)
{
    uint32_t w = wave_max(__float_as_uint(v));      // non-negative floats order like their bits
    if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = __uint_as_float(w);
    __syncthreads();
    float m = sh[0];
#pragma unroll
    for (int i = 1; i < THREADS / kWave; ++i) m = fmaxf(m, sh[i]);
    return m;
}

__device__ __forceinline__ float weight_factor(float amax, int bits)
{
    return amax == 0.0f ? 1.0f : amax / (float)((1 << (bits - 1)) - 1);
}

// One block per output channel n (row of W[N,K]): Sec. 3, Eq. 1 applied to the row.  The general form: any K, the row is
// read twice.
template <bool INT4>
__global__ __launch_bounds__(kPrepThreads) void quantize_weight_kernel(
    const float* __restrict__ w, uint8_t* __restrict__ wq, float* __restrict__ s_w, int64_t K)
{
    __shared__ float sh[kPrepThreads / kWave];
    const int64_t n = blockIdx.x;
    const float* row = w + n * K;
    float amax = 0.0f;
    for (int64_t k = threadIdx.x; k < K; k += kPrepThreads) amax = fmaxf(amax, fabsf(row[k]));
    amax = block_max<kPrepThreads>(amax, sh);
    const int bits = INT4 ? 4 : 8;
    const float sw = weight_factor(amax, bits);
    if (threadIdx.x == 0) s_w[n] = sw;
    const QConst kc = make_qconst(sw, bits);
    if (INT4) {
        uint8_t* out = wq + n * (K / 2);
        for (int64_t j = threadIdx.x; j < K / 2; j += kPrepThreads) {
            int lo = code_of(quantize(row[2 * j], kc));
            int hi = code_of(quantize(row[2 * j + 1], kc));
            out[j] = (uint8_t)((lo & 15) | ((hi & 15) << 4));
        }
    } else {
        uint8_t* out = wq + n * K;
        for (int64_t k = threadIdx.x; k < K; k += kPrepThreads)
            out[k] = (uint8_t)(code_of(quantize(row[k], kc)) & 0xFF);
    }
}

// The same for rows of whole 128-bit pieces (K % 4 == 0) that fit a block's registers, R pieces per thread: the row is read
// once, all of it in flight, and the codes leave four at a time.  Bound by the 5 bytes a weight
// moves: 11008 x 4096 and 4096 x 11008 37 us each, 6.1 TB/s (the general kernel, one float per load and one byte per store: 96).
template <bool INT4, int THREADS, int R>
__global__ __launch_bounds__(THREADS) void quantize_weight_vec_kernel(
    const f32x4* __restrict__ w, uint8_t* __restrict__ wq, float* __restrict__ s_w, int pieces)
{
    __shared__ float sh[THREADS / kWave];
    const int64_t n = blockIdx.x;
    const f32x4* row = w + n * pieces;
    f32x4 v[R];
#pragma unroll
    for (int j = 0; j < R; ++j)                       // past the end: the last piece again, which cannot change a maximum
        v[j] = __builtin_nontemporal_load(&row[min(j * THREADS + (int)threadIdx.x, pieces - 1)]);
    float amax = 0.0f;
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) amax = fmaxf(amax, fabsf(v[j][e]));
    amax = block_max<THREADS>(amax, sh);
    const int bits = INT4 ? 4 : 8;
    const float sw = weight_factor(amax, bits);
    if (threadIdx.x == 0) s_w[n] = sw;
    const QConst kc = make_qconst(sw, bits);
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int i = j * THREADS + (int)threadIdx.x;
        if (i >= pieces) break;
        const uint32_t c = pack_codes4(quantize(v[j][0], kc).c, quantize(v[j][1], kc).c, quantize(v[j][2], kc).c, quantize(v[j][3], kc).c);
        if (INT4)
            reinterpret_cast<uint16_t*>(wq)[n * pieces + i] =
                (uint16_t)((c & 0xFu) | ((c >> 4) & 0xF0u) | ((c >> 8) & 0xF00u) | ((c >> 12) & 0xF000u));
        else
            reinterpret_cast<uint32_t*>(wq)[n * pieces + i] = c;
    }
}

// Re-arrange row-major int8 weight codes [N,K] into the GEMM's operand blocks: 16 rows x 64
// K-bytes per 1 KB block, block (nb, kb) at (nb * K/64 + kb) * 1024, the 16-byte chunk c of row
// r at 16 * (4r + (c ^ swz(r))), swz(r) = ((r >> 1) & 3) ^ ((r >> 3) & 1).  One thread per
// destination chunk; rows past N are zero.
__global__ __launch_bounds__(kPrepThreads) void pack_weight_i8_kernel(
    const uint8_t* __restrict__ wq, u32x4* __restrict__ out, int64_t N, int64_t K, int64_t nchunks)
{
    const int64_t i = (int64_t)blockIdx.x * kPrepThreads + threadIdx.x;
    if (i >= nchunks) return;
    const int64_t blk = i >> 6, KT = K >> 6;
    const int sl = (int)(i & 63), r = sl >> 2;
    const int ch = (sl & 3) ^ (((r >> 1) & 3) ^ ((r >> 3) & 1));
    const int64_t n = (blk / KT) * 16 + r, k0 = (blk % KT) * 64 + ch * 16;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (n < N) v = *reinterpret_cast<const u32x4*>(wq + n * K + k0);
    out[i] = v;
}

// Re-arrange row-major packed int4 weight codes [N,K/2] into 1 KB blocks of 32 rows x 64 k:
// block (nb, kb) at (nb * K/64 + kb) * 1024; the 16 codes k = 64 kb + 32 kk + 16 g + (0..15) of
// row r are the 8 bytes at 512 kk + 256 g + 8 r; in them byte b of the first dword holds code b
// (low nibble) and 4 + b (high nibble), byte b of the second dword codes 8 + b and 12 + b.
// One thread per 8 destination bytes; rows past N are zero.
__global__ __launch_bounds__(kPrepThreads) void pack_weight_i4_kernel(
    const uint8_t* __restrict__ wq, u32x2* __restrict__ out, int64_t N, int64_t K, int64_t nslots)
{
    const int64_t i = (int64_t)blockIdx.x * kPrepThreads + threadIdx.x;
    if (i >= nslots) return;
    const int64_t blk = i >> 7, KT = K >> 6;
    const int sl = (int)(i & 127), kk = sl >> 6, g = (sl >> 5) & 1, r = sl & 31;
    const int64_t n = (blk / KT) * 32 + r, k0 = (blk % KT) * 64 + 32 * kk + 16 * g;
    u32x2 o = {0u, 0u};
    if (n < N) {
        const u32x2 sv = *reinterpret_cast<const u32x2*>(wq + n * (K / 2) + k0 / 2);
        const uint64_t src = (uint64_t)sv[0] | ((uint64_t)sv[1] << 32);     // code j at bits 4j
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t c0 = (uint32_t)(src >> (4 * b)) & 15u, c4 = (uint32_t)(src >> (4 * (4 + b))) & 15u;
            const uint32_t c8 = (uint32_t)(src >> (4 * (8 + b))) & 15u, c12 = (uint32_t)(src >> (4 * (12 + b))) & 15u;
            o[0] |= (c0 | (c4 << 4)) << (8 * b);
            o[1] |= (c8 | (c12 << 4)) << (8 * b);
        }
    }
    out[i] = o;
}

// max |x| over a flat 16-bit tensor: magnitudes of finite values and infinities order like their
// 15 low bits, so the reduction is an integer max (exact and order-independent).  Bound by memory latency and the ticket tail:
// each block keeps the next kAbsmaxUnroll loads per thread in flight under the current ones, and there is one block per CU, as
// every block adds its ticket to one address.  45 MB 13 us, 17 MB 9 (one load at a time from 2048 blocks: 34 and 18; 256
// threads with eight loads but no loads ahead: 19 and 6; the set-up of a 7B MLP as a whole: 270 us with 512 blocks of those,
// 262 with 256, 260 with this).
// ONCE: every thread's loads are in flight at once and there is no loop; smaller blocks, as there is little to keep them busy.
// Measured, us, looping | once: 8 values 4.4 | 3.7, 64 x 4096 5.0 | 4.5, 128 x 4096 5.2 | 4.8, 256 x 4096 (128 blocks) 5.8 | 5.7,
// 512 x 4096 6.4 | 7.0.
template <int DT, int THREADS, bool ONCE>
__global__ __launch_bounds__(THREADS) void absmax_kernel(
    const uint16_t* __restrict__ x, float* __restrict__ s, uint32_t* __restrict__ ws_head,
    uint32_t* __restrict__ partials, int64_t n, int bits)
{
    using S = Store16<DT>;
    uint32_t m = 0;
    const int64_t nvec = n / 8;
    const u32x4* xv = reinterpret_cast<const u32x4*>(x);
    if (nvec > 0) {
        const int64_t step = (int64_t)gridDim.x * THREADS * kAbsmaxUnroll;
        int64_t base = (int64_t)blockIdx.x * THREADS * kAbsmaxUnroll + threadIdx.x;
        u32x4 cur[kAbsmaxUnroll], next[kAbsmaxUnroll];
        auto load = [&](u32x4 (&v)[kAbsmaxUnroll], int64_t from) {
#pragma unroll
            for (int u = 0; u < kAbsmaxUnroll; ++u)      // past the end: the last vector again, which cannot change a maximum
                v[u] = __builtin_nontemporal_load(&xv[min(from + u * THREADS, nvec - 1)]);
        };
        auto take = [&](const u32x4 (&v)[kAbsmaxUnroll]) {
#pragma unroll
            for (int u = 0; u < kAbsmaxUnroll; ++u)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    uint32_t lo = v[u][w] & 0x7FFFu, hi = (v[u][w] >> 16) & 0x7FFFu;
                    m = lo > m ? lo : m;
                    m = hi > m ? hi : m;
                }
        };
        load(cur, base);
        if (ONCE) {
            take(cur);
        } else {
            for (; base - (int64_t)threadIdx.x < nvec; base += step) {
                load(next, base + step);
                take(cur);
#pragma unroll
                for (int u = 0; u < kAbsmaxUnroll; ++u) cur[u] = next[u];
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < (unsigned)(n - nvec * 8)) {
        uint32_t a = x[nvec * 8 + threadIdx.x] & 0x7FFFu;
        m = a > m ? a : m;
    }
    __shared__ uint32_t sh[THREADS / kWave];
    __shared__ bool is_last;
    m = wave_max(m);
    if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < THREADS / kWave; ++i) m = sh[i] > m ? sh[i] : m;
        const uint32_t ticket = publish_then_ticket(&partials[blockIdx.x], m, &ws_head[0]);
        is_last = (ticket == kTicketBase + gridDim.x - 1);
        if (ticket - kTicketBase >= gridDim.x) *s = __uint_as_float(0x7FC00000u);
    }
    __syncthreads();
    if (!is_last) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    static_assert(kAbsmaxBlocks <= THREADS, "one partial per thread");
    uint32_t t = __hip_atomic_load(&partials[threadIdx.x < gridDim.x ? threadIdx.x : 0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    t = wave_max(t);                                              // a duplicate of partial 0 cannot change a max
    __syncthreads();
    if (threadIdx.x % kWave == 0) sh[threadIdx.x / kWave] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 0; i < THREADS / kWave; ++i) t = sh[i] > t ? sh[i] : t;
        float amax = S::one((uint16_t)t);
        *s = amax / (float)((1 << (bits - 1)) - 1);
        __hip_atomic_store(&ws_head[0], kTicketBase, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Rows of up to 256 weights: one wave, which needs no barrier (20000 x 64 6.9 us, with 256 threads 12.7, as many as with the
// general kernel), up to 8192: 256 threads, up to 32768: 1024 (eight pieces per thread at most); longer or ragged ones, and
// more rows than a launch holds workgroups of 1024 threads, take the general kernel.
template <bool INT4>
static void quantize_weight(const float* w, uint8_t* wq, float* s_w, int64_t N, int64_t K, hipStream_t st)
{
    if ((K & 3) || K > 32768 || (K > 8192 && N >= INT64_C(1) << 22)) {
        quantize_weight_kernel<INT4><<<(int)N, kPrepThreads, 0, st>>>(w, wq, s_w, K);
        return;
    }
    const int pieces = (int)(K >> 2);
    auto launch = [&](auto threads_tag, auto r_tag) {
        constexpr int T = decltype(threads_tag)::value, R = decltype(r_tag)::value;
        quantize_weight_vec_kernel<INT4, T, R><<<(int)N, T, 0, st>>>(reinterpret_cast<const f32x4*>(w), wq, s_w, pieces);
    };
    auto by_pieces = [&](auto threads_tag) {
        constexpr int T = decltype(threads_tag)::value;
        switch ((pieces + T - 1) / T) {
            case 1: launch(threads_tag, std::integral_constant<int, 1>{}); break;
            case 2: launch(threads_tag, std::integral_constant<int, 2>{}); break;
            case 3: launch(threads_tag, std::integral_constant<int, 3>{}); break;
            case 4: launch(threads_tag, std::integral_constant<int, 4>{}); break;
            case 5: launch(threads_tag, std::integral_constant<int, 5>{}); break;
            case 6: launch(threads_tag, std::integral_constant<int, 6>{}); break;
            case 7: launch(threads_tag, std::integral_constant<int, 7>{}); break;
            default: launch(threads_tag, std::integral_constant<int, 8>{}); break;
        }
    };
    if (K <= 256) launch(std::integral_constant<int, kWave>{}, std::integral_constant<int, 1>{});
    else if (K <= 8192) by_pieces(std::integral_constant<int, 256>{});
    else           by_pieces(std::integral_constant<int, 1024>{});
}

}  // namespace sasq

using namespace sasq;

extern "C" const char* sasq_status_string(int status)
{
    switch (status) {
        case SASQ_OK: return "SASQ_OK";
        case SASQ_ERR_NULL: return "SASQ_ERR_NULL: a required pointer is NULL";
        case SASQ_ERR_SHAPE: return "SASQ_ERR_SHAPE: bad size";
        case SASQ_ERR_ALIGN: return "SASQ_ERR_ALIGN: pointer not 16-byte aligned";
        case SASQ_ERR_UNSUPPORTED: return "SASQ_ERR_UNSUPPORTED: unknown enum or bits outside [2,8]";
        case SASQ_ERR_WORKSPACE: return "SASQ_ERR_WORKSPACE: workspace missing or too small";
        case SASQ_ERR_LAUNCH: return "SASQ_ERR_LAUNCH: HIP launch error";
        default: return "unknown sasq_status";
    }
}

extern "C" int sasq_version(void) { return 200; }

namespace sasq { int g_tuning[SASQ_TUNE_COUNT] = {0}; }

extern "C" int sasq_set_tuning(int knob, int value)
{
    static const int kMax[SASQ_TUNE_COUNT] = {2, 3, 2, 3, 2};
    if (knob < 0 || knob >= SASQ_TUNE_COUNT || value < 0 || value > kMax[knob]) return SASQ_ERR_UNSUPPORTED;
    sasq::g_tuning[knob] = value;
    return SASQ_OK;
}

extern "C" int sasq_workspace_init(void* workspace, size_t workspace_bytes, void* stream)
{
    if (!workspace) return SASQ_ERR_NULL;
    if (workspace_bytes < kWsMinBytes) return SASQ_ERR_WORKSPACE;
    if (!aligned16(workspace)) return SASQ_ERR_ALIGN;
    const int64_t words = (int64_t)((workspace_bytes < kWsHeaderBytes ? workspace_bytes : kWsHeaderBytes) / 4);
    fill_zero_kernel<<<1, 256, 0, as_stream(stream)>>>(static_cast<uint32_t*>(workspace), words);
    return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
}

extern "C" int sasq_quantize_weight(const float* w, void* wq, float* s_w, int64_t N, int64_t K,
                                    sasq_wfmt wf, void* stream)
{
    if (!w || !wq || !s_w) return SASQ_ERR_NULL;
    if (N <= 0 || K <= 0 || N > 0x7FFFFFFF || N > (INT64_C(1) << 40) / K) return SASQ_ERR_SHAPE;
    if (wf != SASQ_W_INT8 && wf != SASQ_W_INT4_PACKED) return SASQ_ERR_UNSUPPORTED;
    if (wf == SASQ_W_INT4_PACKED && (K & 1)) return SASQ_ERR_SHAPE;
    if (!aligned16(w) || !aligned16(wq)) return SASQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);
    if (wf == SASQ_W_INT8) quantize_weight<false>(w, static_cast<uint8_t*>(wq), s_w, N, K, st);
    else                   quantize_weight<true>(w, static_cast<uint8_t*>(wq), s_w, N, K, st);
    return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
}

extern "C" size_t sasq_packed_weight_bytes(int64_t N, int64_t K, sasq_wfmt wf)
{
    if (N <= 0 || K <= 0 || (K % 64) != 0) return 0;
    if (wf == SASQ_W_INT8_BLOCKED) return (size_t)((N + 15) / 16 * 16) * (size_t)K;
    if (wf == SASQ_W_INT4_BLOCKED) return (size_t)((N + 31) / 32 * 32) * (size_t)(K / 2);
    return 0;
}

extern "C" int sasq_pack_weight(const void* wq, void* packed, int64_t N, int64_t K, sasq_wfmt wf_src, void* stream)
{
    if (!wq || !packed) return SASQ_ERR_NULL;
    if (N <= 0 || K <= 0 || N > 0x7FFFFFFF || N > (INT64_C(1) << 40) / K) return SASQ_ERR_SHAPE;
    if (wf_src != SASQ_W_INT8 && wf_src != SASQ_W_INT4_PACKED) return SASQ_ERR_UNSUPPORTED;
    if (K % 64) return SASQ_ERR_SHAPE;
    if (!aligned16(wq) || !aligned16(packed)) return SASQ_ERR_ALIGN;
    hipStream_t st = as_stream(stream);
    if (wf_src == SASQ_W_INT8) {
        const int64_t nchunks = (int64_t)(sasq_packed_weight_bytes(N, K, SASQ_W_INT8_BLOCKED) / 16);
        pack_weight_i8_kernel<<<(unsigned)((nchunks + kPrepThreads - 1) / kPrepThreads), kPrepThreads, 0, st>>>(
            static_cast<const uint8_t*>(wq), static_cast<u32x4*>(packed), N, K, nchunks);
    } else {
        const int64_t nslots = (int64_t)(sasq_packed_weight_bytes(N, K, SASQ_W_INT4_BLOCKED) / 8);
        pack_weight_i4_kernel<<<(unsigned)((nslots + kPrepThreads - 1) / kPrepThreads), kPrepThreads, 0, st>>>(
            static_cast<const uint8_t*>(wq), static_cast<u32x2*>(packed), N, K, nslots);
    }
    return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
}

extern "C" size_t sasq_absmax_scale_workspace(int64_t rows, int64_t cols)
{
    (void)rows; (void)cols;
    return kWsHeaderBytes + sizeof(uint32_t) * kMaxAbsmaxBlocks;
}

extern "C" int sasq_absmax_scale(const void* x, float* s, int64_t rows, int64_t cols, int bits,
                                 sasq_dtype dt, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !s) return SASQ_ERR_NULL;
    if (rows <= 0 || cols <= 0 || rows > (INT64_C(1) << 40) / cols) return SASQ_ERR_SHAPE;
    if (bits < 2 || bits > 8) return SASQ_ERR_UNSUPPORTED;
    if (dt != SASQ_F16 && dt != SASQ_BF16) return SASQ_ERR_UNSUPPORTED;
    if (!aligned16(x)) return SASQ_ERR_ALIGN;
    if (!workspace || workspace_bytes < sasq_absmax_scale_workspace(rows, cols)) return SASQ_ERR_WORKSPACE;
    if (!aligned16(workspace)) return SASQ_ERR_ALIGN;
    const int64_t n = rows * cols;
    auto blocks = [&](int threads) { return (n / 8 + threads * kAbsmaxUnroll - 1) / (threads * kAbsmaxUnroll); };
    auto head = static_cast<uint32_t*>(workspace);
    auto parts = reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + kWsHeaderBytes);
    hipStream_t st = as_stream(stream);
    auto launch = [&](auto dt_tag, auto threads_tag, auto once_tag) {
        constexpr int T = decltype(threads_tag)::value;
        const int64_t need = blocks(T);
        const int grid = (int)(need < 1 ? 1 : (need > kAbsmaxBlocks ? kAbsmaxBlocks : need));
        absmax_kernel<decltype(dt_tag)::value, T, decltype(once_tag)::value><<<grid, T, 0, st>>>(
            static_cast<const uint16_t*>(x), s, head, parts, n, bits);
    };
    auto by_size = [&](auto dt_tag) {
        if (blocks(kAbsmaxThreadsOnce) <= kAbsmaxBlocksOnce) launch(dt_tag, std::integral_constant<int, kAbsmaxThreadsOnce>{}, std::true_type{});
        else                                             launch(dt_tag, std::integral_constant<int, kAbsmaxThreads>{}, std::false_type{});
    };
    if (dt == SASQ_F16) by_size(std::integral_constant<int, SASQ_F16>{});
    else                by_size(std::integral_constant<int, SASQ_BF16>{});
    return hipGetLastError() == hipSuccess ? SASQ_OK : SASQ_ERR_LAUNCH;
}

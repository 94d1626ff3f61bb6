// Grouped-factor linear (Sec. 3, Eq. 3) for calls of few output tiles: the contraction split over a workgroup's waves.
//
// What bounds such a call is not work but its length: with one tile of outputs per wave or workgroup the whole contraction goes by
// in one K loop of dependent steps (load, barrier, group sum, fold), on a part of the chip.  The chain of fused multiply-adds over the
// groups has to be in order, but the group sums, integers, do not: here the waves take the K tiles of a phase side by side, form
// their groups' sums on the matrix units and put them into LDS, and the chain, then one LDS read and one multiply-add per output
// and group, runs through them in order while the next phase's operands are on their way.  Two LDS buffers in turn, one barrier a
// phase.  Groups of 4, 8, 16 and 32 channels: a K tile of 64 channels is multiplied once per group, with the activation operand's other
// channels zeroed (lane l of an operand holds the 16 channels 16 (l / 16) .. + 15).
// Measured, us with the pre-pass, before | here: 16 x 1024 x 1024 (rows, K, N) groups of 4 15.0 | 10.9, 16 13.6 | 6.2, 32 18.1 | 5.8;
// 16 x 2048 x 4096 groups of 4 26.4 | 17.8, 16 23.4 | 8.3, 32 30.3 | 7.4; 128 x 4096 x 4096 pre-arranged, groups of 64 34.4 | 18.2,
// 128 27.2 | 17.6, 512 20.6 | 16.3.
#include "sasq_device.h"
#include "gemm_tile.h"
#include "gemm_k64.h"
#include <type_traits>

namespace sasq {

constexpr int kSplitFactors = 2048;                // factors of a call, kept in LDS

// G: channels of a group; 64 stands for every multiple of 64, `group_tiles` K tiles.  BLOCKED: pre-arranged int8 weights.
template <int DT, int G, bool BLOCKED, int MT, int NT, int NW>
__global__ __launch_bounds__(64 * NW) void linear_group_split_kernel(
    const int8_t* __restrict__ xq, const uint8_t* __restrict__ wq, const float* __restrict__ s_g,
    const float* __restrict__ s_w, const float* __restrict__ bias, uint16_t* __restrict__ y,
    float* __restrict__ f_out, int M, int N, int K, int group_tiles, int tiles_m, int tiles_n)
{
    using S = Store16<DT>;
    constexpr int kPer = 64 / G;                                    // groups of a K tile
    constexpr int kPhase = NW * kPer, kTiles = MT * NT;             // groups of a phase
    constexpr int kOut = kTiles * 256, kThreads = 64 * NW, kMine = (kOut + kThreads - 1) / kThreads;
    __shared__ __attribute__((aligned(16))) float part[2][kPhase][kOut];
    __shared__ __attribute__((aligned(16))) float factors[kSplitFactors];

    // Eight neighbours in the id go to the eight XCDs: the row tiles of one run of columns stay on one, 8 ids apart.
    const int id = (int)blockIdx.x, octet = id >> 3;
    const int mblk = octet % tiles_m, nblk = octet / tiles_m * 8 + (id & 7);
    if (nblk >= tiles_n) return;
    const int m0 = mblk * 16 * MT, n0 = nblk * 16 * NT;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int frow = lane & 15, fq = lane >> 4;
    const int KT = K >> 6;
    const int groups = G < 64 ? KT * kPer : KT / group_tiles;

    const int8_t* xrow[MT];
    const uint8_t* wrow[NT];
#pragma unroll
    for (int b = 0; b < MT; ++b) xrow[b] = xq + (int64_t)min(m0 + 16 * b + frow, M - 1) * K + 16 * fq;
#pragma unroll
    for (int g = 0; g < NT; ++g) {
        if (BLOCKED) wrow[g] = wq + (int64_t)min((n0 >> 4) + g, (N - 1) >> 4) * KT * 1024 + (4 * frow + (fq ^ swz64(frow))) * 16;
        else         wrow[g] = wq + (int64_t)min(n0 + 16 * g + frow, N - 1) * K + 16 * fq;
    }
    constexpr int kWStep = BLOCKED ? 1024 : 64;
    struct Frag { i32x4 x[MT], w[NT]; };
    auto load = [&](Frag& f, int t) {
#pragma unroll
        for (int b = 0; b < MT; ++b) f.x[b] = *reinterpret_cast<const i32x4*>(xrow[b] + (int64_t)t * 64);
#pragma unroll
        for (int g = 0; g < NT; ++g) f.w[g] = *reinterpret_cast<const i32x4*>(wrow[g] + (int64_t)t * kWStep);
    };
    // This wave's K tiles in order: tile j of the group (phase NW + wave).
    const int gt = G < 64 ? 1 : group_tiles;
    auto tile_of = [&](int phase, int j) { return (phase * NW + wave) * gt + j; };
    const int phases = (groups + kPhase - 1) / kPhase;
    Frag next;
    if (tile_of(0, 0) < KT) load(next, tile_of(0, 0));

    for (int i = tid; i < groups; i += kThreads) factors[i] = s_g[i];

    float f[kMine];
#pragma unroll
    for (int o = 0; o < kMine; ++o) f[o] = 0.0f;
    for (int p = 0; p < phases; ++p) {
        float (*buf)[kOut] = part[p & 1];
        if (tile_of(p, 0) < KT) {
            if constexpr (G < 64) {
                const Frag cur = next;
                if (tile_of(p + 1, 0) < KT) load(next, tile_of(p + 1, 0));
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
#pragma unroll
                    for (int b = 0; b < MT; ++b) {
                        i32x4 x = {0, 0, 0, 0};
                        if constexpr (G == 4) {
                            x[q & 3] = fq == q >> 2 ? cur.x[b][q & 3] : 0;
                        } else if constexpr (G == 8) {
                            x[2 * (q & 1)] = fq == q >> 1 ? cur.x[b][2 * (q & 1)] : 0;
                            x[2 * (q & 1) + 1] = fq == q >> 1 ? cur.x[b][2 * (q & 1) + 1] : 0;
                        }
                        else if constexpr (G == 16) x = fq == q ? cur.x[b] : x;
                        else                        x = fq >> 1 == q ? cur.x[b] : x;
#pragma unroll
                        for (int g = 0; g < NT; ++g) {
                            const i32x4 sum = __builtin_amdgcn_mfma_i32_16x16x64_i8(cur.w[g], x, i32x4{0, 0, 0, 0}, 0, 0, 0);
                            *reinterpret_cast<f32x4*>(&buf[wave * kPer + q][(b * NT + g) * 256 + 4 * lane]) =
                                f32x4{(float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]};
                        }
                    }
                }
            } else {
                i32x4 acc[MT][NT];
#pragma unroll
                for (int b = 0; b < MT; ++b)
#pragma unroll
                    for (int g = 0; g < NT; ++g) acc[b][g] = i32x4{0, 0, 0, 0};
                for (int j = 0; j < gt; ++j) {
                    const Frag cur = next;
                    const int t = j + 1 < gt ? tile_of(p, j + 1) : tile_of(p + 1, 0);
                    if (t < KT) load(next, t);
#pragma unroll
                    for (int b = 0; b < MT; ++b)
#pragma unroll
                        for (int g = 0; g < NT; ++g) acc[b][g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(cur.w[g], cur.x[b], acc[b][g], 0, 0, 0);
                }
#pragma unroll
                for (int b = 0; b < MT; ++b)
#pragma unroll
                    for (int g = 0; g < NT; ++g)
                        *reinterpret_cast<f32x4*>(&buf[wave][(b * NT + g) * 256 + 4 * lane]) =
                            f32x4{(float)acc[b][g][0], (float)acc[b][g][1], (float)acc[b][g][2], (float)acc[b][g][3]};
            }
        }
        // The sums of this phase are there; the other buffer's readers (the phase before) have passed as well.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (wave * 64 < kOut) {
            const int count = min(kPhase, groups - p * kPhase);
            const float* fac = &factors[p * kPhase];
            auto chain = [&](int g, float s) {
#pragma unroll
                for (int o = 0; o < kMine; ++o) f[o] = __builtin_fmaf(buf[g][tid + o * kThreads], s, f[o]);
            };
            int g = 0;
            if constexpr (kPhase >= 8) {
                for (; g + 8 <= count; g += 8) {
                    const f32x4 s0 = *reinterpret_cast<const f32x4*>(fac + g), s1 = *reinterpret_cast<const f32x4*>(fac + g + 4);
#pragma unroll
                    for (int e = 0; e < 8; ++e) chain(g + e, e < 4 ? s0[e & 3] : s1[e & 3]);
                }
            }
            for (; g < count; ++g) chain(g, fac[g]);
        }
    }

    // Output o of a 16 x 16 tile: register o % 4 of lane o / 4, column 4 (lane / 16) + register, row lane % 16.
    if (wave * 64 >= kOut) return;
#pragma unroll
    for (int o = 0; o < kMine; ++o) {
        const int i = tid + o * kThreads, tile = i >> 8, l = (i & 255) >> 2;
        const int m = m0 + 16 * (tile / NT) + (l & 15), n = n0 + 16 * (tile % NT) + 4 * (l >> 4) + (i & 3);
        if (m >= M || n >= N) continue;
        float yv = f[o] * s_w[n];
        if (bias) yv = yv + bias[n];
        const int64_t at = (int64_t)m * N + n;
        y[at] = S::enc(yv);
        if (f_out) f_out[at] = f[o];
    }
}

template <int DT, int G, bool BLOCKED, int MT, int NT, int NW>
static void launch_split(const GemmK64Args& a, int64_t group, hipStream_t st)
{
    const int tm = (int)((a.M + 16 * MT - 1) / (16 * MT)), tn = (int)((a.N + 16 * NT - 1) / (16 * NT));
    linear_group_split_kernel<DT, G, BLOCKED, MT, NT, NW><<<(unsigned)((tn + 7) / 8 * 8 * tm), 64 * NW, 0, st>>>(
        a.xq, a.wq, a.s, a.s_w, a.bias, a.y, reinterpret_cast<float*>(a.acc_out), (int)a.M, (int)a.N, (int)a.K, (int)(group / 64), tm, tn);
}

// 0: the other kernels; rows / 16 and columns / 16 of a workgroup: 1: 1, 1, 2: 2, 2, 3: 1, 2.
// A workgroup of many outputs reads its operands less often, one of few leaves room for more of them; the other kernels' time is their K
// loop's, at any fill.  So the line is a number of 16 x 16 output tiles.  Measured, us, before | 1 | 2 | 3, with that number:
//   groups of 4 (one workgroup a CU for its LDS: one round):  64 x 1024 x 1024 (256) 15.2 | 11.3, 200 x 1024 x 1024 (832) 15.6 | 32.9
//   16:  64 x 2048 x 4096 (1024) 23.8 | 15.2 | 16.5 | 16.3, 200 x 4096 x 1500 (1222) 48.4 | 30.7 | 50.5 | 37.7, 512 x 1024 x 1024 (2048)
//     16.3 | 17.4 | 18.2 | 18.0, 200 x 2048 x 4096 (3328) 32.6 | 39.1 | 53.5 | 45.4
//   32:  16 x 4096 x 1000 (63) 54.7 | 10.6 | 15.3 | 13.5, 64 x 2048 x 4096 (1024) 30.3 | 12.8 | 11.2 | 10.9, 200 x 2048 x 4096 30.9 |
//     30.7 | 30.8 | 28.0, 512 x 2048 x 4096 (8192) 31.3 | 64.8 | 60.3 | 58.2
//   64, row-major:  128 x 1024 x 1024 (512) 13.8 | 6.9 | 7.4 | 6.6, 128 x 4096 x 4096 (2048) 34.3 | 35.3 | 21.0 | 28.5, 300 x 4096 x 4096
//     (4864) 34.5 | 73.5 | 50.2 | 59.8; pre-arranged 13.8 | 6.3 | 6.8 | 6.0, 34.4 | 24.9 | 17.4 | 18.2, 35.6 | 50.4 | 37.9 | 35.8
//   128, pre-arranged:  128 x 4096 x 4096 27.2 | 24.6 | 16.5 | 17.6, 300 x 4096 x 4096 28.1 | 49.6 | 35.1 | 34.5
//   512, row-major and pre-arranged:  300 x 2048 x 1024 (1216) 14.4 | 14.9 | 12.7 | 13.4, 14.1 | 12.8 | 10.3 | 9.7, 300 x 4096 x 4096 22.1 |
//     71.5 | 44.2 | 58.1, 21.5 | 48.3 | 32.3 | 33.4
int grouped_takes_split(int64_t M, int64_t N, int64_t K, int64_t group, bool blocked)
{
    if (K % 64 != 0 || K / group > kSplitFactors) return 0;
    const int64_t tiles = (M + 15) / 16 * ((N + 15) / 16);
    if (group == 4) return tiles <= 256 ? 1 : 0;
    if (group == 8) return tiles <= 512 ? 1 : 0;
    if (group == 16) return tiles <= 1800 ? 1 : 0;
    if (group == 32) return tiles <= 512 ? 1 : tiles <= 3500 ? 3 : 0;
    if (group % 64 != 0) return 0;
    // the other kernel's K tile, with its share of a fold, costs 0.19 us + 0.24 a group, this one's 0.105 ns an output tile, row-major 0.14
    const double most = (0.19 + 0.24 * 64.0 / (double)group) / (blocked ? 0.105e-3 : 0.14e-3);
    if ((double)tiles > most) return 0;
    return tiles < 256 ? 1 : !blocked && tiles >= 1500 ? 2 : 3;
}

template <int DT, int G, bool BLOCKED>
static void launch_split_g(const GemmK64Args& a, int64_t group, int form, hipStream_t st)
{
    if constexpr (G == 4)                launch_split<DT, G, BLOCKED, 1, 1, 4>(a, group, st);
    else if (G < 32 || form == 1)        launch_split<DT, G, BLOCKED, 1, 1, 8>(a, group, st);
    else if constexpr (G == 64) {
        if (form == 2) launch_split<DT, G, BLOCKED, 2, 2, 8>(a, group, st);
        else           launch_split<DT, G, BLOCKED, 1, 2, 8>(a, group, st);
    } else if constexpr (G == 32)        launch_split<DT, G, BLOCKED, 1, 2, 8>(a, group, st);
}

template <int DT>
static void launch_split_dt(const GemmK64Args& a, bool blocked, int64_t group, int form, hipStream_t st)
{
    auto by_group = [&](auto blocked_tag) {
        constexpr bool B = decltype(blocked_tag)::value;
        // pre-arranged weights come with groups of 32 channels and more only
        if constexpr (!B) {
            if (group == 4)  { launch_split_g<DT, 4, B>(a, group, form, st); return; }
            if (group == 8)  { launch_split_g<DT, 8, B>(a, group, form, st); return; }
            if (group == 16) { launch_split_g<DT, 16, B>(a, group, form, st); return; }
        }
        if (group == 32) launch_split_g<DT, 32, B>(a, group, form, st);
        else                  launch_split_g<DT, 64, B>(a, group, form, st);
    };
    if (blocked) by_group(std::true_type{});
    else         by_group(std::false_type{});
}

void launch_grouped_split(const GemmK64Args& a, sasq_dtype dt, bool blocked, int64_t group, int form, hipStream_t st)
{
    if (dt == SASQ_F16) launch_split_dt<SASQ_F16>(a, blocked, group, form, st);
    else                launch_split_dt<SASQ_BF16>(a, blocked, group, form, st);
}

}  // namespace sasq

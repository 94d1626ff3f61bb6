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
#include <cmath>
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
// loop's, at any fill.  A launch's workgroups count with the runs of columns rounded up to the eight XCDs, as the XCD with the most of them
// ends the call.
// Outputs whose rows are not whole 16-byte stores cost the other kernels more, 1.5 us a round or a quarter of the workgroups below.
// Groups of 4 to 32: lines, drawn through 2700 calls of K from 64 to 8192 on weights that the caches have not seen.  us, before | here:
//   4 (one workgroup a CU for its LDS: one round):  64 x 1024 x 1024 (rows, K, columns; 256 workgroups) 15.2 | 11.3, 94 x 1920 x 664 (288)
//     25.3 | 30.5; 5 x 192 x 1424 6.4 | 5.9, shorter K 1.04 to 1.12 of the time
//   8 (one a CU as well, but eight waves of half the chain): up to 256 workgroups 0.95 to 0.4 of the time, up to 384 0.94 at K = 256 to 511 and
//     1.15 under it, up to 512 0.85 at K = 512, 0.72 at 1024, up to 700 0.87 from K = 2048 on
//   16: 1.0 of the time at 400 workgroups and K = 128, 900 and 384, 1450 and 768, 2000 and 1500; 443 x 512 x 920 (1792) 10.7 | 11.7
//     12 x 64 x 56 4.2 | 4.8, as at all sizes of a single K tile
//   32 (16 x 32 outputs): 1.0 at 950 and K = 128, 1650 and 384, 1900 to 2100 from K = 512 on; up to 512 tiles of 16 x 16 those, as a few
//     columns of 32 fill a few XCDs only: 1076 x 5312 x 24 18.0 as 16 x 16, 27.9 as 16 x 32
// Multiples of 64: the line is a number of 16 x 16 output tiles: the other kernel's K tile, with its share of a fold, costs 0.19 us + 0.24 a
// group, this one's 0.105 ns an output tile, row-major 0.14.  That is a mean over calls of some groups and whole rounds: a wave takes whole
// groups, so that few of them leave waves without any, and a round is as many workgroups as the CUs' LDS and waves hold.  Both sides' time
// is therefore estimated as well, in us, by least squares over 10700 calls of 1 to 128 groups of 64 to 1024 channels, K from 64 to 8192
// (rms error: 4 % of the other kernel's 128x128 tiles, which go two to a CU, 8 to 10 % here): another form is taken where it is 15 %
// shorter, and none where all of them are 7 % longer than the tiles.  The calls then take 0.70 of what they take on the tiles, 0.04 % of
// them more than 1.1 (0.6 % by the line alone).  A single K tile leaves nothing to split but the outputs: 16 x 64 x 256 6.1 | 4.0, 296 x 64 x
// 3144 7.3 | 8.5, in one round only.  us, before | here: one group, 128 x 512 x 2048 9.1 | 7.0, 1094 x 1024 x 384 11.2 | 15.4; two, 128 x
// 2048 x 1024 13.6 | 9.5; 290 x 6656 x 1664, groups of 128 40.7 | 45.2, 323 x 5120 x 1104, of 256 29.3 | 33.7 (16 x 32), 25.1 (32 x 32).
struct SplitTime { double call, round, k_tile, phase, k_fill; };
static const SplitTime kSplitTime[2][3] = {                          // row-major, pre-arranged; forms 1, 2, 3
    {{4.72, 0.28, 0.170, 0.166, 0.0497}, {4.53, 0.41, 0.213, 0.417, 0.1131}, {4.54, 0.19, 0.202, 0.328, 0.0810}},
    {{4.52, 0.55, 0.189, 0.193, 0.0285}, {4.44, 0.58, 0.224, 0.462, 0.0689}, {4.51, 0.49, 0.204, 0.332, 0.0407}}};

int grouped_takes_split(int64_t M, int64_t N, int64_t K, int64_t group, bool blocked)
{
    if (K % 64 != 0 || K / group > kSplitFactors) return 0;
    auto workgroups = [&](int64_t mt, int64_t nt) { return (M + 16 * mt - 1) / (16 * mt) * ((N + 128 * nt - 1) / (128 * nt) * 8); };
    const int64_t tiles16 = (M + 15) / 16 * ((N + 15) / 16), tiles = (M + 127) / 128 * ((N + 127) / 128);
    const double k = (double)K, ragged = N % 8 ? 1.25 : 1.0;
    if (group == 4)  return K >= 192 && workgroups(1, 1) <= 256 ? 1 : 0;
    if (group == 8)  return K >= 128 && tiles16 <= 512 && workgroups(1, 1) <= (K >= 2048 ? 700 : K >= 512 ? 512 : K >= 256 ? 384 : 256) ? 1 : 0;
    if (group == 16) return K >= 128 && tiles16 <= 1800 && (double)workgroups(1, 1) <= ragged * (200.0 + 1.6 * k) ? 1 : 0;
    if (group == 32) return tiles16 <= 512 ? 1 : tiles16 <= 3500 && (double)workgroups(1, 2) <= ragged * fmin(2050.0, 500.0 + 3.0 * k) ? 3 : 0;
    if (group % 64 != 0 || (K < 128 && N % 8 == 0 && workgroups(1, 2) > 1024)) return 0;
    const double kt = (double)(K / 64), per_group = (double)(group / 64), phases = (double)((K / group + 7) / 8);
    if ((double)tiles16 > (0.19 + 0.24 / per_group) / (blocked ? 0.105e-3 : 0.14e-3)) return 0;
    const double tile_kt = (blocked ? 0.201 : 0.215) + (blocked ? 0.241 : 0.221) / per_group + (blocked ? 0.040 : 0.054) * (double)(tiles < 512 ? tiles : 512) / 256.0;
    const double tile_us = 7.5 + (double)((tiles + 511) / 512) * (kt * tile_kt + (N % 8 ? 1.5 : 0.0));
    double us[4];
    for (int f = 1; f <= 3; ++f) {
        const int64_t count = f == 1 ? workgroups(1, 1) : f == 2 ? workgroups(2, 2) : workgroups(1, 2);
        const int64_t resident = f == 2 ? 512 : 1024, rest = count % resident;
        const SplitTime& t = kSplitTime[blocked][f - 1];
        auto round = [&](int64_t n) { return t.round + phases * (per_group * t.k_tile + t.phase) + kt * t.k_fill * (double)(n < 128 ? 128 : n) / 256.0; };
        us[f] = t.call + (double)(count / resident) * round(resident) + (rest ? round(rest) : 0.0);
    }
    int form = tiles16 < 256 ? 1 : !blocked && tiles16 >= 1500 ? 2 : 3;
    const int least = us[1] <= us[2] && us[1] <= us[3] ? 1 : us[2] <= us[3] ? 2 : 3;
    if (us[least] < 0.85 * us[form]) form = least;
    return us[form] > 1.07 * tile_us ? 0 : form;
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

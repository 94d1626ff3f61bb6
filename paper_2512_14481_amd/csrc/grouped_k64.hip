// Static linear with one activation factor per group of channels (Sec. 3, Eq. 3) on the 16x16x64 GEMM body: groups of 32 channels and of
// whole K tiles.
#include "sasq_device.h"
#include "gemm_tile.h"
#include "gemm_k64.h"
#include "gemm_k64_body.h"

namespace sasq {

template <int DT, int WMODE, int BM, int BN, int GMODE>
__global__ __launch_bounds__(kGemmThreads)
__attribute__((amdgpu_waves_per_eu(Tile<BM, BN>::kWavesPerSimd, Tile<BM, BN>::kWavesPerSimd)))
void gemm_k64_grouped_kernel(const int8_t* __restrict__ xq, const uint8_t* __restrict__ wq,
                             const float* __restrict__ s_g, const float* __restrict__ s_w,
                             const float* __restrict__ bias, uint16_t* __restrict__ y,
                             int32_t* __restrict__ f_out, int M, int N, int K, int tiles_m, int tiles_n, int group_tiles)
{
    __shared__ __attribute__((aligned(1024))) char lds[lds_bytes_k64<BM, BN>()];
    int tm, tn;
    if (!tile_of_block((int)blockIdx.x, tiles_m, tiles_n, tm, tn)) return;
    gemm_k64_body<DT, WMODE, BM, BN, false, GMODE>(xq, wq, s_g, s_w, bias, y, f_out, M, N, K, tm, tn, lds, group_tiles);
}

template <int DT, int WMODE, int BM, int BN>
static void launch_grouped_one(const GemmK64Args& a, int group_tiles, hipStream_t st)
{
    const int tiles_m = (int)((a.M + BM - 1) / BM), tiles_n = (int)((a.N + BN - 1) / BN);
    const int grid = ((tiles_m * tiles_n + 7) / 8) * 8;
    auto launch = [&](auto mode_tag) {
        gemm_k64_grouped_kernel<DT, WMODE, BM, BN, decltype(mode_tag)::value><<<grid, kGemmThreads, 0, st>>>(
            a.xq, a.wq, a.s, a.s_w, a.bias, a.y, a.acc_out, (int)a.M, (int)a.N, (int)a.K, tiles_m, tiles_n, group_tiles);
    };
    // 128x256 tiles, for tests, have the two general forms only
    if (group_tiles == 0) {
        if constexpr (BN == 128) launch(std::integral_constant<int, GR_HALF>{});
    } else if (group_tiles % 4 == 0) launch(std::integral_constant<int, BN == 128 ? GR_FOURS : GR_EVEN>{});
    else if (group_tiles == 2)     launch(std::integral_constant<int, BN == 128 ? GR_TWO : GR_EVEN>{});
    else if (group_tiles == 1)     launch(std::integral_constant<int, BN == 128 ? GR_ONE : GR_ODD>{});
    else if (group_tiles % 2 == 0) launch(std::integral_constant<int, GR_EVEN>{});
    else                           launch(std::integral_constant<int, GR_ODD>{});
}

template <int DT, int WMODE>
static void launch_grouped_w(const GemmK64Args& a, int tile, int group_tiles, hipStream_t st)
{
    if (tile == 1 && group_tiles != 0) launch_grouped_one<DT, WMODE, 128, 256>(a, group_tiles, st);
    else                               launch_grouped_one<DT, WMODE, 128, 128>(a, group_tiles, st);
}

template <int DT>
static void launch_grouped_dt(const GemmK64Args& a, int wmode, int tile, int group_tiles, hipStream_t st)
{
    if (wmode == KW_I8B)      launch_grouped_w<DT, KW_I8B>(a, tile, group_tiles, st);
    else if (wmode == KW_I4B) launch_grouped_w<DT, KW_I4B>(a, tile, group_tiles, st);
    else                      launch_grouped_w<DT, KW_I8>(a, tile, group_tiles, st);
}

void launch_gemm_k64_grouped(const GemmK64Args& a, sasq_dtype dt, int wmode, int tile, int group_tiles, hipStream_t st)
{
    if (dt == SASQ_F16) launch_grouped_dt<SASQ_F16>(a, wmode, tile, group_tiles, st);
    else                launch_grouped_dt<SASQ_BF16>(a, wmode, tile, group_tiles, st);
}

}  // namespace sasq

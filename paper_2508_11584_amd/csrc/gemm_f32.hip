// fp32 GEMMs (on the bf16 matrix instructions, Split3 in split3.h): instantiations and choice of tiling, plus the dtype
// dispatch.
#include <cstdlib>

#include "gemm_dma.h"
#include "kernels.h"
#include "tile_model.h"
namespace vpe {
hipError_t launch_gemm_bf16(const GemmArgs& a, int amode, hipStream_t s);
int stats_columns_bf16(const GemmArgs& a);
namespace {
// Tilings, with their time models (tile_model.h), fitted to QKV, out-projection, fc1 and fc2 of widths 384 and 768 with 145 ... 12000
// tokens and to 3x3 convolutions as in gemm_bf16.hip: 1.0 % over the measured best in the geometric mean, 14 % at most.
//   0:  64 x 64, 64-deep k-tiles, 8 waves in four k-step groups (64 x 32 wave tiles), two workgroups per CU
//   1:  64 x 128, 64-deep, 8 waves in four groups (64 x 64), one per CU
//   2:  64 x 128, 32-deep, 4 waves in two groups (64 x 64), three stages, two per CU
//   3: 128 x 128, 32-deep, 4 waves (64 x 64), two per CU
//   4:  32 x 64, 64-deep, 4 waves in four groups (32 x 64), three stages, two per CU;  5: two stages, three per CU.  A step is a chain of
//       LDS read, split and twelve products; on half as many rows twice as many workgroups walk it (us, 0 / 4: ViT-S 257 tokens
//       fc2 23.8 / 14.4, out-projection 9.3 / 6.4, fc1 10.6 / 7.8; 256 channels on 34 x 45 36 / 24)
//   6:  32 x 32, 64-deep, 4 waves in four groups, four stages, two per CU: the residual epilogue alone (GemmArgs::st_group = 32).  Half a step's products and two
//       thirds of its splits, on twice the CUs, as long as each has one tile (us, 4 / 6, out-projection and fc2: ViT-S 257 tokens, 108
//       tiles, 6.05 14.07 / 4.97 10.05, 785, 300, 6.27 14.2 / 6.93 15.2; ViT-B 257, 216, 8.69 24.8 / 6.72 17.2, 485, 384, 9.07 24.9 /
//       10.0 26.3)
// With a 32-deep tile and two groups 0 takes 30 instead of 25 us for ViT-S fc2: a group's step is a chain of LDS read, split
// and products, and the barrier and the chain's start are paid once per two steps instead of every one.
// Against the register-staged kernels on v_mfma_f32_32x32x2_f32 that were here first (us, those / now): ViT-S 1531 tokens QKV
// 20.9 / 16.0, out-projection 12.8 / 9.6, fc2 36.1 / 24.5; 3x3 convolutions 256 -> 256 on 34 x 45 55 / 24, 272 x 360 901 / 615 (188
// TFLOP/s, 6 x that on the matrix pipes: 1.13 PFLOP/s, near what the card sustains on bf16 operands; the fp32 instructions
// reach 128 there).
// Tuning aids, read when an engine is created: VPE_GEMM_TILE_F32 = 0 ... 6 forces a tiling, VPE_NO_SPLITK leaves those with
// several wave groups out.
int g_forced_tile_f32 = -1;
bool g_no_splitk_f32 = false;
constexpr TileModel kTiles[] = {
    {0, 64, 64, 2, {5.21f, 5.52f, 4.48f}, 0.52001f, 0.01302f, 0.01128f, 5.48f},
    {1, 64, 128, 1, {7.22f, 7.55f, 6.99f}, 0.00067f, 0.01890f, 0.01000f, 12.87f},
    {2, 64, 128, 2, {7.88f, 7.97f, 6.28f}, 0.54850f, 0.02167f, 0.01948f, 6.18f},
    {3, 128, 128, 2, {8.47f, 11.30f, 8.63f}, 1.93f, 0.03970f, 0.03514f, 19.75f},
    {4, 32, 64, 2, {4.02f, 3.62f, 3.04f}, 0.0f, 0.00857f, 0.00663f, 0.00f},
    {5, 32, 64, 3, {4.25f, 4.28f, 3.59f}, 0.0f, 0.00931f, 0.00685f, 0.00f},
};
constexpr TileModel kNarrow = {6, 32, 32, 2, {3.10f, 3.10f, 3.10f}, 0.0f, 0.00500f, 0.00450f, 0.00f};

hipError_t launch_f32(int kind, const GemmArgs& a, int amode, hipStream_t s, bool configure_only = false) {
    switch (kind) {
        case 0: return launch_gemm_dma<float, 64, 64, 2, 1, 2, 2, 64, 4>(a, amode, s, configure_only);
        case 1: return launch_gemm_dma<float, 128, 64, 2, 1, 2, 1, 64, 4>(a, amode, s, configure_only);
        case 2: return launch_gemm_dma<float, 128, 32, 3, 1, 2, 2, 64, 2>(a, amode, s, configure_only);
        case 4: return launch_gemm_dma<float, 64, 64, 3, 1, 1, 2, 32, 4>(a, amode, s, configure_only);
        case 5: return launch_gemm_dma<float, 64, 64, 2, 1, 1, 2, 32, 4>(a, amode, s, configure_only);
        case 6: return launch_gemm_dma<float, 32, 64, 4, 1, 1, 2, 32, 4>(a, amode, s, configure_only);
        default: return launch_gemm_dma<float, 128, 32, 2, 2, 2, 2, 128>(a, amode, s, configure_only);
    }
}
int pick_f32(const GemmArgs& a, int amode, float& best_cost) {
    int best = 3;
    best_cost = 0.0f;
    for (const TileModel& c : kTiles) {
        if (g_no_splitk_f32 && c.kind != 3) continue;
        const float cost = tile_time(c, tile_count(c, a), a.K, amode == A_CONV3 ? 0 : epilogue_weight(a));
        if (best_cost == 0.0f || cost < best_cost) { best_cost = cost; best = c.kind; }
    }
    return best;
}
}  // namespace

hipError_t launch_gemm(int dtype, const GemmArgs& a, int amode, hipStream_t s) {
    // the k loops have no remainder, and a k-tile of a convolution belongs to one tap
    if (a.K < 64 || a.K % 64 || (amode == A_CONV3 && (a.cC % 64 || a.K != 9 * a.cC))) return hipErrorInvalidValue;
    // convolution kernels carry the epilogues that convolutions have, the others all but the projection; the folded LayerNorm belongs to
    // the epilogues without a residual stream
    if (amode == A_PLAIN && (a.epi < EPI_STORE || a.epi > EPI_PATCH)) return hipErrorInvalidValue;
    if (a.ln_stats && (a.epi == EPI_RESID || a.epi == EPI_PATCH)) return hipErrorInvalidValue;
    if (amode == A_CONV3 && ((a.epi != EPI_STORE && a.epi != EPI_ROWDOT) || a.ln_stats)) return hipErrorInvalidValue;
    if (dtype) return launch_gemm_bf16(a, amode, s);
    if (a.st_group == 32) return amode == A_PLAIN && a.epi == EPI_RESID ? launch_f32(6, a, amode, s) : hipErrorInvalidValue;
    float cost;
    const int best = pick_f32(a, amode, cost);
    return launch_f32(g_forced_tile_f32 < 0 ? best : g_forced_tile_f32 == 6 ? 4 : g_forced_tile_f32, a, amode, s);
}

int stats_columns(int dtype, const GemmArgs& a) {
    if (dtype) return stats_columns_bf16(a);
    if (a.epi != EPI_RESID || (g_forced_tile_f32 >= 0 && g_forced_tile_f32 != 6) || g_no_splitk_f32) return 64;
    float cost;
    pick_f32(a, A_PLAIN, cost);
    return g_forced_tile_f32 == 6 || tile_time(kNarrow, tile_count(kNarrow, a), a.K, epilogue_weight(a)) < cost ? 32 : 64;
}

// LDS opt-in of the fp32 tilings and the tuning aids; called at engine creation, outside any stream capture.
hipError_t configure_gemm_f32() {
    const char* env = getenv("VPE_GEMM_TILE_F32");
    g_forced_tile_f32 = env && env[0] >= '0' && env[0] <= '6' && !env[1] ? env[0] - '0' : -1;
    g_no_splitk_f32 = getenv("VPE_NO_SPLITK") != nullptr;
    GemmArgs a{};
    hipError_t rc = launch_f32(kNarrow.kind, a, A_PLAIN, nullptr, true);
    for (const TileModel& c : kTiles)
        if (rc == hipSuccess) rc = launch_f32(c.kind, a, A_PLAIN, nullptr, true);
    return rc;
}
}  // namespace vpe

// fp32 GEMMs (on the bf16 matrix instructions, Split3 in split3.h): instantiations and choice of tiling, plus the dtype
// dispatch.
#include <cstdlib>

#include "gemm_dma.h"
#include "kernels.h"
namespace vpe {
hipError_t launch_gemm_bf16(const GemmArgs& a, int amode, hipStream_t s);
namespace {
// Tilings and the time model of gemm_bf16.hip (t = alpha max(r, 1) + beta r bm bn K / 1e6, r = ceil(tiles / 256) / held),
// fitted to 39 measured shapes (5-7 % rms per tiling; the pick costs 1.1 % more than the measured best in total time):
//   0:  64 x 64, 64-deep k-tiles, 8 waves in four k-step groups (64 x 32 wave tiles), two workgroups per CU
//   1:  64 x 128, 64-deep, 8 waves in four groups (64 x 64), one per CU
//   2:  64 x 128, 32-deep, 4 waves in two groups (64 x 64), three stages, two per CU
//   3: 128 x 128, 32-deep, 4 waves (64 x 64), two per CU
// With a 32-deep tile and two groups 0 takes 30 instead of 25 us for ViT-S fc2: a group's step is a chain of LDS read, split
// and products, and the barrier and the chain's start are paid once per two steps instead of every one.
// Against the register-staged kernels on v_mfma_f32_32x32x2_f32 before it (us, old / new): ViT-S 1531 tokens QKV 20.9 / 16.2,
// out-projection 12.8 / 10.2, fc1 29.0 / 24.8, fc2 36.1 / 25.0; ViT-B 1370 tokens fc2 103 / 70; 3x3 convolutions 256 -> 256 on
// 34 x 45 55 / 39, 136 x 180 307 / 207, 272 x 360 901 / 642 (180 TFLOP/s, 6 x that on the matrix pipes: 1.08 PFLOP/s, near what
// the card sustains on bf16 operands; the fp32 instructions reach 128 there).
// Tuning aids, read when an engine is created: VPE_GEMM_TILE_F32 = 0 ... 3 forces a tiling, VPE_NO_SPLITK leaves those with
// several wave groups out.
int g_forced_tile_f32 = -1;
bool g_no_splitk_f32 = false;
struct Cand { int bm, bn, held; float alpha, beta; };
constexpr Cand kCands[] = {{64, 64, 2, 5.25f, 6.325f}, {64, 128, 1, 6.75f, 2.649f}, {64, 128, 2, 7.78f, 5.883f}, {128, 128, 2, 10.01f, 5.504f}};

hipError_t launch_f32(int kind, const GemmArgs& a, int amode, hipStream_t s, bool configure_only = false) {
    switch (kind) {
        case 0: return launch_gemm_dma<float, 64, 64, 2, 1, 2, 2, 64, 4>(a, amode, s, configure_only);
        case 1: return launch_gemm_dma<float, 128, 64, 2, 1, 2, 1, 64, 4>(a, amode, s, configure_only);
        case 2: return launch_gemm_dma<float, 128, 32, 3, 1, 2, 2, 64, 2>(a, amode, s, configure_only);
        default: return launch_gemm_dma<float, 128, 32, 2, 2, 2, 2, 128>(a, amode, s, configure_only);
    }
}
}  // namespace

hipError_t launch_gemm(int dtype, const GemmArgs& a, int amode, hipStream_t s) {
    // the k loops have no remainder, and a k-tile of a convolution belongs to one tap
    if (a.K < 64 || a.K % 64 || (amode == A_CONV3 && (a.cC % 64 || a.K != 9 * a.cC))) return hipErrorInvalidValue;
    // convolution kernels carry the epilogues that convolutions have
    if (amode == A_CONV3 && ((a.epi != EPI_STORE && a.epi != EPI_ROWDOT) || a.ln_stats)) return hipErrorInvalidValue;
    if (dtype) return launch_gemm_bf16(a, amode, s);
    int best = 3;
    float best_cost = 0.0f;
    for (int k = 0; k < 4; ++k) {
        if (g_no_splitk_f32 && k != 3) continue;
        const Cand& c = kCands[k];
        const int64_t tiles = (int64_t)cdiv(a.M, c.bm) * cdiv(a.N, c.bn) * (a.nz > 1 ? a.nz : 1);
        const float r = (float)cdiv(tiles, 256) / c.held;
        const float cost = c.alpha * (r > 1.0f ? r : 1.0f) + c.beta * r * (1e-6f * c.bm * c.bn * a.K);
        if (best_cost == 0.0f || cost < best_cost) { best_cost = cost; best = k; }
    }
    return launch_f32(g_forced_tile_f32 >= 0 ? g_forced_tile_f32 : best, a, amode, s);
}

// LDS opt-in of the fp32 tilings and the tuning aids; called at engine creation, outside any stream capture.
hipError_t configure_gemm_f32() {
    const char* env = getenv("VPE_GEMM_TILE_F32");
    g_forced_tile_f32 = env && env[0] >= '0' && env[0] <= '3' && !env[1] ? env[0] - '0' : -1;
    g_no_splitk_f32 = getenv("VPE_NO_SPLITK") != nullptr;
    GemmArgs a{};
    for (int k = 0; k < 4; ++k) {
        const hipError_t rc = launch_f32(k, a, A_PLAIN, nullptr, true);
        if (rc != hipSuccess) return rc;
    }
    return hipSuccess;
}
}  // namespace vpe

// Instantiations of the bf16 direct-to-LDS GEMM and of the strip convolution.
#include <cstdlib>

#include "conv_strip.h"
#include "gemm_dma.h"
#include "kernels.h"
namespace vpe {
// Tilings, with 64-deep k-tiles (128-byte rows: a k-tile of 64-byte rows loads at half the rate, 20 against 43 bytes
// per clock and CU in a load-only probe) except where said:
//   384: 384 x 256, 32-deep k-tiles (two 64-deep stages would not fit the LDS), 8 waves (96 x 128 wave tiles), one workgroup per CU
//   256: 256 x 256, 8 waves (64 x 128), operand tiles in a ring of five units, one workgroup per CU
//    20: 128 x 128, 4 waves (64 x 64), ring, two workgroups per CU;  2: the same with 8 waves (32 x 64).  One workgroup's epilogue has
//        the other's k loop beside it; fewer operand bytes through LDS per product than any 64-row tile.  8 waves have the shorter
//        epilogue, 4 read fewer operands (us, best of the others / 2 / 20): ViT-S 4110 tokens fc1 15.4 / 14.5 / 15.9, ViT-L 2748 fc1
//        38.1 / 34.5 / 36.8, ViT-L 5496 fc2 63.1 / 67.6 / 61.7, ViT-g 4110 fc2 67.4 / 71.4 / 63.9.  (They also took the place of 256 x 128 tiles.)
//    65:  64 x 128, 4 waves (32 x 64), two stages, three workgroups per CU;  64: 64 x 64, 4 waves (32 x 32), two stages
//     5:  64 x 128, 8 waves in two groups that halve the k-steps of every k-tile (32 x 64 wave tiles), three stages
//     6:  64 x 128, 8 waves in four groups (64 x 64 wave tiles), four stages, one workgroup per CU: long k loops on up to 256 tiles
//     4:  64 x 64, 8 waves in four groups (64 x 32 wave tiles), four stages;  43: the same with 128-deep k-tiles, three stages, one
//        workgroup per CU: half the barriers
//    34:  32 x 32, 4 waves in four groups, 128-deep k-tiles, four stages, two per CU: residual epilogue only, one tile per CU (gemm_bf16.hip)
//     3:  32 x 64, 4 waves in four groups (32 x 64 wave tiles), four stages, three per CU;  33: 128-deep k-tiles, three stages, two per CU
// 3 to 6 are for problems with few tiles per CU, where a workgroup's own loop is the time: fixed cost (alpha of the time models in
// gemm_bf16.hip, by epilogue: 3.1-4.0 us for the 32-row tiles, 3.7-4.3 for 64 x 64, 5.1-5.6 for 64 x 128) and the rate at which one CU loads (40-56 bytes a clock).  us, 64 x 64 in four
// groups (4) / 32 x 64 (33): ViT-S 257 tokens QKV 5.2 / 4.9, out-projection 4.6 / 3.8, fc1 5.3 / 4.8, fc2 7.4 / 6.0; 3x3 convolution of
// 256 channels on 34 x 45 12.4 / 9.1; ViT-S detection towers there 17.4, with 43 14.9; ViT-L 1370 tokens fc2 22.6 with 5, 21.1 with 6.
// The one-per-CU shapes run in lockstep rounds, so they pay for a partly filled last round in full; which
// shape wins depends on how the tile count divides by the 256 CUs (see launch_gemm_bf16).
hipError_t launch_gemm_dma_bf16(int kind, const GemmArgs& a, int amode, hipStream_t s, bool configure_only) {
    switch (kind) {
        case 384: return launch_gemm_dma<bf16, 256, 32, 2, 4, 2, 1, 384>(a, amode, s, configure_only);
        case 256: return launch_gemm_dma<bf16, 256, 64, 2, 4, 2, 1, 256, 1, true>(a, amode, s, configure_only);
        case 20: return launch_gemm_dma<bf16, 128, 64, 2, 2, 2, 2, 128, 1, true>(a, amode, s, configure_only);
        case 65: return launch_gemm_dma<bf16, 128, 64, 2, 2, 2, 3, 64>(a, amode, s, configure_only);
        case 64: return launch_gemm_dma<bf16, 64, 64, 2, 2, 2, 4, 64>(a, amode, s, configure_only);
        case 6: return launch_gemm_dma<bf16, 128, 64, 4, 1, 2, 1, 64, 4>(a, amode, s, configure_only);
        case 5: return launch_gemm_dma<bf16, 128, 64, 3, 2, 2, 2, 64, 2>(a, amode, s, configure_only);
        case 43: return launch_gemm_dma<bf16, 64, 128, 3, 1, 2, 1, 64, 4>(a, amode, s, configure_only);
        case 4: return launch_gemm_dma<bf16, 64, 64, 4, 1, 2, 2, 64, 4>(a, amode, s, configure_only);
        case 34: return launch_gemm_dma<bf16, 32, 128, 4, 1, 1, 2, 32, 4>(a, amode, s, configure_only);
        case 33: return launch_gemm_dma<bf16, 64, 128, 3, 1, 1, 2, 32, 4>(a, amode, s, configure_only);
        case 3: return launch_gemm_dma<bf16, 64, 64, 4, 1, 1, 2, 32, 4>(a, amode, s, configure_only);
        default: return launch_gemm_dma<bf16, 128, 64, 2, 4, 2, 2, 128, 1, true>(a, amode, s, configure_only);
    }
}
// 3x3 convolution from an input strip in LDS (conv_strip.h), 96 x 128 wave tiles: 768 x 128 tiles (eight waves on top
// of each other; per 16-channel chunk a tile loads a strip of 768 + 2 (W + 1) + 2 positions and 128 x 9 weight rows: at
// W = 360, 22 % fewer bytes through the direct-to-LDS path than the 384 x 256 shape) or 384 x 256 tiles (4 x 2 waves).
// Returns the shape to use (0: none, 1: 384 x 256, 2: 768 x 128) and its tile count.  VPE_STRIP_SHAPE = 1 / 2 in the
// environment (read at engine creation) keeps to one of them.
static int g_strip_shape = 0;
static int64_t strip_tiles(const GemmArgs& a, int bm, int bn) {
    return (strip_positions(a.M / (a.cH * a.cW), a.cH, a.cW) + bm - 1) / bm * cdiv(a.N, bn) * (a.nz > 1 ? a.nz : 1);
}
int conv_strip_shape(const GemmArgs& a, bool any_size, int64_t* tiles) {
    const bool one_round_only = !any_size;
    for (int shape = 2; shape >= 1; --shape) {
        if (g_strip_shape && g_strip_shape != shape) continue;
        const bool fits = shape == 2 ? conv_strip_fits<768, 128>(a) : conv_strip_fits<384, 256>(a);
        if (!fits) continue;
        const int64_t t = shape == 2 ? strip_tiles(a, 768, 128) : strip_tiles(a, 384, 256);
        if (one_round_only && !(t > 192 && t <= 256)) continue;    // one well-filled round of the 256 CUs
        if (tiles) *tiles = t;
        return shape;
    }
    return 0;
}
hipError_t launch_conv_strip_bf16(int shape, const GemmArgs& a, hipStream_t s) {
    const bool rd = a.epi == EPI_ROWDOT;
    if (shape == 2) return rd ? launch_conv_strip<768, 128, 8, 1, 1, true>(a, s) : launch_conv_strip<768, 128, 8, 1, 1, false>(a, s);
    return rd ? launch_conv_strip<384, 256, 4, 2, 1, true>(a, s) : launch_conv_strip<384, 256, 4, 2, 1, false>(a, s);
}

// LDS opt-in (more than 64 KB) where needed; called once at engine creation.
hipError_t configure_gemm() {
    GemmArgs a{};
    const char* env = getenv("VPE_STRIP_SHAPE");
    g_strip_shape = env ? atoi(env) : 0;
    hipError_t rc = launch_conv_strip<384, 256, 4, 2, 1, true>(a, nullptr, true);
    if (rc == hipSuccess) rc = launch_conv_strip<384, 256, 4, 2, 1, false>(a, nullptr, true);
    if (rc == hipSuccess) rc = launch_conv_strip<768, 128, 8, 1, 1, true>(a, nullptr, true);
    if (rc == hipSuccess) rc = launch_conv_strip<768, 128, 8, 1, 1, false>(a, nullptr, true);
    for (int kind : {384, 256, 20, 2, 65, 64, 6, 5, 43, 4, 33, 3, 34})
        if (rc == hipSuccess) rc = launch_gemm_dma_bf16(kind, a, A_PLAIN, nullptr, true);
    return rc;
}
}  // namespace vpe

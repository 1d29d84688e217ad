// Instantiations of the large-tile direct-to-LDS GEMM.
#include <cstdlib>

#include "conv_strip.h"
#include "gemm_dma.h"
#include "kernels.h"
namespace vpe {
// Tilings, all with 64-deep k-tiles (128-byte rows: a k-tile of 64-byte rows loads at half the rate, 20 against 43 bytes
// per clock and CU in a load-only probe) but for 384, whose two 64-deep stages would not fit the LDS, and 129:
//   384: 384 x 256, 32-deep k-tiles, 8 waves (96 x 128 wave tiles), one workgroup per CU
//   256: 256 x 256, 8 waves (64 x 128), operand tiles in a ring of five units, one workgroup per CU
//   128: 256 x 128, 8 waves (64 x 64), three stages, one workgroup per CU
//   129: the same with 32-deep k-tiles, two workgroups per CU: a large convolution of 128 channels has no wider tile to fall back on,
//        and products of many rows with short k loops are mostly epilogue, which has the other workgroup's k loop beside it (us, best
//        of the others / 129: 128 -> 128 on 320x320 57.8 / 50.6, on 480x520 118.7 / 100.2; ViT-S 25000 tokens fc1 78 / 71,
//        33000 QKV 61 / 54, out-projection 37 / 34.5)
//    65:  64 x 128, 4 waves (32 x 64),  two stages, two workgroups per CU;  64: 64 x 64, 4 waves (32 x 32), two stages
//     5:  64 x 128, 8 waves in two groups that halve the k-steps of every k-tile (32 x 64 wave tiles), three stages
//     4:  64 x 64, 8 waves in four groups (64 x 32 wave tiles), four stages
// 4 and 5 are for problems with few tiles per CU, where a workgroup's own loop is the time: what it waits for is the LDS
// (operand reads + landing loads) and the loads in flight.  Two groups at 64 x 64 read 32 KB of fragments per 16 KB k-tile, four
// groups of twice as wide wave tiles 24 KB.  Against the register-staged two-group kernel that served these problems (us, its
// old / new): ViT-S 1531 tokens fc2 12.2 / 8.4, out-projection 6.8 / 5.6; 257 tokens QKV 6.1 / 5.6, fc2 11.3 / 7.5; 3x3 convolutions
// 34 x 45 256 -> 256 17.3 / 15.3, towers 24.3 / 21.2.  5 against the register-staged 64 x 128 tiles: ViT-B 1370 tokens fc2
// 30.4 / 20.8, ViT-L 1374 tokens fc2 38.2 / 27.1; against 64: 68 x 90 convolution 23.7 / 20.4.
// The one-per-CU shapes run in lockstep rounds, so they pay for a partly filled last round in full; which
// shape wins depends on how the tile count divides by the 256 CUs (see launch_gemm_bf16).
hipError_t launch_gemm_dma_bf16(int kind, const GemmArgs& a, int amode, hipStream_t s) {
    switch (kind) {
        case 4: return launch_gemm_dma<bf16, 64, 64, 4, 1, 2, 2, 64, 4>(a, amode, s);
        case 5: return launch_gemm_dma<bf16, 128, 64, 3, 2, 2, 2, 64, 2>(a, amode, s);
        case 64: return launch_gemm_dma<bf16, 64, 64, 2, 2, 2, 2, 64>(a, amode, s);
        case 65: return launch_gemm_dma<bf16, 128, 64, 2, 2, 2, 2, 64>(a, amode, s);
        case 129: return launch_gemm_dma<bf16, 128, 32, 3, 4, 2, 2>(a, amode, s);
        case 384: return launch_gemm_dma<bf16, 256, 32, 2, 4, 2, 1, 384>(a, amode, s);
        case 256: return launch_gemm_dma<bf16, 256, 64, 2, 4, 2, 1, 256, 1, true>(a, amode, s);
        default: return launch_gemm_dma<bf16, 128, 64, 3, 4, 2, 1>(a, amode, s);
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
    if (rc == hipSuccess) rc = launch_gemm_dma<bf16, 256, 32, 2, 4, 2, 1, 384>(a, A_PLAIN, nullptr, true);
    if (rc == hipSuccess) rc = launch_gemm_dma<bf16, 256, 64, 2, 4, 2, 1, 256, 1, true>(a, A_PLAIN, nullptr, true);
    if (rc == hipSuccess) rc = launch_gemm_dma<bf16, 128, 32, 3, 4, 2, 2>(a, A_PLAIN, nullptr, true);
    if (rc == hipSuccess) rc = launch_gemm_dma<bf16, 64, 64, 4, 1, 2, 2, 64, 4>(a, A_PLAIN, nullptr, true);
    if (rc == hipSuccess) rc = launch_gemm_dma<bf16, 128, 64, 3, 2, 2, 2, 64, 2>(a, A_PLAIN, nullptr, true);
    if (rc == hipSuccess) rc = launch_gemm_dma<bf16, 64, 64, 2, 2, 2, 2, 64>(a, A_PLAIN, nullptr, true);
    if (rc == hipSuccess) rc = launch_gemm_dma<bf16, 128, 64, 2, 2, 2, 2, 64>(a, A_PLAIN, nullptr, true);
    return rc != hipSuccess ? rc : launch_gemm_dma<bf16, 128, 64, 3, 4, 2, 1>(a, A_PLAIN, nullptr, true);
}
}  // namespace vpe

// The choice of tiling for the bf16 GEMMs.
#include <cstdlib>

#include "kernels.h"
#include "tile_model.h"
namespace vpe {
hipError_t launch_gemm_dma_bf16(int kind, const GemmArgs& a, int amode, hipStream_t s, bool configure_only = false);
int conv_strip_shape(const GemmArgs& a, bool any_size, int64_t* tiles);
hipError_t launch_conv_strip_bf16(int shape, const GemmArgs& a, hipStream_t s);

namespace {
// Tuning aids, read from the environment when an engine is created (configure_gemm_bf16), never per launch:
// VPE_GEMM_TILE forces a tiling, VPE_NO_SMALL_DMA leaves the two small one-group direct-to-LDS shapes out, VPE_NO_SPLITK
// the shapes with several wave groups, VPE_NO_STRIP the strip convolution, VPE_NO_ROW_SPLIT the two-launch form of a GEMM whose tile
// count is just above a whole number of rounds.
int g_forced_tile = 0;
bool g_no_small = false, g_no_splitk = false, g_no_strip = false, g_no_split = false;
// The tilings (launch_gemm_dma_bf16 describes them) with their time models (tile_model.h).
// Plain GEMMs: fitted to QKV, out-projection, fc1 and fc2 of widths 384, 768, 1024 and 1536 (SwiGLU) with 145 ... 26000 tokens: 264
// shapes, over which the picks cost 1.0 % more than the measured best in the geometric mean, more than 5 % on 23 of them and 15 % at
// most (a model without the epilogue's weight, fitted to launches of one shape with its weights in the L2s: 7 %).  Fitted before the
// residual epilogue of 2 and 65 had four rows in flight and before 384 and 5 kept their LayerNorm statistics in registers: the third
// alpha of 2 and 65 is 1.2-2.4 us high, the first of 384 2, the second of 5 0.4-1.
constexpr TileModel kPlain[] = {
    {256, 256, 256, 1, {13.69f, 16.34f, 20.09f}, 0.0f, 0.01249f, 0.00100f, 40.28f},
    {384, 384, 256, 1, {18.55f, 21.79f, 25.72f}, 0.0f, 0.02775f, 0.01000f, 52.75f},
    {20, 128, 128, 2, {6.98f, 7.83f, 10.36f}, 0.81022f, 0.00588f, 0.00532f, 4.62f},
    {2, 128, 128, 2, {5.95f, 6.71f, 10.14f}, 0.08001f, 0.00599f, 0.00589f, 5.52f},
    {65, 64, 128, 3, {5.18f, 5.82f, 9.05f}, 0.01749f, 0.00624f, 0.00429f, 0.00f},
    {64, 64, 64, 4, {4.23f, 3.98f, 4.51f}, 0.37123f, 0.00518f, 0.0f, 4.35f},
    {6, 64, 128, 1, {5.62f, 5.23f, 5.43f}, 0.00002f, 0.00002f, 0.00340f, 3.13f},
    {5, 64, 128, 2, {5.13f, 5.09f, 5.53f}, 0.20248f, 0.00369f, 0.00363f, 2.61f},
    {43, 64, 64, 1, {4.11f, 4.06f, 3.68f}, 0.00242f, 0.00002f, 0.00244f, 0.54f},
    {4, 64, 64, 2, {4.27f, 4.32f, 4.09f}, 0.37973f, 0.00231f, 0.00230f, 1.26f},
    {33, 32, 64, 2, {3.98f, 3.78f, 3.11f}, 0.0f, 0.00198f, 0.00159f, 0.00f},
    {3, 32, 64, 3, {3.22f, 3.22f, 3.28f}, 0.0f, 0.00163f, 0.0f, 5.06f},
};
// 3x3 convolutions: 95 of them (64 ... 512 channels on 12x12 ... 400x500 grids, detection towers of 384 ... 1536 channels), 0.1 % over
// the measured best (before: 20 %, most of it on tilings that were not there).
constexpr TileModel kConv[] = {
    {256, 256, 256, 1, {11.35f, 11.35f, 11.35f}, 0.50000f, 0.01716f, 0.00500f, 23.17f},
    {384, 384, 256, 1, {15.46f, 15.46f, 15.46f}, 0.50000f, 0.03182f, 0.00400f, 27.20f},
    {20, 128, 128, 2, {5.74f, 5.74f, 5.74f}, 0.0f, 0.00963f, 0.00738f, 0.00f},
    {2, 128, 128, 2, {4.55f, 4.55f, 4.55f}, 0.0f, 0.00839f, 0.00683f, 3.48f},
    {65, 64, 128, 3, {4.39f, 4.39f, 4.39f}, 0.11007f, 0.00848f, 0.00402f, 1.50f},
    {64, 64, 64, 4, {3.68f, 3.68f, 3.68f}, 0.0f, 0.00735f, 0.00192f, 1.83f},
    {6, 64, 128, 1, {4.65f, 4.65f, 4.65f}, 0.50000f, 0.0f, 0.00461f, 0.00f},
    {5, 64, 128, 2, {4.38f, 4.38f, 4.38f}, 0.18948f, 0.00471f, 0.00401f, 1.39f},
    {43, 64, 64, 1, {3.75f, 3.75f, 3.75f}, 0.50000f, 0.00307f, 0.00100f, 0.00f},
    {4, 64, 64, 2, {3.73f, 3.73f, 3.73f}, 0.14808f, 0.00379f, 0.00311f, 0.03f},
    {33, 32, 64, 2, {3.59f, 3.59f, 3.59f}, 0.0f, 0.00225f, 0.00179f, 0.00f},
    {3, 32, 64, 3, {3.60f, 3.60f, 3.60f}, 0.0f, 0.00242f, 0.00188f, 0.00f},
};
// 32 x 32 tiles, for the residual epilogue alone (GemmArgs::st_group = 32): faster than 33 exactly where a CU has one of them (us, 33 / 34,
// out-projection and fc2: ViT-S 257 tokens, 108 tiles, 3.69 5.41 / 3.41 4.52, 485, 192, 3.76 5.48 / 3.49 4.63, 785, 300, 3.86 5.66 / 4.02 6.52;
// ViT-B 257, 216, 4.42 8.74 / 3.98 7.31; ViT-L 261, 288, 4.87 10.33 / 5.46 13.71; launches with their weights in the L2s, in a frame
// both take longer).
constexpr TileModel kNarrow = {34, 32, 32, 2, {3.10f, 3.10f, 3.10f}, 0.0f, 0.00105f, 0.00115f, 1.50f};
// What a convolution's tile of up to 64 rows has to be faster by, alone, to be taken over a larger one, whatever else runs (the launcher
// does not know): a head's convolutions run beside encoder kernels, where operand traffic costs more than the time alone shows (ViT-S 476x630 frames of two lanes:
// 609 us without this, 591 with it; 256 -> 256 on 136x180 takes 37.7 us with 64 x 128 tiles and 40.5 with 128 x 128).
constexpr float kConvShared = 1.12f;
}  // namespace

static bool narrow_fits(const GemmArgs& a) { return a.epi == EPI_RESID && a.m_begin == 0 && a.K % 128 == 0; }

// Can (and, with the tuning aids, may) a tiling take this problem?
static bool admissible(const TileModel& c, const GemmArgs& a, int amode) {
    // k-tiles of 128 need whole ones (in a convolution within a tap); where there are, the 64-deep 32 x 64 shape is never faster
    const bool deep = amode == A_CONV3 ? a.cC % 128 == 0 : a.K % 128 == 0;
    if (g_no_small && (c.kind == 64 || c.kind == 65)) return false;
    if (g_no_splitk && c.bm <= 64 && c.kind != 64 && c.kind != 65) return false;
    if ((c.kind == 33 || c.kind == 43) && !deep) return false;
    return !(c.kind == 3 && deep);
}

// What `tiles` tiles of a tiling count as, in us: a whole launch, a leading part and a tail by the same measure.
static float tile_cost(const TileModel& c, const GemmArgs& a, int amode, int64_t tiles) {
    return tile_time(c, tiles, a.K, epilogue_weight(a)) * (amode == A_CONV3 && c.bm <= 64 ? kConvShared : 1.0f);
}

// The model's pick for rows m_begin .. M - 1 of `a` and its predicted time in us.
template <int NC>
static int pick_tile(const TileModel (&cands)[NC], const GemmArgs& a, int amode, float& best_cost) {
    int best = 2;
    best_cost = 0.0f;
    for (const TileModel& c : cands) {
        if (!admissible(c, a, amode)) continue;
        const float cost = tile_cost(c, a, amode, tile_count(c, a));
        if (best_cost == 0.0f || cost < best_cost) { best_cost = cost; best = c.kind; }
    }
    return best;
}

template <int NC>
static GemmPlan plan_among(const TileModel (&cands)[NC], const GemmArgs& a, int amode) {
    float cost;
    GemmPlan plan{0, 0, pick_tile(cands, a, amode, cost)};
    // The one-per-CU tiles run in lockstep rounds of 256 and pay for a partly filled last round in full (ViT-g, 8
    // views: fc2 and the out-projection have 43 x 6 = 258 tiles of 256 x 256, QKV 774).  Two launches instead: whole
    // rounds of the large tile over the leading rows, then the remaining rows with whatever the model picks for them.
    if (g_forced_tile == 0 && !g_no_split && a.nz <= 1 && a.m_begin == 0) {
        for (const TileModel& c : cands) {
            if (c.held != 1 || !admissible(c, a, amode)) continue;
            const int tn = cdiv(a.N, c.bn), tm = cdiv(a.M, c.bm);
            const int64_t tiles = (int64_t)tm * tn;
            const int rounds = (int)(tiles / 256);
            if (rounds < 1 || tiles % 256 == 0) continue;
            const int tm_main = rounds * 256 / tn;              // whole tile rows in `rounds` rounds
            if (tm_main < 1 || tm_main >= tm) continue;
            const float main_cost = tile_cost(c, a, amode, (int64_t)tm_main * tn);
            GemmArgs tail = a;
            tail.m_begin = tm_main * c.bm;
            float tail_cost;
            const int tail_kind = pick_tile(cands, tail, amode, tail_cost);
            if (main_cost + tail_cost < 0.93f * cost) {         // a second launch costs a few us the model does not see
                cost = main_cost + tail_cost;
                plan = GemmPlan{c.kind, tail.m_begin, tail_kind};
            }
        }
    }
    return plan;
}

GemmPlan plan_gemm_bf16(const GemmArgs& a, int amode) { return amode == A_CONV3 ? plan_among(kConv, a, amode) : plan_among(kPlain, a, amode); }

static hipError_t launch_picked(const GemmArgs& a, int amode, hipStream_t s, int best);

hipError_t launch_gemm_bf16(const GemmArgs& a, int amode, hipStream_t s) {
    if (a.st_group == 32) return amode == A_PLAIN && narrow_fits(a) ? launch_gemm_dma_bf16(34, a, amode, s) : hipErrorInvalidValue;
    const GemmPlan plan = plan_gemm_bf16(a, amode);
    if (!plan.lead_kind) return launch_picked(a, amode, s, plan.kind);
    GemmArgs lead = a, tail = a;
    lead.M = tail.m_begin = plan.lead_rows;
    const hipError_t rc = launch_gemm_dma_bf16(plan.lead_kind, lead, amode, s);
    return rc != hipSuccess ? rc : launch_picked(tail, amode, s, plan.kind);
}

int stats_columns_bf16(const GemmArgs& a) {
    if (!narrow_fits(a) || (g_forced_tile && g_forced_tile != 34) || g_no_splitk) return 64;
    float cost = 0.0f;
    pick_tile(kPlain, a, A_PLAIN, cost);
    return g_forced_tile == 34 || tile_cost(kNarrow, a, A_PLAIN, tile_count(kNarrow, a)) < cost ? 32 : 64;
}

static hipError_t launch_picked(const GemmArgs& a, int amode, hipStream_t s, int best) {
    const int forced = g_forced_tile;
    // 3x3 convolutions: the strip kernel (conv_strip.h) where its 384 x 256 tiles make one well-filled round of the
    // 256 CUs (measured on 272 x 360 x 256 -> 256, 256 tiles: 128 against 144 us for the generic 384 x 256 kernel on the
    // same box; with several rounds -- 4 x 296 x 296: 477 against 443 us -- the generic kernels stay ahead).
    // VPE_GEMM_TILE=9 forces it wherever it applies, any other forced tile switches it off.
    if (a.m_begin == 0 && amode == A_CONV3 && (forced == 9 || (forced == 0 && !g_no_strip)) && a.epi != EPI_SWIGLU) {
        const int shape = conv_strip_shape(a, forced == 9, nullptr);
        if (shape) return launch_conv_strip_bf16(shape, a, s);
    }
    if (forced && forced != 9) {
        const bool deep = amode == A_CONV3 ? a.cC % 128 == 0 : a.K % 128 == 0;
        best = forced == 33 && !deep ? 3 : forced == 43 && !deep ? 4 : forced == 34 ? (deep ? 33 : 3) : forced;
    }
    return launch_gemm_dma_bf16(best, a, amode, s);
}

// Reads the tuning aids; called at engine creation, outside any stream capture.
hipError_t configure_gemm_bf16() {
    const char* env = getenv("VPE_GEMM_TILE");
    g_forced_tile = 0;
    for (int kind : {384, 256, 20, 2, 65, 64, 6, 5, 43, 4, 33, 3, 34, 9}) if (env && atoi(env) == kind) g_forced_tile = kind;      // (anything else: no tile forced)
    if (env && (atoi(env) == 128 || atoi(env) == 129)) g_forced_tile = 2;                     // (the 256 x 128 shapes that 128 x 128 replaced)
    g_no_small = getenv("VPE_NO_SMALL_DMA") != nullptr;
    g_no_splitk = getenv("VPE_NO_SPLITK") != nullptr;
    g_no_strip = getenv("VPE_NO_STRIP") != nullptr;
    g_no_split = getenv("VPE_NO_ROW_SPLIT") != nullptr;
    return hipSuccess;
}
}  // namespace vpe

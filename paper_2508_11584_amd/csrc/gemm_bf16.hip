// The choice of tiling for the bf16 GEMMs.
#include <cstdlib>

#include "kernels.h"
namespace vpe {
hipError_t launch_gemm_dma_bf16(int bn, const GemmArgs& a, int amode, hipStream_t s);
int conv_strip_shape(const GemmArgs& a, bool any_size, int64_t* tiles);
hipError_t launch_conv_strip_bf16(int shape, const GemmArgs& a, hipStream_t s);

namespace {
// Candidate tilings: tile, workgroups a CU holds at once, and the two coefficients of the time model
//     t [us] = alpha * max(r, 1) + beta * r * (bm * bn * K / 1e6),     r = ceil(tiles / 256) / held,
// r being the number of "rounds" on the busiest of the 256 CUs (it gets ceil(tiles / 256) tiles and works on
// `held` of them at a time); alpha is the cost a workgroup pays whatever its size (first loads, epilogue), not
// discounted on a partly filled chip.  Fitted (relative least squares) to 66 measured shapes on MI355X with random bf16 data and
// the layers' own epilogues: the QKV / proj / fc1 / fc2 GEMMs of ViT-S (257, 900, 1531, 4097, 12000 tokens), -B (1370, 1572, 4110),
// -L (300, 1374, 2748, 5496) and -g (1374, 4122, 10992), and 3x3 convolutions at 34x45 ... 136x180 grids.
// Over 264 shapes of those layers (17 token counts, 145 to 10992) the picks cost 1.1 % more than the measured best in the geometric
// mean, more than 5 % on 24 of them and 14 % at most.  Predictions near the best are within 4-12 % rms, except that one
// alpha for all epilogues is 16-22 % low for the one-per-CU tiles with GELU or the residual epilogue (ViT-L x 4 fc1 on
// 384 x 256: 57 us predicted, 73 measured).  Coefficients per epilogue predict those to 8 % and pick within 0.4 % of the
// best, and frames got slower with them (ViT-g, 663 tokens: 4404 -> 4638 us with QKV and fc1 on 64 x 128; ViT-L x 4 on two lanes
// 6370 -> 6680 with fc2 on 64 x 128 in two groups): a shape timed over and over has its weights in the caches and the chip to itself.
// Tuning aids, read from the environment when an engine is created (configure_gemm_bf16), never per launch:
// VPE_GEMM_TILE forces a tiling, VPE_NO_SMALL_DMA leaves the two small one-group direct-to-LDS shapes out, VPE_NO_SPLITK
// the shapes with several wave groups, VPE_NO_STRIP the strip convolution, VPE_NO_ROW_SPLIT the two-launch form of a GEMM whose tile
// count is just above a whole number of rounds.
int g_forced_tile = 0;
bool g_no_small = false, g_no_splitk = false, g_no_strip = false, g_no_split = false;
struct Cand { int kind, bm, bn, held; float alpha, beta; };
constexpr Cand kCands[] = {
    {256, 256, 256, 1, 15.83f, 0.300f},   // direct-to-LDS (launch_gemm_dma_bf16 describes the shapes)
    {384, 384, 256, 1, 22.58f, 0.344f},
    {128, 256, 128, 1, 10.33f, 0.406f},
    {129, 256, 128, 2, 12.91f, 0.924f},   // (fitted to 158 shapes of 40 ... 33000 tokens, times 0.98: picked from 20000 on)
    {65, 64, 128, 3, 6.58f, 2.001f},
    {64, 64, 64, 4, 5.28f, 3.287f},
    {5, 64, 128, 2, 5.87f, 1.222f},
    {4, 64, 64, 2, 4.79f, 1.411f},
};
// 3x3 convolutions have long k loops, where a CU's rounds are told apart better than by r: with q = ceil(tiles / 256) tiles on the
// busiest CU, floor(q / held) full rounds and one of the q % held tiles that are left, a round of n tiles taking
//     t(n) [us] = alpha + next (n - 1) + K max(chain, rate n)
// (next: what a further workgroup adds to the fixed time; chain: one workgroup's own time per k; rate: the CU's time per k and tile
// when its workgroups share it).  Fitted to 174 convolutions (64-512 channels on 16x16 ... 600x600 grids, detection towers of
// 384-1536 channels), 3-8 % rms per tiling.  Under the model above 64 x 64 tiles in four groups were taken for 257-768
// tiles, up to 31 % slower than 64 x 128 in two (us): 512 -> 512 on 68x90 64.8 / 52.3, 256 -> 256 on 96x96 34.7 / 26.9, ViT-S
// towers on 74x74 49.5 / 38.0, ViT-g towers there 171 / 126; the picks cost 2.7 % over the measured best, now 0.2 %.
struct ConvCand { int kind, bm, bn, held; float alpha, next, chain, rate; };
constexpr ConvCand kConvCands[] = {
    {256, 256, 256, 1, 19.79f, 0.0f, 0.02239f, 0.0f},
    {384, 384, 256, 1, 24.60f, 0.0f, 0.03818f, 0.0f},
    {128, 256, 128, 1, 10.87f, 0.0f, 0.01573f, 0.0f},
    {129, 256, 128, 2, 10.50f, 2.24f, 0.01760f, 0.01570f},
    {65, 64, 128, 3, 4.50f, 0.56f, 0.00829f, 0.00535f},
    {64, 64, 64, 4, 4.88f, 0.0f, 0.00585f, 0.00352f},
    {5, 64, 128, 2, 5.33f, 1.59f, 0.00617f, 0.00453f},
    {4, 64, 64, 4, 4.68f, 1.54f, 0.00458f, 0.00362f},
};
// What a tile of 64 rows has to be faster by, alone, to be taken over one of 256 or more: a head's
// convolutions run beside encoder kernels, where operand traffic costs more than the time alone shows.  256 -> 256 on
// 136x180: 46.6 us with 64 x 128 tiles, 50.4 with 256 x 128, but a ViT-S 476x630 frame takes 856 us with the first and 848 with
// the second, and 631 and 620 as a stream of two lanes.
constexpr float kConvShared = 1.12f;

float predicted(const Cand& c, int64_t tiles, int K) {
    const float r = (float)cdiv(tiles, 256) / c.held;
    return c.alpha * (r > 1.0f ? r : 1.0f) + c.beta * r * (1e-6f * c.bm * c.bn * K);
}
float predicted(const ConvCand& c, int64_t tiles, int K) {
    auto round = [&](int n) { return n == 0 ? 0.0f : c.alpha + c.next * (n - 1) + K * (c.chain > c.rate * n ? c.chain : c.rate * n); };
    const int q = cdiv(tiles, 256);
    return (c.bm == 64 ? kConvShared : 1.0f) * ((float)(q / c.held) * round(c.held) + round(q % c.held));
}
}  // namespace

// The model's pick for rows m_begin .. M - 1 of `a` and its predicted time in us.
template <typename C, int NC>
static int pick_tile(const C (&cands)[NC], const GemmArgs& a, float& best_cost) {
    int best = 128;
    best_cost = 0.0f;
    const int rows = a.M - a.m_begin;
    for (const C& c : cands) {
        if (g_no_small && (c.kind == 64 || c.kind == 65)) continue;
        if (g_no_splitk && (c.kind == 4 || c.kind == 5)) continue;
        // 64-column tiles can do SwiGLU (gate and partner columns meet in the block-level epilogue) but were slower wherever they were
        // timed (ViT-g fc1, us, 64 x 64 in one and four groups against 64 x 128: 400 tokens 23.5, 27.0 / 20.4, 900 45.4, 52.2 / 41.1)
        if (c.bn == 64 && a.epi == EPI_SWIGLU) continue;
        const int64_t tiles = (int64_t)cdiv(rows, c.bm) * cdiv(a.N, c.bn) * (a.nz > 1 ? a.nz : 1);
        // Two workgroups of 64 x 64 with four wave groups share a CU like four of one group do; with a short k loop that is
        // where their partial sums cost more than the groups gain (432 tiles at K = 384: 8.2 against 7.7 us, 264 at K = 768:
        // 9.7 against 9.3; 352 at K = 1024: 11.4 against 11.3, 264 at K = 3072: 23.2 against 26.3)
        if (c.kind == 4 && tiles > 256 && a.K < 1024) continue;
        const float cost = predicted(c, tiles, a.K);
        if (best_cost == 0.0f || cost < best_cost) { best_cost = cost; best = c.kind; }
    }
    return best;
}

static hipError_t launch_picked(const GemmArgs& a, int amode, hipStream_t s, int best);

template <typename C, int NC>
static hipError_t launch_chosen(const C (&cands)[NC], const GemmArgs& a, int amode, hipStream_t s) {
    float whole_cost;
    const int whole = pick_tile(cands, a, whole_cost);
    // The one-per-CU tiles run in lockstep rounds of 256 and pay for a partly filled last round in full (ViT-g, 8
    // views: fc2 and the out-projection have 43 x 6 = 258 tiles of 256 x 256, QKV 774).  Two launches instead: whole
    // rounds of the large tile over the leading rows, then the remaining rows with whatever the model picks for them.
    if (g_forced_tile == 0 && !g_no_split && a.nz <= 1 && a.m_begin == 0) {
        float split_cost = whole_cost;
        int split_kind = 0, split_rows = 0;
        for (const C& c : cands) {
            if (c.held != 1) continue;
            const int tn = cdiv(a.N, c.bn), tm = cdiv(a.M, c.bm);
            const int64_t tiles = (int64_t)tm * tn;
            const int rounds = (int)(tiles / 256);
            if (rounds < 1 || tiles % 256 == 0) continue;
            const int tm_main = rounds * 256 / tn;              // whole tile rows in `rounds` rounds
            if (tm_main < 1 || tm_main >= tm) continue;
            const float main_cost = predicted(c, (int64_t)tm_main * tn, a.K);
            GemmArgs tail = a;
            tail.m_begin = tm_main * c.bm;
            float tail_cost;
            pick_tile(cands, tail, tail_cost);
            if (main_cost + tail_cost < 0.93f * split_cost) {   // a second launch costs a few us the model does not see
                split_cost = main_cost + tail_cost;
                split_kind = c.kind;
                split_rows = tm_main * c.bm;
            }
        }
        if (split_kind) {
            GemmArgs main = a, tail = a;
            main.M = split_rows;
            tail.m_begin = split_rows;
            hipError_t rc = launch_gemm_dma_bf16(split_kind, main, amode, s);
            if (rc != hipSuccess) return rc;
            float unused;
            return launch_picked(tail, amode, s, pick_tile(cands, tail, unused));
        }
    }
    return launch_picked(a, amode, s, whole);
}

hipError_t launch_gemm_bf16(const GemmArgs& a, int amode, hipStream_t s) {
    return amode == A_CONV3 ? launch_chosen(kConvCands, a, amode, s) : launch_chosen(kCands, a, amode, s);
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
    if (forced == 384 || forced == 256 || forced == 128 || forced == 129 || forced == 65 || forced == 5) best = forced;
    if (forced == 4) best = a.epi == EPI_SWIGLU ? 5 : 4;
    if (forced == 64) best = a.epi == EPI_SWIGLU ? 65 : 64;
    return launch_gemm_dma_bf16(best, a, amode, s);
}

// Reads the tuning aids; called at engine creation, outside any stream capture.
hipError_t configure_gemm_bf16() {
    const char* env = getenv("VPE_GEMM_TILE");
    g_forced_tile = 0;
    for (int kind : {384, 256, 128, 129, 65, 64, 5, 4, 9}) if (env && atoi(env) == kind) g_forced_tile = kind;      // (anything else: no tile forced)
    g_no_small = getenv("VPE_NO_SMALL_DMA") != nullptr;
    g_no_splitk = getenv("VPE_NO_SPLITK") != nullptr;
    g_no_strip = getenv("VPE_NO_STRIP") != nullptr;
    g_no_split = getenv("VPE_NO_ROW_SPLIT") != nullptr;
    return hipSuccess;
}
}  // namespace vpe

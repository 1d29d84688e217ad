// Time model of the GEMM tilings (host side): what the launchers choose a tiling by.
#pragma once
#include "gemm.h"

namespace vpe {

// With q = ceil(tiles / 256) tiles on the busiest of the 256 CUs, which works on `held` of them at a time, a problem takes
// q / held full rounds and one of the q % held tiles that are left; a round of n tiles takes
//     t(n) [us] = alpha + next (n - 1) + K max(chain, rate n)
// (alpha: first loads and epilogue, by the epilogue's weight; next: what a further workgroup adds to them; chain: one
// workgroup's own time per k; rate: the CU's time per k and tile when its workgroups share it), and all of them
// together take shared * tiles * K * 1e-6 at what the CUs share (L2 and memory side).
// The coefficients are fitted, per tiling, to times of the kernels on MI355X with random data, the layers' own epilogues and weights
// that change from launch to launch (a model's weights do not stay in the L2s), tilings within some 15 % of
// a shape's best weighing most.
struct TileModel {
    int kind, bm, bn, held;
    float alpha[3], next, chain, rate, shared;
};

// Weight of an epilogue: results only (QKV, plain and ReLU stores), GELU and SwiGLU, the residual stream (fp32 read and written).
static inline int epilogue_weight(const GemmArgs& a) {
    if (a.epi == EPI_RESID || a.epi == EPI_PATCH) return 2;
    return a.epi == EPI_SWIGLU || a.act == ACT_GELU ? 1 : 0;
}

static inline float tile_time(const TileModel& c, int64_t tiles, int K, int weight) {
    auto round = [&](int n) { return n == 0 ? 0.0f : c.alpha[weight] + c.next * (n - 1) + K * (c.chain > c.rate * n ? c.chain : c.rate * n); };
    const int q = (int)((tiles + 255) / 256);
    return (float)(q / c.held) * round(c.held) + round(q % c.held) + c.shared * (float)tiles * (1e-6f * K);
}

static inline int64_t tile_count(const TileModel& c, const GemmArgs& a) {
    return (int64_t)cdiv(a.M - a.m_begin, c.bm) * cdiv(a.N, c.bn) * (a.nz > 1 ? a.nz : 1);
}

}  // namespace vpe

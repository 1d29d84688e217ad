// MFMA GEMM for gfx950 with direct global->LDS loads (global_load_lds_dwordx4).
//
// Operands go from global memory straight into the swizzled LDS tile (no VGPR staging, no ds_write: on MI355X register
// staging stops at 750-840 TFLOP/s with 128 x 128 tiles, its LDS write path and load issue cannot keep four MFMA pipes fed),
// later k-tiles' loads are in flight during the current tile's MFMAs, the LDS reads of k-step s + 1 are interleaved with the
// MFMAs of step s (sched_group_barrier), and the accumulators leave through LDS with 16-byte coalesced stores.
// A CU draws at most 56 bytes per clock through this path (load-only probe, 128-byte rows, operands in L2; 40-45 from
// the memory-side cache with two 32 KB stages in flight).
//
// bf16, and fp32 on the bf16 instructions (Split3).  A modes and epilogues: gemm.h.
#pragma once
#include <type_traits>

#include "gemm.h"
#include "split3.h"

namespace vpe {

#define VPE_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define VPE_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

// s_waitcnt immediate that waits for vmcnt <= n only (gfx9 encoding: vmcnt in bits 3:0 and 15:14,
// expcnt 6:4 and lgkmcnt 11:8 left at their maxima)
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// Workgroup barrier of the load pipelines: this wave's LDS reads are done (lgkmcnt 0) and all but its N youngest
// direct-to-LDS loads have landed, then s_barrier.  __syncthreads() would not do: its fence waits for vmcnt(0), so every
// barrier drains the loads still in flight and any number of LDS stages works like two (measured: 8 waves streaming
// 32 KB stages of 128-byte rows, operands in the memory-side cache: 1360 clocks a stage with __syncthreads at one, two or
// three stages in flight; 794 / 715 at two / three without the drain).
template <int N>
__device__ __forceinline__ void pipeline_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(N) & ~0x0F00);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Row index of a tile row in the output.  PADDED (the strip convolution): tile rows run over the padded pixel index
// ((image (H + 1) + y + 1) (W + 1) + x: one zero column behind every image row, one zero row between images); pad
// positions have no output (returned as a row past M).
template <bool PADDED>
__device__ __forceinline__ int epilogue_row(const GemmArgs& p, int r) {
    if (!PADDED) return r;
    const int wp = p.cW + 1, hp = p.cH + 1;
    const int line = r / wp, x = r - line * wp;
    const int img = line / hp, y = line - img * hp - 1;
    return (x < p.cW && y >= 0) ? (img * p.cH + y) * p.cW + x : 0x7fffffff;
}

// The same map for tile rows visited in increasing order with a fixed step: one pair of divisions at the start, then
// additions and compares (a ROWDOT lane visits every 64 / CG-th row of its wave tile).
template <bool PADDED>
struct EpilogueRows {
    int r, x, y, img, wp, hp;          // tile row; PADDED: its column, line within the image's H + 1 lines, image
    __device__ __forceinline__ EpilogueRows(const GemmArgs& p, int r0) : r(r0), x(0), y(0), img(0), wp(p.cW + 1), hp(p.cH + 1) {
        if (PADDED) {
            const int line = r0 / wp;
            x = r0 - line * wp;
            img = line / hp;
            y = line - img * hp;
        }
    }
    __device__ __forceinline__ int row(const GemmArgs& p) const {
        if (!PADDED) return r;
        return (x < p.cW && y >= 1) ? (img * p.cH + y - 1) * p.cW + x : 0x7fffffff;
    }
    __device__ __forceinline__ void advance(int step) {
        r += step;
        if (PADDED) {
            x += step;
            while (x >= wp) {
                x -= wp;
                if (++y == hp) { y = 0; ++img; }
            }
        }
    }
};

// Epilogue of the wave-tiled kernels: each wave stages its MI x NI accumulator blocks 32 rows at a time in its own
// 32 x WN fp32 block of LDS (the operand buffers are free by now; the caller has put a barrier behind its last
// read of them) and leaves with 8-column chunks per lane.  The MFMAs took the W operand first: a lane holds one row of
// each block (row lane % 32, columns 8 (v / 4) + 4 (lane / 32) + v % 4 of every 32), so a block is staged with 16-byte writes, a quarter of
// the instructions of a layout with a column per lane, and the folded LayerNorm is applied where the chunks are read.
// lnrow: LDS for (mean, rstd) per tile row.  LN: a folded LayerNorm is possible (convolutions have none).
template <typename T, int EPI, int BM, int MI, int NI, int WM, int WN, bool LN, bool PADDED = false>
__device__ __forceinline__ void wave_tile_epilogue(const GemmArgs& p, f32x16 (&acc)[MI][NI], char* smem, float* lnrow,
                                                   int wave, int wm, int wn, int tid, int m0, int n0) {
    const int lane = tid & 63, g = lane >> 5, li = lane & 31;
    float* sC = reinterpret_cast<float*>(smem) + wave * (32 * WN);
    const int wrow0 = m0 + wm * WM, wcol0 = n0 + wn * WN;
    const bool has_ln = LN && EPI != EPI_RESID && EPI != EPI_PATCH && p.ln_stats;
    // 4-column groups of a row are exchanged by the row: 16 consecutive rows writing one group, and the four 8-row blocks
    // that a transposed value read takes at once, fall on different banks
    auto at = [&](int row, int col) { return row * WN + (col ^ ((((row & 15) ^ ((row >> 3) << 2)) & 15) << 2)); };
    auto stage = [&](auto I) {
        constexpr int i = decltype(I)::value;
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4*>(sC + at(li, j * 32 + 8 * q + 4 * g)) =
                    f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    };
    auto chunk8 = [&](int row, int col, float* v) {
        const f32x4 lo = *reinterpret_cast<const f32x4*>(sC + at(row, col)), hi = *reinterpret_cast<const f32x4*>(sC + at(row, col + 4));
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = lo[e]; v[4 + e] = hi[e]; }
    };
    auto row_stats = [&](int row) { return *reinterpret_cast<const f32x2*>(lnrow + 2 * row); };     // (of a tile row)
    // The row-chunk paths: a lane keeps one 8-column chunk (64 is a multiple of the chunks per row) for all its rows
    // Four rows at a time (one at a time cost 128 x 128 tiles of eight waves 1.2-2.1 us a launch, 64 x 128 ones 1.2-2.2: ViT-L 1370 tokens
    // out-projection 14.9 / 12.8 and 11.7 / 10.3; their k loops need more registers than the rows do).  96 x 128 wave
    // tiles have registers for two, and none for the columns while all blocks wait.
    constexpr int CG = WN / 8, ITS = 32 * CG / 64, NB = MI * NI >= 12 ? 2 : ITS < 4 ? ITS : 4;
    static_assert(64 % CG == 0 && ITS % NB == 0, "a lane keeps its column chunk");
    // One pass per 32-row block of the wave tile; the block index is a compile-time constant of each pass (a loop over the
    // blocks turns the accumulators into an indexed array in scratch, or spills them).
    // (rows without operands of their own go one by one: nothing to wait for, and the short loop keeps its code small)
    const bool batched = EPI == EPI_RESID || EPI == EPI_PATCH || (EPI == EPI_STORE && p.add1);
    auto pass = [&](int i) {
        const int rblk = wrow0 + i * 32, tblk = wm * WM + i * 32;
        if constexpr (EPI == EPI_SWIGLU) {
            // groups of 64 physical columns: 32 gate columns, then their 32 linear partners
            constexpr int GG = WN / 16;                  // 8-wide gate chunks per row
            T* out = reinterpret_cast<T*>(p.out);
            const int gg = lane % GG, grp = gg >> 2, j0 = (gg & 3) * 8, ca = wcol0 + grp * 64 + j0;
            if (ca + 40 <= p.N) {
                const EpiCols ka = epilogue_cols<EPI>(p, ca), kb = epilogue_cols<EPI>(p, ca + 32);
#pragma unroll 1
                for (int rr = lane / GG; rr < 32; rr += 64 / GG) {
                    const int r = epilogue_row<PADDED>(p, rblk + rr);
                    float va[8], vb[8], h[8];
                    chunk8(rr, grp * 64 + j0, va);
                    chunk8(rr, grp * 64 + j0 + 32, vb);
                    if (has_ln) {
                        const f32x2 st = row_stats(tblk + rr);
                        ln_apply(st, ka.g0, ka.g1, va);
                        ln_apply(st, kb.g0, kb.g1, vb);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        h[e] = swiglu_for<T>(va[e] + ka.b0[e], vb[e] + kb.b0[e]);
                        h[4 + e] = swiglu_for<T>(va[4 + e] + ka.b1[e], vb[4 + e] + kb.b1[e]);
                    }
                    if (r < p.M) store8(out + (int64_t)r * p.ldo + (ca >> 6) * 32 + j0, h);
                }
            }
        } else if (EPI == EPI_QKV && wcol0 >= 2 * p.dim) {
            // value columns, written transposed: one column and 8 consecutive tokens per lane.  All rows and columns of the QKV
            // epilogue are written out and the biases fetched first: it has no arithmetic to hide a round's LDS and
            // store latency behind (over 66 QKV shapes 256 x 256 and 384 x 256 tiles 6 % faster, 64 x 128 3 %)
            T* vt = reinterpret_cast<T*>(p.out2);
            float bias[WN / 16], cs[WN / 16];
#pragma unroll
            for (int n = 0; n < WN / 16; ++n) {
                const int c = wcol0 + (lane >> 2) + 16 * n;
                bias[n] = c < p.N ? p.bias[c] : 0.0f;
                cs[n] = has_ln && c < p.N ? p.ln_colsum[c] : 0.0f;
            }
            const int rr = (lane & 3) * 8, r = epilogue_row<PADDED>(p, rblk + rr);      // 4 lanes = 32 consecutive tokens of a column
            f32x2 st[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) st[k] = has_ln ? row_stats(tblk + rr + k) : f32x2{0.0f, 1.0f};
#pragma unroll
            for (int n = 0; n < WN / 16; ++n) {
                const int cc = (lane >> 2) + 16 * n;
                if (r < p.M && wcol0 + cc < p.N) {
                    float v[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) v[k] = st[k][1] * (sC[at(rr + k, cc)] - st[k][0] * cs[n]) + bias[n];
                    store_tokens8<T>(p, vt, r, wcol0 + cc - 2 * p.dim, v);
                }
            }
        } else if constexpr (EPI == EPI_QKV) {
            const EpiCols cols = epilogue_cols<EPI>(p, wcol0 + (lane % CG) * 8);
            const float f = cols.c < p.dim ? p.q_scale : 1.0f;
#pragma unroll
            for (int n = 0; n < ITS; ++n) {
                const int rr = lane / CG + n * (64 / CG), r = epilogue_row<PADDED>(p, rblk + rr);
                float v[8];
                chunk8(rr, (lane % CG) * 8, v);
                if (has_ln) ln_apply(row_stats(tblk + rr), cols.g0, cols.g1, v);
#pragma unroll
                for (int e = 0; e < 4; ++e) { v[e] = (v[e] + cols.b0[e]) * f; v[4 + e] = (v[4 + e] + cols.b1[e]) * f; }
                if (r < p.M && cols.nv > 0) store8(reinterpret_cast<T*>(p.out) + (int64_t)r * p.ldo + cols.c, v);
            }
        } else if (batched) {
            const EpiCols cols = epilogue_cols<EPI>(p, wcol0 + (lane % CG) * 8);
#pragma unroll 1
            for (int b = 0; b < ITS; b += NB) {
                EpiRow rows[NB];
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    const int r = epilogue_row<PADDED>(p, rblk + lane / CG + (b + n) * (64 / CG));
                    rows[n] = epilogue_row_operands<EPI>(p, cols, r, r < p.M && cols.nv > 0);
                }
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    const int rr = lane / CG + (b + n) * (64 / CG);
                    const bool active = epilogue_row<PADDED>(p, rblk + rr) < p.M && cols.nv > 0;
                    float v[8];
                    chunk8(rr, (lane % CG) * 8, v);
                    if (has_ln) ln_apply(row_stats(tblk + rr), cols.g0, cols.g1, v);
                    if (active) epilogue_chunk<T, EPI>(p, cols, rows[n], v);
                    if constexpr (WN % 64 == 0) {        // (8 consecutive lanes hold the 8 chunks of a 64-column statistics group)
                        if (EPI == EPI_RESID || EPI == EPI_PATCH) group_stats<T>(p, cols, rows[n], v, active, lane & 7);
                    }
                }
            }
        } else {
            const EpiCols cols = epilogue_cols<EPI>(p, wcol0 + (lane % CG) * 8);
#pragma unroll 1
            for (int rr = lane / CG; rr < 32; rr += 64 / CG) {
                const int r = epilogue_row<PADDED>(p, rblk + rr);
                if (r < p.M && cols.nv > 0) {
                    float v[8];
                    chunk8(rr, (lane % CG) * 8, v);
                    if (has_ln) ln_apply(row_stats(tblk + rr), cols.g0, cols.g1, v);
                    epilogue_chunk<T, EPI>(p, cols, epilogue_row_operands<EPI>(p, cols, r, true), v);
                }
            }
        }
    };
    if (has_ln) {
        // (the statistics of 96 x 128 wave tiles find registers when the first block has left its own; before it, 68 bytes a lane went to
        // scratch: 384 x 256 tiles, QKV of ViT-L 5496 tokens 60.8 us, now 58.5, ViT-g 10992 225 / 216)
        LnTile<BM> ln;
        if (MI * NI < 12) ln.ask(p, m0, tid);
        stage(std::integral_constant<int, 0>{});
        if (MI * NI >= 12) ln.ask(p, m0, tid);
        ln.leave(p, lnrow, m0, n0, tid);
        __syncthreads();
    } else {
        stage(std::integral_constant<int, 0>{});
    }
    pass(0);
    if constexpr (MI > 1) { stage(std::integral_constant<int, 1>{}); pass(1); }
    if constexpr (MI > 2) { stage(std::integral_constant<int, 2>{}); pass(2); }
    if constexpr (MI > 3) { stage(std::integral_constant<int, 3>{}); pass(3); }
    static_assert(MI <= 4, "passes are written out up to four row blocks");
}

// Sum of a value over the two halves of a wave (lane l and lane l ^ 32), in both.
__device__ __forceinline__ float wave_halves_sum(float v) {
    const uint32_t u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Projection epilogue (EPI_ROWDOT) of a wave tile: a lane's accumulators are
// one tile row's columns (row = lane % 32 of a 32-row block, column 8 (v / 4) + 4 (lane / 32) + v % 4 of a 32-column
// block), so out[r][c / 64] = sum over the 64 columns of act(acc + bias) * w is a sum inside the lane plus one
// exchange between the lane halves, and the accumulators never go through LDS (staging a 384 x 256 tile there and
// reading it back, eight waves at once at the LDS's 128 bytes per clock, took 9 of 121 us).  Bias and projection vector
// of the tile's columns go to LDS first (the operand buffers are free; the caller's barrier is behind their last read)
// and come back by broadcast reads of four consecutive columns.
template <int MI, int NI, int WM, int WN, int BN, int THREADS, bool PADDED>
__device__ __forceinline__ void rowdot_epilogue_transposed(const GemmArgs& p, f32x16 (&acc)[MI][NI], char* smem, int wm, int wn,
                                                           int tid, int m0, int n0) {
    static_assert(NI % 2 == 0 && 2 * BN <= THREADS, "whole 64-column groups per wave; one value per thread");
    const int lane = tid & 63, g = lane >> 5, li = lane & 31;
    float* sbw = reinterpret_cast<float*>(smem);
    if (tid < BN) sbw[tid] = n0 + tid < p.N ? p.bias[n0 + tid] : 0.0f;
    else if (tid < 2 * BN) sbw[tid] = n0 + tid - BN < p.N ? p.gamma[n0 + tid - BN] : 0.0f;
    __syncthreads();
    float* out = reinterpret_cast<float*>(p.out);
    EpilogueRows<PADDED> rows(p, m0 + wm * WM + li);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int r = rows.row(p);
        rows.advance(32);
        float sum[NI / 2];
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            float sj = 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ch = wn * WN + j * 32 + 8 * q + 4 * g;
                const f32x4 b4 = *reinterpret_cast<const f32x4*>(sbw + ch), w4 = *reinterpret_cast<const f32x4*>(sbw + BN + ch);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float a = acc[i][j][4 * q + e] + b4[e];
                    if (p.act == ACT_RELU) a = fmaxf(a, 0.0f);
                    sj += a * w4[e];
                }
            }
            if (j & 1) sum[j >> 1] += sj; else sum[j >> 1] = sj;
            __builtin_amdgcn_sched_barrier(0);       // (keeps the scheduler from lifting every block's reads to the top: no registers for that)
        }
#pragma unroll
        for (int k = 0; k < NI / 2; ++k) {
            const float tot = wave_halves_sum(sum[k]);
            const int c = n0 + wn * WN + 64 * k;
            if (g == (k & 1) && r < p.M && c < p.N) out[(int64_t)r * p.ldo + (c >> 6)] = tot;
        }
    }
}

// BM x BN tiles, BK elements per k-tile (LDS rows of 64, 128 or 256 bytes), S LDS stages: the loads of tile kt + S - 1 are
// in flight while tile kt is multiplied, so a load has S - 1 tile times to arrive.  WGM x WGN waves share a tile (BM / WGM
// rows and BN / WGN columns each); OCC workgroups per CU (the launch bound is in waves per SIMD: OCC * waves / 4).
// EPI: one instantiation per epilogue (with all of them behind run-time branches the kernels were two to four times as large).
// KG: groups of WGM x WGN waves that share the tile's loads and take KS / KG of the k-steps of every k-tile each; their
// partial sums are added in LDS in a fixed order by the block-level epilogue.
// RING: the operand tiles of a k-tile are units of their own in a ring of five (A0 B0 A1 B1 A2 ...), see the main loop.
template <typename T, int BN, int BK, int S, int WGM, int WGN, int OCC, int AMODE, int EPI, int BM_ = 256, int KG = 1, bool RING = false>
__global__ __launch_bounds__(64 * WGM * WGN * KG, OCC * WGM * WGN * KG / 4) void gemm_dma_kernel(const GemmArgs args) {
    const GemmArgs p = select_problem(args);
    constexpr int BM = BM_, CE = Elem<T>::CE, ESZ = sizeof(T), NW = WGN * WGM * KG;
    static_assert((BM * BK * ESZ) % (1024 * NW) == 0 && (BN * BK * ESZ) % (1024 * NW) == 0 && BM % (32 * WGM) == 0, "loader / wave tiling");
    constexpr int WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NI = WN / 32;
    constexpr int ROWB = BK * ESZ, CPR = BK / CE, RPI = 64 / CPR;   // row bytes, chunks per row, rows per DMA instruction
    constexpr int KS = BK / 16 / KG;                    // k-steps of a k-tile that a wave takes
    constexpr int A_BYTES = BM * ROWB, B_BYTES = BN * ROWB, STAGE = A_BYTES + B_BYTES;
    static_assert((BK / 16) % KG == 0 && (!RING || (A_BYTES == B_BYTES && KG == 1 && S == 2)), "k-step groups / ring units");
    constexpr int A_SLOTS = A_BYTES / (1024 * NW), B_SLOTS = B_BYTES / (1024 * NW);   // 1 KB DMA instructions per wave per k-tile
    constexpr int PD = S - 1;
    // chunk swizzle: 256 bytes of LDS (64 banks) hold one row of 256 bytes, 2 rows of 128 or 4 rows of 64
    constexpr int SW_SHIFT = ROWB == 256 ? 0 : ROWB == 128 ? 1 : 2, SW_MASK = CPR - 1;
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = KG > 1 ? wave / (WGM * WGN) : 0;
    const int wm = (KG > 1 ? wave % (WGM * WGN) : wave) / WGN, wn = wave % WGN;
    const int g = lane >> 5, li = lane & 31;

    int tm, tn;
    tile_coords(blockIdx.x, p.map, tm, tn);
    const int m0 = p.m_begin + tm * BM, n0 = tn * BN;

    // folded LayerNorm: (mean, rstd) of this tile's rows, written and read in the epilogue, live behind its staging blocks
    constexpr int EPI_BYTES = KG > 1 ? KG * BM * BN * 4 : WN % 64 ? BM * BN * 4 : NW * 32 * WN * 4;
    float* lnrow = reinterpret_cast<float*>(smem + EPI_BYTES);
    constexpr int OPERANDS = RING ? 5 * A_BYTES : S * STAGE;
    int* redo_flags = reinterpret_cast<int*>(smem + (OPERANDS > EPI_BYTES + BM * 8 ? OPERANDS : EPI_BYTES + BM * 8));    // fp32: one per wave, behind both

    // --- loader state.  DMA instruction `slot` of this wave fills 1 KB of LDS = RPI consecutive rows of
    // the A (or B) tile, row group rg = wave + NW slot: lane l lands on row rg*RPI + l/CPR, physical
    // chunk l%CPR, so it must fetch the logical chunk (l%CPR) ^ swizzle(row) of that row.  Byte offsets are 32-bit, from
    // the tile's first row (whose place in the tensor is a 64-bit one).
    const int hw = p.cH * p.cW;
    auto a_row = [&](int r) -> int64_t {        // row of A that row r of the problem reads (conv: centre pixel)
        if (AMODE == A_PLAIN) return p.a_rpi >= p.M ? (int64_t)p.a_off + r : (int64_t)(r / p.a_rpi) * p.a_istride + p.a_off + r % p.a_rpi;
        return (int64_t)(r / hw) * p.a_istride + p.a_off + r % hw;
    };
    const int64_t a_first = a_row(m0 < p.M ? m0 : p.M - 1);
    const char* __restrict__ A = reinterpret_cast<const char*>(p.A) + a_first * p.lda * ESZ;
    const char* __restrict__ W = reinterpret_cast<const char*>(p.W) + (int64_t)n0 * p.K * ESZ;
    int aoff[A_SLOTS];          // byte offset of the lane's chunk from A (k = 0; conv: centre pixel)
    int ay[A_SLOTS], ax[A_SLOTS];
    int boff[B_SLOTS];
#pragma unroll
    for (int s = 0; s < A_SLOTS; ++s) {
        const int row = (wave + NW * s) * RPI + lane / CPR;
        const int c = (lane % CPR) ^ ((row >> SW_SHIFT) & SW_MASK);
        int r = m0 + row;
        r = r < p.M ? r : p.M - 1;
        ay[s] = ax[s] = 0;
        aoff[s] = (int)(((a_row(r) - a_first) * p.lda + c * CE) * ESZ);
        if (AMODE == A_CONV3) {
            const int pix = r % hw;
            ay[s] = pix / p.cW;
            ax[s] = pix % p.cW;
        }
    }
#pragma unroll
    for (int s = 0; s < B_SLOTS; ++s) {
        const int row = (wave + NW * s) * RPI + lane / CPR;
        const int c = (lane % CPR) ^ ((row >> SW_SHIFT) & SW_MASK);
        boff[s] = (row * p.K + c * CE) * ESZ;
    }
    const char* zptr = reinterpret_cast<const char*>(p.zeros);

    auto dma_a = [&](char* sA, int kt) {
        if (AMODE == A_PLAIN) {
            const int k0 = kt * BK;
#pragma unroll
            for (int s = 0; s < A_SLOTS; ++s)
                __builtin_amdgcn_global_load_lds(VPE_GPTR(A + aoff[s] + k0 * ESZ), VPE_LPTR(sA + (wave + NW * s) * 1024), 16, 0, 0);
        } else {
            const int cc = kt / 9, tap = kt - cc * 9, c0 = cc * BK;    // chunk-major, tap-minor k order
            const int dy = tap / 3 - 1, dx = tap % 3 - 1;
            const int shift = ((dy * p.cW + dx) * (int)p.lda + c0) * ESZ;
#pragma unroll
            for (int s = 0; s < A_SLOTS; ++s) {
                const int yy = ay[s] + dy, xx = ax[s] + dx;
                const bool ok = yy >= 0 && yy < p.cH && xx >= 0 && xx < p.cW;
                const uint64_t mask = ok ? ~uint64_t(0) : uint64_t(0);
                const uint64_t addr = (reinterpret_cast<uint64_t>(A + aoff[s] + shift) & mask) |
                                      (reinterpret_cast<uint64_t>(zptr) & ~mask);
                __builtin_amdgcn_global_load_lds(VPE_GPTR(addr), VPE_LPTR(sA + (wave + NW * s) * 1024), 16, 0, 0);
            }
        }
    };
    auto dma_b = [&](char* sB, int kt) {
        const int kw = AMODE == A_PLAIN ? kt * BK : (kt % 9) * p.cC + (kt / 9) * BK;   // weight column of this k-tile
#pragma unroll
        for (int s = 0; s < B_SLOTS; ++s)
            __builtin_amdgcn_global_load_lds(VPE_GPTR(W + boff[s] + kw * ESZ), VPE_LPTR(sB + (wave + NW * s) * 1024), 16, 0, 0);
    };
    auto dma = [&](int stage, int kt) {
        dma_a(smem + stage * STAGE, kt);
        dma_b(smem + stage * STAGE + A_BYTES, kt);
    };

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // --- MFMA operand reads.  Rows of one lane differ by multiples of 32, so the swizzle term is the
    // same for all of them: one lane offset per k-step, rows by immediates.
    const int arow0 = wm * WM + li, brow0 = wn * WN + li;
    const int asw = (arow0 >> SW_SHIFT) & SW_MASK, bsw = (brow0 >> SW_SHIFT) & SW_MASK;
    // Wave tiles of up to 6 fragments per k-step keep two fragment sets (the reads of step ks + 1 are in
    // flight during the MFMAs of step ks); larger wave tiles have no registers for the second set and read
    // each step's fragments just before its MFMAs (two waves per SIMD cover for each other).
    constexpr bool FRAG_DB = ESZ == 2 && MI + NI <= 6;
    const int ks0 = kg * KS;                                        // first k-step of this wave's group
    // fp32: a lane's eight k elements of a step are two chunks of its row
    auto chunk = [&](const char* base, int ks, int sw, int half) {
        return *reinterpret_cast<const f32x4*>(base + ((4 * (ks0 + ks) + 2 * g + half) ^ sw) * 16);
    };
    auto compute_f32 = [&](const char* tile_a, const char* tile_b) {       // on v_mfma_f32_32x32x2_f32
        const char* sA = tile_a + arow0 * ROWB;
        const char* sB = tile_b + brow0 * ROWB;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                f32x4 ra[MI], rb[NI];
#pragma unroll
                for (int i = 0; i < MI; ++i) ra[i] = chunk(sA + i * 32 * ROWB, ks, asw, half);
#pragma unroll
                for (int j = 0; j < NI; ++j) rb[j] = chunk(sB + j * 32 * ROWB, ks, bsw, half);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < MI; ++i)
#pragma unroll
                        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(rb[j][e], ra[i][e], acc[i][j], 0, 0, 0);
            }
    };
    // Fragments of k-step ks of a tile into set `set` (fp32: one set of raw values, split before the next read overwrites it).
    bf16x8 fa[FRAG_DB ? 2 : 1][MI], fb[FRAG_DB ? 2 : 1][NI];
    f32x4 ra[ESZ == 4 ? MI : 1][2], rb[ESZ == 4 ? NI : 1][2];
    auto fetch = [&](const char* tile_a, const char* tile_b, int ks, int set) {
        const char* sA = tile_a + arow0 * ROWB;
        const char* sB = tile_b + brow0 * ROWB;
        if constexpr (ESZ == 4) {
#pragma unroll
            for (int i = 0; i < MI; ++i) { ra[i][0] = chunk(sA + i * 32 * ROWB, ks, asw, 0); ra[i][1] = chunk(sA + i * 32 * ROWB, ks, asw, 1); }
#pragma unroll
            for (int j = 0; j < NI; ++j) { rb[j][0] = chunk(sB + j * 32 * ROWB, ks, bsw, 0); rb[j][1] = chunk(sB + j * 32 * ROWB, ks, bsw, 1); }
        } else {
            const int ca = ((2 * (ks0 + ks) + g) ^ asw) * 16, cb = ((2 * (ks0 + ks) + g) ^ bsw) * 16;
#pragma unroll
            for (int i = 0; i < MI; ++i) fa[set][i] = *reinterpret_cast<const bf16x8*>(sA + i * 32 * ROWB + ca);
#pragma unroll
            for (int j = 0; j < NI; ++j) fb[set][j] = *reinterpret_cast<const bf16x8*>(sB + j * 32 * ROWB + cb);
        }
    };
    auto multiply = [&](int set) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
    };
    // One k-tile.  The fragments of a step are read during the step before it, across the tile boundary too, so no step begins
    // with an LDS latency.  The tile's one barrier stands in front of its LAST step: by then every wave has read
    // all of the tile (its stage is free for the loads of a later one) and the next tile has landed, so the last step's MFMAs run
    // beside the first reads of the next tile and the issue of the loads.  `turn` does that: waits, barrier, loads, and then the
    // reads it is given.  PAR: the set of the first step.
    constexpr bool SMALL = MI * NI <= 2;
    auto k_tile = [&](const char* tile_a, const char* tile_b, const char* next_a, const char* next_b, auto PAR, auto&& between, auto&& turn) {
        constexpr int par = decltype(PAR)::value;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int cur = (par + ks) & 1;
            if constexpr (ESZ == 4) {
                Split3 sa[MI], sb[NI];
#pragma unroll
                for (int i = 0; i < MI; ++i) sa[i] = split3(ra[i][0], ra[i][1]);
#pragma unroll
                for (int j = 0; j < NI; ++j) sb[j] = split3(rb[j][0], rb[j][1]);
                if (ks + 1 < KS) {
                    fetch(tile_a, tile_b, ks + 1, 0);
                } else {
                    turn([&] { fetch(next_a, next_b, 0, 0); });
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int t = 0; t < 6; ++t)
#pragma unroll
                    for (int i = 0; i < MI; ++i)
#pragma unroll
                        for (int j = 0; j < NI; ++j) acc[i][j] = split_mma(t, sb[j], sa[i], acc[i][j]);
            } else {
                if (RING && ks == 1) between();
                if (ks + 1 < KS) {
                    fetch(tile_a, tile_b, ks + 1, cur ^ 1);
                } else {
                    __builtin_amdgcn_sched_barrier(0);
                    turn([&] { fetch(next_a, next_b, 0, cur ^ 1); });
                    if (SMALL) __builtin_amdgcn_sched_barrier(0);
                }
                multiply(cur);
                if (SMALL && ks + 1 == KS) { __builtin_amdgcn_sched_barrier(0); continue; }
                // Issue order for the scheduler: the reads of the next step are spread between the MFMAs of this one (one read
                // per PER MFMAs), so a wave never waits on LDS with an empty matrix pipe.  0x100 = DS read, 0x008 = MFMA.
                constexpr int PER = (MI * NI) / (MI + NI) > 0 ? (MI * NI) / (MI + NI) : 1;
                constexpr int GROUPS = (MI * NI) / PER < MI + NI ? (MI * NI) / PER : MI + NI;
#pragma unroll
                for (int n = 0; n < GROUPS; ++n) {
                    __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, MI + NI - GROUPS, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, MI * NI - GROUPS * PER, 0);
            }
        }
    };
    // The same without a second fragment set: every step's fragments are read just before its MFMAs.
    auto k_tile_single = [&](const char* tile_a, const char* tile_b) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            fetch(tile_a, tile_b, ks, 0);
            multiply(0);
            __builtin_amdgcn_sched_group_barrier(0x100, MI + NI, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, MI * NI, 0);
        }
    };

    constexpr bool BLOCK = WN % 64 != 0 || KG > 1;            // small tiles: a wave does not hold whole 64-column groups, or only partial sums

    // --- main loop over the k-tiles
    const int KT = p.K / BK;
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, KS & 1> odd{};                  // (an even number of steps: every tile begins on the same set)
    auto none = [] {};
    if constexpr (RING) {
        // Two whole stages of a 256 x 256 tile leave 32 KB of the LDS unused and give a load one tile time to arrive (about
        // 2100 clocks, as long as the loads of a tile take by themselves).  Five units of 32 KB instead, A and B of a tile one each:
        // during tile kt A of tile kt + 2 is issued between the MFMAs, B of kt + 2 behind the tile's barrier.
        char* unit[5] = {smem, smem + A_BYTES, smem + 2 * A_BYTES, smem + 3 * A_BYTES, smem + 4 * A_BYTES};
        dma_a(unit[0], 0);
        dma_b(unit[1], 0);
        __builtin_amdgcn_sched_barrier(0);                    // (the counted waits go by the order of issue)
        dma_a(unit[2], KT > 1 ? 1 : 0);
        dma_b(unit[3], KT > 1 ? 1 : 0);
        __builtin_amdgcn_sched_barrier(0);
        pipeline_barrier<A_SLOTS + B_SLOTS>();
        fetch(unit[0], unit[1], 0, 0);
        auto tile = [&](int kt, auto PAR) {
            k_tile(unit[0], unit[1], unit[2], unit[3], PAR,
                   [&] { __builtin_amdgcn_sched_barrier(0); if (kt + 2 < KT) dma_a(unit[4], kt + 2); __builtin_amdgcn_sched_barrier(0); },
                   [&](auto&& reads) {
                       if (kt + 2 < KT) {
                           pipeline_barrier<A_SLOTS>();
                           dma_b(unit[0], kt + 2);
                       } else {
                           pipeline_barrier<0>();
                       }
                       __builtin_amdgcn_sched_barrier(0);
                       reads();
                   });
            char* const u0 = unit[0];
            char* const u1 = unit[1];
            unit[0] = unit[2]; unit[1] = unit[3]; unit[2] = unit[4]; unit[3] = u0; unit[4] = u1;
        };
        static_assert(KS >= 2 && KS % 2 == 0, "A is issued in the second step, tiles begin on set 0");
        for (int kt = 0; kt < KT; ++kt) tile(kt, even);
    } else if constexpr (FRAG_DB || ESZ == 4) {
        // S stages: the tile's barrier waits for tile kt + 1 (kt + 2 ... kt + S - 1 may be on their way), the loads of tile kt + S go
        // into the stage that tile kt leaves.
        constexpr int L = A_SLOTS + B_SLOTS;
#pragma unroll
        for (int s = 0; s < PD; ++s) {
            dma(s, s < KT ? s : KT - 1);                      // (unconditional, so that the wait for older loads can be counted)
            __builtin_amdgcn_sched_barrier(0);                // (the counted waits go by the order of issue)
        }
        pipeline_barrier<(PD - 1) * L>();
        fetch(smem, smem + A_BYTES, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (PD < KT) dma(PD, PD);                             // (the last stage is filled behind the first reads)
        __builtin_amdgcn_sched_barrier(0);
        int cur = 0;                                          // stage of tile kt
        auto tile = [&](auto PAR, auto&& turn) {
            const int nxt = cur + 1 == S ? 0 : cur + 1;
            const char* a = smem + cur * STAGE;
            const char* n = smem + nxt * STAGE;
            k_tile(a, a + A_BYTES, n, n + A_BYTES, PAR, none, turn);
            cur = nxt;
        };
        auto full = [&](int kt, auto PAR) {                   // a tile with all loads in flight
            tile(PAR, [&](auto&& reads) {
                pipeline_barrier<(S - 2) * L>();
                dma(cur, kt + S);
                __builtin_amdgcn_sched_barrier(0);
                reads();
            });
        };
        auto tail = [&](int kt, auto PAR) {                   // one of the last S or S + 1
            tile(PAR, [&](auto&& reads) {
                if (kt + 1 == KT) return;
                if (kt + S <= KT) pipeline_barrier<(S - 2) * L>();
                else pipeline_barrier<0>();
                if (kt + S < KT) dma(cur, kt + S);
                __builtin_amdgcn_sched_barrier(0);
                reads();
            });
        };
        int kt = 0;
        for (; kt + 1 + S < KT; kt += 2) { full(kt, even); full(kt + 1, odd); }
        for (; kt < KT; kt += 2) {
            tail(kt, even);
            if (kt + 1 < KT) tail(kt + 1, odd);
        }
    } else {
        // Tile kt + S - 1 is issued when tile kt has landed and everyone is done with the stage of tile kt - 1.
        auto last = [&](int kt) { return kt < KT ? kt : KT - 1; };     // (prefetches are unconditional: every path has the same loads in flight)
#pragma unroll
        for (int s = 0; s < PD; ++s) {
            dma(s, last(s));
            __builtin_amdgcn_sched_barrier(0);
        }
        int cur = 0, nxt = PD;                                // stages of tiles kt and kt + PD
        for (int kt = 0; kt < KT; ++kt) {
            pipeline_barrier<(PD - 1) * (A_SLOTS + B_SLOTS)>();
            dma(nxt, last(kt + PD));
            __builtin_amdgcn_sched_barrier(0);
            k_tile_single(smem + cur * STAGE, smem + cur * STAGE + A_BYTES);
            cur = cur + 1 == S ? 0 : cur + 1;
            nxt = nxt + 1 == S ? 0 : nxt + 1;
        }
    }
    if constexpr (ESZ == 4) {
        float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};                // NaN if any of the lane's sums is infinite or NaN
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) t[v & 3] = fmaf(acc[i][j][v], 0.0f, t[v & 3]);
        const float all = (t[0] + t[1]) + (t[2] + t[3]);
        const int any = __any(all != all);
        if (lane == 0) redo_flags[wave] = any;
    }
    pipeline_barrier<0>();                                    // everyone is done with the operands: LDS is reused
    if constexpr (ESZ == 4) {
        // The split holds neither infinities nor finite values above 3.396e38 (they round to infinity in bf16): their rests, and
        // with them every sum that they enter, are NaN.  A tile with such a sum is computed again on the fp32
        // instructions, without prefetching: infinities, NaN and overflow come out as those instructions give them.  The check
        // costs 0.4 us a launch (ViT-S 224x224: 926 -> 945 us a frame, 476x630: 2519 -> 2537-2568).
        int redo = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) redo |= redo_flags[w];
        if (__builtin_amdgcn_readfirstlane(redo)) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
            for (int kt = 0; kt < KT; ++kt) {
                dma(0, kt);
                pipeline_barrier<0>();
                compute_f32(smem, smem + A_BYTES);
                pipeline_barrier<0>();
            }
        }
    }
    if constexpr (BLOCK) {                                    // (whole tile staged in LDS)
        block_epilogue<T, EPI, BM, BN, WGM, WGN, KG, AMODE == A_PLAIN>(p, acc, smem, lnrow, m0, n0);
    } else if constexpr (EPI == EPI_ROWDOT) {
        rowdot_epilogue_transposed<MI, NI, WM, WN, BN, 64 * NW, false>(p, acc, smem, wm, wn, tid, m0, n0);
    } else {
        wave_tile_epilogue<T, EPI, BM, MI, NI, WM, WN, AMODE == A_PLAIN>(p, acc, smem, lnrow, wave, wm, wn, tid, m0, n0);
    }
}

template <typename T, int BN, int BK, int S, int WGM = 2, int WGN = 2, int OCC = 1, int BM = 256, int KG = 1, bool RING = false>
static inline hipError_t launch_gemm_dma(const GemmArgs& a, int amode, hipStream_t s, bool configure_only = false) {
    constexpr int nt = 64 * WGM * WGN * KG;
    constexpr int stage_b = (RING ? 5 * BM : S * (BM + BN)) * BK * (int)sizeof(T);
    constexpr int epi_b = (KG > 1 ? KG * BM * BN * 4 : BN / WGN % 64 ? BM * BN * 4 : WGM * WGN * 32 * (BN / WGN) * 4) + BM * 8;   // and (mean, rstd) of the rows
    constexpr int lds = (stage_b > epi_b ? stage_b : epi_b) + (sizeof(T) == 4 ? 64 : 0);        // fp32: a flag per wave
    static_assert(lds * OCC <= 160 * 1024 && nt <= 1024 && lds % 16 == 0, "LDS budget of one CU, workgroup size");
    typedef void (*Kernel)(const GemmArgs);
    // (tiles of 32 columns: the residual epilogue only)
    constexpr auto kernel_for = [](auto mode, auto epi) -> Kernel {
        if constexpr (BN % 64 && !(mode == A_PLAIN && epi == EPI_RESID)) return nullptr;
        else return &gemm_dma_kernel<T, BN, BK, S, WGM, WGN, OCC, decltype(mode)::value, decltype(epi)::value, BM, KG, RING>;
    };
#define VPE_KERNEL(mode, epi) kernel_for(std::integral_constant<int, mode>{}, std::integral_constant<int, epi>{})
    static const Kernel plain[] = {VPE_KERNEL(A_PLAIN, EPI_STORE), VPE_KERNEL(A_PLAIN, EPI_RESID), VPE_KERNEL(A_PLAIN, EPI_SWIGLU),
                                   VPE_KERNEL(A_PLAIN, EPI_QKV), VPE_KERNEL(A_PLAIN, EPI_PATCH)};
    static const Kernel conv[] = {VPE_KERNEL(A_CONV3, EPI_STORE), VPE_KERNEL(A_CONV3, EPI_ROWDOT)};
#undef VPE_KERNEL
    static bool configured = false;
    if (!configured) {
        auto opt_in = [&](Kernel k) {
            return k ? hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, lds) : hipSuccess;
        };
        hipError_t rc = hipSuccess;
        for (Kernel k : plain) if (rc == hipSuccess) rc = opt_in(k);
        for (Kernel k : conv) if (rc == hipSuccess) rc = opt_in(k);
        if (rc != hipSuccess) return rc;
        configured = true;
    }
    if (configure_only) return hipSuccess;
    if (a.K < BK || a.K % BK || (amode == A_CONV3 && a.cC % BK)) return hipErrorInvalidValue;      // the k loop has no remainder
    if (amode == A_CONV3 ? a.epi != EPI_STORE && a.epi != EPI_ROWDOT : a.epi < EPI_STORE || a.epi > EPI_PATCH) return hipErrorInvalidValue;
    const Kernel k = amode == A_CONV3 ? conv[a.epi == EPI_ROWDOT] : plain[a.epi];
    if (!k) return hipErrorInvalidValue;
    GemmArgs args = a;
    args.map = TileMap::make(cdiv(a.M - a.m_begin, BM), cdiv(a.N, BN));
    hipLaunchKernelGGL(k, dim3(args.map.tiles, a.nz > 1 ? a.nz : 1), dim3(nt), lds, s, args);
    return hipGetLastError();
}

}  // namespace vpe

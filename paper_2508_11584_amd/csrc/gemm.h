// Tiled MFMA GEMM for gfx950:  C[M][N] = A[M][K] * W^T  with W stored [N][K] (K contiguous),
// fp32 accumulation, and the layer's epilogue applied to the accumulators: the arguments, the tile order and the
// epilogues.  The kernel is gemm_dma_kernel (gemm_dma.h).
//
// It serves every dense contraction of the encoder and the heads (ViT blocks: fused
// QKV, out-projection, MLP; patch embedding after im2col; the heads' 1x1 and 3x3 convolutions):
//   * A operand: plain rows (optionally re-mapped so that only patch tokens of each image are
//     read) or an implicit im2col of a channels-last grid for 3x3 / pad 1 convolutions.
//   * operands in bf16, or fp32 split into three bf16 terms each; v_mfma_f32_32x32x16_bf16 either way.
#pragma once
#include "common.h"

namespace vpe {

enum AMode { A_PLAIN = 0, A_CONV3 = 1 };
enum Epi { EPI_STORE = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_QKV = 3, EPI_PATCH = 4, EPI_ROWDOT = 5 };
enum Act { ACT_NONE = 0, ACT_RELU = 1, ACT_GELU = 2 };

// Where the tiles of a launch lie, worked out on the host (TileMap::make): the kernel's divisions by these numbers are products
// with their reciprocals.  (The prologue of a 64 x 64 workgroup was 290 instructions, four divisions among them.)
struct TileMap {
    int tiles, tiles_m, per_group;       // workgroups per problem, tile rows, tiles in a group of GM tile rows
    uint32_t inv_group, inv_last;        // ceil(2^32 / d) for d = per_group and the rows of the last group (0: divide)
    static constexpr int GM = 8;
    static uint32_t reciprocal(int64_t d, int64_t most) { return d > 1 && d * most < (int64_t(1) << 32) ? (uint32_t)(((uint64_t(1) << 32) + d - 1) / d) : 0; }
    static TileMap make(int tiles_m, int tiles_n) {
        TileMap t{tiles_m * tiles_n, tiles_m, GM * tiles_n, 0, 0};
        t.inv_group = reciprocal(t.per_group, t.tiles);
        t.inv_last = reciprocal(tiles_m % GM, t.per_group);
        return t;
    }
};

struct GemmArgs {
    const void* A;       // T
    int64_t lda;         // elements between consecutive A rows (PLAIN) / pixels (CONV3)
    const void* W;       // T [N rounded up to 256][K]
    const float* bias;   // [N] in the physical column order of W, may be null
    int M, N, K;         // K multiple of 64 (k-tiles are whole; anything else is refused)
    int m_begin;         // a launch covers rows m_begin .. M - 1 (row indices stay those of the whole problem)
    int nz;              // problems of a batched launch (see z_a below)
    TileMap map;         // (filled in by the launchers)
    // PLAIN: logical row r reads A row (r / a_rpi) * a_istride + a_off + r % a_rpi
    // CONV3: pixel (b, y, x) is A row b * a_istride + a_off + y * cW + x
    int a_rpi, a_istride, a_off;
    int cH, cW, cC;      // CONV3 grid and channels (K = 9 cC, cC multiple of 64)
    const void* zeros;   // CONV3: >= 16 bytes of zeros, read in place of out-of-image taps
    int epi, act, out_f32;         // (CONV3: STORE or ROWDOT, without a folded LayerNorm; PLAIN: all but ROWDOT)
    void* out;           // T or float (out_f32); RESID/PATCH: float residual stream
    int64_t ldo;
    int o_rpi, o_istride, o_off;   // output row map, as for A
    const float* gamma;  // RESID: LayerScale vector.  ROWDOT: projection vector w[N]; the tile itself is not stored,
                         //   out (float) receives out[r * ldo + c / 64] = sum over the 64 columns of group c / 64 of
                         //   act(acc + bias)[col] * w[col]  (N multiple of 64; the caller adds the N / 64 partial sums)
    const float* pos;    // PATCH: positional rows [o_rpi][N]
    void* out2;          // QKV: transposed values  vt[(b * dim + c)][npad]
    int ntok, npad, dim; // QKV
    float q_scale;       // QKV: factor of the query columns (after the bias, before they are rounded)
    // LayerNorm folded into this GEMM (consumer side): A holds the UN-normalised rows (plain row map), W has
    // been scaled by the LayerNorm gain along k and bias holds b + beta W; the accumulator of (row r, column c)
    // becomes rstd_r * (acc - mean_r * ln_colsum[c]) before bias / activation, with ln_colsum[c] = sum_k W[c][k].
    // ln_stats [M][ln_groups][2]: (mean, sum of squared deviations from it) of every group of K / ln_groups columns of row r,
    // as written by the producer below; both sides work with differences, never with raw squares.  Not with RESID or PATCH.
    const float* ln_stats;     // null: no LayerNorm
    const float* ln_colsum;
    int ln_groups;             // groups of a row and their width: K / 64 of 64 columns, or K / 32 of 32 (the producer's st_group)
    float ln_width;
    float ln_eps;
    // A may hold the rows minus a per-row level (LayerNorm does not see a level common to a row, and a 16-bit
    // copy of x - level keeps its precision when the row sits far from zero): ln_level[r] is that level (null:
    // 0).  ln_level_out (may be null) receives the rows' means, written by the tiles of the first column
    // block: the level for the NEXT copy of these rows -- a different buffer from ln_level, which the other
    // column tiles are still reading.
    const float* ln_level;
    float* ln_level_out;
    // Producer side (RESID / PATCH, N a multiple of 64): besides the fp32 rows, write their copy in T
    // (xb_out, [rows][N], may be null) and the group statistics of the updated rows (st_out, [rows][N / group][2], may be null:
    // groups of 64 columns, or, with st_group = 32, of 32: RESID alone, in tiles of 32 columns)
    void* xb_out;
    float* st_out;
    int st_group;
    const float* xb_level;     // xb_out holds x - xb_level[row] (null: 0); statistics are of x itself
    // STORE only (N and ldo multiples of 8): fp32 tensors added after the activation, read through the output
    // row map with the output's row pitch (null: none); and a second copy of the result in T, optionally
    // through ReLU (the operand of a following convolution), same map and pitch (null: none)
    const float* add1;
    const float* add2;
    void* twin;
    int twin_relu;
    // batch of nz independent problems of the same shape in one launch (blockIdx.y = z): problem z uses
    // A + z * z_a, W + z * z_w, out + z * z_out (byte strides, may be negative) and bias + z * z_bias (elements);
    // with z_inner > 0 the output alone is addressed in two levels, out + (z % z_inner) * z_out + (z / z_inner) * z_out2
    int64_t z_a, z_w, z_out, z_bias;
    int z_inner;
    int64_t z_out2;
};

// The arguments of problem blockIdx.y of a batched launch (a plain copy when the launch is not batched).
__device__ __forceinline__ GemmArgs select_problem(const GemmArgs& in) {
    GemmArgs p = in;
    if (in.nz <= 1) return p;
    const int64_t z = blockIdx.y;
    p.A = reinterpret_cast<const char*>(in.A) + z * in.z_a;
    p.W = reinterpret_cast<const char*>(in.W) + z * in.z_w;
    p.out = in.z_inner > 0 ? reinterpret_cast<char*>(in.out) + (z % in.z_inner) * in.z_out + (z / in.z_inner) * in.z_out2
                           : reinterpret_cast<char*>(in.out) + z * in.z_out;
    if (in.bias) p.bias = in.bias + z * in.z_bias;
    return p;
}


// GELU in its exact (erf) form.  erf by the Abramowitz-Stegun 7.1.26 rational approximation
// (|error| <= 1.5e-7, i.e. fp32 rounding level): one reciprocal, one exponential and six FMAs
// instead of the ~40-instruction library erff, which made the GELU epilogue of a 256 x 256 tile as
// long as its k loop.
__device__ __forceinline__ float gelu_erf(float v) {
    const float x = fabsf(v) * 0.70710678118654752f;
    const float t = __frcp_rn(fmaf(0.3275911f, x, 1.0f));
    float poly = fmaf(1.061405429f, t, -1.453152027f);
    poly = fmaf(poly, t, 1.421413741f);
    poly = fmaf(poly, t, -0.284496736f);
    poly = fmaf(poly, t, 0.254829592f);
    const float erf_abs = 1.0f - poly * t * __expf(-x * x);
    return 0.5f * v * (1.0f + copysignf(erf_abs, v));
}

// The same function for results that are rounded to bf16: v Phi(v) with the normal distribution function as a logistic one,
// Phi(v) = 1 / (1 + 2^(v q(v^2))), q of degree 5 on |v| <= 5.5; beyond 5.5 the value there, 1.6e-7 from 0 or 1.  Least maximum
// error of Phi (linear program) relative to an envelope that is 1.6e-8 at 0, where most of fc1's results lie, 1e-6 from 2 on: a fit of
// degree 4 without it had 1.7e-7 rms on |v| < 0.25.  The result differs from the exact form by at most 6.4e-7 |v| (rms, before
// rounding: 1.1e-8 on |v| < 0.25, 1.8e-7 up to 1, 6.4e-7 up to 2, 1.7e-6 beyond; 1.2 % of the result at -4), less on every interval
// than erf as an odd polynomial of degree 19 on |x| <= 3 (1.7e-8, 4.0e-7, 3.1e-6, 9.3e-6 up to 4) in 14 issue slots (8 clocks for
// v_exp_f32 and v_rcp_f32, 4 for the others) instead of 18: an epilogue has the vector ALU to itself while the matrix pipes of its
// workgroup idle, at 64 values a clock and CU.  -inf gives -inf, +inf +inf (the exact form gives NaN for -inf).
constexpr float GELU_LIMIT = 5.5f;
__host__ __device__ __forceinline__ float gelu_exponent(float x) {        // x q(x^2), |x| <= GELU_LIMIT
    const float t = x * x;
    float q = fmaf(1.61200518e-07f, t, -8.30406134e-06f);
    q = fmaf(q, t, 1.41446319e-04f);
    q = fmaf(q, t, 1.36013434e-04f);
    q = fmaf(q, t, -1.04866788e-01f);
    q = fmaf(q, t, -2.30220509e+00f);
    return q * x;
}
__device__ __forceinline__ float gelu_erf_bf16(float v) {
    return v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(gelu_exponent(__builtin_amdgcn_fmed3f(v, -GELU_LIMIT, GELU_LIMIT))));
}
template <typename T>
__device__ __forceinline__ float gelu_for(float v) { return sizeof(T) == 2 ? gelu_erf_bf16(v) : gelu_erf(v); }
// SiLU(a) * b.  For results rounded to bf16 the quotient is one v_rcp_f32 (1 ulp) and a product instead of the
// correctly rounded division sequence (about ten instructions).
template <typename T>
__device__ __forceinline__ float swiglu_for(float a, float b) {
    const float d = 1.0f + __expf(-a);
    return sizeof(T) == 2 ? a * __builtin_amdgcn_rcpf(d) * b : a / d * b;
}

// Spread consecutive block ids (which the hardware deals round-robin to the 8 XCDs) so that
// each XCD works on one contiguous range of tiles and its L2 sees neighbouring A/W panels.
__device__ __forceinline__ int xcd_contiguous(int bid, int nb) {
    const int xcd = bid & 7, idx = bid >> 3, base = nb >> 3, rem = nb & 7;
    return xcd * base + (xcd < rem ? xcd : rem) + idx;
}

// Linear tile index -> (tile row, tile column) in groups of GM tile rows: the ~32 workgroups an XCD
// runs at a time then cover a GM x (32 / GM) block of tiles instead of one row of 32, so each A
// k-slice fetched into that XCD's L2 serves 32 / GM workgroups and each W k-slice GM of them.
// (Measured on the large tiles: with row-major order the loads ran at the XCD <-> memory-side
// fabric rate, about 13 TB/s in aggregate, not at the L2 rate.)
__device__ __forceinline__ uint32_t quotient(uint32_t x, uint32_t d, uint32_t inv) { return inv ? __umulhi(x, inv) : x / d; }
__device__ __forceinline__ void tile_coords(int bid, const TileMap& t, int& tm, int& tn) {
    constexpr int GM = TileMap::GM;
    const int lin = xcd_contiguous(bid, t.tiles);
    const int group = quotient(lin, t.per_group, t.inv_group), rem = lin - group * t.per_group;
    const int first = group * GM;
    const int rows = t.tiles_m - first;
    tn = rows >= GM ? rem / GM : rows == 1 ? rem : quotient(rem, rows, t.inv_last);
    tm = first + rem - tn * (rows >= GM ? GM : rows);
}

// 8 consecutive values of T (16 bytes of bf16, 32 bytes of fp32) to global memory.
__device__ __forceinline__ void store8(bf16* dst, const float* v) {
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (bf16)v[i];
    *reinterpret_cast<bf16x8*>(dst) = o;
}
__device__ __forceinline__ void store8(float* dst, const float* v) {
    *reinterpret_cast<f32x4*>(dst) = f32x4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f32x4*>(dst + 4) = f32x4{v[4], v[5], v[6], v[7]};
}

// Epilogue of row chunks: a lane keeps eight consecutive columns and visits several rows.  What it needs of the columns is
// loaded once (EpiCols); what it needs of a row (residual values, positional row, added maps: EpiRow) is loaded for a
// whole batch of rows before the first of them is stored.  Taken row by row -- the compiler cannot move a row's loads
// above the previous row's stores -- every row pays a memory latency: a 256 x 256 tile spent 21 us on its 16 dependent
// rows per lane (bias, LayerScale and the residual values fetched behind each other), a 64 x 128 tile 3.5 us.
struct EpiCols { f32x4 b0, b1, g0, g1; int c, nv; };      // bias; LayerScale (RESID) or the folded LayerNorm's column sums; nv: columns
                                                          // of the chunk that exist (8, fewer at a ragged edge, <= 0: none)
struct EpiRow { int orow; f32x4 a0, a1; float lev; };

__device__ __forceinline__ void load_columns(const float* src, int c, int nv, f32x4& lo, f32x4& hi) {
    lo = hi = f32x4{0, 0, 0, 0};
    if (!src) return;
    if (nv == 8) {
        lo = *reinterpret_cast<const f32x4*>(src + c);
        hi = *reinterpret_cast<const f32x4*>(src + c + 4);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i < nv) lo[i] = src[c + i];
            if (4 + i < nv) hi[i] = src[c + 4 + i];
        }
    }
}
template <int EPI>
__device__ __forceinline__ EpiCols epilogue_cols(const GemmArgs& p, int c) {
    EpiCols k;
    k.c = c;
    k.nv = p.N - c < 8 ? p.N - c : 8;
    load_columns(p.bias, c, k.nv, k.b0, k.b1);
    load_columns(EPI == EPI_RESID ? p.gamma : EPI != EPI_PATCH && p.ln_stats ? p.ln_colsum : nullptr, c, k.nv, k.g0, k.g1);
    return k;
}
// The folded LayerNorm on eight columns of a row: st = (mean, rstd), cs the column sums.
__device__ __forceinline__ void ln_apply(const f32x2& st, const f32x4& cs0, const f32x4& cs1, float* v) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[i] = st[1] * (v[i] - st[0] * cs0[i]); v[4 + i] = st[1] * (v[4 + i] - st[0] * cs1[i]); }
}

// Row r of the output: its place under the row map and the operands of its chunk (loads only; ok: r < M and the chunk exists).
template <int EPI>
__device__ __forceinline__ EpiRow epilogue_row_operands(const GemmArgs& p, const EpiCols& k, int r, bool ok) {
    EpiRow e;
    e.orow = r;
    e.a0 = e.a1 = f32x4{0, 0, 0, 0};
    e.lev = 0.0f;
    if (!ok) return e;
    const float* src = nullptr;
    if (EPI == EPI_STORE) {
        // (the plain map, one run of rows, needs no division)
        e.orow = p.o_rpi >= p.M ? p.o_off + r : (r / p.o_rpi) * p.o_istride + p.o_off + r % p.o_rpi;
        if (p.add1) src = p.add1 + (int64_t)e.orow * p.ldo + k.c;
    } else if (EPI == EPI_RESID) {
        src = reinterpret_cast<const float*>(p.out) + (int64_t)e.orow * p.ldo + k.c;
    } else if (EPI == EPI_PATCH) {
        const int b = r / p.o_rpi, pp = r - b * p.o_rpi;
        e.orow = b * p.o_istride + p.o_off + pp;
        src = p.pos + (int64_t)pp * p.N + k.c;
    }
    if (src) {
        e.a0 = *reinterpret_cast<const f32x4*>(src);
        e.a1 = *reinterpret_cast<const f32x4*>(src + 4);
    }
    if (p.xb_level) e.lev = p.xb_level[e.orow];
    return e;
}

// Columns k.c .. of the row of `e`, the raw accumulators in v.  Full, aligned chunks go out as 16-byte stores; ragged
// ones element by element.  RESID / PATCH leave the updated residual values in v.
template <typename T, int EPI>
__device__ __forceinline__ void epilogue_chunk(const GemmArgs& p, const EpiCols& k, const EpiRow& e, float* v) {
    const int nv = k.nv;
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[i] += k.b0[i]; v[4 + i] += k.b1[i]; }
    if (EPI == EPI_STORE) {
        if (p.act == ACT_RELU) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = fmaxf(v[i], 0.0f);
        } else if (p.act == ACT_GELU) {
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = gelu_for<T>(v[i]);
        }
        if (p.add1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[i] += e.a0[i]; v[4 + i] += e.a1[i]; }
        }
        if (p.add2) {
            const float* a = p.add2 + (int64_t)e.orow * p.ldo + k.c;
            const f32x4 a0 = *reinterpret_cast<const f32x4*>(a), a1 = *reinterpret_cast<const f32x4*>(a + 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[i] += a0[i]; v[4 + i] += a1[i]; }
        }
        if (p.twin) {
            float t[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = p.twin_relu ? fmaxf(v[i], 0.0f) : v[i];
            store8(reinterpret_cast<T*>(p.twin) + (int64_t)e.orow * p.ldo + k.c, t);
        }
        if (p.out_f32) {
            float* dst = reinterpret_cast<float*>(p.out) + (int64_t)e.orow * p.ldo + k.c;
            if (nv == 8 && (p.ldo & 3) == 0) store8(dst, v);
            else {
#pragma unroll
                for (int i = 0; i < 8; ++i) if (i < nv) dst[i] = v[i];
            }
        } else {
            T* dst = reinterpret_cast<T*>(p.out) + (int64_t)e.orow * p.ldo + k.c;
            if (nv == 8 && (p.ldo & 7) == 0) store8(dst, v);
            else {
#pragma unroll
                for (int i = 0; i < 8; ++i) if (i < nv) dst[i] = from_f32<T>(v[i]);
            }
        }
    } else if (EPI == EPI_RESID || EPI == EPI_PATCH) {
        // fp32 residual stream, N = ldo = model width (multiple of 64): always full aligned chunks
        if (EPI == EPI_PATCH) {
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[i] += e.a0[i]; v[4 + i] += e.a1[i]; }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[i] = e.a0[i] + k.g0[i] * v[i]; v[4 + i] = e.a1[i] + k.g1[i] * v[4 + i]; }
        }
        store8(reinterpret_cast<float*>(p.out) + (int64_t)e.orow * p.ldo + k.c, v);
        if (p.xb_out) {
            float rel[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) rel[i] = v[i] - e.lev;
            store8(reinterpret_cast<T*>(p.xb_out) + (int64_t)e.orow * p.ldo + k.c, rel);
        }
    } else {   // EPI_QKV, query / key columns
        const float f = k.c < p.dim ? p.q_scale : 1.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] *= f;
        store8(reinterpret_cast<T*>(p.out) + (int64_t)e.orow * p.ldo + k.c, v);
    }
}

// ROWDOT: contribution of 8 consecutive columns (starting at c) of one row to the row's projection.
__device__ __forceinline__ float rowdot_chunk(const GemmArgs& p, int c, const float* v) {
    const f32x4 b0 = *reinterpret_cast<const f32x4*>(p.bias + c), b1 = *reinterpret_cast<const f32x4*>(p.bias + c + 4);
    const f32x4 w0 = *reinterpret_cast<const f32x4*>(p.gamma + c), w1 = *reinterpret_cast<const f32x4*>(p.gamma + c + 4);
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = v[i] + b0[i], b = v[4 + i] + b1[i];
        if (p.act == ACT_RELU) { a = fmaxf(a, 0.0f); b = fmaxf(b, 0.0f); }
        s += a * w0[i] + b * w1[i];
    }
    return s;
}

// QKV epilogue, value columns: tokens r .. r + 7 (r a multiple of 8) of value column c2 go to the transposed
// buffer vt[(image * dim + c2)][token in image].  With several images whose token count is not a multiple of
// 8 the group starts at an odd offset inside its image: still one run of 8 when it does not cross into the
// next image, written with the widest stores its alignment allows; only a group that straddles two images
// (or the end of the matrix) goes element by element.
template <typename T>
__device__ __forceinline__ void store_tokens8(const GemmArgs& p, T* vt, int r, int c2, const float* v) {
    const int b = p.M <= p.ntok ? 0 : r / p.ntok, n = r - b * p.ntok;     // (one image: no division)
    T* dst = vt + ((int64_t)b * p.dim + c2) * p.npad + n;
    if (n + 8 <= p.ntok && r + 8 <= p.M) {
        if ((n & 7) == 0) {
            store8(dst, v);
        } else if (sizeof(T) == 2 && (n & 1) == 0) {
#pragma unroll
            for (int k = 0; k < 8; k += 2) {
                const T lo = from_f32<T>(v[k]), hi = from_f32<T>(v[k + 1]);
                uint32_t w;
                w = (uint32_t)(*reinterpret_cast<const uint16_t*>(&lo)) | ((uint32_t)(*reinterpret_cast<const uint16_t*>(&hi)) << 16);
                *reinterpret_cast<uint32_t*>(dst + k) = w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) dst[k] = from_f32<T>(v[k]);
        }
    } else {
        // (an image's end or the matrix's: the place moves on by comparison, not by a division per token)
        int image = b, at = n;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (at == p.ntok) { at = 0; ++image; }
            if (r + k < p.M) vt[((int64_t)image * p.dim + c2) * p.npad + at] = from_f32<T>(v[k]);
            ++at;
        }
    }
}

// (mean, rstd) of a row from its group statistics (mean_g, M2_g = sum of squared deviations from mean_g, of
// each group of 64 or 32 columns), one thread per tile row.  Groups are merged around the first group's mean, so a level common to
// the whole row cancels before anything is squared:
//   mean = m_0 + avg_g (m_g - m_0),   M2 = sum_g M2_g + W (sum_g (m_g - m_0)^2 - G (mean - m_0)^2),  G groups of W columns.
// In two parts, so that the loads are under way while the accumulators are staged: `fetch` asks for the statistics, `merge`
// uses them.  Both belong to the epilogue: while loads into LDS are in flight the compiler waits for all of them before it
// uses any other loaded value, so in front of the k loop the statistics cost a drained pipeline (us before the first
// barrier with / without them, ViT-S 1.9 / 1.0, ViT-g 3.7 / 1.3).
// Rows of up to 24 groups (width 1536; 768 in groups of 32) go in one batch; more follow in `merge`.
struct LnRow {
    f32x4 v[12];                    // two groups each
    float odd_mean, odd_m2, level;  // the last group of an odd number; what A was stored against

    template <int N>
    __device__ __forceinline__ void fetch_pairs(const float* st, int pairs) {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = *reinterpret_cast<const f32x4*>(st + 4 * (k < pairs ? k : 0));
    }
    __device__ __forceinline__ void fetch(const GemmArgs& p, int r) {
        const float* st = p.ln_stats + (int64_t)r * p.ln_groups * 2;
        const int pairs = p.ln_groups >> 1;
        odd_mean = st[2 * (p.ln_groups - 1)];
        odd_m2 = st[2 * (p.ln_groups - 1) + 1];
        level = p.ln_level ? p.ln_level[r] : 0.0f;
        if (pairs == 0) v[0] = f32x4{odd_mean, 0.0f, 0.0f, 0.0f};
        else if (pairs <= 3) fetch_pairs<3>(st, pairs);
        else if (pairs <= 6) fetch_pairs<6>(st, pairs);
        else if (pairs <= 8) fetch_pairs<8>(st, pairs);
        else fetch_pairs<12>(st, pairs);
    }
    __device__ __forceinline__ void merge(const GemmArgs& p, int r, float& mean, float& rstd) const {
        const float m0 = v[0][0];
        float sd = 0.0f, sdd = 0.0f, sm2 = 0.0f;
        auto add = [&](const f32x4& u) {
            const float d0 = u[0] - m0, d1 = u[2] - m0;
            sd += d0 + d1;
            sdd += d0 * d0 + d1 * d1;
            sm2 += u[1] + u[3];
        };
        const int pairs = p.ln_groups >> 1;
#pragma unroll
        for (int k = 0; k < 12; ++k)
            if (k < pairs) add(v[k]);
        const float* st = p.ln_stats + (int64_t)r * p.ln_groups * 2;
        for (int k = 12; k < pairs; ++k) add(*reinterpret_cast<const f32x4*>(st + 4 * k));
        if (p.ln_groups & 1) {
            const float d = odd_mean - m0;
            sd += d; sdd += d * d; sm2 += odd_m2;
        }
        const float G = (float)p.ln_groups, dm = sd / G;
        mean = m0 + dm;
        const float m2 = sm2 + p.ln_width * fmaxf(sdd - G * dm * dm, 0.0f);
        rstd = 1.0f / sqrtf(m2 / (p.ln_width * G) + p.ln_eps);
    }
};

// The value of the lane 1, 2 or (for values equal within every four lanes) 4 away among eight consecutive lanes, on the
// vector ALU (row permutations; an exchange through the LDS crossbar takes ~100 clocks, six of them in a row per chunk).
template <int O>
__device__ __forceinline__ float lane_across(float v) {
    static_assert(O == 1 || O == 2 || O == 4, "");
    constexpr int ctrl = O == 1 ? 0xB1 : O == 2 ? 0x4E : 0x141;     // quad_perm [1,0,3,2], [2,3,0,1]; mirror within eight
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, true));
}

// Statistics (mean, sum of squared deviations) of a W-column group (64 or 32) of the row of `e`, for the LayerNorm that follows.
// Called by all W / 8 lanes that hold the group's chunks (consecutive lanes, chunk index = lane % (W / 8)).  Each lane takes its
// eight values around the first of them, then the lanes' means and sums are merged pairwise: only differences are
// squared, so the level of the data cancels.
template <typename T, int W = 64>
__device__ __forceinline__ void group_stats(const GemmArgs& p, const EpiCols& k, const EpiRow& e, const float* v, bool active, int chunk) {
    if (!p.st_out) return;
    float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
    for (int i = 1; i < 8; ++i) {
        const float d = v[i] - v[0];
        s1 += d;
        s2 += d * d;
    }
    float mean = v[0] + s1 * 0.125f, m2 = fmaxf(s2 - s1 * s1 * 0.125f, 0.0f);
    float d = lane_across<1>(mean) - mean;
    m2 += lane_across<1>(m2) + 4.0f * d * d;
    mean += 0.5f * d;
    d = lane_across<2>(mean) - mean;
    m2 += lane_across<2>(m2) + 8.0f * d * d;
    mean += 0.5f * d;
    if constexpr (W == 64) {
        d = lane_across<4>(mean) - mean;
        m2 += lane_across<4>(m2) + 16.0f * d * d;
        mean += 0.5f * d;
    }
    if (active && chunk == 0)
        *reinterpret_cast<f32x2*>(p.st_out + ((int64_t)e.orow * (p.N >> (W == 64 ? 6 : 5)) + (k.c >> (W == 64 ? 6 : 5))) * 2) = f32x2{mean, m2};
}

// The folded LayerNorm's (mean, rstd) of the tile's rows into lnrow[2 row] (LDS), one thread per row: `ask` in front of other
// epilogue work, `leave` behind it and in front of a barrier.  The means are relative to the level A was stored against; the
// means themselves are handed on as the next level by the first column block's tiles.
template <int BM>
struct LnTile {
    LnRow row;
    __device__ __forceinline__ int place(const GemmArgs& p, int m0, int tid) const { return m0 + tid < p.M ? m0 + tid : p.M - 1; }
    __device__ __forceinline__ void ask(const GemmArgs& p, int m0, int tid) {
        if (tid < BM) row.fetch(p, place(p, m0, tid));
    }
    __device__ __forceinline__ void leave(const GemmArgs& p, float* lnrow, int m0, int n0, int tid) const {
        if (tid >= BM) return;
        float mean, rstd;
        row.merge(p, place(p, m0, tid), mean, rstd);
        if (p.ln_level_out && n0 == 0 && m0 + tid < p.M) p.ln_level_out[m0 + tid] = mean;
        *reinterpret_cast<f32x2*>(lnrow + 2 * tid) = f32x2{mean - row.level, rstd};
    }
};

// Block-level epilogue of the tiles whose waves hold less than whole 64-column groups or partial sums.  The accumulators go through LDS
// (`smem`, free after the k loop, at least BM * BN * 4 bytes) as a row-major fp32 tile, so that
// each thread then owns 8 consecutive columns of a row: one row-index computation and 16-byte
// coalesced global accesses per chunk.  The MFMAs took the W operand first, so a lane holds one tile row and of every block of
// 32 columns four runs of four: accumulator element v of lane (g, li) in block (i, j) is row 32 i + li, column
// 32 j + 8 (v / 4) + 4 g + v % 4, and the tile is written 16 bytes at a time.
// KG > 1: the workgroup holds KG groups of WGM x WGN waves, each with the partial sums of its share of the k
// range for the same tile; each leaves them in a tile of its own in LDS (KG * BM * BN * 4 bytes), they are added in a
// fixed order (group 0, then 1, ...) where they are read, and all KG groups' threads share the chunk work below.  (Added
// into one tile group by group, with a barrier each, four groups cost 1.3 us more than two at 64 x 64.)  The folded
// LayerNorm is applied to the sums: on the partial sums it was done once per group and element.  LN: it is possible
// (convolutions have none).  The first rows' operands are then asked for when its statistics have left their registers, so that
// nothing goes to scratch (64 x 128 tiles in two groups, fc1 of ViT-S 1531 tokens 9.6 / 8.9 us, ViT-B 1370 18.4 / 17.2): of
// those epilogues only a plain store with add1 has any.
template <typename T, int EPI, int BM, int BN, int WGM, int WGN, int KG, bool LN>
__device__ __forceinline__ void block_epilogue(const GemmArgs& p, f32x16 (&acc)[BM / WGM / 32][BN / WGN / 32],
                                               char* smem, float* lnrow, int m0, int n0) {
    constexpr int NTG = 64 * WGM * WGN, NT = NTG * KG;
    constexpr int WM = BM / WGM, WN = BN / WGN, MI = WM / 32, NI = WN / 32;
    const int tid = threadIdx.x, lane = tid & 63, wave = (tid % NTG) >> 6;
    const int kg = KG > 1 ? tid / NTG : 0;
    const int wm = wave / WGN, wn = wave % WGN;
    const int g = lane >> 5, li = lane & 31;
    float* sC = reinterpret_cast<float*>(smem);
    constexpr bool LNE = LN && EPI != EPI_RESID && EPI != EPI_PATCH && EPI != EPI_ROWDOT;
    const bool has_ln = LNE && p.ln_stats;
    LnTile<BM> ln;
    if (has_ln) ln.ask(p, m0, tid);
    // the lane's columns for the row-chunk paths, and its first rows' operands: on their way while the tile is staged
    // (32 x 32 tiles have fewer chunks than the workgroup threads: the others stand by)
    constexpr int CG = BN / 8, RPASS = NT / CG < BM ? NT / CG : BM, PASSES = BM / RPASS, NB = PASSES < 4 ? PASSES : 4;
    constexpr bool SPARE = NT / CG > BM;
    static_assert(BM % RPASS == 0 && PASSES % NB == 0, "whole passes over the tile's rows");
    static_assert(BN % 64 == 0 || EPI == EPI_RESID, "tiles of 32 columns are for the residual epilogue");
    const int cg = tid % CG, rr0 = tid / CG;
    const bool values = EPI == EPI_QKV && n0 >= 2 * p.dim;            // value columns of QKV
    const bool chunks = EPI != EPI_SWIGLU && EPI != EPI_ROWDOT && !values;
    EpiCols cols;
    EpiRow rows[NB];
    auto first_rows = [&] {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const int r = m0 + rr0 + n * RPASS;
            rows[n] = epilogue_row_operands<EPI>(p, cols, r, r < p.M && cols.nv > 0 && !(SPARE && rr0 >= BM));
        }
    };
    if (chunks) {
        cols = epilogue_cols<EPI>(p, n0 + cg * 8);
        if (!LNE) first_rows();
    }
    // 4-column groups of a row are exchanged by the row: 16 consecutive rows writing one group, and eight lanes reading one
    // column of eight 8-row blocks (the transposed value store), fall on different banks
    constexpr int GROUPS = BN / 4 < 16 ? BN / 4 : 16;
    auto at = [&](int row, int col) { return row * BN + (col ^ (((row ^ (row >> 3)) & (GROUPS - 1)) << 2)); };
    {
        float* own = sC + kg * BM * BN;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<f32x4*>(own + at(wm * WM + i * 32 + li, wn * WN + j * 32 + 8 * q + 4 * g)) =
                        f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    }
    if (has_ln) ln.leave(p, lnrow, m0, n0, tid);
    if (LNE && chunks) first_rows();
    __syncthreads();
    auto tile8 = [&](int row, int col, float* v) {           // columns col .. col + 7 of a tile row, the groups' partial sums added in order
#pragma unroll
        for (int k = 0; k < KG; ++k) {
            const f32x4 lo = *reinterpret_cast<const f32x4*>(sC + k * BM * BN + at(row, col));
            const f32x4 hi = *reinterpret_cast<const f32x4*>(sC + k * BM * BN + at(row, col + 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = k == 0 ? lo[e] : v[e] + lo[e];
                v[4 + e] = k == 0 ? hi[e] : v[4 + e] + hi[e];
            }
        }
    };
    auto row_stats = [&](int row) { return *reinterpret_cast<const f32x2*>(lnrow + 2 * row); };

    if constexpr (EPI == EPI_SWIGLU) {
        // physical columns come in groups of 64: 32 gate columns, then their 32 linear partners;
        // a thread takes 8 gate columns and their partners and writes 8 hidden units
        constexpr int GG = BN / 16, GPASS = NT / GG;
        const int gg = tid % GG, grp = gg >> 2, j0 = (gg & 3) * 8;
        const int ca = n0 + grp * 64 + j0;            // physical gate column
        if (ca + 40 <= p.N) {
            const int oc = (ca >> 6) * 32 + j0;       // hidden unit index
            T* out = reinterpret_cast<T*>(p.out);
            const EpiCols ka = epilogue_cols<EPI>(p, ca), kb = epilogue_cols<EPI>(p, ca + 32);
            for (int rr = tid / GG; rr < BM; rr += GPASS) {
                const int r = m0 + rr;
                if (r >= p.M) break;
                float va[8], vb[8], h[8];
                tile8(rr, grp * 64 + j0, va);
                tile8(rr, grp * 64 + j0 + 32, vb);
                if (has_ln) {
                    const f32x2 st = row_stats(rr);
                    ln_apply(st, ka.g0, ka.g1, va);
                    ln_apply(st, kb.g0, kb.g1, vb);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    h[i] = swiglu_for<T>(va[i] + ka.b0[i], vb[i] + kb.b0[i]);
                    h[4 + i] = swiglu_for<T>(va[4 + i] + ka.b1[i], vb[4 + i] + kb.b1[i]);
                }
                store8(out + (int64_t)r * p.ldo + oc, h);
            }
        }
        return;
    }
    if (EPI == EPI_QKV && values) {
        // value columns: written transposed, vt[(b dim + c)][token].  A thread takes one column and 8
        // consecutive tokens (one 16-byte store); consecutive threads take consecutive token groups of
        // the same column, so a column's BM tokens leave as one contiguous run.
        constexpr int RGN = BM / 8;
        T* vt = reinterpret_cast<T*>(p.out2);
        for (int it = tid; it < BN * RGN; it += NT) {
            const int cc = it / RGN, rr = (it % RGN) * 8;
            const int r = m0 + rr, c2 = n0 + cc - 2 * p.dim;
            if (r >= p.M || n0 + cc >= p.N) continue;     // (128-column tiles: the last one of an odd multiple of 64 is half empty)
            const float bias = p.bias[n0 + cc], cs = has_ln ? p.ln_colsum[n0 + cc] : 0.0f;
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                v[k] = sC[at(rr + k, cc)];
#pragma unroll
                for (int q = 1; q < KG; ++q) v[k] += sC[q * BM * BN + at(rr + k, cc)];
                if (has_ln) {
                    const f32x2 st = row_stats(rr + k);
                    v[k] = st[1] * (v[k] - st[0] * cs);
                }
                v[k] += bias;
            }
            store_tokens8<T>(p, vt, r, c2, v);
        }
        return;
    }
    if constexpr (EPI == EPI_ROWDOT) {
        // 8 consecutive lanes hold the 8 chunks of one 64-column group of a row: every lane takes part in
        // the exchange (out-of-range rows / columns contribute zero), the first lane of a group writes
        const int c = n0 + cg * 8;
        float* out = reinterpret_cast<float*>(p.out);
        for (int rr = rr0; rr < BM; rr += RPASS) {
            const int r = m0 + rr;
            float sum = 0.0f;
            if (r < p.M && c < p.N) {
                float v[8];
                tile8(rr, cg * 8, v);
                sum = rowdot_chunk(p, c, v);
            }
            sum += __shfl_xor(sum, 1);
            sum += __shfl_xor(sum, 2);
            sum += __shfl_xor(sum, 4);
            if ((cg & 7) == 0 && r < p.M && c < p.N) out[(int64_t)r * p.ldo + (c >> 6)] = sum;
        }
        return;
    }
    if (SPARE && rr0 >= BM) return;
#pragma unroll 1
    for (int b = 0; b < PASSES; b += NB) {
        EpiRow now[NB];
#pragma unroll
        for (int n = 0; n < NB; ++n) now[n] = rows[n];
        if (b + NB < PASSES) {                           // the next batch's operands, ahead of this batch's stores
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                const int r = m0 + rr0 + (b + NB + n) * RPASS;
                rows[n] = epilogue_row_operands<EPI>(p, cols, r, r < p.M && cols.nv > 0);
            }
        }
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            const int rr = rr0 + (b + n) * RPASS;
            const bool active = m0 + rr < p.M && cols.nv > 0;
            float v[8];
            tile8(rr, cg * 8, v);
            if (has_ln) ln_apply(row_stats(rr), cols.g0, cols.g1, v);
            if (active) epilogue_chunk<T, EPI>(p, cols, now[n], v);
            if (EPI == EPI_RESID || EPI == EPI_PATCH) group_stats<T, BN % 64 ? 32 : 64>(p, cols, now[n], v, active, cg & (BN % 64 ? 3 : 7));
        }
    }
}

}  // namespace vpe

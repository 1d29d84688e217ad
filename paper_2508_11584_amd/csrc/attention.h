// Flash-style softmax attention for head_dim 64 on gfx950 (non-causal, all keys).
//
// Each wave owns 32 queries and walks the keys in tiles of 64.  The score tile is computed
// TRANSPOSED, S^T = K Q^T, so that in the 32x32 MFMA accumulator layout a lane holds 16 keys of
// ONE query (its column): the running max / sum of the online softmax are then in-lane
// reductions plus a single exchange between the two lane halves.  The probabilities stay in
// registers and feed the second product O^T = V^T P^T directly as its B operand; the A operand
// V^T comes from the transposed value buffer the QKV GEMM epilogue wrote (keys contiguous).
//
//   qk  [B*N][2*dim]  queries | keys, head h at columns 64h..64h+63 of each half
//   vt  [B*dim][npad] values transposed, npad = N rounded up to 64, padding columns zero
//   out [B*N][dim]
#pragma once
#include <type_traits>

#include "common.h"
#include "gemm.h"
#include "layernorm.h"
#include "split3.h"

namespace vpe {

// The loader prefetches one iteration (KW key tiles) ahead without clamping, so a workgroup with KW key waves
// reads up to 2 KW 64 key rows past the last token of qk and as many elements past the end of vt (tiles that do
// not exist); both buffers must be readable that far.  What is read there is never used.  `pad` states how many
// rows of qk / elements of vt past their ends the caller made readable; a launch whose shape needs more is refused.
constexpr int ATTN_MAX_KW = 4;                        // widest key split of any instantiation
constexpr int ATTN_PAD = 2 * ATTN_MAX_KW * 64;        // rows / elements a caller has to provide for any shape
// LayerNorm of rows that the launch normalises beside the attention, with workgroups of its own behind the others (x null: none):
// a feature map is tapped between two blocks, and the residual stream stands still until the next block's out-projection.
struct RowNorm {
    const float* x;      // [rows][D]
    const float* gain;
    const float* bias;
    void* out;           // T [rows][D]
    int rows, D;
    float eps;
    int blocks;          // (filled in by the launcher)
};
// Memory that the launch reads once for the sake of the memory-side cache, with workgroups of its own: the weights of the products that
// follow, of models whose weights do not stay there from frame to frame.  Whole KB each (the rest of a KB is not read).
struct Touch {
    const void* at[3];
    uint32_t kb[3];
    int blocks;          // 0: none
};
struct AttnArgs {
    const void* qk;
    const void* vt;
    void* out;
    int B, N, npad, dim, heads;
    float scale_log2e;   // (1 / sqrt(64)) * log2(e): factor of the raw scores; 1 where the queries carry it already (bf16: GemmArgs::q_scale)
    int pad;             // readable rows of qk / elements of vt past their ends
    int shared_gpu;      // the launch runs beside other streams' kernels (several encoder lanes): prefer a shape that
                         // leaves room on its CUs over the fastest one on an empty GPU
    RowNorm norm;
    Touch touch;
};

// Exchange between the two halves of a wave without going through LDS (v_permlane32_swap): both operands are the
// lane's own value, after the swap one holds the lower half's values in all 64 lanes and the other the upper half's.
__device__ __forceinline__ float halves_max(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float halves_sum(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// --- per-type pieces: fragments for S^T = K Q^T and O^T = V^T P^T over a block of 32 keys
template <typename T> struct AttnMma;

template <> struct AttnMma<bf16> {
    static constexpr int QF = 4;                  // q fragments per lane (4 k-steps of 16 over dh = 64)
    typedef bf16x8 QFrag;
    static constexpr int ROWB = 128;              // bytes per 64-element row
    static __device__ __forceinline__ int chunk_at(int row, int chunk) { return swz(row, chunk); }   // where a row's chunk is stored
    static __device__ __forceinline__ QFrag load_q(const bf16* qrow, int ks, int g) {
        return *reinterpret_cast<const QFrag*>(qrow + 16 * ks + 8 * g);
    }
    static __device__ __forceinline__ QFrag zero_q() { return QFrag{0, 0, 0, 0, 0, 0, 0, 0}; }
    // Both 32-key blocks of a tile at once: S0^T, S1^T = K[0..31], K[32..63] times Q^T.  The two accumulation chains
    // alternate (consecutive MFMAs are independent) and the K fragments of k-step ks + 1 are read while the MFMAs of
    // step ks run, instead of read - wait - multiply eight times in a row.
    static __device__ __forceinline__ void qk2(f32x16& s0, f32x16& s1, const char* sK, int li, const QFrag* q, int g) {
        // Accumulator row r of the score block is fed from key row pi(r) = r with bits 2 and 3 exchanged: lane half g
        // then holds, for k-step s of the second product, the eight CONSECUTIVE keys 16 s + 8 g .. + 7 (see pv_tile)
        const int kr = (li & 0x13) | ((li & 8) >> 1) | ((li & 4) << 1);
        const int sw = (kr >> 1) & 7;                      // rows kr and kr + 32 share the swizzle term
        const char* r0 = sK + kr * 128;
        const char* r1 = r0 + 32 * 128;
        bf16x8 a[2][2];
        a[0][0] = *reinterpret_cast<const bf16x8*>(r0 + ((g ^ sw) * 16));
        a[0][1] = *reinterpret_cast<const bf16x8*>(r1 + ((g ^ sw) * 16));
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            if (ks < 3) {
                a[(ks + 1) & 1][0] = *reinterpret_cast<const bf16x8*>(r0 + (((2 * ks + 2 + g) ^ sw) * 16));
                a[(ks + 1) & 1][1] = *reinterpret_cast<const bf16x8*>(r1 + (((2 * ks + 2 + g) ^ sw) * 16));
            }
            __builtin_amdgcn_sched_barrier(0);         // the reads above stay ahead of the MFMAs below
            s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks & 1][0], q[ks], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks & 1][1], q[ks], s1, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // Key (within its 32-key block) of accumulator element v of the score block in lane half g, under the row
    // permutation of qk2.
    static __device__ __forceinline__ int key_of(int v, int g) { return 16 * (v >> 3) + 8 * g + (v & 7); }
    // O^T (64 dh x 32 queries, two accumulators) += V^T[dh][64 keys] P^T, and the row sums of P.  Four k-steps of 16
    // keys; the k slot (g, kk) of step (kb, s) is key 32 kb + 16 s + 8 g + kk -- where accumulator element
    // v = 8 s + kk of score block kb sits, so P needs no shuffle, and a lane's eight keys are one 16-byte chunk of
    // a V^T row (one conflict-free ds_read_b128 per accumulator and step).  The reads of step + 1 are issued before
    // the MFMAs of step.
    // Row sums (sum2) take the same rounded probabilities as the numerator, two keys per instruction.  On the matrix pipe,
    // as a product with ones, they were a fifth of its work and 20 registers (ViT-g x 8, references that move: 122.2 -> 116.6 us, with the
    // vector work before, between and behind the MFMAs below instead of behind each of them 116.1).
    // `sc` holds the raw scores; element e becomes 2^(sc[e] * scale - ref), DONE: 2^sc[e].  The exponentials of step + 1 are issued
    // behind the MFMAs of step, so the vector pipe works on them while the matrix pipe runs.  psum
    // receives the lane's sum of probabilities.
    static __device__ __forceinline__ float sum2(bf16x8 b, float sum) {
        const bf16x2 one = {(bf16)1.0f, (bf16)1.0f};
#pragma unroll
        for (int kk = 0; kk < 8; kk += 2) sum = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{b[kk], b[kk + 1]}, one, sum, false);
        return sum;
    }
    template <bool DONE = false>
    static __device__ __forceinline__ void pv_tile(f32x16& o0, f32x16& o1, float& psum, const char* sV, int li,
                                                   f32x16* sc, float scale, float ref, int g) {
        const int sw = (li >> 1) & 7;                      // rows li and li + 32 share the swizzle term
        const char* r0 = sV + li * 128;
        const char* r1 = r0 + 32 * 128;
        auto probs = [&](int st) {
            bf16x8 b;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const float x = sc[st >> 1][8 * (st & 1) + kk];
                const float e = __builtin_amdgcn_exp2f(DONE ? x : fmaf(x, scale, -ref));
                b[kk] = (bf16)e;
            }
            psum = sum2(b, psum);
            return b;
        };
        bf16x8 a[2][2], b[2];
        a[0][0] = *reinterpret_cast<const bf16x8*>(r0 + ((g ^ sw) * 16));
        a[0][1] = *reinterpret_cast<const bf16x8*>(r1 + ((g ^ sw) * 16));
        b[0] = probs(0);
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            if (st < 3) {
                a[(st + 1) & 1][0] = *reinterpret_cast<const bf16x8*>(r0 + (((2 * st + 2 + g) ^ sw) * 16));
                a[(st + 1) & 1][1] = *reinterpret_cast<const bf16x8*>(r1 + (((2 * st + 2 + g) ^ sw) * 16));
            }
            __builtin_amdgcn_sched_barrier(0);
            o0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[st & 1][0], b[st & 1], o0, 0, 0, 0);
            o1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[st & 1][1], b[st & 1], o1, 0, 0, 0);
            if (st < 3) b[(st + 1) & 1] = probs(st + 1);
            // the next step's exponentials, conversions and sums before, between and behind the two MFMAs
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x402, 4, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x402, 8, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// fp32: every operand as three bf16 terms (Split3), six MFMAs per product block.  Queries are split once, keys and values by
// each wave as it reads them, probabilities in registers.  The score block's rows are permuted as in the bf16 form, so a
// lane's eight probabilities of a k-step are eight consecutive keys here too.  With v_mfma_f32_32x32x2_f32 a 64-key tile
// is 8192 clocks of a wave's matrix pipe, split 3072 and about 750 vector instructions.
template <> struct AttnMma<float> {
    static constexpr int QF = 4;                  // 4 steps of 16 dh
    typedef Split3 QFrag;
    static constexpr int ROWB = 256;
    // a row covers all 64 banks: 16 rows of one logical chunk fall on 16 different 16-byte groups
    static __device__ __forceinline__ int chunk_at(int row, int chunk) { return chunk ^ (row & 15); }
    static __device__ __forceinline__ Split3 load_split(const char* tile, int row, int chunk) {
        return split3(*reinterpret_cast<const f32x4*>(tile + (row * 16 + chunk_at(row, chunk)) * 16),
                      *reinterpret_cast<const f32x4*>(tile + (row * 16 + chunk_at(row, chunk + 1)) * 16));
    }
    static __device__ __forceinline__ QFrag load_q(const float* qrow, int ks, int g) {
        return split3(*reinterpret_cast<const f32x4*>(qrow + 16 * ks + 8 * g), *reinterpret_cast<const f32x4*>(qrow + 16 * ks + 8 * g + 4));
    }
    static __device__ __forceinline__ QFrag zero_q() { return split3(f32x4{0, 0, 0, 0}, f32x4{0, 0, 0, 0}); }
    static __device__ __forceinline__ void qk2(f32x16& s0, f32x16& s1, const char* sK, int li, const QFrag* q, int g) {
        const int kr = (li & 0x13) | ((li & 8) >> 1) | ((li & 4) << 1);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const Split3 a0 = load_split(sK, kr, 4 * ks + 2 * g), a1 = load_split(sK, kr + 32, 4 * ks + 2 * g);
#pragma unroll
            for (int t = 0; t < 6; ++t) {
                s0 = split_mma(t, a0, q[ks], s0);
                s1 = split_mma(t, a1, q[ks], s1);
            }
        }
    }
    static __device__ __forceinline__ int key_of(int v, int g) { return 16 * (v >> 3) + 8 * g + (v & 7); }
    static __device__ __forceinline__ void pv_tile(f32x16& o0, f32x16& o1, float& psum, const char* sV, int li,
                                                   f32x16* sc, float scale, float ref, int g) {
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            f32x4 p[2];
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const float e = __builtin_amdgcn_exp2f(fmaf(sc[st >> 1][8 * (st & 1) + kk], scale, -ref));
                psum += e;
                p[kk >> 2][kk & 3] = e;
            }
            const Split3 b = split3(p[0], p[1]);
            const Split3 a0 = load_split(sV, li, 4 * st + 2 * g), a1 = load_split(sV, li + 32, 4 * st + 2 * g);
#pragma unroll
            for (int t = 0; t < 6; ++t) {
                o0 = split_mma(t, a0, b, o0);
                o1 = split_mma(t, a1, b, o1);
            }
        }
    }
};

// The same blocks on v_mfma_f32_32x32x2_f32, one instruction per k element of a lane half: for workgroups whose values the
// split does not hold.
struct AttnMmaF32 : AttnMma<float> {
    struct QFrag { f32x4 c[2]; };
    static __device__ __forceinline__ f32x4 load_chunk(const char* tile, int row, int chunk) {
        return *reinterpret_cast<const f32x4*>(tile + (row * 16 + chunk_at(row, chunk)) * 16);
    }
    static __device__ __forceinline__ QFrag load_q(const float* qrow, int ks, int g) {
        return {{*reinterpret_cast<const f32x4*>(qrow + 16 * ks + 8 * g), *reinterpret_cast<const f32x4*>(qrow + 16 * ks + 8 * g + 4)}};
    }
    static __device__ __forceinline__ QFrag zero_q() { return {{f32x4{0, 0, 0, 0}, f32x4{0, 0, 0, 0}}}; }
    static __device__ __forceinline__ void qk2(f32x16& s0, f32x16& s1, const char* sK, int li, const QFrag* q, int g) {
        const int kr = (li & 0x13) | ((li & 8) >> 1) | ((li & 4) << 1);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const f32x4 a0 = load_chunk(sK, kr, 4 * (c >> 1) + 2 * g + (c & 1)), a1 = load_chunk(sK, kr + 32, 4 * (c >> 1) + 2 * g + (c & 1));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[e], q[c >> 1].c[c & 1][e], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[e], q[c >> 1].c[c & 1][e], s1, 0, 0, 0);
            }
        }
    }
    static __device__ __forceinline__ void pv_tile(f32x16& o0, f32x16& o1, float& psum, const char* sV, int li,
                                                   f32x16* sc, float scale, float ref, int g) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const f32x4 a0 = load_chunk(sV, li, 4 * (c >> 1) + 2 * g + (c & 1)), a1 = load_chunk(sV, li + 32, 4 * (c >> 1) + 2 * g + (c & 1));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float pe = __builtin_amdgcn_exp2f(fmaf(sc[c >> 2][4 * (c & 3) + e], scale, -ref));
                psum += pe;
                o0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[e], pe, o0, 0, 0, 0);
                o1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[e], pe, o1, 0, 0, 0);
            }
        }
    }
};

// Workgroup shape: QW x KW waves.  Wave (qw, kw) owns QB blocks of 32 queries (query group qw) and
// the key tiles t with t % KW == kw.  Each iteration stages KW key tiles and KW value tiles in LDS,
// loaded by all threads; waves of the same kw share their tile across query groups.  At the end
// the KW partial results of a query group are merged in LDS (fixed order, so results are
// deterministic): by its kw = 0 wave for two, a share by each wave for four.  KW > 1 gives small problems
// enough waves to fill 1024 SIMDs; QW > 1 and QB = 2 cut the L2 -> LDS traffic per query on large ones.
// Launch bound: at least two waves per SIMD wherever the kernel fits 256 registers.  Besides the occupancy, this
// is what makes the compiler keep the MFMA accumulators in ordinary vector registers: with up to 512 registers
// allowed it places them in the accumulation-register file, and since the softmax works on the scores with
// vector instructions every tile then pays ~190 register-file moves per lane (measured on the four-wave shapes:
// 158 + 48 registers and 300 vector instructions per tile without the bound, 164 + 0 and 105 with it).  (2,1,4)
// would spill under the bound and keeps the old one.  The bf16 (1,4,1) shape has LDS for five workgroups on a CU and
// is held to 168 registers, three waves per SIMD (at 128 a query block's references have to be subtracted from the scores: ViT-L x 4
// 42.4 us against 39.3, ViT-g x 8 113 against 108).
template <typename T, int KW>
constexpr bool attn_double_buffered() { return 2 * KW * 2 * 64 * AttnMma<T>::ROWB <= 128 * 1024; }

// LDS of the tiles or, when they are done with, of the merge; fp32 shapes have a flag per wave behind it.
template <typename T, int QB, int QW, int KW>
constexpr int attn_lds() {
    constexpr int kv = (attn_double_buffered<T, KW>() ? 2 : 1) * KW * 2 * 64 * AttnMma<T>::ROWB, red = KW > 1 ? KW * QW * QB * 34 * 64 * 4 : 0;
    return kv > red ? kv : red;
}

// Do a query's exponentials keep the reference of its wave's first tile (bf16; two blocks of queries have no registers for it)?
template <typename T, int QB>
constexpr bool attn_fixed_reference() { return sizeof(T) == 2 && QB == 1; }

template <typename T, int QB, int QW, int KW>
constexpr int attn_min_waves() {
    return QW * KW == 4 && QB == 2 ? 1 : sizeof(T) == 2 && QB == 1 && KW == 1 ? 3 : 2;
}

// RIDERS: with a RowNorm's or a Touch's workgroups (an instantiation of its own: the look at their number is 0.25 us of every launch).
template <typename T, int QB, int QW, int KW, bool FIXED, bool RIDERS>
__global__ __launch_bounds__(64 * QW * KW, (attn_min_waves<T, QB, QW, KW>())) void attention_kernel(const AttnArgs p) {
    constexpr int NW = QW * KW, NT = 64 * NW;
    static_assert(KW <= ATTN_MAX_KW, "the loader's overshoot is budgeted for at most ATTN_MAX_KW key waves");
    constexpr int CE = Elem<T>::CE;
    constexpr int CPR = 64 / CE;                 // 16-byte chunks per 64-element row
    constexpr int ROWB = AttnMma<T>::ROWB;
    constexpr int TILE = 64 * ROWB;
    constexpr int STAGE = KW * 2 * TILE;         // K and V tiles of one iteration
    constexpr bool DB = attn_double_buffered<T, KW>();
    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qw = wave % QW, kw = wave / QW;
    const int g = lane >> 5, li = lane & 31;
    // One-dimensional grid, (image, head)-major: the hardware deals consecutive workgroups round-robin to the 8 XCDs,
    // so ids are remapped to give each XCD one contiguous range -- all query blocks of an (image, head) pair then run
    // on the same XCD and its keys and values are fetched into that L2 once, not into all eight (measured at ViT-g x8:
    // 615 MB fetched per launch against 135 MB of operands before the remapping).
    const int nqb = cdiv(p.N, 32 * QB * QW), tasks = gridDim.x - (RIDERS ? p.touch.blocks + p.norm.blocks : 0);
    if (RIDERS && (int)blockIdx.x >= tasks) {
        const int rider = blockIdx.x - tasks;
        if (rider < p.touch.blocks) {
            // straight to LDS, one KB of it a wave: no registers, up to 63 loads of a wave on their way
#pragma unroll 1
            for (int s = 0; s < 3; ++s)
                for (uint32_t k = rider * NW + wave; k < p.touch.kb[s]; k += p.touch.blocks * NW)
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(reinterpret_cast<const char*>(p.touch.at[s]) + k * 1024ull + lane * 16),
                                                     (__attribute__((address_space(3))) void*)(smem + wave * 1024), 16, 0, 0);
            __builtin_amdgcn_s_waitcnt(0x0F70);            // (the LDS is this workgroup's until the loads have landed)
            return;
        }
        for (int row = (rider - p.touch.blocks) * NW + wave; row < p.norm.rows; row += p.norm.blocks * NW)
            layernorm_row(p.norm.x, row, p.norm.D, p.norm.gain, p.norm.bias, p.norm.eps, reinterpret_cast<T*>(p.norm.out), lane);
        return;
    }
    const int lin = xcd_contiguous(blockIdx.x, tasks);
    const int bh = lin / nqb, b = bh / p.heads, h = bh % p.heads;
    const int q0 = (lin % nqb) * (32 * QB * QW) + qw * 32 * QB;
    const int ld = 2 * p.dim;

    const T* __restrict__ qk = reinterpret_cast<const T*>(p.qk) + (int64_t)b * p.N * ld + h * 64;
    const T* kbase = qk + p.dim;
    const T* vt = reinterpret_cast<const T*>(p.vt) + ((int64_t)b * p.dim + h * 64) * p.npad;

    f32x16 o[QB][2];
    float m_run[QB], l_run[QB];                        // (denominators: per lane half)

    const int KT = p.npad / 64;
    const int NIT = (KT + KW - 1) / KW;
    // Tiles are loaded straight into LDS (global_load_lds_dwordx4: no staging registers, no ds_write).
    // One instruction of a wave fills 1 KB = RPI consecutive rows of a tile; lane l lands on row l / CPR, physical
    // chunk l % CPR of that row group, so it fetches the logical chunk that belongs there under the swizzle.
    // Instruction i of wave w fills slot w + NW i of the stage (tile i / PPT, pass i % PPT over its row groups):
    // a lane's row within the tile is (w + NW pass) RPI + l / CPR -- the passes differ by multiples of 16 rows, which
    // leave the swizzle term unchanged, so one logical chunk and two thread pointers serve every instruction.
    constexpr int RPI = 1024 / ROWB, G = TILE / 1024;  // rows per instruction, instructions per tile
    constexpr int PPT = G / NW > 0 ? G / NW : 1;       // passes of the workgroup over one tile
    constexpr int NDMA = KW * 2 * G / NW;              // instructions per wave per iteration
    constexpr int KEYS = 1, VALUES = 2;
    static_assert(G % NW == 0 && (NW * RPI) % 16 == 0, "loader mapping: a tile is whole passes of the workgroup");
    const int drow = wave * RPI + lane / CPR;
    const int dlc = AttnMma<T>::chunk_at(drow, lane % CPR);          // (exclusive or with the row's term: its own inverse)
    // Scalar addresses of the rows and 32 bits of a lane's own offset.  As constants of the key loop the compiler keeps an iteration's
    // row addresses and places in LDS in scalar registers; of 16 and more instructions it spills up to 149 of them, 64 moves an
    // iteration of fp32 (1,1,4).  There they run (RUN): keys down their rows, values down a tile's rows and on to the next tile,
    // opaque after every step (us, held / running: fp32 54 pairs 12.6 / 11.9, 288 41.8 / 41.4, 1032 117.2 / 115.9; bf16 54 pairs
    // 5.9 / 5.6).  Shapes of up to eight are faster with held ones (fp32 (1,4,1) 3096 pairs 716 / 721, bf16 (1,2,2) 516 16.6 / 16.7).
    constexpr bool RUN = NDMA > 8;
    typedef __attribute__((address_space(3))) char LdsChar;
    const uint32_t koff = (uint32_t)(drow * ld + dlc * CE) * sizeof(T), voff = (uint32_t)(drow * p.npad + dlc * CE) * (uint32_t)sizeof(T);
    auto load = [&](const char* src, LdsChar* dst) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    };
    auto dma = [&](char* base, int it, int kinds) {    // tiles of iteration `it` into the stage at `base`: KEYS, VALUES or both
        const int64_t ka = (int64_t)it * KW * 64 * ld;
        const int va = it * KW * 64;
        if constexpr (RUN) {
            const int64_t kstep = (int64_t)NW * RPI * ld, vstep = (int64_t)NW * RPI * p.npad;
            const T* krow = kbase + ka;
            const T* vtile = vt + va;
            const T* vrow = vtile;
            LdsChar* dst = (LdsChar*)(base + wave * 1024);
#pragma unroll
            for (int i = 0; i < NDMA; ++i, dst += NW * 1024) {
                const int which = (i / PPT) & 1, pass = i % PPT;
                if (!((kinds >> which) & 1)) continue;
                asm("" : "+s"(dst));
                load(reinterpret_cast<const char*>(which ? vrow : krow) + (which ? voff : koff), dst);
                if (!which) {
                    krow += kstep;
                    asm("" : "+s"(krow));
                } else if (pass + 1 < PPT) {
                    vrow += vstep;
                    asm("" : "+s"(vrow));
                } else {
                    vtile += 64;
                    vrow = vtile;
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < NDMA; ++i) {
                const int ti = i / PPT, j = ti >> 1, which = ti & 1, r0 = (i % PPT) * NW * RPI;
                if (!((kinds >> which) & 1)) continue;
                const T* row = which ? vt + (int64_t)r0 * p.npad + j * 64 + va : kbase + (int64_t)(j * 64 + r0) * ld + ka;
                load(reinterpret_cast<const char*>(row) + (which ? voff : koff), (LdsChar*)(base + (wave + NW * i) * 1024));
            }
        }
    };
    // Two buffers: the loads of iteration it + 1 are issued at the top of iteration it into the buffer that was read
    // in iteration it - 1, and one barrier per iteration is enough (everyone has finished reading buffer b, and the
    // loads into buffer b ^ 1 have landed).  Shapes whose two buffers would not fit the CU's LDS have one, and each half of it
    // is loaded while the other is multiplied: behind the barrier that ends the scores the next keys, behind the one that
    // ends the values the next values (staged in registers, 128 of a lane's 422, fp32 ViT-S 224x224 took 13.85 us, now 12.65).
    // All tiles from the start: scores, softmax and values with the product blocks of M.
    // FIXED (the kernel's first sweep; `fixed` here): every query's reference is the maximum of its wave's first tile and stays.  A probability only has to be
    // representable: up to 2^64 above the reference fp32 sums and bf16 probabilities are as precise as at 2^0, so no later tile looks for a
    // maximum, and the reference is what its products start from (-reference in the accumulators: the scores leave the matrix pipe as
    // exponents).  A workgroup that met more than that starts again with references that move.  A wave of ViT-g (22 tiles) issues
    // 2717 vector instructions instead of 3710, its 352 products included (us, references that move / that stay: ViT-S
    // 1531 tokens 12.4 / 11.5, ViT-B 1370 17.0 / 15.6, ViT-L 1374 17.8 / 16.8, x 4 43.1 / 39.3, ViT-g x 8 118 / 108).
    // Not further than 2^64: waves' sums meet in a merge whose factors, 2^(difference of references), underflow from 2^-126 on, and
    // a sum that is dropped there has to be nothing beside the other's.
    // Starting again costs the launch a second sweep, as long as a workgroup of every round of the CUs does it (us, flat scores / one query
    // of every head above 2^64 / all; with references that move always: ViT-S 476x476 9.0 / 15.6 / 16.1; 9.3, 476x630 11.9 / 20.9 / 21.3; 12.6,
    // ViT-B 518x518 16.1 / 25.1 / 29.6; 17.3, ViT-L x 4 39.9 / 54.0 / 74.3; 43.3, ViT-g x 8 108 / 130 / 219; 120).  It takes a score 44
    // (64 in log2 units) above all of a wave's first 64 keys.
    auto sweep = [&](auto mma, auto fixed) {
        using M = decltype(mma);
        constexpr bool FIRST = decltype(fixed)::value;
        f32x16 start[FIRST ? QB : 1];                   // -reference, what a score block's products start from
        typename M::QFrag q[QB][4];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int qi = q0 + qb * 32 + li;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                q[qb][ks] = qi < p.N ? M::load_q(qk + (int64_t)qi * ld, ks, g) : M::zero_q();
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            m_run[qb] = -INFINITY;
            l_run[qb] = 0.0f;
            if constexpr (FIRST) {
#pragma unroll
                for (int v = 0; v < 16; ++v) start[qb][v] = 0.0f;
            }
#pragma unroll
            for (int d = 0; d < 2; ++d)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[qb][d][v] = 0.0f;
        }
        if constexpr (DB) dma(smem, 0, KEYS | VALUES); else dma(smem, 0, KEYS);
        __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): the loads into LDS have landed
        __syncthreads();
        if constexpr (!DB) dma(smem, 0, VALUES);
        // Scores of query block qb against tile t, and the reference that their exponentials are taken against
        auto scores = [&](f32x16* s, int qb, int t, const char* sK) {
            const bool last = t == KT - 1;                 // keys past N only exist in the last tile
            if constexpr (FIRST) {
                s[0] = s[1] = start[qb];
            } else {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int v = 0; v < 16; ++v) s[kb][v] = 0.0f;
            }
            // Waves of a SIMD are in different phases: the one with products to issue goes first, the second products with
            // the exponentials among them before the first (no priorities / these, us: ViT-B 518x518 18.3 / 17.3,
            // ViT-L 19.2 / 18.4, x 4 49.2 / 47.8, ViT-g x 8 136.7 / 137.6, fp32 ViT-S 518x518 x 4 128.9 / 121.5).
            __builtin_amdgcn_s_setprio(1);
            M::qk2(s[0], s[1], sK, li, q[qb], g);
            if (last) {
                // (opaque: the 32 comparisons with it stay here and do not hold registers through the loop)
                int left = p.N - t * 64 - M::key_of(0, g);
                asm volatile("" : "+v"(left));
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        if (kb * 32 + M::key_of(v, 0) >= left) s[kb][v] = -INFINITY;
                    }
            }
            __builtin_amdgcn_s_setprio(0);
            if (FIRST && t >= KW) return;                  // (a wave's first tile is tile kw)
            float mx = s[0][0];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[kb][v]);
            mx = halves_max(mx);
            if constexpr (FIRST) {
                m_run[qb] = mx;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    start[qb][v] = -mx;
                    s[0][v] -= mx;
                    s[1][v] -= mx;
                }
                return;
            }
            // Lazy rescaling: m_run is the reference the exponentials are taken against (in log2 units), not
            // necessarily the running maximum.  It only moves when a query's maximum has grown by more than 8
            // (probabilities stay <= 2^8, exact in fp32 and harmless in bf16), which after the first tile is
            // rare -- and then the whole wave skips the 32 multiplications of the accumulator.  On the first
            // tile the reference is -inf, alpha = 0 and the (zero) accumulators are overwritten.
            const float mxs = mx * p.scale_log2e;
            const bool grow = mxs > m_run[qb] + 8.0f;
            if (__any(grow)) {
                const float m_new = grow ? mxs : m_run[qb];
                const float alpha = __builtin_amdgcn_exp2f(m_run[qb] - m_new);
                l_run[qb] *= alpha;
                m_run[qb] = m_new;
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v) o[qb][d][v] *= alpha;
            }
        };
        auto values = [&](f32x16* s, int qb, const char* sV) {
            float psum = 0.0f;
            __builtin_amdgcn_s_setprio(2);
            if constexpr (FIRST) M::template pv_tile<true>(o[qb][0], o[qb][1], psum, sV, li, s, 1.0f, 0.0f, g);
            else M::pv_tile(o[qb][0], o[qb][1], psum, sV, li, s, p.scale_log2e, m_run[qb], g);
            l_run[qb] += psum;
            __builtin_amdgcn_s_setprio(0);
        };
        // Eight waves issue 64 loads an iteration, 1024 clocks of the CU's address unit: keys and values apart, so that waves multiply
        // meanwhile (1531 tokens, 288 pairs 12.0 -> 11.6 us; shapes of four waves are faster with all loads ahead: 516 pairs 15.8 / 16.3)
        constexpr bool APART = NW > 4;
        for (int it = 0; it < NIT; ++it) {
            // (a wave without a tile in the last iteration still takes part in the barriers)
            if constexpr (DB) {
                const char* stage = smem + (it & 1) * STAGE;
                char* const next = smem + ((it + 1) & 1) * STAGE;
                if (it + 1 < NIT) dma(next, it + 1, APART ? KEYS : KEYS | VALUES);
                const int t = it * KW + kw;
                if (t < KT) {
                    const char* sK = stage + (kw * 2) * TILE;
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) {
                        f32x16 s[2];
                        scores(s, qb, t, sK);
                        if (APART && qb == 0 && it + 1 < NIT) dma(next, it + 1, VALUES);
                        values(s, qb, sK + TILE);
                    }
                } else if (APART && it + 1 < NIT) {
                    dma(next, it + 1, VALUES);
                }
            } else {
                static_assert(DB || QB == 1, "the scores of a query block wait for the values");
                const int t = it * KW + kw;
                const char* sK = smem + (kw * 2) * TILE;
                f32x16 s[2];
                if (t < KT) scores(s, 0, t, sK);
                __builtin_amdgcn_s_waitcnt(0x0F70);
                __syncthreads();
                if (it + 1 < NIT) dma(smem, it + 1, KEYS);
                if (t < KT) values(s, 0, sK + TILE);
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            if constexpr (!DB) {
                if (it + 1 < NIT) dma(smem, it + 1, VALUES);
            }
        }
    };
    sweep(AttnMma<T>{}, std::integral_constant<bool, FIXED>{});
    // A workgroup with a sum that the first sweep does not hold starts again.  FIXED: a row sum above 2^64 (a later tile's score
    // far above the reference) or an infinite or NaN one.  fp32: the split holds neither infinities nor finite values above
    // 3.396e38, NaN among their terms and with them in the sums; it starts again on the fp32 instructions.
    // Every wave leaves a flag; with four key waves their merge's barrier stands behind it (a barrier of its own: ViT-S 224x224
    // 5.6 -> 5.8 us).
    constexpr bool CHECKED = FIXED || sizeof(T) == 4;
    constexpr int PER = QB * (32 + 2) * 64;              // floats per wave that a merge takes: O (32 per lane), m, l
    constexpr int FLAGS = sizeof(T) == 4 ? attn_lds<T, QB, QW, KW>() : KW > 2 ? KW * QW * PER * 4 : 0;
    static_assert(!FIXED || FLAGS + 4 * NW <= attn_lds<T, QB, QW, KW>(), "flags lie behind what a merge writes");
    int* flags = reinterpret_cast<int*>(smem + FLAGS);
    auto leave_flag = [&] {
        float t[4] = {0.0f, 0.0f, 0.0f, 0.0f};            // NaN if any of the lane's sums is infinite or NaN
        bool again = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            t[0] = fmaf(l_run[qb], 0.0f, t[0]);
            if (FIXED) again |= l_run[qb] > 0x1p64f;
#pragma unroll
            for (int d = 0; d < 2; ++d)
#pragma unroll
                for (int v = 0; v < 16; ++v) t[v & 3] = fmaf(o[qb][d][v], 0.0f, t[v & 3]);
        }
        const float all = (t[0] + t[1]) + (t[2] + t[3]);
        const int any = __any(again || all != all);
        if (lane == 0) flags[wave] = any;
    };
    auto flagged = [&] {                                  // (behind a barrier)
        int redo = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) redo |= flags[w];
        return __builtin_amdgcn_readfirstlane(redo) != 0;
    };
    auto sweep_again = [&] {
        asm volatile("" : "+s"(kbase), "+s"(vt));         // (nothing of the first sweep's addresses is held for this one)
        __syncthreads();                                  // everyone has read the flags
        if constexpr (sizeof(T) == 4) sweep(AttnMmaF32{}, std::false_type{});
        else sweep(AttnMma<T>{}, std::false_type{});
    };

    if constexpr (KW > 2) {
        // Merge the KW partial (max, sum, O) triples of each query group, lane by lane and in a fixed order.  Every wave
        // leaves its triple in LDS and finishes 1 / KW of the group's output (one wave merging and storing it all left the
        // others idle; us, before / now: ViT-S 224x224 7.3 / 6.9, 476x630 13.7 / 13.3, fp32 224x224 13.9 / 13.3).
        constexpr int SL = 32 / KW;
        static_assert(SL % 4 == 0, "a wave's share is whole groups of four channels");
        float* red = reinterpret_cast<float*>(smem) + lane;
        float* own = red + (kw * QW + qw) * PER;
        auto leave_triple = [&] {                         // (every wave is done with the tiles: a sweep ends with a barrier)
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v) own[(qb * 34 + d * 16 + v) * 64] = o[qb][d][v];
                own[(qb * 34 + 32) * 64] = m_run[qb];
                own[(qb * 34 + 33) * 64] = l_run[qb];
            }
        };
        if (CHECKED) leave_flag();
        leave_triple();
        __syncthreads();
        if (CHECKED && __builtin_expect(flagged(), 0)) {
            sweep_again();
            leave_triple();
            __syncthreads();
        }
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const float* src = red + qw * PER + qb * 34 * 64;          // wave k's triple: + k QW PER
            float f[KW], m = -INFINITY, l = 0.0f, r[SL];
#pragma unroll
            for (int k = 0; k < KW; ++k) { f[k] = src[k * QW * PER + 32 * 64]; m = fmaxf(m, f[k]); }
#pragma unroll
            for (int k = 0; k < KW; ++k) {
                f[k] = __builtin_amdgcn_exp2f(f[k] - m);               // references are in log2 units
                l += src[k * QW * PER + 33 * 64] * f[k];
            }
#pragma unroll
            for (int e = 0; e < SL; ++e) {
                r[e] = 0.0f;
#pragma unroll
                for (int k = 0; k < KW; ++k) r[e] += src[k * QW * PER + (kw * SL + e) * 64] * f[k];
            }
            const float inv = 1.0f / halves_sum(l);
            const int qi = q0 + qb * 32 + li;
            if (qi < p.N) {
                T* orow = reinterpret_cast<T*>(p.out) + ((int64_t)b * p.N + qi) * p.dim + h * 64;
#pragma unroll
                for (int e = 0; e < SL; e += 4) {
                    const int c = kw * SL + e;                         // accumulator element: O^T row 32 (c / 16) + 8 (c % 16 / 4) + 4 g + c % 4
                    T* dst = orow + 32 * (c >> 4) + 8 * ((c & 15) >> 2) + 4 * g;
#pragma unroll
                    for (int i = 0; i < 4; ++i) dst[i] = from_f32<T>(r[e + i] * inv);
                }
            }
        }
        return;
    }

    if constexpr (CHECKED) {
        leave_flag();
        __syncthreads();
        if (__builtin_expect(flagged(), 0)) sweep_again();
    }

    if constexpr (KW == 2) {
        // two triples: the second wave's through LDS, merged and stored by the first (shared as above: ViT-B 20.0 against 19.7 us)
        float* red = reinterpret_cast<float*>(smem);
        __syncthreads();
        if (kw > 0) {
            float* dst = red + ((kw - 1) * QW + qw) * PER + lane;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v) dst[(qb * 34 + d * 16 + v) * 64] = o[qb][d][v];
                dst[(qb * 34 + 32) * 64] = m_run[qb];
                dst[(qb * 34 + 33) * 64] = l_run[qb];
            }
        }
        __syncthreads();
        if (kw > 0) return;
        for (int k = 1; k < KW; ++k) {
            const float* src = red + ((k - 1) * QW + qw) * PER + lane;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const float mk = src[(qb * 34 + 32) * 64], lk = src[(qb * 34 + 33) * 64];
                const float m_new = fmaxf(m_run[qb], mk);
                const float a = __builtin_amdgcn_exp2f(m_run[qb] - m_new);      // references are in log2 units
                const float bsc = __builtin_amdgcn_exp2f(mk - m_new);
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        o[qb][d][v] = o[qb][d][v] * a + src[(qb * 34 + d * 16 + v) * 64] * bsc;
                l_run[qb] = l_run[qb] * a + lk * bsc;
                m_run[qb] = m_new;
            }
        }
    }

    // each lane half summed its own keys; the query's denominator is the sum of both halves
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float l_tot = halves_sum(l_run[qb]);
        const float inv = 1.0f / l_tot;
        const int qi = q0 + qb * 32 + li;
        if (qi < p.N) {
            T* orow = reinterpret_cast<T*>(p.out) + ((int64_t)b * p.N + qi) * p.dim + h * 64;
#pragma unroll
            for (int d = 0; d < 2; ++d)
#pragma unroll
                for (int v4 = 0; v4 < 4; ++v4) {
                    // O^T rows (dh) 32 d + 8 v4 + 4 g .. + 3 of this lane's query
                    T* dst = orow + 32 * d + 8 * v4 + 4 * g;
#pragma unroll
                    for (int i = 0; i < 4; ++i) dst[i] = from_f32<T>(o[qb][d][4 * v4 + i] * inv);
                }
        }
    }
}

template <typename T, int QB, int QW, int KW, bool FIXED = attn_fixed_reference<T, QB>()>
static inline hipError_t launch_attention_variant(const AttnArgs& a, hipStream_t s, bool configure_only) {
    constexpr int lds = attn_lds<T, QB, QW, KW>() + (sizeof(T) == 4 ? 64 : 0);
    typedef void (*Kernel)(const AttnArgs);
    static const Kernel kernels[] = {&attention_kernel<T, QB, QW, KW, FIXED, false>, &attention_kernel<T, QB, QW, KW, FIXED, true>};
    static bool configured = false;       // opt in to more than 64 KB of LDS once per instantiation
    if (!configured) {
        for (Kernel k : kernels) {
            hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (rc != hipSuccess) return rc;
        }
        configured = true;
    }
    if (configure_only) return hipSuccess;
    if (a.pad < 2 * KW * 64 || a.npad % 64 || a.npad < a.N || a.dim != a.heads * 64) return hipErrorInvalidValue;
    AttnArgs args = a;
    args.norm.blocks = !a.norm.x ? 0 : cdiv(a.norm.rows, QW * KW) < 512 ? cdiv(a.norm.rows, QW * KW) : 512;       // a row per wave up to two per CU
    const int riders = args.norm.blocks + args.touch.blocks;
    hipLaunchKernelGGL(kernels[riders > 0], dim3(cdiv(a.N, 32 * QB * QW) * a.B * a.heads + riders), dim3(64 * QW * KW), lds, s, args);
    return hipGetLastError();
}

}  // namespace vpe

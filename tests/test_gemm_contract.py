"""Host-side checks of the GEMMs: k extents that the kernels' loops cannot do, and epilogues that the convolution kernels do
not carry, are refused before anything is launched; tile maps; the GELU of results that are rounded to bf16."""
import os
import subprocess

import paper_2508_11584_amd as vpe

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2508_11584_amd")

PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
using namespace vpe;
int main() {
    struct { int amode, K, cC; } refused[] = {{A_PLAIN, 32, 0}, {A_PLAIN, 96, 0}, {A_PLAIN, 0, 0}, {A_PLAIN, 608, 0},
                                              {A_CONV3, 9 * 32, 32}, {A_CONV3, 9 * 96, 96}, {A_CONV3, 576, 128}, {A_CONV3, 576, 32}};
    int bad = 0;
    for (auto& r : refused)
        for (int dtype = 0; dtype < 2; ++dtype) {
            GemmArgs a{};
            a.M = a.N = 64;
            a.K = r.K; a.cC = r.cC; a.cH = a.cW = 8;
            a.lda = a.ldo = 64; a.a_rpi = a.o_rpi = 64; a.nz = 1;
            const hipError_t rc = launch_gemm(dtype, a, r.amode, nullptr);
            if (rc != hipErrorInvalidValue) { printf("dtype %d mode %d K %d cC %d: %d\n", dtype, r.amode, r.K, r.cC, (int)rc); ++bad; }
        }
    for (int epi : {EPI_RESID, EPI_SWIGLU, EPI_QKV, EPI_PATCH}) {
        GemmArgs a{};
        a.M = a.N = 64;
        a.cC = 64; a.K = 9 * a.cC; a.cH = a.cW = 8;
        a.lda = a.ldo = 64; a.a_rpi = a.o_rpi = 64; a.nz = 1; a.epi = epi;
        const hipError_t rc = launch_gemm(1, a, A_CONV3, nullptr);
        if (rc != hipErrorInvalidValue) { printf("convolution with epilogue %d: %d\n", epi, (int)rc); ++bad; }
    }
    // the projection epilogue belongs to convolutions, the folded LayerNorm to the epilogues without a residual stream
    const float stats[2] = {0.0f, 1.0f};
    for (int epi : {EPI_RESID, EPI_PATCH, EPI_ROWDOT})
        for (int dtype = 0; dtype < 2; ++dtype) {
            GemmArgs a{};
            a.M = a.N = a.K = 64;
            a.lda = a.ldo = 64; a.a_rpi = a.o_rpi = 64; a.nz = 1; a.epi = epi;
            if (epi != EPI_ROWDOT) { a.ln_stats = stats; a.ln_groups = 1; }
            const hipError_t rc = launch_gemm(dtype, a, A_PLAIN, nullptr);
            if (rc != hipErrorInvalidValue) { printf("dtype %d, epilogue %d of a plain product: %d\n", dtype, epi, (int)rc); ++bad; }
        }
    return bad;
}
"""


def run_host_program(tmp_path, program, optimize="-O1"):
    """Compiles the host side of `program` against the kernels' headers, links it with the library and runs it: exit code 0."""
    vpe.load_library()                                   # (built already, or an error that says so)
    src, exe = tmp_path / "program.cpp", tmp_path / "program"
    src.write_text(program)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", optimize, "-w", "-I" + os.path.join(PKG, "csrc"), str(src),
                    "-x", "none", os.path.join(PKG, "libvpe.so"), "-Wl,-rpath," + PKG, "-o", str(exe)], check=True, capture_output=True)
    # no device: what is checked must come from the arguments alone, with a device as without one
    r = subprocess.run([str(exe)], capture_output=True, text=True, env={**os.environ, "HIP_VISIBLE_DEVICES": ""})
    assert r.returncode == 0, r.stdout + r.stderr


def test_gemm_launcher_refuses_what_its_kernels_do_not_have(tmp_path):
    run_host_program(tmp_path, PROGRAM, "-O0")


MAP_PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
using namespace vpe;
int main() {
    // every tile of a launch exactly once: the map's divisions by reciprocals, as the kernel does them, against divisions
    int bad = 0;
    for (int tiles_m : {1, 2, 5, 7, 8, 9, 15, 16, 17, 43, 250, 1023, 5000})
        for (int tiles_n : {1, 2, 3, 6, 18, 64, 129}) {
            const TileMap t = TileMap::make(tiles_m, tiles_n);
            auto quotient = [](uint32_t x, uint32_t d, uint32_t inv) { return inv ? (uint32_t)(((uint64_t)x * inv) >> 32) : x / d; };
            for (int lin = 0; lin < t.tiles; ++lin) {
                const int group = quotient(lin, t.per_group, t.inv_group), rem = lin - group * t.per_group, rows = tiles_m - group * TileMap::GM;
                if (group != lin / t.per_group) ++bad;
                if (rows > 1 && rows < TileMap::GM && (int)quotient(rem, rows, t.inv_last) != rem / rows) ++bad;
            }
        }
    if (TileMap::make(1 << 20, 1 << 10).inv_group) ++bad;      // (products past 32 bits: the kernel divides)
    printf("%d\n", bad);
    return bad != 0;
}
"""


def test_tile_map_reciprocals_are_exact(tmp_path):
    run_host_program(tmp_path, MAP_PROGRAM)


PLAN_PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
using namespace vpe;
int main() {
    int bad = 0, two = 0;
    auto check = [&](const GemmArgs& a, int amode) {
        const GemmPlan p = plan_gemm_bf16(a, amode);
        const int per_tile = amode == A_CONV3 ? a.cC : a.K;                 // what a k-tile has to divide
        for (int kind : {p.lead_kind, p.kind})
            if ((kind == 43 || kind == 33) && per_tile % 128) { printf("mode %d K %d cC %d N %d M %d: kind %d\n", amode, a.K, a.cC, a.N, a.M, kind); ++bad; }
        two += p.lead_kind != 0;
        if (p.lead_kind && (p.lead_rows <= 0 || p.lead_rows >= a.M || p.lead_rows % 32)) { printf("M %d: lead of %d rows\n", a.M, p.lead_rows); ++bad; }
    };
    for (int k = 64; k <= 4096; k += 64)
        for (int n : {21, 64, 128, 192, 256, 320, 576, 960, 1536, 3072})
            for (double m = 40; m < 3e5; m *= 1.07) {
                GemmArgs a{};
                a.M = (int)m; a.N = n; a.K = k; a.nz = 1;
                for (int epi : {EPI_STORE, EPI_RESID}) { a.epi = epi; check(a, A_PLAIN); }
                if (k > 1536) continue;
                a.epi = EPI_STORE; a.cC = k; a.K = 9 * k;
                check(a, A_CONV3);
            }
    printf("%d problems in two launches\n", two);
    return bad ? 1 : two == 0;
}
"""


def test_plans_use_tilings_whose_k_tiles_divide_the_problem(tmp_path):
    # 128-deep k-tiles (kinds 43 and 33) only where they divide K, of a convolution its channels, as the leading part of a
    # two-launch form, too; over k extents of odd and even multiples of 64
    run_host_program(tmp_path, PLAN_PROGRAM)


NARROW_PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
using namespace vpe;
int main() {
    int bad = 0, narrow = 0, wide = 0;
    for (int dtype = 0; dtype < 2; ++dtype)
        for (int k = 64; k <= 4096; k += 64)
            for (int n : {64, 192, 384, 768, 1024, 1536})
                for (double m = 1; m < 2e4; m *= 1.3) {
                    GemmArgs a{};
                    a.M = (int)m; a.N = n; a.K = k; a.nz = 1; a.epi = EPI_RESID;
                    const int group = stats_columns(dtype, a);
                    if (group != 32 && group != 64) ++bad;
                    if (group == 32 && ((dtype && k % 128) || (int64_t)cdiv(a.M, 32) * (n / 32) > 512)) { printf("dtype %d M %d N %d K %d\n", dtype, a.M, n, k); ++bad; }
                    (group == 32 ? narrow : wide) += 1;
                    for (int epi : {EPI_STORE, EPI_PATCH, EPI_QKV}) { a.epi = epi; if (stats_columns(dtype, a) != 64) { printf("epilogue %d\n", epi); ++bad; } }
                }
    // groups of 32 columns are refused where no tile leaves them
    for (int dtype = 0; dtype < 2; ++dtype)
        for (int kind = 0; kind < 3; ++kind) {
            GemmArgs a{};
            a.M = a.N = 64; a.K = kind == 1 ? 192 : 256; a.lda = a.ldo = 64; a.a_rpi = a.o_rpi = 64; a.nz = 1;
            a.epi = kind == 0 ? EPI_STORE : EPI_RESID; a.st_group = 32;
            if (kind == 2) { a.epi = EPI_STORE; a.cC = 64; a.K = 576; a.cH = a.cW = 8; }
            if (kind == 1 && !dtype) continue;                              // (fp32 k-tiles are 64 deep)
            const hipError_t rc = launch_gemm(dtype, a, kind == 2 ? A_CONV3 : A_PLAIN, nullptr);
            if (rc != hipErrorInvalidValue) { printf("dtype %d kind %d: %d\n", dtype, kind, (int)rc); ++bad; }
        }
    printf("%d narrow, %d wide\n", narrow, wide);
    return bad ? 1 : !narrow || !wide;
}
"""


def test_statistics_of_32_columns_only_where_a_tile_leaves_them(tmp_path):
    # residual products of both types over k extents of odd and even multiples of 64, one row to 20000: 32-column groups only for
    # whole k-tiles and up to two 32 x 32 tiles per CU, never for another epilogue; asked for elsewhere they are refused
    run_host_program(tmp_path, NARROW_PROGRAM)


CONV_PLAN_PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
using namespace vpe;
int main() {
    int bad = 0;
    struct { int cC, N, M; bool two; } towers[] = {{768, 512, 4216, false}, {768, 512, 4 * 33 * 33, false}, {1024, 512, 4 * 46 * 46, false},
                                                   {1536, 512, 5776, false}, {1536, 256, 8 * 39 * 39, false}, {1024, 512, 4232, true}};
    for (auto& t : towers) {
        GemmArgs a{};
        a.M = t.M; a.N = t.N; a.cC = t.cC; a.K = 9 * t.cC; a.nz = 1; a.epi = EPI_STORE; a.act = ACT_RELU;
        const GemmPlan p = plan_gemm_bf16(a, A_CONV3);
        if ((p.lead_kind != 0) != t.two) { printf("%d -> %d channels, %d pixels: lead %d of %d rows, rest %d\n", t.cC, t.N, t.M, p.lead_kind, p.lead_rows, p.kind); ++bad; }
    }
    // the two products that tests/test_gpu_parity.py runs in two launches
    for (int conv = 0; conv < 2; ++conv) {
        GemmArgs a{};
        a.M = conv ? 4232 : 2180; a.N = conv ? 512 : 1024; a.cC = 1024; a.K = conv ? 9 * 1024 : 4096; a.nz = 1;
        a.epi = conv ? EPI_STORE : EPI_RESID; a.act = conv ? ACT_RELU : ACT_NONE;
        const GemmPlan p = plan_gemm_bf16(a, conv ? A_CONV3 : A_PLAIN);
        if (p.lead_kind != 6 || p.lead_rows != (conv ? 4096 : 2048) || p.kind != 33) { printf("conv %d: lead %d of %d rows, rest %d\n", conv, p.lead_kind, p.lead_rows, p.kind); ++bad; }
    }
    return bad;
}
"""


def test_leading_parts_of_convolutions_count_what_a_whole_launch_counts(tmp_path):
    # detection towers just above a round of 64 x 128 tiles: their leading part carries the factor that tiles of up to 64
    # rows carry beside an encoder, so that two launches are taken only where they win by it
    run_host_program(tmp_path, CONV_PLAN_PROGRAM)


GELU_PROGRAM = r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include "gemm.h"
// the GELU of bf16 results as the kernel evaluates it (v_exp_f32 and v_rcp_f32: 1 ulp), and the form before it, erf as an odd
// polynomial on |x| <= 3, both in fp32
static float logistic(float v) {
    const float x = fminf(fmaxf(v, -vpe::GELU_LIMIT), vpe::GELU_LIMIT);
    return v * (1.0f / (1.0f + exp2f(vpe::gelu_exponent(x))));
}
static float polynomial(float v) {
    const float c[10] = {-4.469939086e-09f, 2.302152922e-07f, -5.322654488e-06f, 7.394709974e-05f, -7.009955007e-04f,
                         4.897189327e-03f, -2.645343542e-02f, 1.125671491e-01f, -3.760564327e-01f, 1.128376126e+00f};
    const float x = fminf(fabsf(v) * 0.70710678118654752f, 3.0f), t = x * x;
    float p = c[0];
    for (int i = 1; i < 10; ++i) p = fmaf(p, t, c[i]);
    return 0.5f * v * (1.0f + copysignf(fminf(p * x, 1.0f), v));
}
int main() {
    int bad = 0;
    for (int k = 0; k < 28; ++k) {                       // intervals of 0.25 up to 7, both signs
        const int n = 20000;
        double now = 0.0, before = 0.0, most = 0.0;
        for (int i = 0; i < 2 * n; ++i) {
            const float v = (i & 1 ? -1.0f : 1.0f) * (float)(0.25 * (k + (i / 2 + 0.5) / n));
            const double exact = 0.5 * v * erfc(-v / sqrt(2.0)), e = logistic(v) - exact, f = polynomial(v) - exact;
            now += e * e; before += f * f; most = fmax(most, fabs(e / v));
        }
        if (now > before || most > 6.5e-7) { printf("|v| from %g: rms %.2e, before %.2e, largest %.2e |v|\n", 0.25 * k, sqrt(now / (2 * n)), sqrt(before / (2 * n)), most); ++bad; }
    }
    const float inf = INFINITY;
    if (logistic(inf) != inf || logistic(-inf) != -inf || !std::isnan(logistic(NAN))) { printf("infinities or NaN\n"); ++bad; }
    return bad;
}
"""


def test_gelu_of_bf16_results_loses_nothing_on_any_interval(tmp_path):
    # rms error against 64 bits, before rounding to bf16: no larger than the polynomial's on any interval; 6.4e-7 |v| at most
    run_host_program(tmp_path, GELU_PROGRAM)

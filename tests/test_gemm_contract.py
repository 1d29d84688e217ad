"""Host-side checks of the GEMM launcher: k extents that its kernels' loops cannot do, and epilogues that its convolution kernels do
not carry, are refused before anything is launched."""
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
    return bad;
}
"""


def test_gemm_launcher_refuses_what_its_kernels_do_not_have(tmp_path):
    vpe.load_library()                                   # (built already, or an error that says so)
    src, exe = tmp_path / "contract.cpp", tmp_path / "contract"
    src.write_text(PROGRAM)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O0", "-w", "-I" + os.path.join(PKG, "csrc"), str(src),
                    "-x", "none", os.path.join(PKG, "libvpe.so"), "-Wl,-rpath," + PKG, "-o", str(exe)], check=True, capture_output=True)
    # no device: the refusal must come from the arguments alone, with a device as without one
    r = subprocess.run([str(exe)], capture_output=True, text=True, env={**os.environ, "HIP_VISIBLE_DEVICES": ""})
    assert r.returncode == 0, r.stdout + r.stderr


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
    vpe.load_library()
    src, exe = tmp_path / "map.cpp", tmp_path / "map"
    src.write_text(MAP_PROGRAM)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-w", "-I" + os.path.join(PKG, "csrc"), str(src),
                    "-x", "none", os.path.join(PKG, "libvpe.so"), "-Wl,-rpath," + PKG, "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, env={**os.environ, "HIP_VISIBLE_DEVICES": ""})
    assert r.returncode == 0, r.stdout + r.stderr

"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Error measure per tensor: max |gpu - oracle| / max |oracle|.
Gates: fp32 path <= 1e-4; bf16 path <= 2e-2 on features / logits / depth and >= 0.99 agreement
of the segmentation and detection class maps (the oracle's argmax is taken on its fp64 scores).
Depth maps: the same measure; both it and the error relative to the map before its final ReLU are printed,
and a map that the ReLU clips (its maximum below a quarter of the pre-ReLU magnitude: with random weights
that happens) is held to the second form instead (helpers.depth_gate).
"""
import math

import numpy as np
import pytest
import torch

import paper_2508_11584_amd as vpe
import vpe_inputs as vi
from helpers import depth_errs, depth_gate, make_engine, relerr
from oracle import model, ops

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def run_gpu(eng, images, n_heads):
    """One frame through encode + all heads; returns (features [4 x (B,N,D)], head outputs)."""
    img = torch.from_numpy(images).cuda().contiguous()
    fh = eng.encode(img)
    for h in range(n_heads):
        assert eng.run_head(h, fh) == 0
    eng.sync()
    feats = [eng.feat_view(fh, k).float().cpu().numpy() for k in range(4)]
    return fh, feats


def regret(scores, ref_cls, got_cls):
    """max over positions of oracle score of the oracle's class minus oracle score of the GPU's class."""
    s = np.asarray(scores)
    a = np.take_along_axis(s, np.asarray(ref_cls, dtype=np.int64)[None], 0)[0]
    b = np.take_along_axis(s, np.asarray(got_cls, dtype=np.int64)[None], 0)[0]
    return float(np.max(a - b))


def head_outputs(eng, kinds):
    """Host copies of every output of every head: [[output 0, output 1 (class map, if the head has one)], ...]."""
    return [[eng.head_output(hi, which).cpu().numpy().copy() for which in range(2 if kind in ("seg", "det") else 1)]
            for hi, kind in enumerate(kinds)]


def compare_with_oracle(spec, w, hw, kinds, images, feats, outs, batch_check=None):
    """Runs the oracle on the checked batch elements and applies the gates.  feats: four [B][N][D] host arrays;
    outs: as head_outputs returns them."""
    tol = TOL[spec.dtype]
    report = {}
    for b in (range(spec.batch) if batch_check is None else batch_check):
        ofe = model.encode_image(spec, w, images[b])
        for k in range(4):
            report[f"b{b}.feat{k}"] = relerr(feats[k][b], ofe[k])
        for hi, kind in enumerate(kinds):
            if kind == "seg":
                o = model.seg_head(spec, hw[hi], ofe)
                logits = outs[hi][0][b]                                       # [gh][gw][C]
                report[f"b{b}.h{hi}.seg.logits"] = relerr(logits.transpose(2, 0, 1), o["logits"])
                cm = outs[hi][1][b]
                report[f"b{b}.h{hi}.seg.agree"] = float(np.mean(cm == o["classmap"]))
                # a differing pixel is valid only if it is a near-tie: picking class g over the oracle's o
                # implies oracle[o] - oracle[g] <= 2 max |logit error| (interpolation is a convex combination)
                up = ops.bilinear(o["logits"], spec.img_h, spec.img_w)
                err = np.max(np.abs(logits.transpose(2, 0, 1) - o["logits"]))
                report[f"b{b}.h{hi}.seg.regret_ok"] = bool(regret(up, o["classmap"], cm) <= 2 * err + 1e-6)
            elif kind == "det":
                o = model.det_head(spec, hw[hi], ofe)
                out = outs[hi][0][b]                                          # [gh][gw][K+4]
                K = spec.det_classes
                report[f"b{b}.h{hi}.det.logits"] = relerr(out[..., :K].transpose(2, 0, 1), o["logits"])
                report[f"b{b}.h{hi}.det.box"] = relerr(out[..., K:].transpose(2, 0, 1), o["box"])
                cm = outs[hi][1][b]
                report[f"b{b}.h{hi}.det.agree"] = float(np.mean(cm == o["classmap"]))
                err = np.max(np.abs(out[..., :K].transpose(2, 0, 1) - o["logits"]))
                report[f"b{b}.h{hi}.det.regret_ok"] = bool(regret(o["logits"], o["classmap"], cm) <= 2 * err + 1e-6)
            else:
                o = (model.dpt_head if kind == "dpt" else model.depth_head)(spec, hw[hi], ofe)
                d = outs[hi][0][b]
                assert d.min() >= 0.0 and d.shape == (spec.img_h, spec.img_w)
                errs = depth_errs(d, o)
                report.update({f"b{b}.h{hi}.{kind}.{k}": v for k, v in errs.items()})
                report[f"b{b}.h{hi}.{kind}.gate_ok"] = depth_gate(errs, tol)
    print(spec.name, {k: (v if isinstance(v, bool) else round(v, 6) if v < 0.5 else round(v, 4))
                      for k, v in report.items()}, flush=True)
    # class maps: >= 0.99 agreement on maps large enough for the fraction to mean something (one cell of a
    # 165-cell map is already 0.6 %); on small maps >= 0.95, and every disagreement must be a near-tie
    cells = spec.patches
    for k, v in report.items():
        if k.endswith("regret_ok") or k.endswith("gate_ok"):
            assert v, (k, report)
        elif ".depth." in k or ".dpt." in k:
            pass                                # both normalisations are printed; gate_ok carries the decision
        elif k.endswith("agree"):
            floor = 0.999 if spec.dtype == "f32" else 0.99 if (cells >= 1000 or "seg" in k) else 0.95
            assert v >= floor, (k, v)
        else:
            assert v <= tol, (k, v)
    return report


def check_all(spec, seed, img_seed, kinds=("seg", "depth", "det"), flags=0, batch_check=None, lead_frames=0,
              weights_edit=None, on_device=None, **engine_kw):
    """One frame through the engine, then the oracle on the same inputs (the engine is closed before the oracle
    starts: the GPU is not held while the CPU works).  on_device(eng, images, fh, feats, outs) may add device-side
    checks while the engine is alive."""
    if weights_edit is not None:               # same generator, then an in-place change both sides will see
        engine_kw["weights"] = vi.make_backbone_weights(spec, seed)
        weights_edit(engine_kw["weights"])
    eng, w, hw = make_engine(spec, seed, kinds=kinds, flags=flags, **engine_kw)
    images = vi.make_batch(spec, img_seed)
    # optional lead-in: other frames pushed through encode + heads with no host synchronisation, so that the
    # checked frame runs in a filled pipeline (its slot, lane and graph are not the first ones)
    lead = [torch.from_numpy(vi.make_batch(spec, img_seed + 100 + i)).cuda() for i in range(min(lead_frames, 2))]
    for i in range(lead_frames):
        lf = eng.encode(lead[i % len(lead)])
        for h in range(len(kinds)):
            eng.run_head(h, lf)
    fh, feats = run_gpu(eng, images, len(kinds))
    outs = head_outputs(eng, kinds)
    if on_device is not None:
        on_device(eng, images, fh, feats, outs)
    eng.close()
    return compare_with_oracle(spec, w, hw, kinds, images, feats, outs, batch_check)


MEDIUM = dict(dim=128, depth=4, heads=2, mlp_hidden=256, img_h=154, img_w=210, taps=(1, 2, 3, 4), head_ch=64)


def test_medium_fp32_all_heads():
    # 11 x 15 = 165 patches, N = 166: more than one 128-row tile plus a ragged tail
    check_all(vi.ModelSpec("medium_f32", dtype="f32", **MEDIUM), 101, 201)


def test_medium_bf16_all_heads():
    check_all(vi.ModelSpec("medium_bf16", dtype="bf16", **MEDIUM), 102, 202)


def test_swiglu_registers_batch_bf16():
    spec = vi.ModelSpec("swiglu_b3", dtype="bf16", **{**MEDIUM, "mlp_kind": vi.MLP_SWIGLU, "registers": 4, "batch": 3,
                                                       "img_h": 70, "img_w": 98, "seg_classes": 150})
    check_all(spec, 103, 203)


def test_swiglu_registers_batch_fp32():
    spec = vi.ModelSpec("swiglu_b2_f32", dtype="f32", **{**MEDIUM, "mlp_kind": vi.MLP_SWIGLU, "registers": 4,
                                                           "batch": 2, "img_h": 70, "img_w": 98})
    check_all(spec, 104, 204)


def test_single_patch_image():
    # degenerate grid: 1 x 1 patches, N = 2, every bilinear resize clamps everywhere
    for dt in ("f32", "bf16"):
        check_all(vi.ModelSpec("one_patch_" + dt, dtype=dt, **{**MEDIUM, "img_h": 14, "img_w": 14}), 105, 205)


def test_one_row_of_patches():
    check_all(vi.ModelSpec("strip", dtype="bf16", **{**MEDIUM, "img_h": 14, "img_w": 14 * 67}), 106, 206)


def test_widest_supported_model():
    # the limits the library accepts: width 2048 (32 heads: 32 statistics groups per row, LayerNorm rows of 16
    # float2 per lane), 64 register tokens, 255 segmentation classes, 1024 head channels; four blocks, a 2 x 3 grid
    spec = vi.ModelSpec("widest", dtype="bf16", dim=2048, depth=4, heads=32, mlp_hidden=2048, registers=64, img_h=28,
                        img_w=42, taps=(1, 2, 3, 4), seg_classes=255, head_ch=1024)
    check_all(spec, 107, 207)


def test_cfg1_vits_fp32_224_seg():
    # benchmark configuration 1: ViT-S/14 fp32, 224 x 224, linear seg head; gate 1e-4
    spec = vi.CONFIGS["cfg1"]
    check_all(spec, *vi.SEEDS["cfg1"], kinds=("seg",))


def test_cfg2_vits_bf16_476x630_three_heads():
    # benchmark configuration 2 (the headline one), whole, all three heads, as bench.py runs it
    spec = vi.CONFIGS["cfg2"]
    check_all(spec, *vi.SEEDS["cfg2"], flags=vpe.VPE_FLAG_GRAPHS)


def test_residual_stream_with_a_large_common_offset():
    # every token carries a level of +30 (patch bias and CLS) on top of deviations of order 1, and keeps it through
    # all blocks: the in-GEMM LayerNorm statistics must come from differences, not from raw sums of squares
    # (E[x^2] - mean^2 in fp32 would lose four digits here and miss the 1e-4 gate)
    def lift(w, by):
        w["patch_b"] += np.float32(by)
        w["cls"] += np.float32(by)
    check_all(vi.ModelSpec("offset30_f32", dtype="f32", **MEDIUM), 104, 204, weights_edit=lambda w: lift(w, 30.0))
    # the bf16 engine multiplies a 16-bit copy of the stream itself, stored relative to each row's level (the
    # mean the previous LayerNorm saw, or bias + positional row for a fresh frame): the same lift must not
    # cost it its ordinary gate either
    check_all(vi.ModelSpec("offset30_bf16", dtype="bf16", **MEDIUM), 105, 205, weights_edit=lambda w: lift(w, 30.0))


def test_cfg2_in_the_pipelined_configuration_the_benchmark_times():
    # as bench.py launches it: three encoder lanes, a ring of four slots, HIP graphs, frames in flight
    spec = vi.CONFIGS["cfg2"]
    check_all(spec, *vi.SEEDS["cfg2"], flags=vpe.VPE_FLAG_GRAPHS, lead_frames=6, ring_slots=4, encoder_lanes=3)


@pytest.mark.parametrize("tile", ["384", "256", "128", "65", "64", "5", "4"])
def test_direct_to_lds_gemm_variant(tile, monkeypatch):
    # each bf16 GEMM shape (384 x 256, 256 x 256, 64 x 128, 64 x 64 tiles; "5" and "4": 64 x 128 and 64 x 64 whose two and four wave
    # groups share the k-steps of every k-tile; "128": the name of a former shape, which stands for 128 x 128 tiles, "2"), forced
    # for every GEMM of the model,
    # through every epilogue: folded LayerNorm + QKV with transposed values, LayerScale residual with row
    # statistics, GELU and SwiGLU, patch embedding, 1x1 and 3x3 convolutions, the fused 1-channel projection
    monkeypatch.setenv("VPE_GEMM_TILE", tile)
    check_all(vi.ModelSpec("medium_bf16_tile" + tile, dtype="bf16", **MEDIUM), 102, 202)
    spec = vi.ModelSpec("swiglu_tile" + tile, dtype="bf16", **{**MEDIUM, "mlp_kind": vi.MLP_SWIGLU, "registers": 4,
                                                                "batch": 3, "img_h": 70, "img_w": 98})
    check_all(spec, 103, 203)


@pytest.mark.parametrize("tile", ["384", "256", "65", "64", "5", "4"])
def test_direct_to_lds_gemm_with_fewer_k_tiles_than_stages(tile, monkeypatch):
    # one k-tile (width 64), three (MLP of 192) and nine (3x3 convolutions of 64 channels): pipelines whose first loads
    # already run past the last k-tile; 35 + 3 tokens a view, so that tiles and 8-row groups straddle two views; QKV width
    # 192, so that a 128-column tile of value columns is half empty (its other half is the next view's place).  The
    # gates of check_all are those of every bf16 model
    monkeypatch.setenv("VPE_GEMM_TILE", tile)
    check_all(vi.ModelSpec("short_k_tile" + tile, dtype="bf16", dim=64, depth=4, heads=1, mlp_hidden=192, registers=2, batch=2,
                           img_h=70, img_w=98, taps=(1, 2, 3, 4), head_ch=64), 141, 241)


@pytest.mark.parametrize("tile", ["20", "2", "6", "43", "33", "3"])
def test_gemm_tilings_for_few_and_for_many_tiles_per_cu(tile, monkeypatch):
    # 128 x 128 tiles with four and eight waves ("20", "2"), 64 x 128 in four wave groups ("6"), 64 x 64 and 32 x 64 with 128-deep
    # k-tiles ("43", "33") and 32 x 64 ("3"), forced for every GEMM of the models of the two tests above: every epilogue, whole and
    # ragged tiles, 8-row groups that straddle two views, one to nine k-tiles (widths of an odd multiple of 64: the 128-deep ones hand
    # over to "4" and "3").  The gates are those of every bf16 model
    monkeypatch.setenv("VPE_GEMM_TILE", tile)
    check_all(vi.ModelSpec("medium_bf16_tile" + tile, dtype="bf16", **MEDIUM), 102, 202)
    spec = vi.ModelSpec("swiglu_tile" + tile, dtype="bf16", **{**MEDIUM, "mlp_kind": vi.MLP_SWIGLU, "registers": 4,
                                                                "batch": 3, "img_h": 70, "img_w": 98})
    check_all(spec, 103, 203)
    check_all(vi.ModelSpec("short_k_tile" + tile, dtype="bf16", dim=64, depth=4, heads=1, mlp_hidden=192, registers=2, batch=2,
                           img_h=70, img_w=98, taps=(1, 2, 3, 4), head_ch=64), 141, 241)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("width", [320, 1600])
def test_layernorm_statistics_of_odd_and_of_many_groups(width, dtype):
    # 5 and 25 groups of 64 columns: an odd last group, and more than the 24 that are fetched in one batch; the gates are
    # those of every model of the type
    check_all(vi.ModelSpec("groups_%s_%d" % (dtype, width), dtype=dtype, dim=width, depth=4, heads=width // 64, mlp_hidden=320, registers=1,
                           img_h=70, img_w=98, taps=(1, 2, 3, 4), head_ch=64), 148, 248, kinds=("seg",))


@pytest.mark.parametrize("variant", ["114", "141", "124"])
def test_fp32_attention_shapes(variant, monkeypatch):
    # every workgroup shape of the fp32 attention: 38 tokens a view (one ragged key tile, fewer than the key waves), and 166
    # (three tiles, the last of 38 keys: key waves with unequal numbers of tiles); fp32 gates
    monkeypatch.setenv("VPE_ATTN_VARIANT", variant)
    check_all(vi.ModelSpec("attn_f32_" + variant, dtype="f32", **MEDIUM), 143, 243, kinds=("seg",))
    check_all(vi.ModelSpec("attn_f32_short_" + variant, dtype="f32", **{**MEDIUM, "registers": 2, "batch": 2, "img_h": 70, "img_w": 98}),
              144, 244, kinds=("seg",))


@pytest.mark.parametrize("width", [64, 128, 192])
def test_fp32_products_on_short_and_ragged_shapes(width):
    # fp32 operands as three bf16 terms: one to three k-tiles, 38 tokens a view (tiles and 8-row groups straddle two views),
    # a last 128-column tile that is half empty, convolutions from 5 x 7 up to 40 x 56 (one and several tiles per CU);
    # the gates are those of every fp32 model (1e-4)
    check_all(vi.ModelSpec("short_f32_%d" % width, dtype="f32", dim=width, depth=4, heads=width // 64, mlp_hidden=3 * width, registers=2,
                           batch=2, img_h=70, img_w=98, taps=(1, 2, 3, 4), head_ch=2 * width), 142, 242)


@pytest.mark.parametrize("tile", ["0", "1", "2", "3"])
def test_fp32_gemm_tilings(tile, monkeypatch):
    # each fp32 tiling (0: 64 x 64 in four wave groups, 1: 64 x 128 in four, 2: 64 x 128 in two with three stages, 3: 128 x 128, whose
    # waves leave by themselves) forced for every GEMM, through every epilogue: folded LayerNorm + QKV with transposed values,
    # LayerScale residual with row statistics, GELU and SwiGLU, patch embedding, 1x1 and 3x3 convolutions, the fused 1-channel
    # projection, the full DPT head's adds and ReLU copies; 166 tokens, then 38 + 38 (tiles and 8-row groups straddle two views) at
    # one and three k-tiles of 64 and with a half-empty last 128-column tile.  The gates are those of every fp32 model (1e-4)
    monkeypatch.setenv("VPE_GEMM_TILE_F32", tile)
    small = {"registers": 2, "batch": 2, "img_h": 70, "img_w": 98}
    check_all(vi.ModelSpec("medium_f32_tile" + tile, dtype="f32", **MEDIUM), 145, 245)
    check_all(vi.ModelSpec("swiglu_f32_tile" + tile, dtype="f32", **{**MEDIUM, **small, "mlp_kind": vi.MLP_SWIGLU}), 146, 246, kinds=("seg", "dpt"))
    for width in (64, 192):
        check_all(vi.ModelSpec("short_f32_tile%s_%d" % (tile, width), dtype="f32", **{**MEDIUM, **small, "dim": width, "heads": width // 64,
                                                                                      "mlp_hidden": 192}), 147, 247)


@pytest.mark.parametrize("tile", ["4", "5"])
def test_fp32_tilings_of_32_rows(tile, monkeypatch):
    # 32 x 64 tiles in four wave groups, three stages and two, as above: every epilogue, one and three k-tiles, ragged edges, and the
    # second computation of tiles with values that bf16 terms cannot hold (an infinite weight in one row); fp32 gates (1e-4)
    monkeypatch.setenv("VPE_GEMM_TILE_F32", tile)
    small = {"registers": 2, "batch": 2, "img_h": 70, "img_w": 98}
    check_all(vi.ModelSpec("medium_f32_tile" + tile, dtype="f32", **MEDIUM), 145, 245)
    check_all(vi.ModelSpec("swiglu_f32_tile" + tile, dtype="f32", **{**MEDIUM, **small, "mlp_kind": vi.MLP_SWIGLU}), 146, 246, kinds=("seg", "dpt"))
    for width in (64, 192):
        check_all(vi.ModelSpec("short_f32_tile%s_%d" % (tile, width), dtype="f32", **{**MEDIUM, **small, "dim": width, "heads": width // 64,
                                                                                      "mlp_hidden": 192}), 147, 247)
    test_fp32_head_weights_beyond_the_range_of_bf16(tile, monkeypatch)


@pytest.mark.parametrize("dtype,name,tile", [("bf16", "VPE_GEMM_TILE", "34"), ("f32", "VPE_GEMM_TILE_F32", "6")])
def test_tilings_of_32_columns(dtype, name, tile, monkeypatch):
    # 32 x 32 tiles wherever they are allowed (out-projection and fc2; 32 x 64 elsewhere): the LayerNorms that follow read
    # statistics of 32-column groups.  166 tokens, then 38 + 38 (the last row tile holds 12 rows); widths of one, two, three and four
    # groups of 64, with k extents that 128-deep k-tiles do and do not divide (bf16: then one of the two leaves groups of 64), and a
    # level of +30 common to every token; rows of 32 and 48 groups of 32 (24 are fetched in one batch); SwiGLU.  The gates of every model of the type
    monkeypatch.setenv(name, tile)
    small = {"registers": 2, "batch": 2, "img_h": 70, "img_w": 98}
    check_all(vi.ModelSpec("narrow_%s" % dtype, dtype=dtype, **MEDIUM), 148, 248, kinds=("seg",))
    check_all(vi.ModelSpec("narrow_swiglu_%s" % dtype, dtype=dtype, **{**MEDIUM, **small, "mlp_kind": vi.MLP_SWIGLU}), 149, 249, kinds=("seg",))

    def lift(w):
        w["pos"][:] += np.float32(30.0)
    for width, hidden in ((64, 128), (192, 384), (256, 192)):
        check_all(vi.ModelSpec("narrow_%s_%d" % (dtype, width), dtype=dtype, **{**MEDIUM, **small, "dim": width, "heads": width // 64,
                                                                               "mlp_hidden": hidden}), 150, 250, kinds=("seg",), weights_edit=lift)
    # (without the level: fp32 sums of 1024 and 1536 terms of its size are 1.1e-4 to 4.4e-4 off in every tiling, of 32 columns or not)
    for width in (1024, 1536):
        check_all(vi.ModelSpec("narrow_%s_%d" % (dtype, width), dtype=dtype, **{**MEDIUM, **small, "dim": width, "heads": width // 64}), 150, 250, kinds=("seg",))


@pytest.mark.parametrize("shape", ["1", "2"])
def test_strip_convolution_kernel(shape, monkeypatch):
    # the 3x3 convolution that forms its nine taps from one input strip in LDS, in both of its tile shapes (1: 384 x 256,
    # 2: 768 x 128), forced for every convolution it can take (whole tiles of output channels): detection towers reading
    # token rows of two images with register tokens in between, the depth head's four fusion stages on 11x15 ... 88x120
    # grids (tiles that span several image rows, both images and the end of the tensor; taps masked at every edge), the
    # last with the 1-channel projection
    monkeypatch.setenv("VPE_GEMM_TILE", "9")
    monkeypatch.setenv("VPE_STRIP_SHAPE", shape)
    spec = vi.ModelSpec("strip_conv", dtype="bf16", **{**MEDIUM, "head_ch": 256, "batch": 2, "registers": 4})
    check_all(spec, 108, 208)
    # one row of patches (every pixel on the top and bottom edge) and a single patch
    check_all(vi.ModelSpec("strip_conv_row", dtype="bf16", **{**MEDIUM, "head_ch": 256, "img_h": 14, "img_w": 14 * 9}), 109, 209)
    check_all(vi.ModelSpec("strip_conv_1x1", dtype="bf16", **{**MEDIUM, "head_ch": 256, "img_h": 14, "img_w": 14}), 110, 210)


@pytest.mark.parametrize("dtype,batch", [("f32", 104), ("bf16", 208)])
def test_operands_larger_than_two_gib(dtype, batch):
    # convolution inputs of 2.25 GB (11 x 15 patches, 88 x 120 pixels of 512 channels per view): byte offsets from the first view
    # do not fit 32 bits, those from a tile's own first row do.  Three different views in turn, so a wrapped offset meets
    # other data; every view against the same view in an engine of three, by the gates of its type
    spec = vi.ModelSpec("large_" + dtype, dtype=dtype, **{**MEDIUM, "head_ch": 512, "batch": 3})
    views = vi.make_batch(spec, 260)
    results = []
    for n in (3, batch):
        eng, _, _ = make_engine(vi.with_(spec, batch=n), 160, kinds=("depth", "seg"))
        _, feats = run_gpu(eng, np.ascontiguousarray(views[np.arange(n) % 3]), 2)
        results.append([feats[3], eng.head_output(0, 0).cpu().numpy().copy(), eng.head_output(1, 0).cpu().numpy().copy()])
        eng.close()
    for small, large in zip(*results):
        err = max(relerr(large[b], small[b % 3]) for b in range(batch))
        print("large", dtype, small.shape, err, flush=True)
        assert err <= TOL[dtype]


# ---------------------------------------------------------------- full DPT head
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_dpt_head_small_grids_odd_and_even(dtype):
    # 11 x 15 patches: the deepest level is 6 x 8 (odd grid halved with padding), resizes 6x8 -> 11x15 are not x2
    check_all(vi.ModelSpec("dpt_odd_" + dtype, dtype=dtype, **MEDIUM), 131, 231, kinds=("dpt",))
    # two images, registers, an even grid, together with the other heads (shared features)
    spec = vi.ModelSpec("dpt_even_" + dtype, dtype=dtype, **{**MEDIUM, "registers": 4, "batch": 2, "img_h": 112, "img_w": 140})
    check_all(spec, 132, 232, kinds=("seg", "dpt", "det"))


def test_dpt_head_degenerate_grids():
    # one patch (every level at least 1 x 1, resizes from a single sample) and one row of patches
    for dt in ("f32", "bf16"):
        check_all(vi.ModelSpec("dpt_one_patch_" + dt, dtype=dt, **{**MEDIUM, "img_h": 14, "img_w": 14}), 135, 235, kinds=("dpt",))
    check_all(vi.ModelSpec("dpt_strip", dtype="bf16", **{**MEDIUM, "img_h": 14, "img_w": 14 * 23}), 136, 236, kinds=("dpt",))


def test_dpt_head_wider_and_under_graph_replay():
    spec = vi.ModelSpec("dpt_wide", dtype="bf16", **{**MEDIUM, "head_ch": 128, "img_h": 98, "img_w": 126})
    check_all(spec, 133, 233, kinds=("dpt", "depth"), flags=vpe.VPE_FLAG_GRAPHS, lead_frames=3, ring_slots=2)


def test_dpt_head_at_its_widest():
    # width 256 (the DepthAnythingV2-large head shape): reassembled widths 192 .. 1536, no channel padding anywhere
    spec = vi.ModelSpec("dpt_256", dtype="bf16", **{**MEDIUM, "head_ch": 256, "img_h": 70, "img_w": 98, "batch": 2})
    check_all(spec, 134, 234, kinds=("dpt",))


def test_dpt_head_at_the_benchmark_size():
    # ViT-S/14 at 476 x 630 with the DepthAnythingV2-small head shape (width 64, reassembled widths 48 .. 384):
    # levels 136x180, 68x90, 34x45, 17x23; output convolutions on 272x360 and 476x630
    spec = vi.with_(vi.CONFIGS["cfg2"], head_ch=64, name="cfg2_dpt")
    check_all(spec, *vi.SEEDS["cfg2"], kinds=("dpt",), flags=vpe.VPE_FLAG_GRAPHS, lead_frames=2, ring_slots=2)


# ---------------------------------------------------------------- camera-frame transform
@pytest.mark.parametrize("src,dst,batch", [((1080, 1920), (476, 630), 1),      # the paper's camera frames -> cfg 2
                                           ((1080, 1920), (518, 518), 2),      # -> cfgs 3-5, two views
                                           ((37, 53), (98, 154), 1),           # enlargement, odd sizes
                                           ((224, 224), (224, 224), 1),        # same size: conversion only
                                           ((1, 1), (14, 14), 1),              # degenerate source
                                           ((300, 7), (14, 700), 3)])          # ragged: shrink one axis, stretch the other
def test_preprocess_u8_matches_the_oracle(src, dst, batch):
    frames = np.stack([vi.make_camera_frame(src[0], src[1], 40 + b) for b in range(batch)])
    dev = torch.from_numpy(frames).cuda()
    out = torch.full((batch, 3, dst[0], dst[1]), float("nan"), dtype=torch.float32, device="cuda")
    vpe.preprocess_u8(dev, out, vi.CAMERA_MEAN, vi.CAMERA_STD)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    for b in range(batch):
        ref = model.preprocess_u8(frames[b], dst[0], dst[1], vi.CAMERA_MEAN, vi.CAMERA_STD)
        err = float(np.max(np.abs(got[b] - ref)) / np.max(np.abs(ref)))
        print("preprocess", src, dst, b, err, flush=True)
        assert err <= 2e-6                      # exact tap positions; fp32 weights, blend, one scale and one shift


def test_preprocessed_camera_frame_runs_through_the_engine():
    # the transform's output is a valid engine input: same features as feeding the oracle's transform
    spec = vi.small_spec()
    eng, w, _ = make_engine(spec, 7, kinds=("seg",))
    frame = vi.make_camera_frame(90, 160, 77)
    dev = torch.from_numpy(frame[None]).cuda()
    img = torch.empty((1, 3, spec.img_h, spec.img_w), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()                   # the frame upload; from here on the engine's own stream orders the work
    vpe.preprocess_u8(dev, img, vi.CAMERA_MEAN, vi.CAMERA_STD, stream=eng.next_encode_stream())
    fh = eng.encode(img)
    eng.sync()
    got = eng.feat_view(fh, 3).float().cpu().numpy()[0]
    ref_img = model.preprocess_u8(frame, spec.img_h, spec.img_w, vi.CAMERA_MEAN, vi.CAMERA_STD)
    feats = model.encode_image(spec, w, ref_img.astype(np.float32))
    assert relerr(got, feats[3]) <= (1e-4 if spec.dtype == "f32" else 2e-2)
    eng.close()


# ---------------------------------------------------------------- several heads of one kind (paper, Sec. "Parallel
# vs. Sequential Processing" and "Single Backbone vs. Independent Models": k heads of one kind on one backbone)
def test_four_depth_heads_on_one_backbone_each_match_the_oracle():
    # four DPT-lite heads with different weights share the feature slot; more heads than head streams, so two
    # share a stream.  Every replica is compared with the oracle run on its own weights.
    spec = vi.CONFIGS["cfg2"]
    rep = check_all(spec, *vi.SEEDS["cfg2"], kinds=("depth",) * 4)
    assert len({round(rep[f"b0.h{h}.depth.pre_relu"], 9) for h in range(4)}) > 1      # different heads, not copies


def test_eight_detection_heads_in_the_pipelined_configuration():
    spec = vi.CONFIGS["cfg2"]
    check_all(spec, *vi.SEEDS["cfg2"], kinds=("det",) * 8, flags=vpe.VPE_FLAG_GRAPHS, lead_frames=5, ring_slots=4,
              encoder_lanes=3)


# ---------------------------------------------------------------- products in two launches
@pytest.mark.parametrize("gh,gw,batch,kinds", [(33, 33, 2, ("seg",)), (46, 46, 2, ("det",))])
def test_two_launches_with_a_leading_part_of_64_row_tiles(gh, gw, batch, kinds, monkeypatch):
    # width 1024: fc2 of 2180 tokens and a detection tower on 4232 cells (tests/test_gemm_contract.py holds that these shapes go out as
    # 64 x 128 tiles in four wave groups over 2048 and 4096 rows and 32 x 64 tiles over the others).  Against an engine
    # with one launch per product: the gates of every bf16 model, and bit-equal repeats
    spec = vi.ModelSpec("two_launches_%d" % gh, dtype="bf16", dim=1024, depth=4, heads=16, mlp_hidden=4096, img_h=14 * gh, img_w=14 * gw,
                        batch=batch, taps=(1, 2, 3, 4), head_ch=256)
    weights, images = vi.make_backbone_weights(spec, 161), vi.make_batch(spec, 261)
    results = []
    for one_launch in (False, True):
        if one_launch:
            monkeypatch.setenv("VPE_NO_ROW_SPLIT", "1")
        eng, _, _ = make_engine(spec, 161, kinds=kinds, weights=weights)
        got = []
        for _ in range(1 if one_launch else 2):
            _, feats = run_gpu(eng, images, 1)
            got.append((feats[3], head_outputs(eng, kinds)[0][0]))
        eng.close()
        assert all(np.array_equal(a, b) for a, b in zip(got[0], got[-1]))
        results.append(got[0])
    (f2, o2), (f1, o1) = results
    print("features", relerr(f2, f1), "head", relerr(o2, o1), flush=True)
    assert relerr(f2, f1) <= TOL["bf16"] and relerr(o2, o1) <= TOL["bf16"]
    for rows in (slice(0, 64), slice(-64, None)):                # (a lost tail would hide in a maximum over everything)
        a, b = f2.reshape(-1, spec.dim)[rows], f1.reshape(-1, spec.dim)[rows]
        assert relerr(a, b) <= TOL["bf16"]


# ---------------------------------------------------------------- attention far from uniform
SHARP = dict(dim=128, depth=4, heads=2, mlp_hidden=256, img_h=14 * 18, img_w=14 * 20, taps=(1, 2, 3, 4), head_ch=64)


def _sharpen(scale):
    def edit(w):
        # queries and keys (the first two thirds of the fused projection) scaled up: scores grow by scale^2, the
        # softmax concentrates on a few keys per query, and which keys differs from one key tile to the next
        for name in list(w):
            if name.endswith("qkv_w"):
                w[name][:, : 2 * w[name].shape[1] // 3] *= np.float32(scale)
            elif name.endswith("qkv_b"):
                w[name][: 2 * w[name].shape[0] // 3] *= np.float32(scale)
    return edit


@pytest.mark.parametrize("dtype,variant,scale", [("bf16", "124", 16.0), ("bf16", "224", 16.0), ("bf16", "141", 16.0),
                                                 ("bf16", "114", 16.0), ("bf16", "214", 16.0), ("bf16", "122", 16.0),
                                                 ("bf16", "", 16.0),
                                                 ("f32", "114", 32.0), ("f32", "141", 32.0), ("f32", "124", 32.0)])
def test_attention_with_peaked_softmax(dtype, variant, scale, monkeypatch):
    # 361 tokens = six key tiles of 64 (the last with 41 keys): with four key waves two of them own two tiles.
    # With the benchmark's weights every score lies within a fraction of a unit of the others, so the running
    # maximum never grows after the first tile and the partial results of the key waves are nearly equal; here
    # scores spread over tens of units, so rescaling on a growing maximum, the merge of partials taken against
    # different references and the masked tail all carry weight.
    if variant:
        monkeypatch.setenv("VPE_ATTN_VARIANT", variant)
    spec = vi.ModelSpec(f"sharp_{dtype}_{variant or 'auto'}", dtype=dtype, **SHARP)
    rep = check_all(spec, 141, 241, kinds=("seg",), weights_edit=_sharpen(scale))
    assert rep["b0.feat3"] > 0.0


@pytest.mark.parametrize("dtype,gh,gw,batch,lanes", [
    ("bf16", 7, 9, 1, 1), ("bf16", 8, 8, 1, 1), ("bf16", 16, 16, 7, 1), ("bf16", 16, 16, 8, 1), ("bf16", 16, 16, 13, 1), ("bf16", 16, 16, 3, 2),
    ("bf16", 16, 16, 4, 2), ("bf16", 16, 16, 25, 1), ("bf16", 16, 16, 26, 1), ("bf16", 16, 16, 25, 2), ("bf16", 16, 16, 26, 2), ("f32", 16, 16, 7, 1), ("f32", 16, 16, 8, 1),
    ("f32", 16, 16, 21, 2), ("f32", 16, 16, 22, 2), ("f32", 8, 8, 213, 1), ("f32", 8, 8, 214, 1)])
def test_attention_on_both_sides_of_its_shape_lines(dtype, gh, gw, batch, lanes):
    # 64, 65 and 257 tokens of a view: a whole key tile, a key more, one more than a round of four key waves.  Pairs of a head and a
    # block of 32 queries, bf16: 252, 288 and 468: below the line of 256, above it, and above 256 workgroups of 64 queries; 108
    # and 144 beside a second lane (line 128); 500 and 520 workgroups of 64 queries (line 512, with and without a second lane).  fp32: 252 and 288 (256),
    # 756 and 792 beside a second lane (768), 2556 and 2568 (2560).  Sharp scores, so a lost or doubled key shows; the gates
    # of every model of the type.
    spec = vi.ModelSpec("attn_line_%s_%d_%d_%d" % (dtype, gh, gw, batch), dtype=dtype,
                        **{**SHARP, "dim": 256, "heads": 4, "img_h": 14 * gh, "img_w": 14 * gw, "batch": batch})
    rep = check_all(spec, 151, 251, kinds=("seg",), batch_check=sorted({0, batch - 1}), weights_edit=_sharpen(16.0),
                    encoder_lanes=lanes, ring_slots=lanes + 1)
    assert rep["b0.feat3"] > 0.0


ONE_KEY = {**SHARP, "img_h": 14 * 24, "img_w": 14 * 25}


def _one_key(product, one_query):
    D, where, who, big = ONE_KEY["dim"], 5, 77, 300.0

    def edit(w):
        w["pos"][:, where] *= 0.1
        w["pos"][:, who] *= 0.1
        w["pos"][-1, where] = big
        w["pos"][40, who] = big
        for l in range(ONE_KEY["depth"]):
            for h in range(ONE_KEY["heads"]):
                c = 64 * h + 9
                w["blk%d.qkv_w" % l][:, c] = 0.0
                w["blk%d.qkv_w" % l][:, D + c] = 0.0
                w["blk%d.qkv_w" % l][where, D + c] = product / math.sqrt(D) * 16.0 / 8.0
                w["blk%d.qkv_w" % l][who, c] = 8.0 / math.sqrt(D) if one_query else 0.0
                w["blk%d.qkv_b" % l][c] = 0.0 if one_query else 8.0
                w["blk%d.qkv_b" % l][D + c] = 0.0
    return edit


@pytest.mark.parametrize("variant", ["", "114", "124", "122", "141"])
@pytest.mark.parametrize("product,one_query", [(16.0, False), (30.0, False), (48.0, False), (30.0, True), (48.0, True)])
def test_attention_to_one_key_of_a_later_tile(variant, product, one_query, monkeypatch):
    # 601 tokens (19 blocks of 32 queries of two heads: (1,1,4) by itself; more than two tiles a wave, so references stay there, too);
    # the last token (tile 9 of 10, no wave's first) stands out in one channel, which the keys of every head show to a query channel
    # that is constant, or large for token 40 alone: its score is 2 x product (log2 units: 46, 87 and 138) above the others', which
    # the references of the first tiles know nothing of.  Within the 2^64 that sums taken against them hold; above it, but finite; and
    # infinite: there the workgroup starts again, all of them or (one query) one of a head's.  The result of a query that sees the key
    # is that token's value (the next share is below e^-20), whatever rounding does to the scores.
    monkeypatch.setenv("VPE_ATTN_VARIANT", variant or "0")
    rep = check_all(vi.ModelSpec("one_key_" + variant, dtype="bf16", **ONE_KEY), 161, 261, kinds=("seg",), weights_edit=_one_key(product, one_query))
    assert rep["b0.feat3"] > 0.0


# ---------------------------------------------------------------- GELU of bf16 results
def _gelu_exact(v):
    return np.array([0.5 * x * math.erfc(-x / math.sqrt(2.0)) for x in np.asarray(v, dtype=np.float64)])


@pytest.mark.parametrize("lo,hi,gate", [(-3.5, -3.0, 5.5e-6), (-4.2, -3.5, 3.5e-6)])
def test_gelu_of_bf16_results_where_it_is_nearly_zero(lo, hi, gate):
    # One block whose second MLP product is the identity, fed by biases alone: the residual stream is GELU(v) of 256 known
    # v, beside 256 exact anchors between 0 and -0.005 whose straight-line fit undoes the final LayerNorm.  Gate: rms error of
    # the rounded value.  The form itself gives 8e-7 and 1.6e-6, rounding to bf16 3.6e-6 and 0.6e-6, the features' own rounding
    # (2^-9 / sqrt 3 of values up to 2e-3 from the mean) up to 2e-6: 4.2e-6 and 2.6e-6 together, and 1.3 times that as the
    # gate.  erf as an odd polynomial, 6.5e-6 and 1.0e-5 before rounding, gives 7.7e-6 and 1.05e-5 and fails both.
    D = 512
    spec = vi.ModelSpec("gelu_tail", dtype="bf16", dim=D, depth=4, heads=8, mlp_hidden=D, img_h=14, img_w=14, taps=(1, 2, 3, 4))
    w = vi.make_backbone_weights(spec, 1)
    v, anchors = np.linspace(lo, hi, 256).astype(np.float32), np.linspace(0.0, -0.005, 256).astype(np.float32)
    for name in w:
        w[name][...] = 0.0
    w["norm_g"][...] = 1.0
    w["blk0.fc1_b"][:256] = v
    w["blk0.fc2_w"][...] = np.eye(D, dtype=np.float32)
    w["blk0.fc2_b"][256:] = anchors
    w["blk0.ls2"][...] = 1024.0                                  # (so that LayerNorm's epsilon does not count)
    eng, _, _ = make_engine(spec, 1, kinds=("seg",), weights=w)
    _, feats = run_gpu(eng, np.zeros((1, 3, 14, 14), np.float32), 0)
    eng.close()
    y = feats[0][0, 1].astype(np.float64)
    err = np.polyval(np.polyfit(y[256:], anchors, 1), y[:256]) - _gelu_exact(v)
    rms = float(np.sqrt(np.mean(err ** 2)))
    print("gelu", lo, hi, "rms", rms, "max", float(np.max(np.abs(err))), flush=True)
    assert rms <= gate


# ---------------------------------------------------------------- fp32 operands that bf16 terms cannot hold
BIG = np.float32(3.4e38)          # finite in fp32, rounds to infinity in bf16


@pytest.mark.parametrize("tile", ["", "0", "1", "2", "3"])
def test_fp32_head_weights_beyond_the_range_of_bf16(tile, monkeypatch):
    # features within +-1 (a small final LayerNorm gain), so that a weight of 3.4e38 gives finite sums; an infinite one gives
    # infinities of the feature's sign, and the detection tower's ReLU has to keep them and the large values apart from 0
    if tile:
        monkeypatch.setenv("VPE_GEMM_TILE_F32", tile)
    spec = vi.ModelSpec("f32_range", dtype="f32", **MEDIUM)
    backbone = vi.make_backbone_weights(spec, 151)
    backbone["norm_g"][...] = 0.1
    backbone["norm_b"][...] = 0.0

    def edited(spec_, kind, seed, make=vi.make_head_weights):
        hw = make(spec_, kind, seed)
        if kind == vi.HEAD_SEG:
            hw["seg_w"][:2] = 0.0
            hw["seg_w"][0, 5], hw["seg_w"][1, 70] = BIG, np.inf
        else:
            hw["cls_tower_w"][0] = 0.0
            hw["cls_tower_w"][0, 5, 1, 1] = BIG
            hw["cls_w"][:, 0] = np.where(np.arange(spec_.det_classes) % 2, 1e-36, -1e-36)
        return hw

    monkeypatch.setattr(vi, "make_head_weights", edited)
    eng, w, hw = make_engine(spec, 151, kinds=("seg", "det"), weights=backbone)
    images = vi.make_batch(spec, 251)
    _, feats = run_gpu(eng, images, 2)
    outs = head_outputs(eng, ("seg", "det"))
    eng.close()
    f = feats[3][0, 1:].reshape(spec.gh, spec.gw, spec.dim).astype(np.float64)
    logits = outs[0][0][0]
    assert np.max(np.abs(f)) < 1.0
    np.testing.assert_allclose(logits[..., 0], f[..., 5] * float(BIG) + hw[0]["seg_b"][0], rtol=1e-6)
    assert np.array_equal(logits[..., 1], np.inf * np.sign(f[..., 70]))
    assert relerr(logits[..., 2:], f @ hw[0]["seg_w"][2:].T.astype(np.float64) + hw[0]["seg_b"][2:]) <= TOL["f32"]
    o = model.det_head(spec, hw[1], model.encode_image(spec, w, images[0]))
    assert relerr(outs[1][0][0][..., :spec.det_classes].transpose(2, 0, 1), o["logits"]) <= TOL["f32"]


@pytest.mark.parametrize("variant", ["114", "141", "124"])
def test_fp32_attention_keys_beyond_the_range_of_bf16(variant, monkeypatch):
    # one channel of every key at 3.4e38 against 1e-37 in the queries: the same 4.25 in every score, which the softmax does not see
    monkeypatch.setenv("VPE_ATTN_VARIANT", variant)
    D = MEDIUM["dim"]

    def edit(w):
        for c, value in ((3, np.float32(1e-37)), (D + 3, BIG)):
            w["blk1.qkv_w"][:, c] = 0.0
            w["blk1.qkv_b"][c] = value
    check_all(vi.ModelSpec("f32_keys_" + variant, dtype="f32", **MEDIUM), 152, 252, kinds=("seg",), weights_edit=edit)

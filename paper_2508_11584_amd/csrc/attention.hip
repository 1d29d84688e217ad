// Instantiations of the flash-style attention kernel and the choice of workgroup shape.
#include <cstdlib>

#include "kernels.h"
namespace vpe {

// variant = QB * 100 + QW * 10 + KW
template <typename T>
static hipError_t launch_variant(int variant, const AttnArgs& a, hipStream_t s, bool cfg = false) {
    // With up to two tiles a wave the check of references that stay costs more than the maxima (257 tokens, 54 pairs: 5.62 us with
    // references that move, 5.76 with others; 577 tokens 6.74 / 6.71)
    if (sizeof(T) == 2 && variant == 114 && (cfg || a.npad <= 2 * 4 * 64)) {
        const hipError_t rc = launch_attention_variant<T, 1, 1, 4, false>(a, s, cfg);
        if (!cfg || rc != hipSuccess) return rc;
    }
    switch (variant) {
        case 114: return launch_attention_variant<T, 1, 1, 4>(a, s, cfg);
        case 141: return launch_attention_variant<T, 1, 4, 1>(a, s, cfg);
        case 124: return launch_attention_variant<T, 1, 2, 4>(a, s, cfg);
        default: break;
    }
    if constexpr (sizeof(T) == 2) {
        switch (variant) {
            case 214: return launch_attention_variant<T, 2, 1, 4>(a, s, cfg);
            case 122: return launch_attention_variant<T, 1, 2, 2>(a, s, cfg);
            case 224: return launch_attention_variant<T, 2, 2, 4>(a, s, cfg);
            default: break;
        }
    }
    return hipErrorInvalidValue;
}

// VPE_ATTN_VARIANT = 100 QB + 10 QW + KW overrides the choice of shape (tuning aid; read when an engine is created).
static int g_forced_variant = 0;

// LDS opt-in for every instantiation; called once at engine creation, outside any stream capture.
hipError_t configure_attention() {
    const char* env = getenv("VPE_ATTN_VARIANT");
    g_forced_variant = env ? atoi(env) : 0;
    static const int all[] = {114, 141, 214, 122, 124, 224};
    AttnArgs a{};
    for (int v : all) {
        hipError_t rc = launch_variant<bf16>(v, a, nullptr, true);
        if (rc != hipSuccess) return rc;
    }
    for (int v : {114, 124, 141}) {
        hipError_t rc = launch_variant<float>(v, a, nullptr, true);
        if (rc != hipSuccess) return rc;
    }
    return hipSuccess;
}

hipError_t launch_attention(int dtype, const AttnArgs& a, hipStream_t s) {
    const int forced = g_forced_variant;
    // Workgroup shapes measured on MI355X (QB, QW, KW = query blocks per wave, query waves, key waves), us, by pairs of a head
    // and a block of 32 queries:
    //                                        (1,1,4) (1,2,4) (1,2,2) (1,4,1)
    //     54  ViT-S 224x224  (N  257)             5.6     7.0     6.3     7.1
    //    108  ViT-B 224x224                       5.7     7.0     6.4     7.2
    //    222  ViT-S 476x476  (N 1157)             8.9    10.4    11.3    15.7
    //    288  ViT-S 476x630  (N 1531)            17.9    11.6    12.9    18.8
    //    348  ViT-S 602x602  (N 1850)            21.5    13.7    15.3    21.9
    //    444  ViT-B 476x476                      16.5    11.1    12.0    15.9
    //    516  ViT-B 518x518  (N 1370)            26.0    21.4    15.6    17.7
    //    612  ViT-B 252x406 x 3                  17.9    15.4    10.5    10.1
    //    696  ViT-B 602x602                      31.8    26.0    20.5    22.4
    //    928  ViT-L 602x602                      41.9    27.0    22.2    23.1
    //   1548  ViT-B 518x518 x 3                  60.2    42.0    31.0    25.7
    //   2752  ViT-L 518x518 x 4                  95.8    64.8    48.2    39.3
    // The first two hold a CU each, the longest-running split of the keys that one round of the 256 CUs has room for wins
    // (and a merge that four waves share beats one by a single wave); then half a CU each, as long as one round of two to a CU
    // holds them (512 workgroups of 64 queries; beyond, whole frames are 1-4 % faster with (1,4,1): ViT-B 518x518 x 3 on two lanes
    // 11891 / 11611 us, ViT-S 476x630 x 4 1655 / 1610, ViT-L 518x518 x 2 4912 / 4804); more want four query waves sharing each key
    // tile, three to a CU, and no merge.  Wider workgroups (eight query waves, or two query blocks per wave) halve the
    // L2 -> LDS traffic and are slower all the same; narrower ones (two waves) double it and are slower too.
    // Beside another encoder lane's kernels the footprint counts for more than the time alone.  Encoder passes on two lanes, us, in the
    // order of the table:
    //     54  ViT-S 224x224   196  199  201  205        222  ViT-S 476x476       331  306  305  325      1032  ViT-B 518x518 x 2  1275 1163 1102 1075
    //     96  ViT-S 308x308   229  223  228  239        288  ViT-S 476x630       407  362  348  371      1152  ViT-S 476x630 x 4  1033  898  845  812
    //    150  ViT-S 392x392   270  266  269  283        444  ViT-B 476x476       637  560  539  556      1376  ViT-L 518x518 x 2  3410 3085 2955 2855
    //    192  ViT-B 308x308   341  331  334  331        516  ViT-B 518x518       720  636  614  604
    //    688  ViT-L 518x518  1975 1823 1731 1744        696  ViT-B 602x602       935  826  778  772
    // so (1,1,4) where both lanes' workgroups find a CU each, then (1,2,2) up to the line of (1,4,1), above which the last column is.  At 96,
    // 150 and 516 pairs another shape is 1-2.5 % faster.
    const int64_t heads = (int64_t)a.B * a.heads, qblocks = cdiv(a.N, 32) * heads;
    int variant = cdiv(a.N, 64) * heads > 512 ? 141 : qblocks <= (a.shared_gpu ? 128 : 256) ? 114 : a.shared_gpu || cdiv(a.N, 64) * heads > 256 ? 122 : 124;
    if (forced) variant = forced;
    if (dtype) return launch_variant<bf16>(variant, a, s);
    // fp32: a workgroup fills a CU's LDS ((1,4,1): half of it), so what counts is whole rounds of the 256 CUs and waves to overlap:
    // a wave alone on its SIMD splits values and multiplies in turn, of eight waves two share a SIMD.  us, the kernel on fp32
    // instructions / (1,1,4) (1,2,4) (1,4,1), and (1,2,2), which is no longer there, before its masks and addresses changed:
    //   54 pairs (ViT-S 224x224)  15.8 / 12.7 15.5 21.1, 15.2    288 (ViT-S 476x630)  79.0 / 55.7 42.2 83.5, 47.5
    //   348 (ViT-S 602x602)       72.4 53.8 99.9, 58.3           516 (ViT-B 518x518) 116.3 / 84 77 80.6, 91.1
    //   1032 (ViT-S 518x518 x4) 192 / 139 115.5 122.5, 129       2064 (ViT-B 518x518 x4) 280 / 252 196 203, 237
    //   3096 (ViT-S 896x896 x4) 973 763 704
    // Beside another lane's kernels (1,4,1) leaves half a CU.  Frames of two lanes, us, (1,2,4) / (1,4,1), without and with a depth head:
    //   288 1038 / 1366, 2003 / 2273   516 2317 / 2319   576 - , 3395 / 3435   696 2169 / 2187   774 2176 / 2165, 4786 / 4773
    //   864 2390 / 2262   1032 2799 / 2678, 5803 / 5944   1152 3169 / 3077, 6767 / 6634   1290 3300 / 3161, 7292 / 7181   1548
    //   (ViT-B) 5944 / 5771, 8391 / 8267   2064 8084 / 7866, 11510 / 11377
    int v32 = qblocks <= 256 ? 114 : qblocks <= (a.shared_gpu ? 768 : 2560) ? 124 : 141;
    if (forced == 114 || forced == 124 || forced == 141) v32 = forced;
    return launch_variant<float>(v32, a, s);
}
}  // namespace vpe

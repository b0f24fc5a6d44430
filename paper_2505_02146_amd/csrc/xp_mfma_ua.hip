// bf16 variants of the kernel for operands of any alignment (xp_mfma_ua.hpp).
#include "xp_mfma_ua.hpp"

namespace xp {
namespace {

// the three that take convolutions too; at the end of each line the times of ua_cost, in us
#define XP_UA_VARIANT(NAME, SIZE, BM, BN, PF, ...) \
    typedef UaTile<BM, BN, 2, 2, 1, PF> NAME##T; \
    double NAME##_cost(const Problem &q) { return ua_cost<NAME##T>(q, UaTimes{__VA_ARGS__}); } \
    const Variant NAME = {"bf16 " SIZE "x128B waves 2x2 any alignment, through registers, mfma16", ua_can_run<false, NAME##T>, ua_launch<false, NAME##T>, NAME##_cost};

XP_UA_VARIANT(kUa128, "128x128", 128, 128, 2, 3.08, 2.89, 3.18, 0.702, 0.708, 0.088, 0.196, 0.654)
XP_UA_VARIANT(kUa128x64, "128x64", 128, 64, 2, 2.88, 1.78, 1.77, 0.494, 0.489, -0.013, 0.079, 0.754)
XP_UA_VARIANT(kUa64, "64x64", 64, 64, 3, 3.06, 1.56, 0.798, 0.297, 0.321, -0.055, 0.045, 0.652)

#define XP_UA_GEMM_VARIANT(NAME, BM, BN, WM, WN, KG, DEALT, SHIFT, TEXT, ...) \
    typedef UaTile<BM, BN, WM, WN, KG, 2, 2, DEALT, SHIFT> NAME##T; \
    double NAME##_cost(const Problem &q) { return ua_cost<NAME##T>(q, UaTimes{__VA_ARGS__}); } \
    const Variant NAME = {"bf16 " #BM "x" #BN " waves " #WM "x" #WN "x" #KG " unaligned rows" TEXT ", through registers, mfma16", ua_can_run_gemm<false, NAME##T>, \
                          ua_launch<false, NAME##T>, NAME##_cost};

XP_UA_GEMM_VARIANT(kUaDealt128, 128, 128, 2, 2, 1, true, false, ", loads dealt out", 3.02, 3.29, 3.14, 0.638, 0.677, 0.12, 0.089, 0.745)
XP_UA_GEMM_VARIANT(kUa192, 192, 128, 4, 2, 1, false, false, "", 2.68, 2.97, 5.83, 0.837, 0.961, 0.172, 0.076, 0.74)
XP_UA_GEMM_VARIANT(kUa96, 96, 96, 2, 2, 2, true, true, ", from dwords", 2.81, 2.6, 4.2, 0.821, 0.926, 0.114, 0.252, 0.722)
XP_UA_GEMM_VARIANT(kUa64k2, 64, 64, 2, 2, 2, false, false, "", 2.46, 2.19, 1.56, 0.524, 0.565, -0.047, 0.064, 0.671)
XP_UA_GEMM_VARIANT(kUa32x64, 32, 64, 1, 2, 4, false, false, "", 1.26, 3.1, 2.64, 0.821, 0.994, 0.055, 0.061, 0.83)
XP_UA_GEMM_VARIANT(kUa64x32, 64, 32, 2, 1, 4, false, false, "", 1.39, 2.92, 2.66, 0.826, 0.99, -0.032, 0.143, 0.779)

}  // namespace

bool any_alignment_needed(const Problem &q) { return ua_needed(q); }

int ua_variants_bf16(const Variant **out)
{
    out[0] = &kUa128; out[1] = &kUa128x64; out[2] = &kUa64;
    return 3;
}

int ua_gemm_variants_bf16(const Variant **out)
{
    const Variant *v[] = {&kUaDealt128, &kUa192, &kUa96, &kUa64k2, &kUa32x64, &kUa64x32};
    for (size_t i = 0; i < sizeof v / sizeof *v; ++i) out[i] = v[i];
    return (int)(sizeof v / sizeof *v);
}

}  // namespace xp

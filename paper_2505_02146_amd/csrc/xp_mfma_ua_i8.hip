// int8 variants of the kernel for operands of any alignment (xp_mfma_ua.hpp).
#include "xp_mfma_ua.hpp"

namespace xp {
namespace {

// at the end of each line the times of ua_cost, in us
#define XP_UA_VARIANT(NAME, SIZE, BM, BN, PF, ...) \
    typedef UaTile<BM, BN, 2, 2, 1, PF> NAME##T; \
    double NAME##_cost(const Problem &q) { return ua_cost<NAME##T>(q, UaTimes{__VA_ARGS__}); } \
    const Variant NAME = {"i8 " SIZE "x128B waves 2x2 any alignment, through registers, mfma16", ua_can_run<true, NAME##T>, ua_launch<true, NAME##T>, NAME##_cost};

XP_UA_VARIANT(kUa128, "128x128", 128, 128, 2, 4.07, 1.44, 2.62, 0.845, 0.844, 0.067, 0.006, 0.531)
XP_UA_VARIANT(kUa128x64, "128x64", 128, 64, 2, 3.28, 1.2, 1.55, 0.576, 0.575, 0.002, -0.042, 0.512)
XP_UA_VARIANT(kUa64, "64x64", 64, 64, 3, 2.96, 1.49, 0.763, 0.37, 0.367, -0.047, -0.022, 0.846)

#define XP_UA_GEMM_VARIANT(NAME, BM, BN, WM, WN, KG, DEALT, SHIFT, TEXT, ...) \
    typedef UaTile<BM, BN, WM, WN, KG, 2, 2, DEALT, SHIFT> NAME##T; \
    double NAME##_cost(const Problem &q) { return ua_cost<NAME##T>(q, UaTimes{__VA_ARGS__}); } \
    const Variant NAME = {"i8 " #BM "x" #BN " waves " #WM "x" #WN "x" #KG " unaligned rows" TEXT ", through registers, mfma16", ua_can_run_gemm<true, NAME##T>, \
                          ua_launch<true, NAME##T>, NAME##_cost};

XP_UA_GEMM_VARIANT(kUaDealt128, 128, 128, 2, 2, 1, true, false, ", loads dealt out", 4, 1.69, 2.71, 0.768, 0.777, 0.235, -0.085, 0.521)
XP_UA_GEMM_VARIANT(kUa192, 192, 128, 4, 2, 1, false, false, "", 3.59, 1.99, 4.85, 0.975, 1.15, 0.111, -0.093, 0.78)
XP_UA_GEMM_VARIANT(kUa96, 96, 96, 2, 2, 2, true, true, ", from dwords", 2.98, 2.24, 3.69, 0.82, 1.02, 0.111, 0.243, 0.682)
XP_UA_GEMM_VARIANT(kUa64k2, 64, 64, 2, 2, 2, false, false, "", 2.57, 1.6, 1.3, 0.738, 0.705, 0.019, -0.043, 0.778)
XP_UA_GEMM_VARIANT(kUa32x64, 32, 64, 1, 2, 4, false, false, "", 1.24, 2.48, 2.4, 1.23, 1.27, 0.041, -0.026, 0.817)
XP_UA_GEMM_VARIANT(kUa64x32, 64, 32, 2, 1, 4, false, false, "", 1.22, 2.49, 2.26, 1.21, 1.28, 0.033, 0.022, 0.824)

}  // namespace

int ua_variants_i8(const Variant **out)
{
    out[0] = &kUa128; out[1] = &kUa128x64; out[2] = &kUa64;
    return 3;
}

int ua_gemm_variants_i8(const Variant **out)
{
    const Variant *v[] = {&kUaDealt128, &kUa192, &kUa96, &kUa64k2, &kUa32x64, &kUa64x32};
    for (size_t i = 0; i < sizeof v / sizeof *v; ++i) out[i] = v[i];
    return (int)(sizeof v / sizeof *v);
}

}  // namespace xp

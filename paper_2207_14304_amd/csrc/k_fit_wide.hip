// Moment accumulation of the FP32 fit on wide frames (see fit_wide.h).
#include "fit_wide.h"

int fit_accum_launch_wide(argus_ctx *ctx, const argus_fit::FitArgs &fa, int D, dim3 grid) {
    using namespace argus_fit;
    hipError_t err = hipSuccess;
    bool ok = false;
#define ARGUS_FH(DD, HH)                                                                    \
    if (D == DD && fa.h == HH) {                                                            \
        const size_t lds = FitWideLds<DD, HH>::bytes();                                     \
        err = hipFuncSetAttribute((const void *)fit_wide_kernel<DD, HH>,                    \
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);    \
        if (err == hipSuccess)                                                              \
            hipLaunchKernelGGL((fit_wide_kernel<DD, HH>), grid, dim3(1024), lds, ctx->stream, fa); \
        ok = true;                                                                          \
    }
#define ARGUS_FD(DD)                                                                        \
    ARGUS_FH(DD, 1) ARGUS_FH(DD, 2) ARGUS_FH(DD, 3) ARGUS_FH(DD, 4) ARGUS_FH(DD, 5)          \
    ARGUS_FH(DD, 6) ARGUS_FH(DD, 7) ARGUS_FH(DD, 8) ARGUS_FH(DD, 9) ARGUS_FH(DD, 10)         \
    ARGUS_FH(DD, 11) ARGUS_FH(DD, 12) ARGUS_FH(DD, 13) ARGUS_FH(DD, 14) ARGUS_FH(DD, 15)
    ARGUS_FD(1)
    ARGUS_FD(2)
#undef ARGUS_FD
#undef ARGUS_FH
    if (!ok) return argus_fail(ctx, ARGUS_ESHAPE, "unsupported degree %d / half width %d", D, fa.h);
    ARGUS_HIP_CHECK(ctx, err);
    ARGUS_HIP_CHECK(ctx, hipGetLastError());
    return ARGUS_OK;
}

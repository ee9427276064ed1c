// C entry point of the fwd contraction; the kernel template lives in contract_kernel.hpp
#include "contract_kernel.hpp"

using namespace adapt;


extern "C" int adapt_conv_fwd(adapt_ctx *ctx, adapt_conv_desc d, const void *x, adapt_fmt fx, const void *w, adapt_fmt fw,
                              void *y, adapt_epilogue ep)
{
    if (ctx && wants_wide(fx, fw, ep)) {
        if (!conv_ok(d)) return ADAPT_EINVAL;
        if (d.n == 0) return ADAPT_OK;
        if (!check_ptrs(x, w, y)) return ADAPT_EINVAL;
        const int planes = wide_fwd_planes(ctx, d, x, fx, w, fw, y, ep);      // one kernel on byte planes where it applies
        if (planes != ADAPT_EWORKSPACE && planes != ADAPT_EUNSUPPORTED) return planes;
        const int p = (d.h + 2 * d.pad - d.r) / d.stride + 1, q = (d.w + 2 * d.pad - d.s) / d.stride + 1;
        const SubContraction sub = [&](const void *pa, adapt_fmt fpa, const void *pb, adapt_fmt fpb, void *c, adapt_epilogue ex) {
            return adapt_conv_fwd(ctx, d, pa, fpa, pb, fpb, c, ex);
        };
        return wide_contraction(ctx, x, fx, (uint64_t)d.n * d.h * d.w * d.c, w, fw, (uint64_t)d.k * d.r * d.s * d.c, (uint64_t)d.n * p * q * d.k,
                                (int64_t)d.r * d.s * d.c, y, ep, sub);
    }
    if (!ctx || !fmt_ok(fx) || !fmt_ok(fw) || !conv_ok(d)) return ADAPT_EINVAL;
    if (d.n == 0) return ADAPT_OK;
    if (!check_ptrs(x, w, y)) return ADAPT_EINVAL;
    if (!epilogue_ok(ep)) return ADAPT_EINVAL;
    PadJobs pads;
    ContractPlan p;
    if (int s = plan_fwd(ctx, d, x, fx, w, fw, y, ep, scratch_bytes(ctx), pads, p)) return s;
    hipError_t e = launch_pads(ctx, pads);
    if (e == hipSuccess) e = launch_and_finish(ctx, p, launch_planned<OP_FWD>);
    return hip_status(ctx, e);
}

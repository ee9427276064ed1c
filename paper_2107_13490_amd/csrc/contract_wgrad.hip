// C entry point of the wgrad contraction; the kernel template lives in contract_kernel.hpp
#include "contract_kernel.hpp"

using namespace adapt;

namespace adapt {
hipError_t launch_planned_wgrad(adapt_ctx *ctx, const ContractPlan &p) { return launch_planned<OP_WGRAD>(ctx, p); }
}  // namespace adapt


extern "C" int adapt_conv_wgrad(adapt_ctx *ctx, adapt_conv_desc d, const void *dy, adapt_fmt fdy, const void *x,
                                adapt_fmt fx, void *dw, adapt_epilogue ep)
{
    if (ctx && wants_wide(fdy, fx, ep)) {
        if (!conv_ok(d)) return ADAPT_EINVAL;
        if (!dw || !aligned16(dw) || (d.n > 0 && !check_ptrs(dy, x, dw))) return ADAPT_EINVAL;
        if (d.n == 0) return ADAPT_EUNSUPPORTED;             // (an empty batch would only clear dw)
        const int p = (d.h + 2 * d.pad - d.r) / d.stride + 1, q = (d.w + 2 * d.pad - d.s) / d.stride + 1;
        const SubContraction sub = [&](const void *pa, adapt_fmt fpa, const void *pb, adapt_fmt fpb, void *c, adapt_epilogue ex) {
            return adapt_conv_wgrad(ctx, d, pa, fpa, pb, fpb, c, ex);
        };
        return wide_contraction(ctx, dy, fdy, (uint64_t)d.n * p * q * d.k, x, fx, (uint64_t)d.n * d.h * d.w * d.c, (uint64_t)d.k * d.r * d.s * d.c,
                                (int64_t)d.n * p * q, dw, ep, sub);
    }
    if (!ctx || !fmt_ok(fdy) || !fmt_ok(fx) || !conv_ok(d)) return ADAPT_EINVAL;
    if (!dw || !aligned16(dw)) return ADAPT_EINVAL;
    if (d.n > 0 && !check_ptrs(dy, x, dw)) return ADAPT_EINVAL;
    if (!epilogue_ok(ep)) return ADAPT_EINVAL;
    PadJobs pads;
    ContractPlan pd, pw;
    if (int s = plan_gradients(ctx, GRAD_DW, d, dy, fdy, nullptr, fdy, x, fx, nullptr, ep, dw, ep, scratch_bytes(ctx), pads, pd, pw)) return s;
    hipError_t e = launch_pads(ctx, pads);
    if (e == hipSuccess) e = launch_and_finish(ctx, pw, launch_planned<OP_WGRAD>);
    return hip_status(ctx, e);
}

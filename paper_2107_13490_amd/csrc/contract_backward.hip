// C entry point of a layer's backward pass: data gradient and weight gradient of one convolution
// (Alg. 1, the backward-pass line, per layer).  Results are exactly those of adapt_conv_dgrad and
// adapt_conv_wgrad; when both contractions take a vector path with matching tiles (one limb:
// 192-deep stages; two limbs: int16 operands, equal square tiles) they run as one launch.
#include "contract_pair.hpp"

using namespace adapt;

extern "C" int adapt_conv_backward(adapt_ctx *ctx, adapt_conv_desc d, const void *dy, adapt_fmt fdy, const void *w,
                                   adapt_fmt fw, const void *x, adapt_fmt fx, void *dx, adapt_epilogue ep_dx, void *dw,
                                   adapt_epilogue ep_dw)
{
    if (ctx && (wants_wide(fdy, fw, ep_dx) || wants_wide(fdy, fx, ep_dw))) {
        // word lengths above 16: the two contractions one after the other, each composed of its parts
        if (d.n > 0)
            if (int s = adapt_conv_dgrad(ctx, d, dy, fdy, w, fw, dx, ep_dx)) return s;
        return adapt_conv_wgrad(ctx, d, dy, fdy, x, fx, dw, ep_dw);
    }
    if (!ctx || !fmt_ok(fdy) || !fmt_ok(fw) || !fmt_ok(fx) || !conv_ok(d)) return ADAPT_EINVAL;
    if (!dw || !aligned16(dw)) return ADAPT_EINVAL;
    if (d.n > 0 && (!check_ptrs(dy, w, dx) || !check_ptrs(dy, x, dw))) return ADAPT_EINVAL;
    if (!epilogue_ok(ep_dx) || !epilogue_ok(ep_dw)) return ADAPT_EINVAL;
    PadJobs pads;
    ContractPlan pd, pw;
    // an empty batch: dw = 0, no dx
    if (int s = plan_gradients(ctx, d.n > 0 ? GRAD_DX | GRAD_DW : GRAD_DW, d, dy, fdy, w, fw, x, fx, dx, ep_dx, dw, ep_dw, scratch_bytes(ctx), pads, pd, pw))
        return s;
    if (d.n == 0) return hip_status(ctx, launch_and_finish(ctx, pw, launch_planned_wgrad));
    hipError_t e = launch_pads(ctx, pads);
    bool paired = false;
    if (e == hipSuccess && pairs(pd, pw)) {
        if (pd.tile.bm == 64 && pd.tile.bn == 64) e = launch_pair_d64x64(ctx, pd, pw, &paired);
        else if (pd.tile.bm == 128 && pd.tile.bn == 64) e = launch_pair_d128x64(ctx, pd, pw, &paired);
        else if (pd.tile.bm == 64 && pd.tile.bn == 128) e = launch_pair_d64x128(ctx, pd, pw, &paired);
        else e = launch_pair_d128x128(ctx, pd, pw, &paired);
        if (e == hipSuccess && paired) e = finish_planned(ctx, pw);
    }
    if (!paired) {
        // one after the other; both may use the scratch behind the copies from its start because the stream orders them
        if (e == hipSuccess) e = launch_and_finish(ctx, pd, launch_planned_dgrad);
        if (e == hipSuccess) e = launch_and_finish(ctx, pw, launch_planned_wgrad);
    }
    return hip_status(ctx, e);
}

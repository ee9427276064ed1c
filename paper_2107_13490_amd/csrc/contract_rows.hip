// Weight gradients on image rows in LDS (contract_rows.hpp), operands of one and two limbs
#include "contract_rows.hpp"

namespace adapt {

hipError_t launch_rows_both(adapt_ctx *ctx, const ContractPlan &p);

hipError_t launch_rows(adapt_ctx *ctx, const ContractPlan &p)
{
    const ContractArgs &a = p.kern;
    if (a.act_es == 2 && a.wgt_es == 2) return launch_rows_both(ctx, p);
    if (a.act_es == 2) return a.balanced ? launch_rows_modes<3, 1>(ctx, p) : launch_rows_modes<2, 1>(ctx, p);
    return a.balanced ? launch_rows_modes<1, 3>(ctx, p) : launch_rows_modes<1, 2>(ctx, p);
}

}  // namespace adapt

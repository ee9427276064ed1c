// Weight gradients on image rows in LDS (contract_rows.hpp), two operands of two limbs
#include "contract_rows.hpp"

namespace adapt {
hipError_t launch_rows_both(adapt_ctx *ctx, const ContractPlan &p)
{
    return p.kern.balanced ? launch_rows_modes<3, 3>(ctx, p) : launch_rows_modes<2, 2>(ctx, p);
}
}  // namespace adapt

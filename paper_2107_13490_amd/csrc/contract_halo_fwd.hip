// Forward pass of stride-1 convolutions on input patches in LDS (contract_halo.hpp)
#include "contract_halo.hpp"

namespace adapt {
hipError_t launch_halo_fwd(adapt_ctx *ctx, const ContractPlan &p) { return launch_halo<OP_FWD>(ctx, p); }
}  // namespace adapt

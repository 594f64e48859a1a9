// chain kernel instantiations: double components, left factors as GOOMs
#include "goom_chain_kernel.h"

namespace goom_chain {
int dispatch_f64_goom(goom_ctx *ctx, const ChainArgs &args, int dp, int nw, long long grid, const char *label)
{
    return dispatch<double>(ctx, args, dp, nw, grid, label);
}
} // namespace goom_chain

// Backward in five products: element type f16, head dim 64.
#include "sdpa_bwd_chain_kernel.h"

namespace tsdpa {
int launch_bwd_chain_f16_d64(const BwdLaunchArgs &a, int per_claim) { return launch_bwd_chain<_Float16, 64>(a, per_claim); }
}  // namespace tsdpa

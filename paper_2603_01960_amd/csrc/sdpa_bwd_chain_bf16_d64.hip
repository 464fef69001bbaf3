// Backward in five products: element type bf16, head dim 64.
#include "sdpa_bwd_chain_kernel.h"

namespace tsdpa {
int launch_bwd_chain_bf16_d64(const BwdLaunchArgs &a, int per_claim) { return launch_bwd_chain<__bf16, 64>(a, per_claim); }
}  // namespace tsdpa

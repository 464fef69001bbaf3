// Backward in five products: element type f16, head dim 128.
#include "sdpa_bwd_chain_kernel.h"

namespace tsdpa {
int launch_bwd_chain_f16_d128(const BwdLaunchArgs &a, int per_claim) { return launch_bwd_chain<_Float16, 128>(a, per_claim); }
}  // namespace tsdpa

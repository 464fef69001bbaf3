// Decoding-kernel instantiations: element type bf16.
#include <mutex>

#include "sdpa_decode_kernel.h"

namespace tsdpa {
int launch_decode_bf16(int D, const LaunchArgs &a) { return launch_decode<__bf16>(D, a); }
}  // namespace tsdpa

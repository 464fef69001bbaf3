// Decoding-kernel instantiations: element type f16.
#include <mutex>

#include "sdpa_decode_kernel.h"

namespace tsdpa {
int launch_decode_f16(int D, const LaunchArgs &a) { return launch_decode<_Float16>(D, a); }
}  // namespace tsdpa

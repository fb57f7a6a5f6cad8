// Instantiations of the four-row recurrent kernel for k depth 16 (h rows up to 1024 bytes).
#include "quad_kernel.inc.h"

namespace lstm_int {
quad_fn quad_pick_16(int fl) { return quad_pick_ks<16>(fl); }
}  // namespace lstm_int

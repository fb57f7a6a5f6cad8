// Instantiations of the four-row recurrent kernel for k depth 8 (h rows up to 512 bytes).
#include "quad_kernel.inc.h"

namespace lstm_int {
quad_fn quad_pick_8(int fl) { return quad_pick_ks<8>(fl); }
}  // namespace lstm_int

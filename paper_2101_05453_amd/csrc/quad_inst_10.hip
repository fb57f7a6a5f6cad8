// Instantiations of the four-row recurrent kernel for k depth 10 (h rows up to 640 bytes).
#include "quad_kernel.inc.h"

namespace lstm_int {
quad_fn quad_pick_10(int fl) { return quad_pick_ks<10>(fl); }
}  // namespace lstm_int

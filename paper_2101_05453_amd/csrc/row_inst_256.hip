// Instantiations of the kernel with one batch row per workgroup for layers of up to 256 cells and outputs.
#include "row_kernel.inc.h"

namespace lstm_int {
row_fn row_pick_256(int fl, bool own) { return own ? row_pick_size<16, 4, true>(fl) : row_pick_size<16, 4, false>(fl); }
}  // namespace lstm_int

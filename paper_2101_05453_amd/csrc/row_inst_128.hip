// Instantiations of the kernel with one batch row per workgroup for layers of up to 128 cells and outputs.
#include "row_kernel.inc.h"

namespace lstm_int {
row_fn row_pick_128(int fl, bool own) { return own ? row_pick_size<8, 2, true>(fl) : row_pick_size<8, 2, false>(fl); }
}  // namespace lstm_int

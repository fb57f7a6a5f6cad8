// Instantiations of the kernel with one batch row per workgroup for several layers of up to 64 cells and outputs in one launch.
#include "row_kernel.inc.h"

namespace lstm_int {
row_stack_fn row_stack_pick_64(int fl) { return row_pick_size<4, 1, kRowStack, 0>(fl); }
}  // namespace lstm_int

// Instantiations of the kernel with one batch row per workgroup for several layers of up to 128 cells and outputs in one launch.
#include "row_kernel.inc.h"

namespace lstm_int {
row_stack_fn row_stack_pick_128(int fl) { return row_pick_size<8, 2, kRowStack, 0>(fl); }
}  // namespace lstm_int

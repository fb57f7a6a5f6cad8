// Instantiations of the kernel with one batch row per workgroup for several layers in one launch, up to 256 cells and 192 outputs, and,
// with a projection, up to 128 outputs.
#include "row_kernel.inc.h"

namespace lstm_int {
row_stack_fn row_stack_pick_192(int fl) { return row_pick_size<16, 3, kRowStack, 0>(fl); }
row_stack_fn row_stack_pick_256_128(int fl) { return row_pick_size<16, 2, kRowStack, 8>(fl); }
}  // namespace lstm_int

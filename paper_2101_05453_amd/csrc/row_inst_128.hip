// Instantiations of the kernel with one batch row per workgroup for layers of up to 128 cells and outputs.
#include "row_kernel.inc.h"

namespace lstm_int {
row_fn row_pick_128(int fl, bool own) { return own ? row_pick_size<8, 2, kRowOwn, 0>(fl) : row_pick_size<8, 2, kRowTerms, 0>(fl); }
}  // namespace lstm_int

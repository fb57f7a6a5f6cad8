// Instantiations of the kernel with one batch row per workgroup for layers of up to 64 cells and outputs.
#include "row_kernel.inc.h"

namespace lstm_int {
row_fn row_pick_64(int fl, bool own) { return own ? row_pick_size<4, 1, kRowOwn, 0>(fl) : row_pick_size<4, 1, kRowTerms, 0>(fl); }
}  // namespace lstm_int

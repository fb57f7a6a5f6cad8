// Instantiations of the kernel with one batch row per workgroup for layers of 129 to 256 cells or outputs: by the k steps of R h.
#include "row_kernel.inc.h"

namespace lstm_int {
row_fn row_pick_256(int fl, bool own) { return own ? row_pick_size<16, 4, kRowOwn, 0>(fl) : row_pick_size<16, 4, kRowTerms, 0>(fl); }
}  // namespace lstm_int

// Instantiations of the kernel with one batch row per workgroup for layers of 129 to 256 cells and up to 192 outputs, and, with a
// projection, up to 128 outputs.
#include "row_kernel.inc.h"

namespace lstm_int {
row_fn row_pick_192(int fl, bool own) { return own ? row_pick_size<16, 3, kRowOwn, 0>(fl) : row_pick_size<16, 3, kRowTerms, 0>(fl); }
row_fn row_pick_256_128(int fl, bool own) { return own ? row_pick_size<16, 2, kRowOwn, 8>(fl) : row_pick_size<16, 2, kRowTerms, 8>(fl); }
}  // namespace lstm_int

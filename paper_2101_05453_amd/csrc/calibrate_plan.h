// Sizes of the statistics run (calibrate.hip) that the host works out, apart from device code so that they can be checked on
// a CPU.
#pragma once

#include <stdint.h>

namespace lstm_int {

// Rows that one launch of a product takes when a workgroup takes `block` of them: the row blocks are grid.y, which holds
// 65535.
constexpr int64_t calibrate_rows_per_launch(int block) { return (int64_t)65535 * block; }
// Batch rows of one launch of the cell kernels, a workgroup of 512 threads each: grid.x holds less than 2^32 threads.
constexpr int kCalibrateCellRows = 1 << 22;

}  // namespace lstm_int

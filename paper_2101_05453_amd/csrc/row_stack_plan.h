// Which layer and row a workgroup of a launch of several small layers works on (row_kernel.inc.h, kRowStack), apart from device code
// so that it can be checked on a CPU.
#pragma once

#include "lstm_int_math.h"

namespace lstm_int {

// A chain is one row in one direction of time, its links are the layers: rows and directions never interact, so a workgroup waits for
// one other alone, the link below in its chain.  The chain is the workgroup's by its index, the link by the order in which the
// chain's workgroups start (a count in memory that each of them raises once): whoever is waited for is running or has ended
// already, however few workgroups fit the chip and whatever else runs on it.  Links by the index, layer after layer, would not
// have that: workgroups go to the XCDs by turns, each XCD starts its own in their order, and of two launches on two streams each could
// fill the XCD on which the other's lower layer is still to start.  Links by the index -> by the count, us:
// 2 layers of 64 cells, 1 row, 1 step 11.9 -> 11.8; 6 of 64, 4 rows, 40 steps 83.8 -> 81.9; 2 of 256, layer norm, 128 rows, 8 steps 54.3 ->
// 54.8; 2 of 203 cells, 37 rows, peephole, 4 steps 29.4 -> 30.0, 60 steps 123.4 -> 124.8, with a projection too 139.2 -> 139.2.
struct RowStackPlace {
  int chain, dir, row;
};
LSTM_HD RowStackPlace row_stack_place(int block, int rows, int dirs) {
  const int chain = (int)((unsigned)block % (unsigned)(dirs * rows)), dir = chain >= rows ? 1 : 0;  // two directions at most
  return {chain, dir, dir ? chain - rows : chain};
}
// Index of the layer's arguments
LSTM_HD int row_stack_link(int order, int dir, int dirs) { return order * dirs + dir; }

}  // namespace lstm_int

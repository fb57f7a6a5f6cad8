// Choices of the SRU's forward call (sru.hip) that the host makes from sizes alone, apart from device code so that they can be
// checked on a CPU.
#pragma once

#include <stdint.h>

namespace lstm_int {

constexpr int kScanBlock = 256;      // threads per workgroup of the scan (each workgroup holds a table: two per compute unit)
constexpr int kScanBlockFull = 512;  // with the table of all values (128 KB): one workgroup per compute unit

// Whether a scan of `threads` threads (four cells each) takes the table of all values: fewer instructions per step, in
// workgroups twice as large.  Let w be the number of the other form's workgroups.
// Row-major terms: as soon as those have no compute unit each.  One layer, 64 steps, the other form -> this one, us, 2048 cells
// with the identity: w = 256 (128 rows) 45.6 -> 47.1, 258 59 -> 47, 512 65.7 -> 52.8, 520 92.9 -> 92.4, 1024 129 -> 117; with a
// highway matrix: 260 56 -> 42, 512 61 -> 54.  Loading it pays from one step on (w = 512: 7.3 -> 7.2, three steps 9.6 -> 9.5;
// w = 260, five steps 11.9 -> 10.2).
// Tile-ordered terms: memory bounds a full chip and the two are even there (1024 cells with the identity, w = 512: 134.9 ->
// 133.4; 2048 cells with a matrix 93 -> 93); with fewer the small workgroups fill it better (256: 62 -> 120, 288: 119 -> 121).
// Beyond that what counts is the last round, of two small workgroups per compute unit or one large: if small ones have a
// compute unit each in it they end sooner (w = 640: 193 -> 237 and 130 -> 158, 768: 206 -> 248 and 142 -> 168), if not the large
// one does (832: 177 -> 175 with a matrix, 896: 264 -> 260 and 184 -> 180, 1024: 280 -> 267 and 199 -> 186).
inline bool scan_takes_full_table(bool tile, int64_t threads, int cus) {
  const int64_t w = (threads + kScanBlock - 1) / kScanBlock;
  if (cus < 1 || w <= cus) return false;
  if (!tile) return true;
  const int64_t last = w % (2 * cus);
  return w > 2 * cus && (last == 0 || last > cus);
}

}  // namespace lstm_int

// Sizes of the statistics run (calibrate.hip) that the host works out, apart from device code so that they can be checked on
// a CPU.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "../../include/lstm_int.h"

namespace lstm_int {

// Where a call keeps what, in one allocation.  Kept through the call: the statistics, the raw parameters and the vectors of
// a layer (the next layer's are uploaded while this one computes), and the layer inputs and outputs, which change places
// from layer to layer.  The rest belongs to one layer at a time, so the layers share the same bytes, each with a layout of
// its own (the largest of every buffer over the layers at once would take more than any layer needs when they differ).  A
// layer's parameters are there twice, as uploaded and in the order of the products.
struct CalibrateRegion {
  size_t off = 0, bytes = 0;
};
struct CalibrateLayer {
  CalibrateRegion wop, rop, pop, wx, m, h, c, pre, part, amax;
};
struct CalibratePlan {
  CalibrateRegion stats, raw, vec[2], act[2], ext;
  std::vector<CalibrateLayer> layers;
  size_t total = 0;
};

// Workgroups of the cell kernel that share a batch row: up to the 256 compute units, at least 128 cells each.
inline int calibrate_cell_slices(int64_t N, uint32_t flags, int64_t B) {
  const bool whole_row = (flags & LSTM_INT_PEEPHOLE) && (flags & LSTM_INT_LAYER_NORM);
  return whole_row ? 1 : (int)std::max<int64_t>(1, std::min<int64_t>(256 / B, (N + 127) / 128));
}
constexpr int kCalibrateRowMax = 4096;  // cells of the widest row that the cell kernel holds in registers
// Whether a product of M rows and Nout columns runs in blocks of 128 x 128: enough of them to fill half of the chip.
inline bool calibrate_wide_product(int64_t M, int64_t Nout) { return ((M + 127) / 128) * ((Nout + 127) / 128) >= 128; }
// Whether the products of the steps take the layer norm's sums along, so that the cell kernel needs no pass over its row: a
// group of 32 columns lies in one gate, the sum is whole then (a peephole adds to it) and k is split over the waves, which
// store whole groups.
inline bool calibrate_sums_in_product(int64_t N, uint32_t flags, int64_t B) {
  return (flags & LSTM_INT_LAYER_NORM) && !(flags & LSTM_INT_PEEPHOLE) && N % 32 == 0 && N <= kCalibrateRowMax &&
         !calibrate_wide_product(B, (flags & LSTM_INT_CIFG ? 3 : 4) * N);
}
// Running extremes of the cell kernel, a value of each per thread and workgroup in memory, up to 256 batch rows and so 256
// workgroups; beyond, a workgroup reduces its own at every step.  Seven of 512 threads where the kernel takes the gate sums'
// too, three of the 128 that have cells where it does not; 0: none.
constexpr int kCalibrateExtremes = 7;
inline size_t calibrate_extreme_values(int64_t N, uint32_t flags, int64_t B) {
  if (B > 256 || N > kCalibrateRowMax) return 0;
  const bool own_sums = (flags & LSTM_INT_LAYER_NORM) && !calibrate_sums_in_product(N, flags, B);
  return (size_t)B * calibrate_cell_slices(N, flags, B) * (own_sums ? kCalibrateExtremes * 512 : (kCalibrateExtremes - 4) * 128);
}

inline int64_t calibrate_up16(int64_t v) { return (v + 15) / 16 * 16; }

inline CalibratePlan calibrate_plan(const lstm_int_layer_params *layers, int num_layers, int64_t T, int64_t B,
                                    size_t stats_bytes_per_layer) {
  CalibratePlan p;
  p.layers.resize(num_layers);
  size_t off = 0;
  auto place = [&](CalibrateRegion &r, size_t bytes) {
    r.off = off;
    r.bytes = bytes;
    off += (bytes + 255) & ~(size_t)255;
  };
  auto up16 = [](size_t v) { return (size_t)calibrate_up16((int64_t)v); };
  size_t raw = 0, vec = 0, ext = 0, act[2] = {up16((size_t)T * B) * up16(layers[0].input_size), 0};
  for (int l = 0; l < num_layers; ++l) {
    const size_t I = layers[l].input_size, N = layers[l].num_cells, H = layers[l].output_size;
    raw = std::max(raw, 4 * N * (I + H) + ((layers[l].flags & LSTM_INT_PROJECTION) ? H * N : 0));
    vec = std::max(vec, 11 * N + H);
    ext = std::max(ext, calibrate_extreme_values(N, layers[l].flags, B));
    act[(l + 1) & 1] = std::max(act[(l + 1) & 1], up16((size_t)T * B) * up16(H));  // layer l writes what layer l + 1 reads
  }
  // the statistics, and behind them the running extremes they are taken from
  p.ext.off = (stats_bytes_per_layer * num_layers + 255) & ~(size_t)255;
  p.ext.bytes = sizeof(double) * ext;
  place(p.stats, p.ext.off + p.ext.bytes);
  place(p.raw, sizeof(float) * raw);
  for (CalibrateRegion &r : p.vec) place(r, sizeof(float) * vec);
  for (int i = 0; i < 2; ++i) place(p.act[i], sizeof(double) * act[i]);
  const size_t shared = off;
  p.total = off;
  for (int l = 0; l < num_layers; ++l) {
    const size_t I = layers[l].input_size, N = layers[l].num_cells, H = layers[l].output_size;
    CalibrateLayer &r = p.layers[l];
    off = shared;
    place(r.wop, sizeof(float) * up16(4 * N) * up16(I));
    place(r.rop, sizeof(float) * up16(4 * N) * up16(H));
    if (layers[l].flags & LSTM_INT_PROJECTION) place(r.pop, sizeof(float) * up16(H) * up16(N));
    place(r.wx, sizeof(double) * T * B * 4 * N);
    place(r.m, sizeof(double) * up16(B) * up16(N));
    place(r.h, sizeof(double) * up16(B) * up16(H));
    place(r.c, sizeof(double) * B * N);
    place(r.pre, sizeof(double) * B * 4 * N);
    if (calibrate_sums_in_product(N, layers[l].flags, B)) {  // sums and extremes of the gates' groups of 32 cells
      place(r.part, sizeof(double) * 2 * B * (4 * N / 32));
      place(r.amax, sizeof(double) * B * (4 * N / 32));
    }
    p.total = std::max(p.total, off);
  }
  return p;
}

// Rows that one launch of a product takes when a workgroup takes `block` of them: the row blocks are grid.y, which holds
// 65535.
constexpr int64_t calibrate_rows_per_launch(int block) { return (int64_t)65535 * block; }
// Batch rows of one launch of the cell kernels, a workgroup of 512 threads each: grid.x holds less than 2^32 threads.
constexpr int kCalibrateCellRows = 1 << 22;

}  // namespace lstm_int

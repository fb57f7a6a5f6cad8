// Persistent recurrent kernels of the integer GRU (gru_seq.hip): one launch runs all T steps of a layer.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "persistent.h"

namespace lstm_int {

struct GruSeqArgs {
  int32_t B, N, T, Kp;        // Kp: state depth padded to 64
  int32_t GS, groups;         // workgroups per group (tiles of 64 cells); groups of this launch
  int32_t rows_pg, batch0;    // rows per group: 4, 16 or 32; first row of the launch, a multiple of 32
  const int8_t *R16;          // [GS][4 waves][3 gates][Kp / 64][64 lanes][16 B]: lane (c, q) holds bytes 64 k + 16 q .. of the
                              // row of cell 16 wave + c of the tile, an operand of the 16x16x64 MFMA on either side
  const int32_t *bh;          // [3][Nc], Nc = 64 GS
  const int4 *tx2;            // input term in the input GEMM's tile order [(t Bp + b) / 32][tile of 8 cells][half][lane][8 values],
  int32_t tiles, Bp;          //   lane (row, half) value 4 slot + c: gate slot - 1; or NULL:
  const int16_t *tx;          // row-major [T B][3 Nt], 16-byte rows
  int32_t Nt;
  int16_t *h16;               // [B][N] state, written after step T - 1, or NULL; read before step 0 unless zero_state
  int32_t zero_state;
  int8_t *h8;                 // [T][B][Kp] for the layer above, or NULL
  int8_t *y;                  // [T][B][N] or NULL
  int8_t *hx;                 // rows_pg > 4: the exchange buffer, steps or slots of [row tile of 16][Kp / 64][64 lanes][16 B].  32 rows: [T],
  size_t hx_step;             //   every line written once and never read before that; 16: [kGruAllSlots], as many of the first
                              //   kGruSlots as there are steps filled with kMarkFree.  hx_step: bytes of one
  int32_t Mh[3], rh[3];       // 3 <= rh <= 62
  LutWide lut[2];             // sigma, tanh
  uint8_t *sync;              // kGruSyncBytes, zero at launch up to gru_seq_sync_bytes
  int *status;
  int32_t spin_limit, sync_sleep;
  int32_t never;              // test hook: every wait is for something that never comes
};

// gru_rows_kernel, 16 rows: slots that the state of a step passes through by turns, and with the two escape slots (kMarkEscape) behind them
constexpr int kGruSlots = 4, kGruAllSlots = kGruSlots + 2;
// scratch: placement words [8][32 words of 8 B], flags [256 workgroups][2 row tiles][64 B], exchange words [256 workgroups][2][64 words]
constexpr size_t kGruFlagsOff = 2048, kGruWordsOff = kGruFlagsOff + 256 * 128, kGruSyncBytes = kGruWordsOff + 256 * 1024;
inline size_t gru_seq_sync_bytes(const GruSeqArgs &a) {
  return a.rows_pg == 4 ? kGruWordsOff + (size_t)a.groups * a.GS * 1024 : kGruWordsOff;
}

// rows per group for N cells and B rows, 0 = none of the kernels takes the layer; *max_groups: groups one launch can run
int gru_seq_rows(int N, int B, int *max_groups);
hipError_t gru_seq_init();
hipError_t launch_gru_seq(hipStream_t s, const GruSeqArgs &a);

}  // namespace lstm_int

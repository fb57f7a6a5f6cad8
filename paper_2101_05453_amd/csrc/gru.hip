// Integer-only GRU (include/gru_int.h): the recipe assembled from the building
// blocks of arXiv 2101.05453 (Sec. 7 names the GRU; Secs. 3.2.1, 3.2.2, 3.2.4,
// 3.2.7, 3.2.9 and Sec. 6 supply the blocks), offline phase on the host and
// the online phase as HIP kernels for gfx950.
//
// Online phase per layer:
//   1. tx = sat16(rescale(W x + bx')) for all T*B rows: the library's int8
//      MFMA matmul (kernels.hip), gate-major columns [3N].
//   2. per step ONE kernel, gru_step_kernel: R h8 + bh for the three gates on
//      the 32x32x32 int8 MFMA, a workgroup per tile of 32 cells x 32 or 64
//      batch rows, depth split over its four waves, weights and state read in
//      operand order (one contiguous KB per wave load, every byte once per
//      workgroup).  The MFMA leaves a lane with the three gate accumulators of
//      the same cells of one batch row, so the whole elementwise cell
//      (rescale, sigma/tanh tables, reset product, coupled update, the int8
//      form of the new state) follows in the same kernel with one LDS
//      reduction and no exchange between workgroups.
//   3. where the layer fits (up to 2048 cells), steps 2 of all T steps as ONE
//      persistent launch instead (gru_seq.hip): weights in registers, one
//      exchange per step inside an XCD; the input term then comes from the LSTM
//      path's register-resident input GEMM (in_gemm.hip) in its tile order
//      where its depth allows.  (Depths from 1025 to 2048: deep_gemm.hip, in
//      the general matmul's order, on either path.)
// The state is read and written in place (each (row, cell) belongs to one
// thread); its int8 form is written three times: in operand order for the
// next step, row-major for the next layer's matmul, dense for the caller.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/gru_int.h"
#include "gru_seq.h"
#include "kernels.h"
#include "lstm_int_math.h"
#include "model.h"
#include "persistent.h"

namespace lstm_int {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr double kInt32MaxD = 2147483647.0;

struct GruLayerHost {
  int32_t I = 0, N = 0, zp_x = 0;
  double s_x = 0, s_W[3] = {0, 0, 0}, s_R[3] = {0, 0, 0};
  int32_t Mx[3] = {0, 0, 0}, ex[3] = {0, 0, 0}, Mh[3] = {0, 0, 0}, eh[3] = {0, 0, 0};
  std::vector<int8_t> Wq, Rq;
  std::vector<int32_t> bxq, bhq, bx_fold;
  int64_t amax_x[3] = {0, 0, 0};  // bounds of the input accumulators
};

// padded extents of one layer on the device
struct GruDims {
  int Ip, Kp, Ncp;   // input depth / state depth (multiples of 64), cells (multiple of 32)
  int Nt, cols_pad;  // columns of a gate in the row-major input terms (multiple of 8: 16-byte pieces), 3 Nt to 128
};
GruDims gru_dims(int I, int N) {
  const int Nt = (N + 7) / 8 * 8;
  return GruDims{(I + 63) / 64 * 64, (N + 63) / 64 * 64, (N + 31) / 32 * 32, Nt, (3 * Nt + 127) / 128 * 128};
}
// bytes of the operand-ordered copy of the int8 state for B rows: whole blocks of 32 rows, an even number of them
size_t hop_bytes(int B, int Kp) { return (size_t)((B + 63) / 64 * 2) * (Kp / 32) * 1024; }

struct GruLayerDev {
  const int8_t *W = nullptr;      // [cols_pad][Ip] gate-major rows, Nt per gate, zero beyond the real extents
  const int32_t *bx = nullptr;    // [cols_pad] folded input bias
  const int8_t *Rop = nullptr;    // [Ncp/32][3][Kp/32][64 lanes][16 B]: operand order of the 32x32x32 MFMA
  const int32_t *bh = nullptr;    // [3][Ncp]
  const int8_t *R16 = nullptr;    // up to 2048 cells: R for the persistent kernels (GruSeqArgs)
  const int32_t *bh64 = nullptr;  // [3][cells to 64]
  // input depth up to 1024: W once more as the register-resident input GEMM reads it (in_gemm.hip): tiles of 8 cells
  // x 4 gate slots (slot 0 empty, slots 1-3 = r, u, n), row 8 slot + cell % 8, [tile][Ip/32][64 lanes][16 B]
  const int8_t *W2f = nullptr;
  const int32_t *bx2 = nullptr;   // [tiles][32]
  int tiles = 0;                  // a multiple of 8 (cells padded to 64)
  // depths beyond that: the form of deep_gemm.hip
  DeepWeights deep;
  const int4 *Wd = nullptr;
  const int32_t *bd = nullptr;
};

bool finite_all(const float *a, size_t n) {
  for (size_t i = 0; i < n; ++i)
    if (!std::isfinite(a[i])) return false;
  return true;
}

// symmetric int8, +-127; scale max|w| / 127 (1 for an all-zero tensor); floor(v / s + 1/2)
double quantize_tensor(const float *src, size_t n, int8_t *dst) {
  double amax = 0.0;
  for (size_t i = 0; i < n; ++i) amax = std::fmax(amax, std::fabs((double)src[i]));
  const double s = amax == 0.0 ? 1.0 : amax / 127.0;
  for (size_t i = 0; i < n; ++i) {
    double r = std::floor((double)src[i] / s + 0.5);
    dst[i] = (int8_t)std::fmin(std::fmax(r, -127.0), 127.0);
  }
  return s;
}

int32_t quantize_bias32(double v, double s) {
  double r = std::floor(v / s + 0.5);
  return (int32_t)std::fmin(std::fmax(r, -kInt32MaxD), kInt32MaxD);
}

int prepare_gru_layer(const gru_int_layer_params &p, bool has_prev, GruLayerHost &q) {
  const int I = p.input_size, N = p.num_cells;
  if (I < 1 || N < 1) return LSTM_INT_E_INVALID_ARG;
  if (I > 32768 || N > 32768) return LSTM_INT_E_UNSUPPORTED;  // accumulation depth, Sec. 3.1.1
  for (int g = 0; g < 3; ++g)
    if (!p.W[g] || !p.R[g] || !p.bx[g] || !p.bh[g]) return LSTM_INT_E_INVALID_ARG;
  q.I = I;
  q.N = N;
  if (has_prev) {  // the int8 form of the state below: scale 2^-7, zero point 0
    q.s_x = std::ldexp(1.0, -7);
    q.zp_x = 0;
  } else {  // asymmetric int8, range widened to 0, nudged zero point (Sec. 3.2.4)
    double lo = p.x_min, hi = p.x_max;
    if (!std::isfinite(lo) || !std::isfinite(hi) || lo > hi) return LSTM_INT_E_BAD_RANGE;
    lo = std::fmin(lo, 0.0);
    hi = std::fmax(hi, 0.0);
    double s = (hi - lo) / 255.0;
    if (s == 0.0) s = 1.0;
    const double z = std::floor(-128.0 - lo / s + 0.5);
    q.s_x = s;
    q.zp_x = (int32_t)std::fmin(std::fmax(z, -128.0), 127.0);
  }
  const double s_h8 = std::ldexp(1.0, -7);
  q.Wq.assign((size_t)3 * N * I, 0);
  q.Rq.assign((size_t)3 * N * N, 0);
  q.bxq.assign((size_t)3 * N, 0);
  q.bhq.assign((size_t)3 * N, 0);
  q.bx_fold.assign((size_t)3 * N, 0);
  for (int g = 0; g < 3; ++g) {
    if (!finite_all(p.W[g], (size_t)N * I) || !finite_all(p.R[g], (size_t)N * N) || !finite_all(p.bx[g], N) ||
        !finite_all(p.bh[g], N))
      return LSTM_INT_E_BAD_RANGE;
    q.s_W[g] = quantize_tensor(p.W[g], (size_t)N * I, q.Wq.data() + (size_t)g * N * I);
    q.s_R[g] = quantize_tensor(p.R[g], (size_t)N * N, q.Rq.data() + (size_t)g * N * N);
    for (int n = 0; n < N; ++n) {  // biases at the scale of their accumulators (Sec. 3.2.4)
      q.bxq[g * N + n] = quantize_bias32(p.bx[g][n], q.s_W[g] * q.s_x);
      q.bhq[g * N + n] = quantize_bias32(p.bh[g][n], q.s_R[g] * s_h8);
    }
    int rc;  // both matmul results go to Q3.12 (Sec. 3.2.4)
    if ((rc = quantize_multiplier(q.s_W[g] * q.s_x * 4096.0, &q.Mx[g], &q.ex[g])) != LSTM_INT_OK) return rc;
    if ((rc = quantize_multiplier(q.s_R[g] * s_h8 * 4096.0, &q.Mh[g], &q.eh[g])) != LSTM_INT_OK) return rc;
    for (int n = 0; n < N; ++n) {  // zero point folded (Sec. 6); accumulators safe for every int8 input
      const int8_t *w = q.Wq.data() + ((size_t)g * N + n) * I;
      int64_t sum = 0, sum_abs = 0;
      for (int k = 0; k < I; ++k) {
        sum += w[k];
        sum_abs += std::abs((int)w[k]);
      }
      const int64_t f = (int64_t)q.bxq[g * N + n] - (int64_t)q.zp_x * sum;
      if (std::llabs(f) + 128 * sum_abs > 2147483647LL) return LSTM_INT_E_UNSUPPORTED;
      q.bx_fold[g * N + n] = (int32_t)f;
      q.amax_x[g] = std::max<int64_t>(q.amax_x[g], std::llabs(f) + 128 * sum_abs);
      const int8_t *r = q.Rq.data() + ((size_t)g * N + n) * N;
      int64_t rabs = 0;
      for (int k = 0; k < N; ++k) rabs += std::abs((int)r[k]);
      if (std::llabs((int64_t)q.bhq[g * N + n]) + 128 * rabs > 2147483647LL) return LSTM_INT_E_UNSUPPORTED;
    }
  }
  return LSTM_INT_OK;
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

typedef int v16i __attribute__((ext_vector_type(16)));

// the int8 form of a state value: sat8(floor((h16 + 128) / 256))
__device__ __forceinline__ int32_t state_i8(int32_t h16) { return sat8((h16 + 128) >> 8); }

// Byte offset of state value (row, k) in the operand-ordered copy of h8 that the step kernel reads:
// [row / 32][k / 32][64 lanes][16 B], lane = 32 ((k / 16) % 2) + row % 32 -- the second operand of the
// 32x32x32 int8 MFMA for 32 rows and one 32-deep k step is one contiguous KB.
__host__ __device__ __forceinline__ size_t hop_offset(int row, int k, int KS32) {
  return ((((size_t)(row >> 5) * KS32 + (k >> 5)) * 64 + (((k >> 4) & 1) << 5) + (row & 31)) << 4) + (k & 15);
}

// Start of a layer: the working state (caller's h_state slice or zeros) is used in place; its int8 form
// goes to the operand-ordered buffer hop0 (columns N..Kp-1 zero).
__global__ void gru_init_kernel(int16_t *h16, int B, int N, int Kp, int8_t *hop0, int zero_state) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)B * Kp) return;
  const int b = (int)(i / Kp), k = (int)(i - (int64_t)b * Kp);
  int32_t v = 0;
  if (k < N) {
    if (zero_state)
      h16[(size_t)b * N + k] = 0;
    else
      v = state_i8(h16[(size_t)b * N + k]);
  }
  hop0[hop_offset(b, k, Kp >> 5)] = (int8_t)v;
}

struct GruStepArgs {
  int32_t B, N, Kp, KS32;     // KS32 = Kp / 32
  int32_t ctiles, rtn;        // tiles of 32 cells; tiles of 32 RB rows
  const int8_t *hop_prev;     // state before the step, operand order
  const int8_t *Rop;          // [ctiles][3][KS32][64 lanes][16 B]
  const int32_t *bh;          // [3][32 ctiles]
  const int16_t *tx;          // [B][3 Nt] of this step, or NULL:
  int32_t Nt;
  const int4 *tx2;            // this step's input terms in the input GEMM's tile order [row block][tile of 8 cells][half][lane][8]
  int32_t tiles;              // tiles of 8 cells per row block of tx2
  int16_t *h16;               // [B][N] in/out
  int8_t *hop_out;            // state after the step, operand order
  int8_t *h8_out;             // [B][Kp] row-major (the next layer's matmul input)
  int8_t *y;                  // [B][N] or NULL
  int32_t Mh[3], rh[3];
  const uint16_t *sig_tab, *tanh_tab;  // [32769] each, Q3.12 inputs
  int16_t *tr_tx, *tr_th, *tr_act, *tr_h16;  // [B][3][N] / [B][N] of this step, or NULL
  int8_t *tr_h8;
};

// One step of one layer.  A workgroup owns 32 cells (their r, u, n rows of R: 96 x Kp bytes) and 32 RB batch
// rows (the library launches RB = 1); its four waves split the depth, each running its quarter of the k steps for all RB x 3 tiles of the
// 32x32x32 int8 MFMA with both operands loaded straight into registers in operand order (every byte of the
// weight slice and of the state tile is loaded once per workgroup, a contiguous KB per wave load), and the four
// partial sums meet in LDS.  The MFMA leaves a lane with 16 cells of one batch row, the same cells in each of
// the three gate tiles, so the elementwise cell needs no further exchange.
// Workgroup w takes cell tile (w % 8) + 8 (w / 8 / rtn): the hardware deals consecutive workgroups out to the
// eight XCDs in turn, and every launch here is a multiple of eight workgroups, so an XCD meets the same eighth
// of R at every step of a sequence and keeps it in its L2 (N = 2048: 1.5 MB of 4 MB).  The mapping only places
// the work; results do not depend on where a workgroup runs.
constexpr int kPartTile = 32 * 33;  // one 32 x 32 tile of partial sums in LDS, row stride 33

template <int RB>
__global__ __launch_bounds__(256) void gru_step_kernel(GruStepArgs a) {
  extern __shared__ __attribute__((aligned(16))) int32_t part[];  // [4 waves][RB][3][kPartTile]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 31, b2 = lane >> 5;
  const int w = blockIdx.x, j = w >> 3;
  const int ct = (w & 7) + 8 * (j / a.rtn), rt = j % a.rtn;
  if (ct >= a.ctiles) return;  // uniform over the workgroup, ahead of every barrier
  const int KS = a.KS32;
  const int rblocks = (a.B + 31) >> 5;  // row blocks that exist in the operand-ordered buffers

  // this thread's share of the elementwise cell, and its W x terms and old state requested now: they come from
  // memory and are not needed before the matmul is done
  const int rsub = threadIdx.x >> 3, cg = threadIdx.x & 7;
  const int N = a.N;
  const int n0 = ct * 32 + 4 * cg;
  const bool vec = (N & 3) == 0;  // runs of four cells are aligned 8-byte pieces of h16
  int rowe[RB];
  int32_t txe[RB][3][4], h16e[RB][4];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    rowe[rb] = (rt * RB + rb) * 32 + rsub;
    const int row = rowe[rb] < a.B ? rowe[rb] : a.B - 1;
    const int16_t *hq = a.h16 + (size_t)row * N + n0;
    if (vec && n0 < N) {
      const short4 h4 = *reinterpret_cast<const short4 *>(hq);
      h16e[rb][0] = h4.x; h16e[rb][1] = h4.y; h16e[rb][2] = h4.z; h16e[rb][3] = h4.w;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) h16e[rb][c] = n0 + c < N ? hq[c] : 0;
    }
    if (a.tx2) {
      // the input term in the register-resident input GEMM's tile order (this step's row blocks): lane
      // (row % 32, half) of tile n / 8 holds value 4 slot + c for cell 8 (n / 8) + 4 half + c; slots 1-3 = r, u, n
      const int4 *tp = a.tx2 + ((size_t)(rt * RB + rb) * a.tiles + (ct * 4 + (cg >> 1))) * 128 + ((cg & 1) << 5) + rsub;
#pragma unroll
      for (int g = 0; g < 3; ++g) {
        const int slot = g + 1;
        const short4 t4 = *reinterpret_cast<const short4 *>(reinterpret_cast<const int16_t *>(tp + (slot >> 1) * 64) + (slot & 1) * 4);
        txe[rb][g][0] = t4.x; txe[rb][g][1] = t4.y; txe[rb][g][2] = t4.z; txe[rb][g][3] = t4.w;
      }
    } else {
      const int16_t *txp = a.tx + (size_t)row * 3 * a.Nt + n0;
#pragma unroll
      for (int g = 0; g < 3; ++g) {
        const short4 t4 = n0 < a.Nt ? *reinterpret_cast<const short4 *>(txp + (size_t)g * a.Nt) : short4{0, 0, 0, 0};
        txe[rb][g][0] = t4.x; txe[rb][g][1] = t4.y; txe[rb][g][2] = t4.z; txe[rb][g][3] = t4.w;
      }
    }
  }

  v16i acc[RB][3];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int g = 0; g < 3; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[rb][g][v] = 0;
  const v4i *wp = reinterpret_cast<const v4i *>(a.Rop) + (size_t)ct * 3 * KS * 64 + lane;
  const v4i *hp[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    int blk = rt * RB + rb;
    blk = blk < rblocks ? blk : rblocks - 1;  // a row block past the batch repeats the last one; never stored
    hp[rb] = reinterpret_cast<const v4i *>(a.hop_prev) + (size_t)blk * KS * 64 + lane;
  }
  const int per = (KS + 3) >> 2;
  const int k0 = wave * per, k1 = k0 + per < KS ? k0 + per : KS;
  // U k steps per batch, all their loads in flight together (one wave per SIMD: nothing else hides the
  // latency); steps past the wave's share re-read its last step against zero weights
  constexpr int U = 8;
  for (int ks = k0; ks < k1; ks += U) {
    v4i hf[U][RB], wf[U][3];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = ks + u < k1 ? ks + u : k1 - 1;
#pragma unroll
      for (int g = 0; g < 3; ++g) wf[u][g] = wp[((size_t)g * KS + kk) * 64];
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) hf[u][rb] = hp[rb][(size_t)kk * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool live = ks + u < k1;
#pragma unroll
      for (int g = 0; g < 3; ++g) {
        const v4i wv = live ? wf[u][g] : v4i{0, 0, 0, 0};
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
          acc[rb][g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wv, hf[u][rb], acc[rb][g], 0, 0, 0);
      }
    }
  }
  // partial sums -> LDS as [wave][rb][gate][2 v + b2][33]: result value v of lane (col, b2) is cell
  // 8 (v / 4) + 4 b2 + v % 4 of the tile for batch row col; the odd stride keeps the transposed reads below
  // at two lanes per bank
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int g = 0; g < 3; ++g)
#pragma unroll
      for (int v = 0; v < 16; ++v) part[((wave * RB + rb) * 3 + g) * kPartTile + (2 * v + b2) * 33 + col] = acc[rb][g][v];
  __syncthreads();

  // The elementwise cell, with the threads laid out along the rows: thread (rsub, cg) takes cells 4 cg .. 4 cg + 3
  // of row rsub in each row block, so that a wave's loads and stores cover runs of 32 consecutive cells of 8 rows
  // (a lane's four cells share the result index v / 4 = cg / 2 and the lane half b2 = cg % 2).
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int row = rowe[rb];
    const bool row_ok = row < a.B;
    int32_t h84[4], hn4[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int n = n0 + c;
      int32_t th[3];
#pragma unroll
      for (int g = 0; g < 3; ++g) {
        const int o = (rb * 3 + g) * kPartTile + (2 * (4 * (cg >> 1) + c) + (cg & 1)) * 33 + rsub;
        const int32_t sum = part[o] + part[o + RB * 3 * kPartTile] + part[o + 2 * RB * 3 * kPartTile] + part[o + 3 * RB * 3 * kPartTile];
        th[g] = sat16(rescale(sum + a.bh[g * 32 * a.ctiles + n], a.Mh[g], a.rh[g]));
      }
      const int32_t r = sigmoid_from_table(a.sig_tab, sat16(txe[rb][0][c] + th[0]));  // Sec. 3.2.1
      const int32_t u = sigmoid_from_table(a.sig_tab, sat16(txe[rb][1][c] + th[1]));
      const int32_t rn = (mul_i24(r, th[2]) + 16384) >> 15;  // Q0.15 x Q3.12 -> Q3.12; |r th| < 2^30
      const int32_t cand = tanh_from_table(a.tanh_tab, sat16(txe[rb][2][c] + rn));
      const int32_t ubar = cifg_input_gate(u);  // 1 - u, Sec. 3.2.9
      const int32_t hn = cell_update32(ubar, cand, u, h16e[rb][c], 0);  // Sec. 3.2.7, both products Q0.30 -> Q0.15
      hn4[c] = hn;
      h84[c] = state_i8(hn);
      if (row_ok && n < N) {
        const size_t row3 = (size_t)row * 3 * N;
        if (a.tr_tx)
          for (int g = 0; g < 3; ++g) a.tr_tx[row3 + (size_t)g * N + n] = (int16_t)txe[rb][g][c];
        if (a.tr_th)
          for (int g = 0; g < 3; ++g) a.tr_th[row3 + (size_t)g * N + n] = (int16_t)th[g];
        if (a.tr_act) {
          a.tr_act[row3 + n] = (int16_t)r;
          a.tr_act[row3 + (size_t)N + n] = (int16_t)u;
          a.tr_act[row3 + (size_t)2 * N + n] = (int16_t)cand;
        }
        if (a.tr_h16) a.tr_h16[(size_t)row * N + n] = (int16_t)hn;
        if (a.tr_h8) a.tr_h8[(size_t)row * N + n] = (int8_t)h84[c];
      }
    }
    if (!row_ok || n0 >= N) continue;
    int16_t *hd = a.h16 + (size_t)row * N + n0;
    if (vec) {
      short4 o4;
      o4.x = (short)hn4[0]; o4.y = (short)hn4[1]; o4.z = (short)hn4[2]; o4.w = (short)hn4[3];
      *reinterpret_cast<short4 *>(hd) = o4;
    } else {
      for (int c = 0; c < 4 && n0 + c < N; ++c) hd[c] = (int16_t)hn4[c];
    }
    // the int8 form: operand order for the next step, row-major for the next layer, dense for the caller
    uint32_t pk = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) pk |= (uint32_t)((n0 + c < N ? h84[c] : 0) & 0xFF) << (8 * c);
    *reinterpret_cast<uint32_t *>(a.hop_out + hop_offset(row, n0, KS)) = pk;  // cells past N hold 0 and meet zero weights
    *reinterpret_cast<uint32_t *>(a.h8_out + (size_t)row * a.Kp + n0) = pk;
    if (a.y) {
      int8_t *yd = a.y + (size_t)row * N + n0;
      if (vec && !(reinterpret_cast<uintptr_t>(a.y) & 3))
        *reinterpret_cast<uint32_t *>(yd) = pk;
      else
        for (int c = 0; c < 4 && n0 + c < N; ++c) yd[c] = (int8_t)h84[c];
    }
  }
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

}  // namespace lstm_int

using namespace lstm_int;

struct GruTimed {  // one timed stretch of launches of a forward call made while profiling
  hipEvent_t start, stop;
  int cls, launches;
};

struct gru_int_model {
  int device = -1;
  bool profiling = false;
  std::vector<GruTimed> timed;
  int persistent = 1;   // layers that fit run all their steps in one launch (gru_seq.hip)
  int spin_limit = 1 << 21, sync_sleep = 4;
  int extra_arrivals = 0;  // test hook (option "barrier_never_completes")
  int *status = nullptr;  // device word: nonzero once a wait inside a persistent kernel gave up (1) or placement failed (2)
  int num_cus = 0;
  std::vector<GruLayerHost> host;
  std::vector<GruLayerDev> dev;
  uint8_t *arena = nullptr;
  const uint16_t *sig_tab = nullptr, *tanh_tab = nullptr;
  LutWide lut[2] = {};     // the same two as the persistent kernels keep them (dom = 0: they do not compress, and none runs)
};

namespace {

// carve-up of the workspace for (T, B)
struct GruWs {
  size_t xpad, tx, out[2], hop[2], h16, sync, hop_seq, total;
};
GruWs gru_workspace(const gru_int_model *m, int64_t T, int64_t B) {
  GruWs w{};
  size_t off = 0, max_tx = 0, max_out = 0, max_hop = 0, sum_h16 = 0;
  for (const GruLayerHost &q : m->host) {
    const GruDims d = gru_dims(q.I, q.N);
    max_tx = std::max(max_tx, (size_t)T * B * 3 * d.Nt * 2);
    // the same terms in the register-resident input GEMM's tile order: rows padded to 32 per step, cells to 64, 4 gate slots
    max_tx = std::max(max_tx, (size_t)T * ((B + 31) / 32 * 32) * ((q.N + 63) / 64 * 64) * 4 * 2);
    max_out = std::max(max_out, ((size_t)T * B + 32) * d.Kp);
    max_hop = std::max(max_hop, hop_bytes((int)B, d.Kp));
    sum_h16 = std::max(sum_h16, (size_t)B * q.N * 2);
  }
  const GruDims d0 = gru_dims(m->host[0].I, m->host[0].N);
  w.xpad = off; off += align256(((size_t)T * B + 32) * d0.Ip);
  w.tx = off; off += align256(max_tx);
  w.out[0] = off; off += align256(max_out);
  w.out[1] = off; off += align256(max_out);
  w.hop[0] = off; off += align256(max_hop);
  w.hop[1] = off; off += align256(max_hop);
  w.h16 = off; off += align256(sum_h16);
  w.sync = off; off += kGruSyncBytes;
  w.hop_seq = off; off += align256(max_hop * (size_t)std::max<int64_t>(T, kGruAllSlots));  // the persistent kernels' exchange buffer
  w.total = off;
  return w;
}

}  // namespace

extern "C" {

int gru_int_prepare(const gru_int_layer_params *layers, int32_t num_layers, int32_t device, gru_int_model **out) {
  if (!layers || !out || num_layers < 1) return LSTM_INT_E_INVALID_ARG;
  *out = nullptr;
  gru_int_model *m = new (std::nothrow) gru_int_model();
  if (!m) return LSTM_INT_E_OUT_OF_MEMORY;
  try {
    m->host.resize(num_layers);
    for (int l = 0; l < num_layers; ++l) {
      if (l > 0 && layers[l].input_size != layers[l - 1].num_cells) {
        delete m;
        return LSTM_INT_E_INVALID_ARG;
      }
      const int rc = prepare_gru_layer(layers[l], l > 0, m->host[l]);
      if (rc != LSTM_INT_OK) {
        delete m;
        return rc;
      }
    }
    m->device = device;
    if (device < 0) {
      *out = m;
      return LSTM_INT_OK;
    }
    // device image: the two Q3.12 tables, then per layer W, bx, R in operand order, bh
    constexpr size_t kTab = 32769;
    std::vector<uint8_t> img;
    auto reserve = [&](size_t bytes) {
      const size_t off = align256(img.size());
      img.resize(off + bytes, 0);
      return off;
    };
    const size_t o_sig = reserve(kTab * 2), o_tanh = reserve(kTab * 2), o_status = reserve(256);
    const size_t o_wide[2] = {reserve(kLutWideBytes), reserve(kLutWideBytes)};
    fill_sigmoid_table(3, reinterpret_cast<uint16_t *>(img.data() + o_sig));
    fill_tanh_table(3, reinterpret_cast<uint16_t *>(img.data() + o_tanh));
    LutWide lut[2] = {};
    for (int i = 0; i < 2; ++i) {
      int has_tail = 0, flat_from = 0;
      const int sh = compress_table_wide(reinterpret_cast<const uint16_t *>(img.data() + (i ? o_tanh : o_sig)),
                                         img.data() + o_wide[i], &has_tail, &flat_from);
      if (sh < 0 || (!has_tail && flat_from + 1 > 32768)) continue;
      lut[i].sh = sh;
      lut[i].tail = has_tail;
      lut[i].dom = has_tail ? 16384 : (flat_from + 1 + 1023) / 1024 * 1024;
    }
    struct Off { size_t W, bx, R, bh, W2f, bx2, R16, bh64, Wd, bd; int tiles; DeepWeights deep; };
    std::vector<Off> offs(num_layers);
    for (int l = 0; l < num_layers; ++l) {
      const GruLayerHost &q = m->host[l];
      const int I = q.I, N = q.N;
      const GruDims d = gru_dims(I, N);
      const int KS = d.Kp / 32;
      Off o;
      o.W = reserve((size_t)d.cols_pad * d.Ip);
      o.bx = reserve((size_t)d.cols_pad * 4);
      o.R = reserve((size_t)(d.Ncp / 32) * 3 * KS * 1024);
      o.bh = reserve((size_t)3 * d.Ncp * 4);
      o.tiles = 0;
      o.W2f = o.bx2 = 0;
      if (d.Ip <= 1024) {
        o.tiles = (N + 63) / 64 * 8;
        o.W2f = reserve((size_t)o.tiles * 32 * d.Ip);
        o.bx2 = reserve((size_t)o.tiles * 32 * 4);
        for (int g = 0; g < 3; ++g)
          for (int n = 0; n < N; ++n) {
            const int tile = n / 8, rho = 8 * (g + 1) + n % 8;
            const int8_t *w = q.Wq.data() + ((size_t)g * N + n) * I;
            for (int k = 0; k < I; ++k)
              img[o.W2f + ((((size_t)tile * (d.Ip / 32) + k / 32) * 64) + rho + 32 * ((k % 32) / 16)) * 16 + k % 16] = (uint8_t)w[k];
            reinterpret_cast<int32_t *>(img.data() + o.bx2)[tile * 32 + rho] = q.bx_fold[g * N + n];
          }
      }
      for (int g = 0; g < 3; ++g) {
        for (int n = 0; n < N; ++n)
          std::memcpy(img.data() + o.W + ((size_t)g * d.Nt + n) * d.Ip, q.Wq.data() + ((size_t)g * N + n) * I, I);
        std::memcpy(img.data() + o.bx + (size_t)g * d.Nt * 4, q.bx_fold.data() + (size_t)g * N, (size_t)N * 4);
      }
      o.deep = deep_weights(d.Ip, 3, d.Nt);
      if (o.deep.stages) {
        o.Wd = reserve(o.deep.bytes());
        o.bd = reserve((size_t)o.deep.cbs * 128 * 4);
        deep_pack(o.deep, 3, d.Nt, d.Ip, reinterpret_cast<int8_t *>(img.data() + o.W), reinterpret_cast<int32_t *>(img.data() + o.bx),
                  reinterpret_cast<int8_t *>(img.data() + o.Wd), reinterpret_cast<int32_t *>(img.data() + o.bd));
      }
      // first operand of the 32x32x32 MFMA: lane (row = lane % 32, half = lane / 32) holds, for k step ks, bytes
      // 32 ks + 16 half .. + 15 of weight row 32 ct + row of gate g (zero beyond N in either direction)
      for (int ct = 0; ct < d.Ncp / 32; ++ct)
        for (int g = 0; g < 3; ++g)
          for (int ks = 0; ks < KS; ++ks)
            for (int lane = 0; lane < 64; ++lane) {
              const int n = ct * 32 + (lane & 31), k0 = ks * 32 + (lane >> 5) * 16;
              uint8_t *dst = img.data() + o.R + ((((size_t)ct * 3 + g) * KS + ks) * 64 + lane) * 16;
              if (n < N)
                for (int j = 0; j < 16 && k0 + j < N; ++j) dst[j] = (uint8_t)q.Rq[((size_t)g * N + n) * N + k0 + j];
            }
      for (int g = 0; g < 3; ++g)
        std::memcpy(img.data() + o.bh + (size_t)g * d.Ncp * 4, q.bhq.data() + (size_t)g * N, (size_t)N * 4);
      o.R16 = o.bh64 = 0;
      if (int cap = 0; gru_seq_rows(N, 1, &cap)) {
        const int K64 = d.Kp / 64;  // = tiles of 64 cells
        o.R16 = reserve((size_t)3 * d.Kp * d.Kp);
        o.bh64 = reserve((size_t)3 * d.Kp * 4);
        uint8_t *dst = img.data() + o.R16;
        for (int n16 = 0; n16 < K64 * 4; ++n16)
          for (int g = 0; g < 3; ++g)
            for (int ks = 0; ks < K64; ++ks)
              for (int lane = 0; lane < 64; ++lane, dst += 16) {
                const int n = n16 * 16 + (lane & 15), k0 = ks * 64 + (lane >> 4) * 16;
                if (n < N && k0 < N) std::memcpy(dst, q.Rq.data() + ((size_t)g * N + n) * N + k0, std::min(16, N - k0));
              }
        for (int g = 0; g < 3; ++g)
          std::memcpy(img.data() + o.bh64 + (size_t)g * d.Kp * 4, q.bhq.data() + (size_t)g * N, (size_t)N * 4);
      }
      offs[l] = o;
    }
    if (hipSetDevice(device) != hipSuccess || in_gemm_init() != hipSuccess || deep_gemm_init() != hipSuccess || gemm_init() != hipSuccess || gru_seq_init() != hipSuccess ||
        hipMalloc(reinterpret_cast<void **>(&m->arena), img.size()) != hipSuccess) {
      m->arena = nullptr;
      delete m;
      return LSTM_INT_E_DEVICE;
    }
    if (hipMemcpy(m->arena, img.data(), img.size(), hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipFree(m->arena);
      delete m;
      return LSTM_INT_E_DEVICE;
    }
    m->status = reinterpret_cast<int *>(m->arena + o_status);
    {
      hipDeviceProp_t prop;
      m->num_cus = hipGetDeviceProperties(&prop, device) == hipSuccess ? prop.multiProcessorCount : 0;
    }
    m->sig_tab = reinterpret_cast<const uint16_t *>(m->arena + o_sig);
    m->tanh_tab = reinterpret_cast<const uint16_t *>(m->arena + o_tanh);
    for (int i = 0; i < 2; ++i) {
      m->lut[i] = lut[i];
      m->lut[i].blob = m->arena + o_wide[i];
    }
    m->dev.resize(num_layers);
    for (int l = 0; l < num_layers; ++l) {
      m->dev[l].W = reinterpret_cast<const int8_t *>(m->arena + offs[l].W);
      m->dev[l].bx = reinterpret_cast<const int32_t *>(m->arena + offs[l].bx);
      m->dev[l].Rop = reinterpret_cast<const int8_t *>(m->arena + offs[l].R);
      m->dev[l].bh = reinterpret_cast<const int32_t *>(m->arena + offs[l].bh);
      if (offs[l].R16) {
        m->dev[l].R16 = reinterpret_cast<const int8_t *>(m->arena + offs[l].R16);
        m->dev[l].bh64 = reinterpret_cast<const int32_t *>(m->arena + offs[l].bh64);
      }
      if (offs[l].tiles) {
        m->dev[l].W2f = reinterpret_cast<const int8_t *>(m->arena + offs[l].W2f);
        m->dev[l].bx2 = reinterpret_cast<const int32_t *>(m->arena + offs[l].bx2);
        m->dev[l].tiles = offs[l].tiles;
      }
      if (offs[l].deep.stages) {
        m->dev[l].deep = offs[l].deep;
        m->dev[l].Wd = reinterpret_cast<const int4 *>(m->arena + offs[l].Wd);
        m->dev[l].bd = reinterpret_cast<const int32_t *>(m->arena + offs[l].bd);
      }
    }
  } catch (const std::bad_alloc &) {
    delete m;
    return LSTM_INT_E_OUT_OF_MEMORY;
  }
  *out = m;
  return LSTM_INT_OK;
}

int gru_int_get_quant(const gru_int_model *m, int32_t layer, gru_int_layer_quant *out) {
  if (!m || !out || layer < 0 || layer >= (int32_t)m->host.size()) return LSTM_INT_E_INVALID_ARG;
  const GruLayerHost &q = m->host[layer];
  out->I = q.I; out->N = q.N; out->zp_x = q.zp_x; out->s_x = q.s_x;
  for (int g = 0; g < 3; ++g) {
    out->s_W[g] = q.s_W[g]; out->s_R[g] = q.s_R[g];
    out->Mx[g] = q.Mx[g]; out->ex[g] = q.ex[g]; out->Mh[g] = q.Mh[g]; out->eh[g] = q.eh[g];
  }
  out->Wq = q.Wq.data(); out->Rq = q.Rq.data();
  out->bxq = q.bxq.data(); out->bhq = q.bhq.data(); out->bx_fold = q.bx_fold.data();
  return LSTM_INT_OK;
}

size_t gru_int_workspace_bytes(const gru_int_model *m, int32_t T, int32_t B) {
  if (!m || T < 0 || B < 0 || m->host.empty()) return 0;
  return gru_workspace(m, T, B).total;
}

int gru_int_forward(const gru_int_model *m, const int8_t *x, int32_t T, int32_t B, int8_t *y, int16_t *h_state,
                    void *workspace, size_t workspace_bytes, void *hip_stream, const gru_int_trace *trace) {
  if (!m || T < 0 || B < 0) return LSTM_INT_E_INVALID_ARG;
  if (T == 0 || B == 0) return LSTM_INT_OK;
  if (!x || !y) return LSTM_INT_E_INVALID_ARG;
  if (m->device < 0) return LSTM_INT_E_DEVICE;
  const int L = (int)m->host.size();
  if (trace && (trace->layer < 0 || trace->layer >= L)) return LSTM_INT_E_INVALID_ARG;
  int64_t widest = 0;
  for (const GruLayerHost &q : m->host) widest = std::max<int64_t>(widest, std::max(3 * (int64_t)q.N, (int64_t)gru_dims(q.I, q.N).Ip));
  if ((int64_t)T * B * widest >= ((int64_t)1 << 31)) return LSTM_INT_E_UNSUPPORTED;  // 32-bit row arithmetic of the matmul
  const GruWs w = gru_workspace(m, T, B);
  if (!workspace || workspace_bytes < w.total || (reinterpret_cast<uintptr_t>(workspace) & 255)) return LSTM_INT_E_WORKSPACE;
  if (hipSetDevice(m->device) != hipSuccess) return LSTM_INT_E_DEVICE;
  hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
  uint8_t *ws = reinterpret_cast<uint8_t *>(workspace);
  const int64_t TB = (int64_t)T * B;

  const int8_t *in = x;
  int ld_in = m->host[0].I;
  size_t h_off = 0;
  for (int l = 0; l < L; ++l) {
    const GruLayerHost &q = m->host[l];
    const GruLayerDev &dv = m->dev[l];
    const int N = q.N;
    const GruDims d = gru_dims(q.I, N);
    int16_t *tx = reinterpret_cast<int16_t *>(ws + w.tx);
    int8_t *out = reinterpret_cast<int8_t *>(ws + w.out[l & 1]);
    int8_t *hop[2] = {reinterpret_cast<int8_t *>(ws + w.hop[0]), reinterpret_cast<int8_t *>(ws + w.hop[1])};
    int16_t *h16 = h_state ? h_state + h_off : reinterpret_cast<int16_t *>(ws + w.h16);
    const gru_int_trace *tr = (trace && trace->layer == l) ? trace : nullptr;

    Requant rq{};
    rq.all_hi = 1;
    for (int g = 0; g < 3; ++g) {
      rq.M[g] = q.Mx[g];
      rq.r[g] = 31 - q.ex[g];
      if (rq.r[g] < 33) rq.all_hi = 0;
    }
    rq.M[3] = rq.M[2];
    rq.r[3] = rq.r[2];
    rq.cols_per_gate = d.Nt;
    rq.zp = 0;
    gru_int_model *mm = const_cast<gru_int_model *>(m);  // the profile is bookkeeping beside the model
    auto timed_begin = [&](int cls, int launches) {
      if (!m->profiling) return;
      GruTimed e{nullptr, nullptr, cls, launches};
      if (hipEventCreate(&e.start) != hipSuccess || hipEventCreate(&e.stop) != hipSuccess) return;
      (void)hipEventRecord(e.start, s);
      mm->timed.push_back(e);
    };
    auto timed_end = [&]() {
      if (m->profiling && !mm->timed.empty()) (void)hipEventRecord(mm->timed.back().stop, s);
    };
    // One launch for all steps where the layer fits (gru_seq.hip), several for batches that do not fit one
    int rows_pg = 0, max_groups = 0;
    if (m->persistent && !tr && m->num_cus == 256 && dv.R16 && m->lut[0].dom && m->lut[1].dom && T < (1 << 20))
      rows_pg = gru_seq_rows(N, B, &max_groups);
    for (int g = 0; g < 3; ++g)
      if (31 - q.eh[g] < 3 || 31 - q.eh[g] > 62) rows_pg = 0;
    const bool seq = rows_pg != 0;
    // The input term: from the LSTM path's input GEMM where the input depth allows (weights resident in registers, depth
    // up to 1024, output in its tile order, which both recurrent kernels read); else, and with a trace, from the
    // general matmul, row-major.
    InGemmArgs ga{};
    ga.A = in; ga.lda = ld_in; ga.cols = in == x ? q.I : 0; ga.T = T; ga.B = B; ga.Bp = (B + 31) / 32 * 32;
    ga.W2f = dv.W2f; ga.kpad = d.Ip; ga.tiles = dv.tiles; ga.bx2 = dv.bx2;
    ga.M[0] = 1 << 30; ga.r[0] = 33;  // the empty gate slot
    for (int g = 0; g < 3; ++g) {
      ga.M[g + 1] = q.Mx[g];
      ga.r[g + 1] = 31 - q.ex[g];
      ga.pre = std::max(ga.pre, preshift_mode(ga.r[g + 1], q.amax_x[g]));
    }
    ga.tx2 = reinterpret_cast<int4 *>(ws + w.tx);
    // (on the launch-per-step path only where the matmul is large: the tile-ordered terms cost the step kernel
    // 0.5 us per step, measured, which 8192 rows and more of a faster matmul pay for)
    const bool ws_gemm = !tr && dv.W2f && m->num_cus == 256 && (seq || TB >= 8192) && in_gemm_ws_supported(ga);
    // depths beyond 1024: the weights in registers as well (deep_gemm.hip; figures in sru.hip, whose layers take it too)
    DeepGemmArgs da{};
    da.lda = d.Ip; da.M = (int)TB; da.kpad = d.Ip; da.Wd = dv.Wd; da.bias = dv.bd;
    da.G = 3; da.N = d.Nt; da.out = tx; da.ldc = 3 * d.Nt;
    for (int g = 0; g < 3; ++g) da.rs[g] = rescale_hi_prepare(q.Mx[g], rq.r[g]);
    da.pre = ga.pre;
    const bool deep = !tr && dv.deep.stages && m->num_cus == 256 && !ws_gemm && deep_gemm_supported(da, rq.r);
    // The register-resident GEMMs read x in place in any batch (rows of 16-byte pieces, the deep one of Ip bytes); the general
    // one takes rows of Ip bytes in whole blocks of 32, a padded copy unless x already has that shape.
    if (l == 0 && !ws_gemm && (d.Ip != q.I || (reinterpret_cast<uintptr_t>(x) & 15) || (!deep && (B & 31)))) {
      int8_t *xp = reinterpret_cast<int8_t *>(ws + w.xpad);
      launch_copy_rows_i8(s, x, q.I, xp, d.Ip, (int)TB, q.I, 0);
      in = xp;
      ld_in = d.Ip;
    }
    da.A = in;  // rows of d.Ip bytes, 16-byte aligned: the caller's, the copy, or the layer below's
    GruSeqArgs sa{};
    size_t mark_bytes = 0;
    if (seq) {
      sa.B = B; sa.N = N; sa.T = T; sa.Kp = d.Kp;
      sa.GS = d.Kp / 64; sa.rows_pg = rows_pg;
      sa.groups = std::min((B + rows_pg - 1) / rows_pg, max_groups);
      sa.R16 = dv.R16; sa.bh = dv.bh64;
      sa.tx2 = ws_gemm ? ga.tx2 : nullptr;
      sa.tiles = dv.tiles; sa.Bp = ga.Bp;
      sa.tx = ws_gemm ? nullptr : tx;
      sa.Nt = d.Nt;
      sa.h16 = h_state ? h16 : nullptr; sa.zero_state = h_state ? 0 : 1;
      sa.h8 = l == L - 1 ? nullptr : out;
      sa.y = l == L - 1 ? y : nullptr;
      sa.hx = reinterpret_cast<int8_t *>(ws + w.hop_seq);
      sa.hx_step = hop_bytes(B, d.Kp);
      mark_bytes = rows_pg == 16 ? sa.hx_step * std::min(T, kGruSlots) : 0;
      for (int g = 0; g < 3; ++g) {
        sa.Mh[g] = q.Mh[g];
        sa.rh[g] = 31 - q.eh[g];
      }
      sa.lut[0] = m->lut[0]; sa.lut[1] = m->lut[1];
      sa.sync = ws + w.sync;
      sa.status = m->status;
      sa.spin_limit = m->spin_limit; sa.sync_sleep = m->sync_sleep;
      sa.never = m->extra_arrivals;
      if (ws_gemm) {  // the input GEMM clears the scratch on the way
        ga.has_init = 1;
        ga.init.sync = reinterpret_cast<int4 *>(sa.sync);
        ga.init.sync_vec = (long long)(gru_seq_sync_bytes(sa) / 16);
        ga.init.mark = reinterpret_cast<int4 *>(sa.hx);
        ga.init.mark_vec = (long long)(mark_bytes / 16);
      }
    }
    timed_begin(GRU_INT_K_INPUT_GEMM, 1);
    if (ws_gemm) {
      launch_in_gemm_ws(s, ga, m->num_cus);
    } else if (deep) {
      launch_deep_gemm(s, da, dv.deep, m->num_cus);
    } else {
      // the matmul's row arithmetic is 32-bit (padded columns may exceed what the call was checked for): in runs of rows
      const int64_t most = (((int64_t)1 << 31) - 1) / std::max(3 * d.Nt, d.Ip);
      for (int64_t r0 = 0; r0 < TB; r0 += most)
        launch_gemm_i16(s, in + r0 * ld_in, ld_in, (int)std::min(most, TB - r0), dv.W, d.Ip, 3 * d.Nt, dv.bx, rq, tx + r0 * 3 * d.Nt, 3 * d.Nt);
    }
    timed_end();
    if (seq) {
      timed_begin(GRU_INT_K_STEP, T);
      for (int b0 = 0; b0 < B; b0 += max_groups * rows_pg) {
        sa.batch0 = b0;
        sa.groups = std::min((B - b0 + rows_pg - 1) / rows_pg, max_groups);
        if (!ws_gemm && mark_bytes)  // groups of 16 rows: one launch has them all
          launch_init_layer(s, nullptr, 0, nullptr, 0, 0, 0, 0, sa.sync, (int64_t)gru_seq_sync_bytes(sa), nullptr, 0, nullptr, 0, sa.hx, (int64_t)mark_bytes);
        else if (!ws_gemm || b0 > 0)
          launch_fill_i16(s, reinterpret_cast<int16_t *>(sa.sync), (int64_t)gru_seq_sync_bytes(sa) / 2, 0);
        if (launch_gru_seq(s, sa) != hipSuccess) return LSTM_INT_E_DEVICE;
      }
      timed_end();
    } else {
    {
      const int64_t n = (int64_t)B * d.Kp;  // the state before step 0 goes where step "-1" would have put it
      hipLaunchKernelGGL(gru_init_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, h16, B, N, d.Kp, hop[1], h_state ? 0 : 1);
    }
    GruStepArgs a{};
    a.B = B; a.N = N; a.Kp = d.Kp; a.KS32 = d.Kp / 32;
    a.ctiles = d.Ncp / 32;
    a.Rop = dv.Rop; a.bh = dv.bh; a.h16 = h16;
    for (int g = 0; g < 3; ++g) {
      a.Mh[g] = q.Mh[g];
      a.rh[g] = 31 - q.eh[g];
    }
    a.sig_tab = m->sig_tab; a.tanh_tab = m->tanh_tab;
    // 32 rows per workgroup (RB = 1): at large batches two workgroups then share a compute unit and one's cell runs
    // under the other's matmul (measured at N = 2048, B = 256: 12.9 us per step against 13.3 with RB = 2)
    constexpr int rb = 1;
    a.rtn = (B + 32 * rb - 1) / (32 * rb);
    const dim3 grid((unsigned)(8 * a.rtn * ((a.ctiles + 7) / 8)));
    const size_t lds = (size_t)4 * rb * 3 * kPartTile * 4;
    timed_begin(GRU_INT_K_STEP, T);
    for (int t = 0; t < T; ++t) {
      const size_t tb = (size_t)t * B;
      a.hop_prev = hop[(t + 1) & 1];
      a.hop_out = hop[t & 1];
      a.tx = ws_gemm ? nullptr : tx + tb * 3 * d.Nt;
      a.Nt = d.Nt;
      a.tx2 = ws_gemm ? ga.tx2 + (size_t)t * (ga.Bp / 32) * dv.tiles * 128 : nullptr;
      a.tiles = dv.tiles;
      a.h8_out = out + tb * d.Kp;
      a.y = l == L - 1 ? y + tb * N : nullptr;
      a.tr_tx = tr && tr->tx ? tr->tx + tb * 3 * N : nullptr;
      a.tr_th = tr && tr->th ? tr->th + tb * 3 * N : nullptr;
      a.tr_act = tr && tr->act ? tr->act + tb * 3 * N : nullptr;
      a.tr_h16 = tr && tr->h16 ? tr->h16 + tb * N : nullptr;
      a.tr_h8 = tr && tr->h8 ? tr->h8 + tb * N : nullptr;
      hipLaunchKernelGGL(gru_step_kernel<rb>, grid, dim3(256), lds, s, a);
    }
    timed_end();
    }
    in = out;
    ld_in = d.Kp;
    h_off += (size_t)B * N;
  }
  return hipGetLastError() == hipSuccess ? LSTM_INT_OK : LSTM_INT_E_DEVICE;
}

int gru_int_set_option(gru_int_model *m, const char *key, int64_t value) {
  if (!m || !key) return LSTM_INT_E_INVALID_ARG;
  if (!strcmp(key, "persistent")) {
    if (value < 0 || value > 1) return LSTM_INT_E_INVALID_ARG;
    m->persistent = (int)value;
    return LSTM_INT_OK;
  }
  if (!strcmp(key, "spin_limit")) {
    if (value < 1 || value > (1 << 30)) return LSTM_INT_E_INVALID_ARG;
    m->spin_limit = (int)value;
    return LSTM_INT_OK;
  }
  if (!strcmp(key, "sync_sleep")) {
    if (value < 0 || value > 1024) return LSTM_INT_E_INVALID_ARG;
    m->sync_sleep = (int)value;
    return LSTM_INT_OK;
  }
  if (!strcmp(key, "barrier_never_completes")) {
    if (value < 0 || value > 1) return LSTM_INT_E_INVALID_ARG;
    m->extra_arrivals = (int)value;
    return LSTM_INT_OK;
  }
  if (!strcmp(key, "reset_status")) {
    if (m->device < 0) return LSTM_INT_E_DEVICE;
    const int zero = 0;
    if (hipSetDevice(m->device) != hipSuccess || hipDeviceSynchronize() != hipSuccess ||
        hipMemcpy(m->status, &zero, sizeof(zero), hipMemcpyHostToDevice) != hipSuccess)
      return LSTM_INT_E_DEVICE;
    return LSTM_INT_OK;
  }
  return LSTM_INT_E_INVALID_ARG;
}

int gru_int_device_status(const gru_int_model *m, int32_t *status) {
  if (!m || !status) return LSTM_INT_E_INVALID_ARG;
  if (m->device < 0) return LSTM_INT_E_DEVICE;
  int v = 0;
  if (hipSetDevice(m->device) != hipSuccess || hipDeviceSynchronize() != hipSuccess ||
      hipMemcpy(&v, m->status, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess)
    return LSTM_INT_E_DEVICE;
  *status = v;
  return LSTM_INT_OK;
}

int gru_int_profile_begin(gru_int_model *m) {
  if (!m) return LSTM_INT_E_INVALID_ARG;
  if (m->device < 0) return LSTM_INT_E_DEVICE;
  for (GruTimed &e : m->timed) {
    (void)hipEventDestroy(e.start);
    (void)hipEventDestroy(e.stop);
  }
  m->timed.clear();
  m->profiling = true;
  return LSTM_INT_OK;
}

int gru_int_profile_end(gru_int_model *m, int64_t launches[GRU_INT_K_COUNT], double total_ms[GRU_INT_K_COUNT]) {
  if (!m || !launches || !total_ms) return LSTM_INT_E_INVALID_ARG;
  if (m->device < 0) return LSTM_INT_E_DEVICE;
  m->profiling = false;
  for (int k = 0; k < GRU_INT_K_COUNT; ++k) {
    launches[k] = 0;
    total_ms[k] = 0.0;
  }
  int rc = LSTM_INT_OK;
  if (hipSetDevice(m->device) != hipSuccess) rc = LSTM_INT_E_DEVICE;
  for (GruTimed &e : m->timed) {
    float ms = 0.f;
    if (rc == LSTM_INT_OK && hipEventSynchronize(e.stop) == hipSuccess && hipEventElapsedTime(&ms, e.start, e.stop) == hipSuccess) {
      launches[e.cls] += e.launches;
      total_ms[e.cls] += ms;
    } else {
      rc = LSTM_INT_E_DEVICE;
    }
    (void)hipEventDestroy(e.start);
    (void)hipEventDestroy(e.stop);
  }
  m->timed.clear();
  return rc;
}

void gru_int_destroy(gru_int_model *m) {
  if (!m) return;
  for (GruTimed &e : m->timed) {
    (void)hipEventDestroy(e.start);
    (void)hipEventDestroy(e.stop);
  }
  if (m->arena) {
    (void)hipSetDevice(m->device);
    (void)hipFree(m->arena);
  }
  delete m;
}

}  // extern "C"

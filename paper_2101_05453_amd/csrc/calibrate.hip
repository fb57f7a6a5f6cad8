// On-GPU collection of the statistics lstm_int_prepare needs (Sec. 4,
// post-training: ranges are logged at the nodes the execution figures mark
// "log"): the float LSTM of Sec. 2 (eqs. 1-7, with the CIFG, peephole,
// layer-norm and projection variants) in double precision over representative
// inputs, with min/max of x, h and m, max |c| and, under layer norm, max |gate
// sum| per gate.  Offline tooling like prepare: it allocates device memory,
// synchronizes, and is not on the integer path.
//
// Shape of the computation: per layer one hoisted GEMM W x over all T*B rows,
// then per step a GEMM R h on top of that step's slice (with the row sums of
// the layer norm), a kernel for layer norm, activations and the cell update,
// and the projection GEMM.  Parameters stay float32 in memory (they are
// float32) and are widened on load; all arithmetic and all activations are
// double.  The products run on the f64 MFMA; while a layer computes, the next
// layer's parameters are uploaded by a second thread on a second stream.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <condition_variable>
#include <functional>
#include <mutex>
#include <new>
#include <system_error>
#include <thread>
#include <type_traits>
#include <vector>

#include "../../include/lstm_int.h"
#include "calibrate_plan.h"

namespace {

using namespace lstm_int;

constexpr int kCifg = LSTM_INT_CIFG, kPeephole = LSTM_INT_PEEPHOLE, kLayerNorm = LSTM_INT_LAYER_NORM,
              kProjection = LSTM_INT_PROJECTION;

// statistics slots in device memory
enum { S_XMIN, S_XMAX, S_HMIN, S_HMAX, S_MMIN, S_MMAX, S_CABS, S_GABS, S_COUNT = S_GABS + 4 };

__device__ void atomic_min_f64(double *addr, double v) {
  unsigned long long *p = reinterpret_cast<unsigned long long *>(addr);
  unsigned long long old = *p;
  while (v < __longlong_as_double((long long)old)) {
    const unsigned long long seen = atomicCAS(p, old, (unsigned long long)__double_as_longlong(v));
    if (seen == old) break;
    old = seen;
  }
}
__device__ void atomic_max_f64(double *addr, double v) {
  unsigned long long *p = reinterpret_cast<unsigned long long *>(addr);
  unsigned long long old = *p;
  while (v > __longlong_as_double((long long)old)) {
    const unsigned long long seen = atomicCAS(p, old, (unsigned long long)__double_as_longlong(v));
    if (seen == old) break;
    old = seen;
  }
}

// ---- reductions over a workgroup of 256 threads (4 wavefronts of 64)
__device__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ double wave_min(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}
// the same over the 16 lanes of a DPP row
template <int CTRL>
__device__ double dpp_f64(double v) {
  const long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
__device__ double row16_sum(double v) {
  v += dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp_f64<0x141>(v);  // mirror in eights
  v += dpp_f64<0x140>(v);  // mirror in sixteens
  return v;
}
__device__ double row16_max(double v) {
  v = fmax(v, dpp_f64<0xB1>(v));
  v = fmax(v, dpp_f64<0x4E>(v));
  v = fmax(v, dpp_f64<0x141>(v));
  return fmax(v, dpp_f64<0x140>(v));
}
// every thread gets the result; red: 4 doubles of LDS
template <int OP>  // 0 sum, 1 max, 2 min
__device__ double block_reduce(double v, double *red) {
  v = OP == 0 ? wave_sum(v) : OP == 1 ? wave_max(v) : wave_min(v);
  __syncthreads();  // red may still be read from the previous reduction
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const double a = red[0], b = red[1], c = red[2], d = red[3];
  return OP == 0 ? (a + b) + (c + d) : OP == 1 ? fmax(fmax(a, b), fmax(c, d)) : fmin(fmin(a, b), fmin(c, d));
}

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

inline int64_t up16(int64_t v) { return calibrate_up16(v); }

// Every activation lies in the order in which the products read it, tiles of 16 rows x 16 columns, [row / 16][column / 16]
// [64 lanes][4]: lane (r, q) = r + 16 q of a tile holds row r, columns 4 q + 0..3, so a wave's operand is 2 KB in a row.
// (From plain rows four neighbouring lanes are in four lines, and the load unit takes them one by one: the projection of
// a step 10.7 us, 6.3 of them that.)  ld: the columns, a multiple of 16.
__device__ __forceinline__ int64_t tiled(int64_t row, int col, int ld) {
  return (row >> 4) * 16 * ld + (col >> 4) * 256 + (((col & 15) >> 2) * 16 + (row & 15)) * 4 + (col & 3);
}
// the row and column of element i
__device__ __forceinline__ void tiled_place(int64_t i, int ld, int64_t *row, int *col) {
  const int64_t tile = i >> 8;
  const int per_row = ld >> 4, in = (int)(i & 255);
  *row = tile / per_row * 16 + ((in >> 2) & 15);
  *col = (int)(tile % per_row) * 16 + (in >> 6) * 4 + (in & 3);
}
// Where a step's rows go: row b of the step's own operand, and row row0 + b of the layer's output (or nowhere else).
struct TileOut {
  double *step, *all;
  int64_t row0;
  int ld;
  __device__ __forceinline__ void put(int64_t b, int col, double v) const {
    step[tiled(b, col, ld)] = v;
    if (all) all[tiled(row0 + b, col, ld)] = v;
  }
  TileOut from(int64_t rows) const { return {step + rows * ld, all, row0 + rows, ld}; }  // rows: a multiple of 16
};

// x float [rows][cols] -> double, tiled with ld columns (those beyond cols zero), and its range
__global__ __launch_bounds__(256) void widen_kernel(const float *x, double *out, int64_t rows, int cols, int ld, double *stats) {
  __shared__ double red[4];
  double lo = INFINITY, hi = -INFINITY;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < (rows + 15) / 16 * 16 * ld; i += (int64_t)gridDim.x * 256) {
    int64_t row;
    int col;
    tiled_place(i, ld, &row, &col);
    double v = 0.0;
    if (row < rows && col < cols) {
      v = x[row * cols + col];
      lo = fmin(lo, v);
      hi = fmax(hi, v);
    }
    out[i] = v;
  }
  lo = block_reduce<2>(lo, red);
  hi = block_reduce<1>(hi, red);
  if (threadIdx.x == 0) {
    atomic_min_f64(stats + S_XMIN, lo);
    atomic_max_f64(stats + S_XMAX, hi);
  }
}

// A layer's ranges: of its output (tiled, `rows` rows, columns below cols), and from what its steps left per thread (ext of
// `wgs` workgroups, the gate sums' too if `sums`) and per group of columns (amax [batch][(4 - g0) * groups]); either of
// these may be absent.
struct Extremes {
  const double *ext;
  int wgs, cell_lanes;  // threads per workgroup that have cells
  bool sums;
  const double *amax;
  int64_t batch;
  int groups, g0;
};
constexpr int kExtremes = kCalibrateExtremes;  // per thread: max |gate sum| of gates 0..3, max |c|, max m, max -m
__global__ __launch_bounds__(256) void range_kernel(const double *v, int64_t rows, int cols, int ld, Extremes x, double *stats) {
  __shared__ double red[4];
  double lo = INFINITY, hi = -INFINITY;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < (rows + 15) / 16 * 16 * ld; i += (int64_t)gridDim.x * 256) {
    int64_t row;
    int col;
    tiled_place(i, ld, &row, &col);
    if (row >= rows || col >= cols) continue;
    lo = fmin(lo, v[i]);
    hi = fmax(hi, v[i]);
  }
  lo = block_reduce<2>(lo, red);
  hi = block_reduce<1>(hi, red);
  if (threadIdx.x == 0) {
    atomic_min_f64(stats + S_HMIN, lo);
    atomic_max_f64(stats + S_HMAX, hi);
  }
  const int per_row = (4 - x.g0) * x.groups;
  const bool has_ext = x.ext && (int)blockIdx.x < x.wgs, has_sums = x.amax && blockIdx.x < x.batch;
  if (!has_ext && !has_sums) return;
  const int from = x.sums ? 0 : 4, lanes = x.sums ? 512 : 128;
  double top[kExtremes];
#pragma unroll
  for (int i = 0; i < kExtremes; ++i) {
    top[i] = -INFINITY;
    if (has_ext && (i >= 4 || x.sums))
      for (int w = blockIdx.x; w < x.wgs; w += gridDim.x)
        for (int l = threadIdx.x; l < (i < 4 ? 512 : x.cell_lanes); l += 256)
          top[i] = fmax(top[i], x.ext[((size_t)w * (kExtremes - from) + i - from) * lanes + l]);
    if (has_sums && i < 4 && i >= x.g0)
      for (int64_t b = blockIdx.x; b < x.batch; b += gridDim.x)
        for (int j = threadIdx.x; j < x.groups; j += 256) top[i] = fmax(top[i], x.amax[b * per_row + (i - x.g0) * x.groups + j]);
  }
#pragma unroll
  for (int i = 0; i < kExtremes; ++i) {
    const bool have = i < 4 ? i >= x.g0 && ((has_ext && x.sums) || has_sums) : has_ext;
    if (!have) continue;
    const double t = block_reduce<1>(top[i], red);
    if (threadIdx.x != 0) continue;
    if (i < 4)
      atomic_max_f64(stats + S_GABS + i, t);
    else if (i == 4)
      atomic_max_f64(stats + S_CABS, t);
    else if (i == 5)
      atomic_max_f64(stats + S_MMAX, t);
    else
      atomic_min_f64(stats + S_MMIN, -t);
  }
}

// a tiled buffer -> plain [rows][cols]
__global__ __launch_bounds__(256) void plain_kernel(const double *v, double *out, int64_t rows, int cols, int ld) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < rows * cols; i += (int64_t)gridDim.x * 256)
    out[i] = v[tiled(i / cols, (int)(i % cols), ld)];
}

// Weights [rows][K] (dense, as the caller has them) -> MFMA order [rows / 16][K / 16][64 lanes][4], zero beyond the
// real extents: lane (r, q) = r + 16 q of chunk c holds W[16 tile + r][16 c + 4 q + 0..3].  A wave's load of one chunk
// is then one contiguous KB, and the product kernels need no edge tests on the weights.  Done once per layer: 21 MB
// in and out at 8192 x 640, about 10 us against 64 steps that read the result.
__global__ __launch_bounds__(256) void repack_kernel(const float *W, float *op, int rows, int K, int64_t vecs) {
  const int chunks = (K + 15) >> 4;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < vecs; i += (int64_t)gridDim.x * 256) {
    const int lane = (int)(i & 63);
    const int64_t tc = i >> 6;
    const int64_t row = tc / chunks * 16 + (lane & 15);
    const int k = (int)(tc % chunks) * 16 + 4 * (lane >> 4);
    v4f v = {0.f, 0.f, 0.f, 0.f};
    if (row < rows) {
      const float *src = W + row * K + k;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k + j < K) v[j] = src[j];
    }
    reinterpret_cast<v4f *>(op)[i] = v;
  }
}

// C[m][n] = (Cin ? Cin[m][n] : 0) + (bias ? bias[n] : 0) + sum_k A[m][k] * W[n][k] on v_mfma_f64_16x16x4: A tiled, with
// zero columns beyond K, W in the order of repack_kernel, C double [M][ldc], or tiled into `to` (ldc = 0).
// A wave computes MT x NT tiles of 16 x 16; the k chunks of 16 are split over WK waves whose sums meet in LDS.  The
// four MFMAs of a chunk take k = 4 q + j, j = 0..3, from lane group q (any assignment of k to the instructions' slots
// gives the same sum), so that a lane's operands are 16 contiguous bytes of W and 32 of A, a wave's 1 and 2 KB.  U chunks
// are loaded together, with PIPE ahead of the U being multiplied.  Result value i of lane (c, q) is row 4 i + q, column c.
// Bound: 2 M Nout K / 70 TFLOP/s (measured for the library's f64 product on this chip) for the hoisted product, the
// latency of one weight read for a step's (its 21 MB come from the Infinity Cache at every step).
// ST: with the product, what the layer norm needs of it per row and 32 columns (RowStats below), the columns of a
// workgroup then: in the wave that stores them a lane holds both of its columns of a row, 16 lanes the row.
struct RowStats {
  double *part;  // [M][columns / 32][2] sum and sum of squares about the mean of the 32
  double *amax;  // [M][columns / 32] running max |value|
  int first;     // the first step: amax holds nothing yet
};

template <int MT, int NT, int WM, int WN, int WK, int U, bool PIPE, bool ST = false>
__global__ __launch_bounds__(64 * WM * WN * WK) void gemm_kernel(const double *A, const float *W, int chunks, double *C,
                                                                 int64_t ldc, TileOut to, const double *Cin,
                                                                 int64_t ldcin, const float *bias, int M, int Nout,
                                                                 RowStats rs) {
  static_assert(!ST || (WM == 1 && WN == 1 && WK > 1 && NT == 2));
  extern __shared__ double part[];  // WK > 1: [WM * WN][WK][MT * NT * 4][64]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int wk = wave % WK, wn = wave / WK % WN, wm = wave / (WK * WN);
  const int m0 = (blockIdx.y * WM + wm) * MT * 16, t0 = (blockIdx.x * WN + wn) * NT;
  const int tiles = (Nout + 15) >> 4;
  const double *ap[MT];
  const v4f *wp[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int m = m0 + 16 * i;  // a tile beyond M repeats the last one; rows beyond M are not stored
    ap[i] = A + ((size_t)((m < M ? m : M - 1) >> 4) * chunks * 64 + lane) * 4;
  }
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int t = t0 + i < tiles ? t0 + i : tiles - 1;
    wp[i] = reinterpret_cast<const v4f *>(W) + (size_t)t * chunks * 64 + lane;
  }
  v4d acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  // what is added to the values this thread stores at the end (WK > 1: value wk + SW * t of the first SW waves), on its
  // way meanwhile
  constexpr int SW = ST ? 4 : WK, OUT = WK > 1 ? MT * NT * 4 / SW : 1;
  double add[OUT];
#pragma unroll
  for (int t = 0; t < OUT; ++t) {
    const int v = wk + SW * t, m = m0 + 16 * (v / (4 * NT)) + 4 * (v & 3) + q, n = (t0 + v / 4 % NT) * 16 + r;
    add[t] = 0.0;
    if (WK > 1 && wk < SW && m < M && n < Nout) {
      if (Cin) add[t] = Cin[m * ldcin + n];
      if (bias) add[t] += (double)bias[n];
    }
  }
  const int per = (chunks + WK - 1) / WK;
  const int c0 = wk * per, c1 = c0 + per < chunks ? c0 + per : chunks;
  v4d a[U][MT];
  v4f w[U][NT];
  auto load = [&](int c, v4d (&av)[U][MT], v4f (&wv)[U][NT]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cc = c + u < c1 ? c + u : c1 - 1;
#pragma unroll
      for (int i = 0; i < NT; ++i) wv[u][i] = wp[i][(size_t)cc * 64];
#pragma unroll
      for (int i = 0; i < MT; ++i) av[u][i] = *reinterpret_cast<const v4d *>(ap[i] + (size_t)cc * 256);
    }
  };
  if (c0 < c1) {
    load(c0, a, w);
    for (int c = c0; c < c1; c += U) {
      v4d an[U][MT];
      v4f wn_[U][NT];
      if (PIPE && c + U < c1) load(c + U, an, wn_);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool live = c + u < c1;  // uniform over the wave
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int n = 0; n < NT; ++n) {
            const double wd = live ? (double)w[u][n][j] : 0.0;
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m][n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][m][j], wd, acc[m][n], 0, 0, 0);
          }
      }
      if constexpr (PIPE) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
          for (int i = 0; i < MT; ++i) a[u][i] = an[u][i];
#pragma unroll
          for (int i = 0; i < NT; ++i) w[u][i] = wn_[u][i];
        }
      } else if (c + U < c1) {
        load(c + U, a, w);
      }
    }
  }
  if constexpr (WK == 1) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = m0 + 16 * mt + 4 * i + q, n = (t0 + nt) * 16 + r;
          if (m >= M || n >= Nout) continue;
          double v = acc[mt][nt][i];
          if (Cin) v += Cin[m * ldcin + n];
          if (bias) v += (double)bias[n];
          if (ldc)
            C[m * ldc + n] = v;
          else
            to.put(m, n, v);
        }
  } else {
    constexpr int V = MT * NT * 4;
    static_assert(V % SW == 0);
    double *mine = part + ((size_t)(wm * WN + wn) * WK) * V * 64 + lane;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) mine[(wk * V + (mt * NT + nt) * 4 + i) * 64] = acc[mt][nt][i];
    __syncthreads();
    if (wk >= SW) return;
    double out[OUT];
#pragma unroll
    for (int t = 0; t < OUT; ++t) {
      const int v = wk + SW * t;
      double sum = 0.0;
#pragma unroll
      for (int k = 0; k < WK; ++k) sum += mine[(k * V + v) * 64];
      out[t] = sum + add[t];
      const int m = m0 + 16 * (v / (4 * NT)) + 4 * (v & 3) + q, n = (t0 + v / 4 % NT) * 16 + r;
      if (m < M && n < Nout) {
        if (ldc)
          C[m * ldc + n] = out[t];
        else
          to.put(m, n, out[t]);
      }
    }
    if constexpr (ST) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const double v0 = out[2 * mt], v1 = out[2 * mt + 1];
        const double s = row16_sum(v0 + v1), mean = s * (1.0 / 32.0);
        const double sq = row16_sum((v0 - mean) * (v0 - mean) + (v1 - mean) * (v1 - mean));
        const double top = row16_max(fmax(fabs(v0), fabs(v1)));
        const int m = m0 + 16 * mt + 4 * wk + q;
        if (r == 0 && m < M) {
          const size_t at = (size_t)m * (Nout >> 5) + blockIdx.x;
          rs.part[2 * at] = s;
          rs.part[2 * at + 1] = sq;
          rs.amax[at] = rs.first ? top : fmax(top, rs.amax[at]);
        }
      }
    }
  }
}

// The projection of a step of up to 16 rows, where k is long and the columns are few: to[m][n] = bias[n] + sum_k A[m][k] *
// W[n][k], four rows x 16 columns per workgroup and k split over 16 waves: v_mfma_f64_4x4x4 in its four blocks, which take
// the same four rows and four columns each, operands as in gemm_kernel.  Lane (r, q) ends with row q, column r.  Bound: the
// operands' way from the L2, 192 KB per workgroup.  One workgroup per 16 x 16 is 40 of them at 640 columns, whose matrix cores
// take 3.4 us; this way there are 160.  2048 -> 640, 16 rows: 10.6 us before (and with plain rows), 5.8 now.
template <int U>
__global__ __launch_bounds__(1024) void thin_gemm_kernel(const double *A, const float *W, int chunks, TileOut to,
                                                         const float *bias, int M, int Nout) {
  __shared__ double part[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int m0 = blockIdx.y * 4, n = blockIdx.x * 16 + r;  // all of one tile of 16 rows
  const double *ap = A + (m0 + (r & 3) + 16 * q) * 4;
  const v4f *wp = reinterpret_cast<const v4f *>(W) + (size_t)blockIdx.x * chunks * 64 + lane;
  const int per = (chunks + 15) / 16;
  const int c0 = wave * per, c1 = c0 + per < chunks ? c0 + per : chunks;
  const double add = wave == 0 && bias && n < Nout ? (double)bias[n] : 0.0;
  double acc[2] = {0.0, 0.0};
  for (int c = c0; c < c1; c += U) {
    v4d a[U];
    v4f w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cc = c + u < c1 ? c + u : c1 - 1;
      w[u] = wp[(size_t)cc * 64];
      a[u] = *reinterpret_cast<const v4d *>(ap + (size_t)cc * 256);
    }
    __builtin_amdgcn_sched_barrier(0);  // else the loads sink to their uses, two in flight
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool live = c + u < c1;  // uniform over the wave
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[j & 1] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[u][j], live ? (double)w[u][j] : 0.0, acc[j & 1], 0, 0, 0);
    }
  }
  part[wave][lane] = acc[0] + acc[1];
  __syncthreads();
  if (wave != 0) return;
  double sum = 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) sum += part[k][lane];
  if (m0 + q < M && n < Nout) to.put(m0 + q, n, sum + add);
}

struct CellArgs {
  double *pre;    // [B][4*N] gate sums W x + R h of this step, slot per gate; overwritten
  double *c;      // [B][N] cell state, in/out
  TileOut m;      // hidden state out (the layer output itself when there is no projection)
  const float *b[4], *P[3], *Lw[4];
  int N, flags;
  double *stats;
  const double *part;  // RowStats of the gate sums, or null
  double *ext;         // running extremes per thread, [workgroup][7][512], or the last three of them of 128, or null
  int first;           // the first step: ext holds nothing yet
};

__device__ double sigmoid_f64(double v) { return 1.0 / (1.0 + exp(-v)); }

// K sums over a workgroup of 8 waves; every thread gets them.  red: K * 8 doubles that nobody still reads.
template <int K>
__device__ void block_sum8(double (&v)[K], double *red) {
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const double s = wave_sum(v[i]);
    if ((threadIdx.x & 63) == 0) red[i * 8 + (threadIdx.x >> 6)] = s;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < K; ++i) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) s += red[i * 8 + w];
    v[i] = s;
  }
}

// Eqs. (1)-(6) of Sec. 2 after the matrix products, for rows of up to 512 E cells.  gridDim.y workgroups share a batch
// row: each takes the layer norm's mean and deviation over the whole row (from the sums of its groups of 32 that the product
// left, merged by one wave per gate, about their common mean; or its values in registers, the gates that do not wait for
// the new cell state in one pair of reductions) and then a slice of the cells -- five double exp / tanh
// per cell are the bulk of the work, and one workgroup per row would leave all but 16 compute units idle at the
// default calibration batch.  With peephole and layer norm the o gate's statistics need the whole new cell state, so
// gridDim.y is 1 there (and without a peephole nobody reads the c of another slice).  The ranges stay with the threads, in
// memory, until range_kernel takes them at the end of the layer.  16 rows of 2048 cells: 14.4 us with a pass over the row and
// a reduction of the ranges at every step (7.4 and 3.7 of it), 5.8 without.
template <int E>
__global__ __launch_bounds__(512) void cell_row_kernel(CellArgs a) {
  __shared__ double red[4][4 * 8], top[7 * 8], act[4][128];
  const int b = blockIdx.x, tid = threadIdx.x, N = a.N, wave = tid >> 6;
  const bool cifg = a.flags & kCifg, ph = a.flags & kPeephole, ln = a.flags & kLayerNorm;
  const double *pre = a.pre + (size_t)b * 4 * N;
  double *crow = a.c + (size_t)b * N;
  const int g0 = cifg ? 1 : 0;
  double amax[4] = {0.0, 0.0, 0.0, 0.0}, mean[4], sd[4];
  // this thread's extremes so far, on their way while the statistics are taken
  const bool late_o = ph && ln;  // gridDim.y == 1
  const bool own_sums = ln && !a.part, cells = late_o || tid < 128;  // which of them this thread has
  const int from = own_sums ? 0 : 4, lanes = own_sums ? 512 : 128;   // (late_o: own_sums)
  double *ext = a.ext ? a.ext + ((size_t)b * gridDim.y + blockIdx.y) * (kExtremes - from) * lanes + tid : nullptr;
  double so_far[kExtremes];
#pragma unroll
  for (int i = 0; i < kExtremes; ++i) {
    so_far[i] = -INFINITY;
    if (ext && !a.first && (i < 4 ? own_sums : cells)) so_far[i] = ext[(i - from) * lanes];
  }
  // gate sum of cell n before the norm; cell: c^{t-1}, or c^t for the o gate
  auto gate_sum = [&](int g, int n, double cell) {
    double v = pre[(size_t)g * N + n];
    if (ph && g != 2) v += (double)a.P[g == 3 ? 2 : g][n] * cell;
    return v;
  };
  // layer-norm statistics of the gates of `mask`: mean, sd (0 where the row is constant)
  auto statistics = [&](int mask, double *r0, double *r1) {
    double v[4][E], s[4] = {0.0, 0.0, 0.0, 0.0}, sq[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int n = tid + 512 * e;
#pragma unroll
      for (int g = 0; g < 4; ++g) v[g][e] = (mask >> g & 1) && n < N ? gate_sum(g, n, ph ? crow[n] : 0.0) : 0.0;
    }
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        s[g] += v[g][e];
        amax[g] = fmax(amax[g], fabs(v[g][e]));
      }
    block_sum8(s, r0);
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (mask >> g & 1) {
        mean[g] = s[g] / N;
#pragma unroll
        for (int e = 0; e < E; ++e)
          if (tid + 512 * e < N) sq[g] += (v[g][e] - mean[g]) * (v[g][e] - mean[g]);
      }
    block_sum8(sq, r1);
#pragma unroll
    for (int g = 0; g < 4; ++g)
      if (mask >> g & 1) sd[g] = sqrt(sq[g] / N);
  };
  auto norm = [&](int g, int n, double v) {
    if (ln) v = sd[g] > 0.0 ? (v - mean[g]) / sd[g] * (double)a.Lw[g][n] : 0.0;
    return v + (double)a.b[g][n];
  };
  if (own_sums) statistics((cifg ? 0 : 1) | 2 | 4 | (ph ? 0 : 8), red[0], red[1]);
  // 128 cells at a time, one gate per wave pair: the activations are long chains of dependent double instructions, so
  // the gates of a cell run side by side and meet in LDS
  const int gate = tid >> 7, cell = tid & 127;
  const int blocks = (N + 127) >> 7;
  double cmax = 0.0, lo = INFINITY, hi = -INFINITY;
  for (int blk = blockIdx.y; blk < blocks; blk += gridDim.y) {
    const int n = blk * 128 + cell;
    const bool live = n < N;
    const double c0 = live ? crow[n] : 0.0;
    const double mine = live && gate >= g0 && (gate != 3 || !ph) ? gate_sum(gate, n, c0) : 0.0;
    if (a.part && blk == (int)blockIdx.y) {
      // one wave per gate: mean and deviation from the sums of the row's groups of 32, while its values are on their way
      if (wave < 4 && wave >= g0) {
        const int groups = N >> 5, lane = tid & 63;  // at most 128
        const double2 *p = reinterpret_cast<const double2 *>(a.part) + ((size_t)b * (4 - g0) + (wave - g0)) * groups;
        const double2 zero = {0.0, 0.0};
        const double2 p0 = lane < groups ? p[lane] : zero, p1 = lane + 64 < groups ? p[lane + 64] : zero;
        const double mu = wave_sum(p0.x + p1.x) / N;
        double sq = p0.y + p1.y;
        if (lane < groups) sq += 32.0 * (p0.x * (1.0 / 32.0) - mu) * (p0.x * (1.0 / 32.0) - mu);
        if (lane + 64 < groups) sq += 32.0 * (p1.x * (1.0 / 32.0) - mu) * (p1.x * (1.0 / 32.0) - mu);
        sq = wave_sum(sq);
        if (lane == 0) {
          red[0][wave] = mu;
          red[1][wave] = sqrt(sq / N);
        }
      }
      __syncthreads();
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        mean[g] = red[0][g];
        sd[g] = red[1][g];
      }
    }
    if (live && gate >= g0 && gate != 3) {
      const double v = norm(gate, n, mine);
      act[gate][cell] = gate == 2 ? tanh(v) : sigmoid_f64(v);
    } else if (live && gate == 3 && !ph) {
      act[3][cell] = sigmoid_f64(norm(3, n, mine));
    }
    __syncthreads();
    if (live && gate == 0) {
      const double f = act[1][cell], i = cifg ? 1.0 - f : act[0][cell];
      const double c = i * act[2][cell] + f * c0;
      crow[n] = c;
      cmax = fmax(cmax, fabs(c));
      if (!late_o) {
        const double o = ph ? sigmoid_f64(norm(3, n, gate_sum(3, n, c))) : act[3][cell];
        const double mv = o * tanh(c);
        a.m.put(b, n, mv);
        lo = fmin(lo, mv);
        hi = fmax(hi, mv);
      }
    }
    __syncthreads();
  }
  if (late_o) {  // every c of the row is there
    statistics(8, red[2], red[3]);
    for (int n = tid; n < N; n += 512) {
      const double c = crow[n];
      const double mv = sigmoid_f64(norm(3, n, gate_sum(3, n, c))) * tanh(c);
      a.m.put(b, n, mv);
      lo = fmin(lo, mv);
      hi = fmax(hi, mv);
    }
  }
  const double t[kExtremes] = {amax[0], amax[1], amax[2], amax[3], cmax, hi, -lo};
  if (ext) {
#pragma unroll
    for (int i = 0; i < kExtremes; ++i)
      if (i < 4 ? own_sums : cells) ext[(i - from) * lanes] = fmax(t[i], so_far[i]);
    return;
  }
  // ranges: one value per wave into LDS, the last step by seven threads
#pragma unroll
  for (int i = 0; i < 7; ++i) {
    const double w = wave_max(t[i]);
    if ((tid & 63) == 0) top[i * 8 + wave] = w;
  }
  __syncthreads();
  if (tid < 7) {
    double w = top[tid * 8];
    for (int i = 1; i < 8; ++i) w = fmax(w, top[tid * 8 + i]);
    if (tid < 4) {
      if (own_sums && tid >= g0) atomic_max_f64(a.stats + S_GABS + tid, w);
    } else if (tid == 4) {
      atomic_max_f64(a.stats + S_CABS, w);
    } else if (tid == 5) {
      atomic_max_f64(a.stats + S_MMAX, w);
    } else {
      atomic_min_f64(a.stats + S_MMIN, -w);
    }
  }
}

// The same as cell_row_kernel for rows too wide for registers: gate by gate through memory.
// Gates f, z, i from c^{t-1}; the cell update; gate o from c^t; m.
__global__ __launch_bounds__(256) void cell_kernel(CellArgs a) {
  __shared__ double red[4];
  const int b = blockIdx.x, tid = threadIdx.x, N = a.N;
  const bool cifg = a.flags & kCifg, ph = a.flags & kPeephole, ln = a.flags & kLayerNorm;
  double *pre = a.pre + (size_t)b * 4 * N;
  double *c = a.c + (size_t)b * N;
  // gate g in place: pre[g] <- activation(norm(pre[g] + P . cell) . L + b)
  auto gate = [&](int g) {
    double *pg = pre + (size_t)g * N;
    const float *pw = (ph && g != 2) ? a.P[g == 3 ? 2 : g] : nullptr;
    double amax = 0.0, sum = 0.0;
    for (int n = tid; n < N; n += 256) {
      double v = pg[n];
      if (pw) v += (double)pw[n] * c[n];
      if (!ln) v += (double)a.b[g][n];
      pg[n] = v;
      amax = fmax(amax, fabs(v));
      sum += v;
    }
    if (ln) {
      amax = block_reduce<1>(amax, red);
      if (tid == 0) atomic_max_f64(a.stats + S_GABS + g, amax);
      const double mean = block_reduce<0>(sum, red) / N;
      double sq = 0.0;
      for (int n = tid; n < N; n += 256) {
        const double d = pg[n] - mean;
        sq += d * d;
      }
      const double sd = sqrt(block_reduce<0>(sq, red) / N);
      for (int n = tid; n < N; n += 256) {
        const double xn = sd > 0.0 ? (pg[n] - mean) / sd : 0.0;
        pg[n] = xn * (double)a.Lw[g][n] + (double)a.b[g][n];
      }
    }
    for (int n = tid; n < N; n += 256) pg[n] = g == 2 ? tanh(pg[n]) : sigmoid_f64(pg[n]);
  };
  gate(1);
  gate(2);
  if (!cifg) gate(0);
  double cmax = 0.0;
  for (int n = tid; n < N; n += 256) {
    const double f = pre[N + n];
    const double i = cifg ? 1.0 - f : pre[n];
    const double cn = i * pre[2 * (size_t)N + n] + f * c[n];
    c[n] = cn;
    cmax = fmax(cmax, fabs(cn));
  }
  cmax = block_reduce<1>(cmax, red);  // also orders the writes of c before gate o reads them
  gate(3);
  double lo = INFINITY, hi = -INFINITY;
  for (int n = tid; n < N; n += 256) {
    const double mv = pre[3 * (size_t)N + n] * tanh(c[n]);
    a.m.put(b, n, mv);
    lo = fmin(lo, mv);
    hi = fmax(hi, mv);
  }
  lo = block_reduce<2>(lo, red);
  hi = block_reduce<1>(hi, red);
  if (tid == 0) {
    atomic_max_f64(a.stats + S_CABS, cmax);
    atomic_min_f64(a.stats + S_MMIN, lo);
    atomic_max_f64(a.stats + S_MMAX, hi);
  }
}

// A thread that uploads the layers' parameters in turn.  Copies from pageable memory hold the thread that asks for them
// (13 ms for the 377 MB of an 8-layer encoder) and a layer's 200 launches take the host another millisecond: one after the
// other they are longer than the layer's 1.6 ms on the device (8 layers of 2048 cells, 16 rows, 64 steps: 20.8 ms a call
// with one thread for both, 17.0 with two).  Layer l may go once the layer before it has freed the raw buffer, which
// the caller says with free_up_to(l).  Without a thread to be had, the caller uploads by itself.
class Uploader {
 public:
  ~Uploader() {
    if (!thread_.joinable()) return;
    {
      std::lock_guard<std::mutex> lock(mutex_);
      stop_ = true;
    }
    changed_.notify_all();
    thread_.join();
  }
  // upload(l) for l = 1 .. layers - 1; false: it returned false
  void start(int device, int layers, std::function<bool(int)> upload) {
    upload_ = std::move(upload);
    try {
      thread_ = std::thread([this, device, layers] {
        bool ok = hipSetDevice(device) == hipSuccess;
        for (int l = 1; l < layers; ++l) {
          {
            std::unique_lock<std::mutex> lock(mutex_);
            changed_.wait(lock, [&] { return stop_ || free_ >= l; });
            if (stop_) return;
          }
          ok = ok && upload_(l);
          {
            std::lock_guard<std::mutex> lock(mutex_);
            done_ = l;
            failed_ = !ok;
          }
          changed_.notify_all();
        }
      });
    } catch (const std::system_error &) {
    }
  }
  void free_up_to(int l) {
    {
      std::lock_guard<std::mutex> lock(mutex_);
      free_ = l;
    }
    changed_.notify_all();
  }
  // until the copies of layer l are on their stream
  bool wait(int l) {
    if (!thread_.joinable()) return upload_(l);
    std::unique_lock<std::mutex> lock(mutex_);
    changed_.wait(lock, [&] { return done_ >= l; });
    return !failed_;
  }

 private:
  std::function<bool(int)> upload_;
  std::thread thread_;
  std::mutex mutex_;
  std::condition_variable changed_;
  int free_ = 0, done_ = 0;
  bool stop_ = false, failed_ = false;
};

// What a call holds on the device and in the runtime; gone when the call ends, in whatever way (nothing may still
// be running on the memory then).
struct Held {
  hipStream_t s = nullptr, copy = nullptr;
  hipEvent_t uploaded = nullptr, repacked = nullptr;
  uint8_t *arena = nullptr;
  ~Held() {
    if (copy) (void)hipStreamSynchronize(copy);
    if (arena) (void)hipStreamSynchronize(s);
    if (uploaded) (void)hipEventDestroy(uploaded);
    if (repacked) (void)hipEventDestroy(repacked);
    if (copy) (void)hipStreamDestroy(copy);
    if (arena) (void)hipFree(arena);
  }
};

// One product, C plain (ldc > 0) or tiled into `to`.  M rows against Nout rows of weights in repack_kernel's order (K =
// the real depth).
//   * Enough 128 x 128 blocks to fill half of the chip: four waves of 64 x 64, the rate of the matrix cores bounds it.
//   * A step's product of up to 16 rows, few columns and a long k: thin_gemm_kernel.
//   * else 16 or 32 rows x 32 columns per workgroup, k split over four waves, or eight where four would need more than one
//     trip for their operands (five chunks each): a step's product at N = 2048 is 256 workgroups, each one weight read
//     deep (four waves and two reads: 9.1 us for 6.9 at 16 rows; at k = 178 eight waves take 6.2, four 5.3).
void launch_gemm(hipStream_t s, const double *A, const float *W, double *C, int64_t ldc, const TileOut &to, const double *Cin,
                 int64_t ldcin, const float *bias, int M, int Nout, int K, const RowStats *rs = nullptr) {
  const int chunks = (K + 15) / 16;
  auto go = [&](auto kernel, int mb, int nb, int waves, size_t lds) {
    const int64_t per = calibrate_rows_per_launch(mb);
    for (int64_t m = 0; m < M; m += per) {
      RowStats part = {};
      if (rs) part = {rs->part + m * (Nout >> 5) * 2, rs->amax + m * (Nout >> 5), rs->first};
      hipLaunchKernelGGL(kernel, dim3((Nout + nb - 1) / nb, (unsigned)((std::min<int64_t>(per, M - m) + mb - 1) / mb)),
                         dim3(64 * waves), lds, s, A + m * 16 * chunks, W, chunks, C + m * ldc, ldc, ldc ? to : to.from(m),
                         Cin ? Cin + m * ldcin : nullptr, ldcin, bias, (int)std::min<int64_t>(per, M - m), Nout, part);
    }
  };
  auto split = [&](auto st) {
    constexpr bool ST = decltype(st)::value;
    const bool deep = chunks > 20;
    if (M > 16 && deep)
      go(gemm_kernel<2, 2, 1, 1, 8, 5, false, ST>, 32, 32, 8, 8 * 16 * 64 * 8);
    else if (M > 16)
      go(gemm_kernel<2, 2, 1, 1, 4, 5, false, ST>, 32, 32, 4, 4 * 16 * 64 * 8);
    else if (deep)
      go(gemm_kernel<1, 2, 1, 1, 8, 5, false, ST>, 16, 32, 8, 8 * 8 * 64 * 8);
    else
      go(gemm_kernel<1, 2, 1, 1, 4, 5, false, ST>, 16, 32, 4, 4 * 8 * 64 * 8);
  };
  if (calibrate_wide_product(M, Nout))
    go(gemm_kernel<4, 4, 2, 2, 1, 1, true>, 128, 128, 4, 0);
  else if (rs)
    split(std::true_type());
  else if (M <= 16 && Nout <= 2048 && K >= 512 && !ldc)
    hipLaunchKernelGGL(thin_gemm_kernel<8>, dim3((Nout + 15) / 16, (M + 3) / 4), dim3(1024), 0, s, A, W, chunks, to, bias, M,
                       Nout);
  else
    split(std::false_type());
}

void launch_cell_rows(hipStream_t s, const CellArgs &a, int B) {
  const dim3 grid(B, calibrate_cell_slices(a.N, a.flags, B)), block(512);
  if (a.N <= 512)
    hipLaunchKernelGGL(cell_row_kernel<1>, grid, block, 0, s, a);
  else if (a.N <= 1024)
    hipLaunchKernelGGL(cell_row_kernel<2>, grid, block, 0, s, a);
  else if (a.N <= 2048)
    hipLaunchKernelGGL(cell_row_kernel<4>, grid, block, 0, s, a);
  else if (a.N <= kCalibrateRowMax)
    hipLaunchKernelGGL(cell_row_kernel<8>, grid, block, 0, s, a);
  else
    hipLaunchKernelGGL(cell_kernel, dim3(B), dim3(256), 0, s, a);
}
void launch_cell(hipStream_t s, const CellArgs &a, int B) {
  CellArgs part = a;
  for (int b = 0; b < B; b += kCalibrateCellRows) {
    const int rows = std::min(B - b, kCalibrateCellRows);
    launch_cell_rows(s, part, rows);
    part.pre += (size_t)rows * 4 * a.N;
    part.c += (size_t)rows * a.N;
    part.m = part.m.from(rows);
  }
}

int calibrate(const lstm_int_layer_params *layers, int32_t num_layers, int32_t device, const float *x, int32_t T, int32_t B,
              void *hip_stream, lstm_int_layer_stats *stats_out, double *y_float) {
  if (!layers || num_layers < 1 || device < 0 || !x || T < 1 || B < 1 || !stats_out) return LSTM_INT_E_INVALID_ARG;
  for (int l = 0; l < num_layers; ++l) {
    const lstm_int_layer_params &p = layers[l];
    const bool cifg = p.flags & kCifg, ph = p.flags & kPeephole, ln = p.flags & kLayerNorm, proj = p.flags & kProjection;
    if (p.input_size < 1 || p.num_cells < 1 || p.output_size < 1 || (p.flags & ~15u)) return LSTM_INT_E_INVALID_ARG;
    if (!proj && p.output_size != p.num_cells) return LSTM_INT_E_INVALID_ARG;
    if (l > 0 && p.input_size != layers[l - 1].output_size) return LSTM_INT_E_INVALID_ARG;
    if ((int64_t)T * B * 4 * p.num_cells >= (1ll << 31) || (int64_t)T * B * p.input_size >= (1ll << 31))
      return LSTM_INT_E_UNSUPPORTED;  // 32-bit row counts times strides in the kernels' index arithmetic
    for (int g = cifg ? 1 : 0; g < 4; ++g) {
      if (!p.W[g] || !p.R[g] || !p.b[g]) return LSTM_INT_E_INVALID_ARG;
      if (ln && !p.Lw[g]) return LSTM_INT_E_INVALID_ARG;
      if (ph && g != 2 && !p.P[g == 3 ? 2 : g]) return LSTM_INT_E_INVALID_ARG;
    }
    if (proj && !p.Wproj) return LSTM_INT_E_INVALID_ARG;
  }
  if (hipSetDevice(device) != hipSuccess) return LSTM_INT_E_DEVICE;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int64_t TB = (int64_t)T * B;

  // One allocation for the whole call: each one costs about 0.1 ms to make and 0.3 ms to give back.
  const CalibratePlan plan = calibrate_plan(layers, num_layers, T, B, sizeof(double) * S_COUNT);
  std::vector<std::vector<float>> vectors(num_layers);  // outlives the copies: declared ahead of what waits for them
  std::vector<double> init((size_t)S_COUNT * num_layers, 0.0);
  Held held;
  held.s = s;
  if (hipMalloc(reinterpret_cast<void **>(&held.arena), plan.total) != hipSuccess) {
    held.arena = nullptr;
    return LSTM_INT_E_OUT_OF_MEMORY;
  }
  if (hipStreamCreateWithFlags(&held.copy, hipStreamNonBlocking) != hipSuccess ||
      hipEventCreateWithFlags(&held.uploaded, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&held.repacked, hipEventDisableTiming) != hipSuccess)
    return LSTM_INT_E_DEVICE;
  auto dbl = [&](const CalibrateRegion &r) { return reinterpret_cast<double *>(held.arena + r.off); };
  auto flt = [&](const CalibrateRegion &r) { return reinterpret_cast<float *>(held.arena + r.off); };
  double *const stats = dbl(plan.stats);
  for (int l = 0; l < num_layers; ++l) {
    double *st = init.data() + (size_t)l * S_COUNT;
    st[S_XMIN] = st[S_HMIN] = st[S_MMIN] = INFINITY;
    st[S_XMAX] = st[S_HMAX] = st[S_MMAX] = -INFINITY;
  }
  if (hipMemcpyAsync(stats, init.data(), init.size() * sizeof(double), hipMemcpyHostToDevice, s) != hipSuccess)
    return LSTM_INT_E_DEVICE;
  const int blocks = 256;  // of the range kernels: each ends with two compare-and-swap loops on the same words
  double *cur = dbl(plan.act[0]), *next = dbl(plan.act[1]);
  hipLaunchKernelGGL(widen_kernel, dim3(blocks), dim3(256), 0, s, x, cur, TB, layers[0].input_size,
                     (int)up16(layers[0].input_size), stats);

  // The layers' vectors: b[4], P[3], Lw[4], bproj
  for (int l = 0; l < num_layers; ++l) {
    const lstm_int_layer_params &p = layers[l];
    const size_t N = p.num_cells, H = p.output_size, first = (p.flags & kCifg) ? 1 : 0;
    std::vector<float> &hv = vectors[l];
    hv.assign(11 * N + H, 0.0f);
    for (size_t g = first; g < 4; ++g) {
      std::copy(p.b[g], p.b[g] + N, hv.begin() + g * N);
      if (p.flags & kLayerNorm) std::copy(p.Lw[g], p.Lw[g] + N, hv.begin() + (7 + g) * N);
      if ((p.flags & kPeephole) && g < 3) std::copy(p.P[g], p.P[g] + N, hv.begin() + (4 + g) * N);
    }
    if ((p.flags & kProjection) && p.bproj) std::copy(p.bproj, p.bproj + H, hv.begin() + 11 * N);
  }
  // Parameters of layer l into the raw buffer, on the copy stream: gates first..3 of W, then of R, then W_proj.
  auto upload = [&, copy = held.copy, uploaded = held.uploaded, repacked = held.repacked](int l) {
    const lstm_int_layer_params &p = layers[l];
    const size_t I = p.input_size, N = p.num_cells, H = p.output_size, first = (p.flags & kCifg) ? 1 : 0;
    bool ok = l == 0 || hipStreamWaitEvent(copy, repacked, 0) == hipSuccess;  // the raw buffer is free again
    auto up = [&](void *dst, const void *src, size_t bytes) {
      ok = ok && hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, copy) == hipSuccess;
    };
    float *raw = flt(plan.raw);
    for (size_t g = first; g < 4; ++g, raw += N * I) up(raw, p.W[g], sizeof(float) * N * I);
    for (size_t g = first; g < 4; ++g, raw += N * H) up(raw, p.R[g], sizeof(float) * N * H);
    if (p.flags & kProjection) up(raw, p.Wproj, sizeof(float) * H * N);
    up(flt(plan.vec[l & 1]), vectors[l].data(), sizeof(float) * vectors[l].size());
    return ok && hipEventRecord(uploaded, copy) == hipSuccess;
  };
  auto repack = [&](const float *src, float *op, int rows, int K) {
    const int64_t vecs = (int64_t)up16(rows) * up16(K) / 4;
    hipLaunchKernelGGL(repack_kernel, dim3((unsigned)std::min<int64_t>((vecs + 255) / 256, 4096)), dim3(256), 0, s, src, op,
                       rows, K, vecs);
  };

  if (!upload(0)) return LSTM_INT_E_DEVICE;
  Uploader uploader;  // ends before what it writes to
  if (num_layers > 1) uploader.start(device, num_layers, upload);
  for (int l = 0; l < num_layers; ++l) {
    const lstm_int_layer_params &p = layers[l];
    const CalibrateLayer &at = plan.layers[l];
    const int I = p.input_size, N = p.num_cells, H = p.output_size, first = (p.flags & kCifg) ? 1 : 0, G = 4 - first;
    const bool proj = p.flags & kProjection;
    const int Np = (int)up16(N), Hp = (int)up16(H);
    double *st = stats + (size_t)l * S_COUNT;
    bool ok = (l == 0 || uploader.wait(l)) && hipStreamWaitEvent(s, held.uploaded, 0) == hipSuccess;
    const float *raw = flt(plan.raw);
    repack(raw, flt(at.wop), G * N, I);
    repack(raw + (size_t)G * N * I, flt(at.rop), G * N, H);
    if (proj) repack(raw + (size_t)G * N * (I + H), flt(at.pop), H, N);
    ok = ok && hipEventRecord(held.repacked, s) == hipSuccess;
    if (ok) uploader.free_up_to(l + 1);
    ok = ok && hipMemsetAsync(dbl(at.c), 0, sizeof(double) * (size_t)B * N, s) == hipSuccess;
    ok = ok && hipMemsetAsync(dbl(at.h), 0, at.h.bytes, s) == hipSuccess;
    if (proj && Np != N) ok = ok && hipMemsetAsync(dbl(at.m), 0, at.m.bytes, s) == hipSuccess;
    if (Hp != H) ok = ok && hipMemsetAsync(next, 0, sizeof(double) * up16(TB) * Hp, s) == hipSuccess;
    if (!ok) return LSTM_INT_E_DEVICE;

    const float *vb = flt(plan.vec[l & 1]);
    double *wx = dbl(at.wx), *pre = dbl(at.pre);
    // W x for all steps (eqs. 1-4, first term), gates first..3 in one product
    launch_gemm(s, cur, flt(at.wop), wx, G * (int64_t)N, TileOut{}, nullptr, 0, nullptr, (int)TB, G * N, I);
    CellArgs ca;
    ca.pre = pre;
    ca.c = dbl(at.c);
    for (int g = 0; g < 4; ++g) {
      ca.b[g] = vb + (size_t)g * N;
      ca.Lw[g] = vb + (size_t)(7 + g) * N;
    }
    for (int j = 0; j < 3; ++j) ca.P[j] = vb + (size_t)(4 + j) * N;
    ca.N = N;
    ca.flags = (int)p.flags;
    ca.stats = st;
    const bool ln = p.flags & kLayerNorm, ph = p.flags & kPeephole;
    const bool sums = calibrate_sums_in_product(N, p.flags, B);
    ca.ext = calibrate_extreme_values(N, p.flags, B) ? dbl(plan.ext) : nullptr;
    ca.part = sums ? dbl(at.part) : nullptr;
    for (int t = 0; t < T; ++t) {
      const TileOut out = {dbl(at.h), next, (int64_t)t * B, Hp};
      // + R h^{t-1}
      const RowStats rs = {dbl(at.part), dbl(at.amax), t == 0};
      launch_gemm(s, dbl(at.h), flt(at.rop), pre + (size_t)first * N, 4 * (int64_t)N, TileOut{}, wx + (size_t)t * B * G * N,
                  G * (int64_t)N, nullptr, B, G * N, H, sums ? &rs : nullptr);
      ca.first = t == 0;
      ca.m = proj ? TileOut{dbl(at.m), nullptr, 0, Np} : out;
      launch_cell(s, ca, B);
      if (proj)  // eq. (7)
        launch_gemm(s, dbl(at.m), flt(at.pop), nullptr, 0, out, nullptr, 0, vb + (size_t)11 * N, B, H, N);
    }
    const Extremes steps = {ca.ext, B * calibrate_cell_slices(N, p.flags, B), ln && ph ? 512 : 128, ln && !sums,
                            sums ? dbl(at.amax) : nullptr, B, N / 32, first};
    hipLaunchKernelGGL(range_kernel, dim3(blocks), dim3(256), 0, s, next, TB, H, Hp, steps, st);
    if (hipGetLastError() != hipSuccess) return LSTM_INT_E_DEVICE;
    if (l + 1 == num_layers && y_float) {
      hipLaunchKernelGGL(plain_kernel, dim3(blocks), dim3(256), 0, s, next, y_float, TB, H, Hp);
      if (hipGetLastError() != hipSuccess) return LSTM_INT_E_DEVICE;
    }
    std::swap(cur, next);  // this layer's output is the next layer's input
  }
  if (hipStreamSynchronize(s) != hipSuccess) return LSTM_INT_E_DEVICE;

  std::vector<double> hs((size_t)S_COUNT * num_layers);
  if (hipMemcpy(hs.data(), stats, hs.size() * sizeof(double), hipMemcpyDeviceToHost) != hipSuccess)
    return LSTM_INT_E_DEVICE;
  for (int l = 0; l < num_layers; ++l) {
    const double *st = hs.data() + (size_t)l * S_COUNT;
    lstm_int_layer_stats &o = stats_out[l];
    // the input of layer l > 0 is the output of layer l - 1
    o.x_min = l == 0 ? st[S_XMIN] : hs[(size_t)(l - 1) * S_COUNT + S_HMIN];
    o.x_max = l == 0 ? st[S_XMAX] : hs[(size_t)(l - 1) * S_COUNT + S_HMAX];
    o.h_min = st[S_HMIN];
    o.h_max = st[S_HMAX];
    o.m_min = st[S_MMIN];
    o.m_max = st[S_MMAX];
    o.c_absmax = st[S_CABS];
    for (int g = 0; g < 4; ++g) o.g_absmax[g] = st[S_GABS + g];
  }
  return LSTM_INT_OK;
}

}  // namespace

extern "C" int lstm_int_calibrate(const lstm_int_layer_params *layers, int32_t num_layers, int32_t device,
                                  const float *x, int32_t T, int32_t B, void *hip_stream,
                                  lstm_int_layer_stats *stats_out, double *y_float) {
  try {
    return calibrate(layers, num_layers, device, x, T, B, hip_stream, stats_out, y_float);
  } catch (const std::bad_alloc &) {
    return LSTM_INT_E_OUT_OF_MEMORY;
  }
}

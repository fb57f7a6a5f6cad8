// Persistent recurrent kernels of the integer GRU for gfx950: all T steps of a layer in one launch, for layers of up to
// 2048 cells.  The batch is cut into groups of rows; the cells of a group are spread over GS = ceil(N / 64) workgroups of
// ONE XCD (one L2), 64 cells each, whose recurrent weights stay in registers, at 2048 cells three quarters of the compute
// unit's.  A step is the product R h8, the elementwise cell
// (reset product, coupled update, all on the lane that holds the product) and one exchange of the int8 state.
//
//  * gru_quad_kernel, groups of 4 rows: a lane has one cell of one row (little work per wave: what bounds a small batch is
//    the number of instructions a wave issues per step and the latency of the exchange).  The state travels as (value,
//    tag) byte pairs, four cells to a 64-bit word, the tag being the step: a reader polls the words it needs.  (Stored at
//    workgroup scope, polled at agent scope; they meet in the L2 of the group's one XCD, see quad_kernel.inc.h.  Stored at
//    agent scope, through the L2 to memory: 512 cells, 16 rows, 100 steps 152 -> 267 us.)
//  * gru_rows_kernel (gru_rows.hip), groups of 16 or 32 rows: eight waves, 16 cells and half of the depth each; a lane
//    finishes two cells of a row.  Groups of 16 rows hand the state on in marked words: one wave stores the workgroup's piece in
//    operand order, every wave fetches an eighth of the tile, global -> LDS, until no word of it is marked as not written.  (Until
//    then a flag raised behind the acknowledgement of the stores, a poll of all flags and the fetch behind it followed each other;
//    100 steps, us: 512 cells, 256 rows 275 -> 213; 333 cells, 333 rows 367 -> 306; 1024 cells, 128 rows 302 -> 256; 2048 cells, 128 rows 420 ->
//    374.  A pause of 4 ahead of the first fetch: 0 and 8 are 1 to 4 % slower.)
//    In groups of 32 rows a workgroup waits for the acknowledgement and raises its flag, a word in a line of its own; one wave
//    polls the flags of all members, then every wave fetches.
//    Groups of 32 rows are two tiles of 16 by turns, the exchange of one under the product and the cell of the other:
//    all that is left of it open is a poll, and marked words cost more than that, asked for before, within or behind the product
//    (1024 cells, 512 rows 528 -> 554 to 590; two layers of 2048 cells, 256 rows, 64 steps 930 -> 1036 to 1130).
//    (A flag per wave, polled by the waves that need it, saves both barriers but four times the polling delays the very
//    stores it waits for: 0.3 to 1.3 us per step slower.  Flags packed into lines: another 1 to 3 us.)
//
// What bounds them: the chain of a step, instruction issue of the cell and the exchange (1 us among 2 to 32 workgroups), not
// the product: 0.65 us of 3.7 at 2048 cells and 64 rows.  Time per step (us), one launch per step, which re-reads the weights
// from L2 (before; up to 1024 cells 3.6 in one launch) -> these kernels:
//    512 cells, 16 rows   3.6 -> 1.3     1024 cells, 128 rows  3.7 -> 2.5     2048 cells, 16 rows   8.4 -> 2.4
//    512 cells, 256 rows  3.7 -> 2.1     1024 cells, 512 rows  10.5 -> 4.3    2048 cells, 256 rows  13.4 -> 5.4
//
// Placement and the waits that end are those of the LSTM's recurrent kernels (rec_kernel.inc.h).
#include "gru_kernel.inc.h"

namespace lstm_int {

namespace {

// ---------------------------------------------------------------------------------------------------------------------
template <int KS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gru_quad_kernel(GruSeqArgs a) {
  constexpr int LS = KS * 64 + 16;  // row stride of the h tiles
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, q = lane >> 4;
  const int GS = a.GS, N = a.N, T = a.T;
  const GruPlace pl = gru_place(a);
  const int member = pl.member;
  if (pl.group >= a.groups) {
    gru_placement_check(a);
    return;
  }
  const int row0 = a.batch0 + pl.group * 4;

  // ---- LDS: two h tiles, the W x terms of two steps, the flag, the tables
  int8_t *hT = reinterpret_cast<int8_t *>(lds);
  int16_t *txL = reinterpret_cast<int16_t *>(lds + 8 * LS);
  int *flag = reinterpret_cast<int *>(lds + 8 * LS + 4096);
  int off = (8 * LS + 4096 + 16 + 1023) & ~1023;
  const GruLut ls = gru_lut_place(a.lut[0], off), lt = gru_lut_place(a.lut[1], off);
  gru_lut_load<4>(a.lut[0], ls, lds, wave, lane);
  gru_lut_load<4>(a.lut[1], lt, lds, wave, lane);

  // W x terms of a step -> LDS, waves 2 and 3.  Tile order: piece ((tile 2 + half) 2 + quad) 4 + row, 8 values; row-major:
  // piece (row 3 + gate) 8 + j, 8 cells
  auto tx_request = [&](int t) {
    if (wave < 2) return;
    const int pc = (wave - 2) * 64 + lane;
    int8_t *dst = reinterpret_cast<int8_t *>(txL) + (t & 1) * 2048 + (wave - 2) * 1024;
    if (a.tx2) {
      const int rr = pc & 3, quad = (pc >> 2) & 1, half = (pc >> 3) & 1, tile = pc >> 4;
      dma16(a.tx2 + ((((size_t)t * a.Bp + row0) >> 5) * (size_t)a.tiles + member * 8 + tile) * 128 + half * 64 + 32 * quad + ((row0 + rr) & 31), dst);
    } else {
      const int rr = pc / 24, g = (pc >> 3) % 3, n = member * 64 + (pc & 7) * 8;
      if (pc < 96 && n < a.Nt)
        dma16(a.tx + ((size_t)t * a.B + (row0 + rr < a.B ? row0 + rr : a.B - 1)) * 3 * a.Nt + g * a.Nt + n, dst);
    }
  };
  int tx_at[3];
#pragma unroll
  for (int g = 0; g < 3; ++g)
    tx_at[g] = a.tx2 ? ((((wave * 2 + (c16 >> 3)) * 2 + ((g + 1) >> 1)) * 2 + ((c16 >> 2) & 1)) * 4 + q) * 8 + ((g + 1) & 1) * 4 + (c16 & 3)
                     : (q * 3 + g) * 64 + wave * 16 + c16;
  tx_request(0);

  v4i Wf[3][KS];
  gru_load_weights<KS, 64>(a, member, wave, 0, lane, Wf);
  const int cell = member * 64 + wave * 16 + c16;
  int32_t bh[3];
  RescaleHi ps[3];
  bool pre = false;
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    bh[g] = a.bh[g * 64 * GS + cell];
    ps[g] = rescale_hi_prepare(a.Mh[g], a.rh[g]);
    pre |= a.rh[g] < 33;
  }
  const bool row_ok = row0 + q < a.B;
  int32_t hreg = !a.zero_state && cell < N ? a.h16[(size_t)(row_ok ? row0 + q : a.B - 1) * N + cell] : 0;
  // the tile before step 0; the other one starts as zeros (columns past the layer's only meet zero weights)
  if (a.zero_state) {
    for (int i = tid; i < 8 * LS / 16; i += 256) reinterpret_cast<int4 *>(hT)[i] = int4{0, 0, 0, 0};
  } else {
    const bool vec = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(a.h16) & 7) == 0;
#pragma unroll 4
    for (int i = tid; i < 8 * LS / 4; i += 256) {
      const int rr = i / (LS / 4), k = 4 * (i - rr * (LS / 4));
      const int16_t *hq = a.h16 + (size_t)(row0 + rr < a.B ? row0 + rr : a.B - 1) * N + k;
      uint32_t w = 0;
      if (rr < 4 && k < N) {
        short4 v{0, 0, 0, 0};
        if (vec) {
          v = *reinterpret_cast<const short4 *>(hq);
        } else {
          v.x = hq[0];
          if (k + 1 < N) v.y = hq[1];
          if (k + 2 < N) v.z = hq[2];
          if (k + 3 < N) v.w = hq[3];
        }
        w = (state_i8(v.x) & 0xFF) | (state_i8(v.y) & 0xFF) << 8 | (state_i8(v.z) & 0xFF) << 16 | (uint32_t)(state_i8(v.w) & 0xFF) << 24;
      }
      reinterpret_cast<uint32_t *>(hT)[i] = w;
    }
  }
  if (tid == 0) flag[0] = 1;
  if (T > 1) tx_request(1);
  const bool y_words = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(a.y) & 3) == 0;
  // exchange words of the group: [2 slots][4 rows][16 GS]
  u64 *const xw = reinterpret_cast<u64 *>(a.sync + kGruWordsOff) + (size_t)pl.group * GS * 128;
  const int row_words = 16 * GS;
  const unsigned never = a.never ? 0x80u : 0;  // a tag nobody stores in so few steps
  wait_vmem();
  __syncthreads();

  const int arow = c16 >> 2;  // result row 4 q of the product is row q of the group; the rows between repeat it
  for (int t = 0; t < T; ++t) {
    const int8_t *hcur = hT + (t & 1) * 4 * LS;
    int8_t *hnext = hT + ((t + 1) & 1) * 4 * LS;
    const unsigned tag = (unsigned)(t + 1) & 0xFF;
    int32_t tx[3], th[3];
#pragma unroll
    for (int g = 0; g < 3; ++g) tx[g] = txL[(t & 1) * 1024 + tx_at[g]];
    {
      v4i acc[3];
#pragma unroll
      for (int g = 0; g < 3; ++g) acc[g] = v4i{bh[g], 0, 0, 0};
      constexpr int U = KS < 8 ? KS : 8;  // operands in flight together
#pragma unroll
      for (int k0 = 0; k0 < KS; k0 += U) {
        v4i hf[U];
#pragma unroll
        for (int u = 0; u < U; ++u) hf[u] = *reinterpret_cast<const v4i *>(hcur + arow * LS + (q << 4) + (k0 + u) * 64);
        // a gate's products one after the other: dependent 16x16x64 MFMAs issue back to back, rotating accumulators do not (with
        // four k steps there is nothing in it)
        if constexpr (KS >= 8) {
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int g = 0; g < 3; ++g)
#pragma unroll
            for (int u = 0; u < U; ++u) acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(hf[u], Wf[g][k0 + u], acc[g], 0, 0, 0);
        } else {
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < 3; ++g) acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(hf[u], Wf[g][k0 + u], acc[g], 0, 0, 0);
        }
      }
      if (pre) {
#pragma unroll
        for (int g = 0; g < 3; ++g) th[g] = rescale_sat16_pre<2>(acc[g][0], ps[g]);
      } else {
#pragma unroll
        for (int g = 0; g < 3; ++g) th[g] = rescale_sat16_pre<0>(acc[g][0], ps[g]);
      }
    }
    const int32_t x[2] = {sat16(tx[0] + th[0]), sat16(tx[1] + th[1])};  // Sec. 3.2.1
    int32_t v[2];
    gru_lookup<2>(lds, ls, x, v);
    const int32_t r = mirror_sigmoid(x[0], v[0]), u = mirror_sigmoid(x[1], v[1]);
    const int32_t xn[1] = {sat16(tx[2] + ((mul_i24(r, th[2]) + 16384) >> 15))};  // Q0.15 x Q3.12 -> Q3.12
    int32_t vn[1];
    gru_lookup<1>(lds, lt, xn, vn);
    hreg = cell_update32(cifg_input_gate(u), mirror_tanh(xn[0], vn[0]), u, hreg, 0);  // 1 - u, Secs. 3.2.9, 3.2.7
    const int32_t h8 = state_i8(hreg);

    // Nobody else reads this state: this workgroup's cells go to the tile directly.  (A single step meets its group all the
    // same: h16 is read by every member and written by each.)
    if (GS == 1 || (t == T - 1 && T > 1)) {
      hnext[q * LS + cell] = (int8_t)h8;
      wait_vmem();
      __syncthreads();
    } else {
      u64 *const words = xw + (size_t)(t & 1) * 4 * row_words;
      {
        const int32_t b = (h8 & 0xFF) | (int32_t)(tag << 8);
        const int32_t w = b | (__builtin_amdgcn_mov_dpp(b, 0xB1, 0xF, 0xF, true) << 16);  // lanes 0, 2 of a quad: cells (0, 1), (2, 3)
        const int32_t w2 = __builtin_amdgcn_mov_dpp(w, 0x4E, 0xF, 0xF, true);              // lane 0: the word of lane 2
        if ((lane & 3) == 0)
          __hip_atomic_store(words + q * row_words + member * 16 + wave * 4 + (c16 >> 2), (u64)(uint32_t)w | (u64)(uint32_t)w2 << 32,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      if constexpr (KS >= 8) {
        // a thread polls its words, two of them per load (poll_pairs), until all carry the tag.  With the products in order and
        // this, 100 steps of 512 cells, 16 rows 149 -> 138 us, 64 of 1024 cells 141 -> 120, of 2048 cells, 32 rows 220 -> 178.
        const int pairs = 2 * row_words;  // a row's words are a multiple of 16
        const uint32_t want = (tag ^ never) * 0x01000100u;
        constexpr int U = KS >= 16 ? 2 : 1;
#pragma unroll 1
        for (int base = 0; base < pairs; base += 256 * U) {
          unsigned at[U];
          v4i w[U];
#pragma unroll
          for (int k = 0; k < U; ++k) at[k] = base + k * 256 + tid < pairs ? (unsigned)(base + k * 256 + tid) * 16 : 0;
          int budget = a.spin_limit;
          for (;;) {
            poll_pairs(words, at, w);
            uint32_t off = 0;
#pragma unroll
            for (int k = 0; k < U; ++k)
#pragma unroll
              for (int i = 0; i < 4; ++i) off |= (uint32_t)w[k][i] ^ want;
            if (__builtin_amdgcn_ballot_w64((off & 0xFF00FF00u) != 0) == 0) break;
            if (gru_spent(a, budget)) {
              __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              flag[0] = 0;
              break;
            }
          }
#pragma unroll
          for (int k = 0; k < U; ++k) {
            const int c = base + k * 256 + tid;
            if (c < pairs) {
              const int half = row_words >> 1, rr = (c >= half) + (c >= 2 * half) + (c >= 3 * half);
              *reinterpret_cast<v2i *>(hnext + rr * LS + 8 * (c - rr * half)) =
                  v2i{(int)__builtin_amdgcn_perm((uint32_t)w[k][1], (uint32_t)w[k][0], 0x06040200u),
                      (int)__builtin_amdgcn_perm((uint32_t)w[k][3], (uint32_t)w[k][2], 0x06040200u)};
            }
          }
        }
      } else {  // up to 256 cells a thread has one word at most (in pairs half of the threads would have none: 2 to 4 % longer)
        const u64 want = (u64)((tag ^ never) * 0x01000100u) << 32 | (u64)((tag ^ never) * 0x01000100u);
        u64 w = want;
        int budget = a.spin_limit;
        for (;;) {
          if (tid < 4 * row_words) w = __hip_atomic_load(words + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (__builtin_amdgcn_ballot_w64((w & 0xFF00FF00FF00FF00ull) != want) == 0) break;
          if (gru_spent(a, budget)) {
            __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            flag[0] = 0;
            break;
          }
        }
        if (tid < 4 * row_words) {
          const int rr = (tid >= row_words) + (tid >= 2 * row_words) + (tid >= 3 * row_words), c = tid - rr * row_words;
          *reinterpret_cast<uint32_t *>(hnext + rr * LS + 4 * c) = __builtin_amdgcn_perm((uint32_t)(w >> 32), (uint32_t)w, 0x06040200u);
        }
      }
      wait_vmem();  // the W x terms asked for a step ago are in LDS (a wave may have had nothing to poll)
      __syncthreads();
      if (flag[0] == 0) return;
    }
    if (t + 2 < T) tx_request(t + 2);
    if (wave == 1) {  // this workgroup's columns of the output: four cells of a row per lane
      const int rr = q, n = member * 64 + 4 * c16;
      if (row0 + rr < a.B) {
        const size_t orow = (size_t)t * a.B + row0 + rr;
        const uint32_t w = *reinterpret_cast<const uint32_t *>(hnext + rr * LS + n);
        if (a.h8) *reinterpret_cast<uint32_t *>(a.h8 + orow * a.Kp + n) = w;
        if (a.y) {
          int8_t *yd = a.y + orow * N + n;
          if (y_words && n < N)
            *reinterpret_cast<uint32_t *>(yd) = w;
          else
            for (int k = 0; k < 4 && n + k < N; ++k) yd[k] = (int8_t)(w >> (8 * k));
        }
      }
    }
  }
  gru_placement_check(a);
  if (a.h16 && row_ok && cell < N) a.h16[(size_t)(row0 + q) * N + cell] = (int16_t)hreg;
}

constexpr int kGruKS[] = {4, 8, 16, 24, 32};
int gru_ks(int Kp) {
  for (int k : kGruKS)
    if (Kp <= 64 * k) return k;
  return 0;
}
gru_fn gru_pick(int ks, int rows) {
  if (rows > 4) return gru_rows_pick(ks, rows);
  switch (ks) {
    case 4: return gru_quad_kernel<4>;
    case 8: return gru_quad_kernel<8>;
    case 16: return gru_quad_kernel<16>;
    case 24: return gru_quad_kernel<24>;
    case 32: return gru_quad_kernel<32>;
    default: return nullptr;
  }
}
size_t gru_lds_bytes(int ks, int rows, const LutWide (&lut)[2]) {
  const int rt = rows / 16;
  size_t n = rows == 4 ? 8 * (size_t)(ks * 64 + 16) + 4096 + 16
                       : (size_t)rt * (ks + 1) * 1024 + kGruTxSlots(rt) * kGruTxBytes + 768 + kGruExchange + 16;
  n = (n + 1023) & ~(size_t)1023;
  for (const LutWide &l : lut) n += (size_t)lut_wide_lds_bytes(l.dom, l.sh, l.tail != 0);
  return n;
}

}  // namespace

// The fewest rows whose groups fit one launch: the fewer rows a group has, the shorter its step (1024 cells: 2.2 us with 4
// rows, 2.5 with 16, 4.3 with 32).  32 is the most that keeps the tile of 2048 cells, the terms of two steps and the tables
// in LDS.
int gru_seq_rows(int N, int B, int *max_groups) {
  if (N < 1 || N > 2048 || B < 1) return 0;
  const int GS = (N + 63) / 64, cap = 8 * (32 / GS);
  *max_groups = cap;
  return (B + 3) / 4 <= cap ? 4 : (B + 15) / 16 <= cap ? 16 : 32;
}

hipError_t gru_seq_init() {
  for (int ks : kGruKS)
    for (int rows : {4, 16, 32}) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(gru_pick(ks, rows)),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

hipError_t launch_gru_seq(hipStream_t s, const GruSeqArgs &a) {
  const int ks = gru_ks(a.Kp);
  int cap = 0;
  if (!ks || a.GS != (a.N + 63) / 64 || a.Kp != 64 * a.GS || !gru_seq_rows(a.N, a.B, &cap) || a.groups < 1 || a.groups > cap ||
      (a.rows_pg != 4 && a.rows_pg != 16 && a.rows_pg != 32) || a.batch0 + (a.groups - 1) * a.rows_pg >= a.B || a.batch0 % 32 != 0 ||
      (!a.tx2 && (!a.tx || a.Nt % 8 != 0)) || (a.tx2 && (a.tiles < 8 * a.GS || a.Bp % 32 != 0)) || (a.rows_pg > 4 && !a.hx) ||
      (!a.zero_state && !a.h16))
    return hipErrorInvalidValue;
  GruSeqArgs args = a;
  // Longer prefixes of the two tables as far as the LDS goes, to |x| < 6: beyond the prefix is a detour for the whole wave
  while (args.lut[0].dom < 24576 || args.lut[1].dom < 24576) {
    LutWide more[2] = {args.lut[0], args.lut[1]};
    for (LutWide &l : more)
      if (l.dom < 24576) l.dom += 1024;
    if (gru_lds_bytes(ks, a.rows_pg, more) > 160 * 1024) break;
    args.lut[0] = more[0];
    args.lut[1] = more[1];
  }
  const size_t lds = gru_lds_bytes(ks, a.rows_pg, args.lut);
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  void *params[] = {&args};
  return hipLaunchKernel(reinterpret_cast<const void *>(gru_pick(ks, a.rows_pg)), dim3(8 * a.GS * ((a.groups + 7) / 8)),
                         dim3(a.rows_pg == 4 ? 256 : 512), params, lds, s);
}

}  // namespace lstm_int

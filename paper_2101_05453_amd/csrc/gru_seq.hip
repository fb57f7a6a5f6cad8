// Persistent recurrent kernels of the integer GRU for gfx950: all T steps of a layer in one launch, for layers of up to
// 2048 cells.  The batch is cut into groups of rows; the cells of a group are spread over GS = ceil(N / 64) workgroups of
// ONE XCD (one L2), 64 cells each, whose recurrent weights stay in registers -- a wave has 16 cells of all three gates
// over the whole depth, at 2048 cells 384 of a lane's 512 registers.  A step is the product R h8, the elementwise cell
// (reset product, coupled update, all on the lane that holds the product) and one exchange of the int8 state.
//
//  * gru_quad_kernel, groups of 4 rows: a lane has one cell of one row (little work per wave: what bounds a small batch is
//    the number of instructions a wave issues per step and the latency of the exchange).  The state travels as (value,
//    tag) byte pairs, four cells to a 64-bit word, the tag being the step: a reader polls the words it needs.  (Stored at
//    workgroup scope, polled at agent scope; they meet in the L2 of the group's one XCD, see quad_kernel.inc.h.  Stored at
//    agent scope, through the L2 to memory: 512 cells, 16 rows, 100 steps 152 -> 267 us.)
//  * gru_rows_kernel, groups of 16 or 32 rows: a lane has four cells of a row.  A workgroup stores its piece of the state
//    in operand order, waits for the acknowledgement and raises its flag, a word in a line of its own; one wave polls the
//    flags of all members, then every wave fetches a quarter of the tile, global -> LDS without a register in between.
//    Groups of 32 rows are two tiles of 16 by turns, the exchange of one under the product and the cell of the other.
//    (A flag per wave, polled by the waves that need it, saves both barriers but four times the polling delays the very
//    stores it waits for: 0.3 to 1.3 us per step slower.  Flags packed into lines: another 1 to 3 us.)
//
// What bounds them: the chain of a step, instruction issue of the cell (about 300 instructions per row tile of 16) and the
// exchange (1 us among 2 to 32 workgroups), not the product: 0.65 us of 3.7 at 2048 cells and 64 rows.  Time per step (us),
// one launch per step, which re-reads the weights from L2 (before; up to 1024 cells 3.6 in one launch) -> these kernels:
//    512 cells, 16 rows   3.6 -> 1.3     1024 cells, 128 rows  3.7 -> 2.9     2048 cells, 16 rows   8.4 -> 2.4
//    512 cells, 256 rows  3.7 -> 2.7     1024 cells, 512 rows  10.5 -> 4.6    2048 cells, 256 rows  13.4 -> 5.7
// (2048 cells, 256 rows, both tiles of 32 rows in one turn: 6.1; without any exchange it would take 4.9)
//
// Placement and the waits that end are those of the LSTM's recurrent kernels (rec_kernel.inc.h).
#include "gru_seq.h"

#include "lstm_int_math.h"
#include "rec_kernel.inc.h"

namespace lstm_int {

namespace {

__device__ __forceinline__ int32_t state_i8(int32_t h16) { return sat8((h16 + 128) >> 8); }

__device__ __forceinline__ void dma16(const void *src, void *dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                   (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// All of this wave's vector memory operations are done.  (The builtin, not an asm: the compiler then knows it too, and adds
// no wait of its own before reads of the LDS that the transfers above filled.)
__device__ __forceinline__ void wait_vmem() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  asm volatile("" ::: "memory");
}

// where a table is in LDS
struct GruLut {
  int32_t dom, sh, D, B, T;
};
__device__ __forceinline__ GruLut gru_lut_place(const LutWide &w, int &off) {
  GruLut l{w.dom, w.sh, off, off + w.dom, 0};
  off += lut_wide_lds_bytes(w.dom, w.sh, false);
  if (w.tail) {
    l.T = off;
    off += 3072;
  }
  return l;
}
__device__ __forceinline__ void gru_lut_load(const LutWide &w, const GruLut &l, uint8_t *lds, int wave, int lane) {
  const int nd = w.dom >> 10, nb = (((w.dom >> w.sh) * 2) + 1023) >> 10, nt = w.tail ? 3 : 0;
  for (int c = wave; c < nd + nb + nt; c += 4) {
    const int so = c < nd ? c * 1024 : (c < nd + nb ? kLutWideBaseOff + (c - nd) * 1024 : kLutWideTailOff + (c - nd - nb) * 1024);
    dma16(w.blob + so + lane * 16, lds + l.D + c * 1024);  // deltas, bases and tail follow each other
  }
}
// table values of |x| for K values at once
template <int K>
__device__ __forceinline__ void gru_lookup(const uint8_t *lds, const GruLut &l, const int32_t (&x)[K], int32_t (&out)[K]) {
  int32_t mag[K];
  uint32_t base[K], delta[K];
  bool over = false;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    mag[k] = abs_i32(x[k]);
    over |= mag[k] >= l.dom;
    const int32_t ai = mag[k] < l.dom ? mag[k] : l.dom - 1;
    base[k] = *reinterpret_cast<const uint16_t *>(lds + l.B + 2 * (ai >> l.sh));
    delta[k] = lds[l.D + ai];
  }
  __builtin_amdgcn_sched_barrier(0);  // all reads before the first sum
#pragma unroll
  for (int k = 0; k < K; ++k) out[k] = (int32_t)(base[k] + delta[k]);
  if (l.T && __builtin_amdgcn_ballot_w64(over) != 0) {
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (mag[k] >= l.dom) out[k] = lut_wide_tail(lds + l.T, mag[k]);
  }
}

// the place of a workgroup: XCC_ID and the hardware's dealing of consecutive workgroups to the XCDs in turn; see rec_kernel
struct GruPlace {
  int group, member;
};
__device__ __forceinline__ int gru_xcc() { return (int)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7); }
__device__ __forceinline__ GruPlace gru_place(const GruSeqArgs &a) {
  const int slot = (int)blockIdx.x >> 3;
  return GruPlace{gru_xcc() + 8 * (slot / a.GS), slot % a.GS};
}
__device__ __forceinline__ void gru_placement_check(const GruSeqArgs &a) {
  if (threadIdx.x != 0) return;
  const unsigned places = gridDim.x >> 3;  // at most 32
  const u64 mine = (1ull << 32) + (1ull << (blockIdx.x >> 3));
  const u64 now = __hip_atomic_fetch_add(reinterpret_cast<u64 *>(a.sync) + gru_xcc() * 32, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine;
  const unsigned count = (unsigned)(now >> 32);
  const unsigned all = places >= 32 ? 0xFFFFFFFFu : (1u << places) - 1;
  if (count > places || (count == places && (unsigned)now != all))
    __hip_atomic_store(a.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool gru_spent(const GruSeqArgs &a, int &budget) {
  --budget;
  return (budget & 15) == 0 && (budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0);
}

// recurrent weights of a wave -> registers, the first 64 operands in accumulation registers; k steps past the layer's zero
template <int KS>
__device__ __forceinline__ void gru_load_weights(const GruSeqArgs &a, int member, int wave, int lane, v4i (&Wf)[3][KS]) {
  const int ks_n = a.Kp >> 6;
  const v4i *src = reinterpret_cast<const v4i *>(a.R16) + (size_t)(member * 4 + wave) * 3 * ks_n * 64 + lane;
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    v4i w[KS];  // a gate's loads in flight together
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) w[ks] = ks < ks_n ? src[((size_t)g * ks_n + ks) * 64] : v4i{0, 0, 0, 0};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      Wf[g][ks] = w[ks];
      if (g * KS + ks < 64)
        asm volatile("" : "+a"(Wf[g][ks]));
      else
        asm volatile("" : "+v"(Wf[g][ks]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

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
  gru_lut_load(a.lut[0], ls, lds, wave, lane);
  gru_lut_load(a.lut[1], lt, lds, wave, lane);

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
  gru_load_weights<KS>(a, member, wave, lane, Wf);
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

// ---------------------------------------------------------------------------------------------------------------------
template <int KS, int RT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void gru_rows_kernel(GruSeqArgs a) {
  constexpr int R = 16 * RT;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, q = lane >> 4;
  const int GS = a.GS, N = a.N, T = a.T, ks_n = a.Kp >> 6;  // ks_n = GS
  const GruPlace pl = gru_place(a);
  const int member = pl.member;
  if (pl.group >= a.groups) {
    gru_placement_check(a);
    return;
  }
  const int row0 = a.batch0 + pl.group * R;

  // ---- LDS: the h tile [row tile][k step][64 lanes][16 B], the W x terms of two steps, biases, the flag, the tables
  v4i *hT = reinterpret_cast<v4i *>(lds);
  constexpr int TX = R * 512;  // bytes of a step's W x terms
  uint8_t *txL = lds + RT * KS * 1024;
  int32_t *bhL = reinterpret_cast<int32_t *>(txL + 2 * TX);  // [3][64]
  v4i *stage = reinterpret_cast<v4i *>(bhL + 192);           // [row tile][64 lanes]: this workgroup's piece of the new state
  int *flag = reinterpret_cast<int *>(stage + RT * 64);
  int off = (RT * KS * 1024 + 2 * TX + 768 + RT * 1024 + 16 + 1023) & ~1023;
  const GruLut ls = gru_lut_place(a.lut[0], off), lt = gru_lut_place(a.lut[1], off);
  gru_lut_load(a.lut[0], ls, lds, wave, lane);
  gru_lut_load(a.lut[1], lt, lds, wave, lane);
  if (tid < 192) bhL[tid] = a.bh[(tid >> 6) * 64 * GS + member * 64 + (tid & 63)];

  // W x terms of a step -> LDS, by waves 1 to 3: the poll of wave 0 would wait behind them.
  // Tile order: piece ((tile 2 + half) 2 + quad) R + row; row-major: piece (row 3 + gate) 8 + j
  const int8_t *tx_src;  // of the first step; a piece's offset from it is the same in every step
  size_t tx_step;
  constexpr int NTX = (8 * RT + 2) / 3;
  unsigned tx_off[NTX];
  unsigned tx_has = 0;
  if (a.tx2) {
    tx_src = reinterpret_cast<const int8_t *>(a.tx2 + ((size_t)(row0 >> 5) * a.tiles + member * 8) * 128);
    tx_step = (size_t)(a.Bp >> 5) * a.tiles * 2048;
  } else {
    tx_src = reinterpret_cast<const int8_t *>(a.tx + (size_t)row0 * 3 * a.Nt);
    tx_step = (size_t)a.B * 3 * a.Nt * 2;
  }
#pragma unroll
  for (int i = 0; i < NTX; ++i) {
    const int pc = (wave - 1 + 3 * i) * 64 + lane;
    if (wave == 0 || pc >= 8 * RT * 64) continue;
    if (a.tx2) {
      const int rr = pc & (R - 1), quad = (pc / R) & 1, half = (pc / (2 * R)) & 1, tile = pc / (4 * R);
      tx_off[i] = (unsigned)(tile * 128 + half * 64 + 32 * quad + (row0 & 31) + rr) * 16;
      tx_has |= 1u << i;
    } else {
      const int rr = pc / 24, g = (pc >> 3) % 3, n = member * 64 + (pc & 7) * 8;
      tx_off[i] = (unsigned)(((row0 + rr < a.B ? rr : a.B - 1 - row0) * 3 + g) * a.Nt + n) * 2;
      if (rr < R && n < a.Nt) tx_has |= 1u << i;
    }
  }
  auto tx_request = [&](int t) {
    const int8_t *src = tx_src + (size_t)t * tx_step;
#pragma unroll
    for (int i = 0; i < NTX; ++i)
      if (tx_has >> i & 1) dma16(src + tx_off[i], txL + (t & 1) * TX + (wave - 1 + 3 * i) * 1024);
  };
  // byte offset of a lane's four terms of a gate, row tile 0; row tile rt: tx_row rt further
  int tx_at[3];
#pragma unroll
  for (int g = 0; g < 3; ++g)
    tx_at[g] = a.tx2 ? ((((wave * 2 + (q >> 1)) * 2 + ((g + 1) >> 1)) * 2 + (q & 1)) * R + c16) * 16 + ((g + 1) & 1) * 8
                     : ((c16 * 3 + g) * 64 + wave * 16 + 4 * q) * 2;
  const int tx_row = a.tx2 ? 256 : 16 * 3 * 128;
  tx_request(0);

  v4i Wf[3][KS];
  gru_load_weights<KS>(a, member, wave, lane, Wf);
  RescaleHi ps[3];
  bool pre = false;
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    ps[g] = rescale_hi_prepare(a.Mh[g], a.rh[g]);
    pre |= a.rh[g] < 33;
  }
  const int n0 = member * 64 + wave * 16 + 4 * q;  // this lane's four cells
  int32_t hreg[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int row = row0 + rt * 16 + c16 < a.B ? row0 + rt * 16 + c16 : a.B - 1;
#pragma unroll
    for (int c = 0; c < 4; ++c) hreg[rt][c] = !a.zero_state && n0 + c < N ? a.h16[(size_t)row * N + n0 + c] : 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(hreg[rt][c]));  // wait here, not at the first use in the loop
  }
  // the tile before step 0: 16 cells of a row per piece
  {
    const bool vec = (N & 7) == 0 && (reinterpret_cast<uintptr_t>(a.h16) & 15) == 0;
    for (int i = tid; i < RT * KS * 64; i += 256) {
      const int l = i & 63, ks = (i >> 6) % KS, rt = (i >> 6) / KS;
      const int row = row0 + rt * 16 + (l & 15), k = ks * 64 + (l >> 4) * 16;
      int32_t w[4] = {0, 0, 0, 0};
      if (!a.zero_state && k < N) {
        const int16_t *hq = a.h16 + (size_t)(row < a.B ? row : a.B - 1) * N + k;
        int16_t v[16];
        if (vec) {
          const int4 lo = *reinterpret_cast<const int4 *>(hq), hi = k + 8 < N ? *reinterpret_cast<const int4 *>(hq + 8) : int4{0, 0, 0, 0};
          __builtin_memcpy(v, &lo, 16);
          __builtin_memcpy(v + 8, &hi, 16);
        } else {
#pragma unroll
          for (int j = 0; j < 16; ++j) v[j] = k + j < N ? hq[j] : 0;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j >> 2] |= (int32_t)((uint32_t)(state_i8(v[j]) & 0xFF) << (8 * (j & 3)));
      }
      hT[i] = v4i{w[0], w[1], w[2], w[3]};
    }
  }
  if (tid == 0) flag[0] = 1;
  const bool y_vec = (N & 15) == 0 && (reinterpret_cast<uintptr_t>(a.y) & 15) == 0;
  const bool y_words = (N & 3) == 0 && (reinterpret_cast<uintptr_t>(a.y) & 3) == 0;
  unsigned *const flags = reinterpret_cast<unsigned *>(a.sync + kGruFlagsOff) + pl.group * RT * GS * 16;  // [row tile][member], a line each
  const int per = (GS + 3) >> 2, m0 = wave * per < GS ? wave * per : GS, m1 = m0 + per < GS ? m0 + per : GS;  // members whose pieces this wave fetches
  // group's part of a step of the exchange buffer, in rows of 16: tiles of ks_n KB
  int8_t *const hx0 = a.hx + (size_t)(a.batch0 / 16 + pl.group * RT) * ks_n * 1024;
  wait_vmem();
  __syncthreads();

  // The terms of a step.  (Read in an asm: behind an ordinary read of memory that transfers fill, the compiler waits for
  // every operation on global memory before it, here the stores of the output of the step before.)
  auto read_tx = [&](int t, int rt, short4 (&tx4)[3]) {
    const unsigned at = (unsigned)(RT * KS * 1024 + (t & 1) * TX + rt * tx_row);
    asm volatile("ds_read_b64 %0, %3\n ds_read_b64 %1, %4\n ds_read_b64 %2, %5\n s_waitcnt lgkmcnt(0)"
                 : "=&v"(tx4[0]), "=&v"(tx4[1]), "=&v"(tx4[2])
                 : "v"(at + tx_at[0]), "v"(at + tx_at[1]), "v"(at + tx_at[2])
                 : "memory");
  };
  auto product = [&](int rt, v4i (&acc)[3]) {
#pragma unroll
    for (int g = 0; g < 3; ++g) acc[g] = *reinterpret_cast<const v4i *>(bhL + g * 64 + wave * 16 + 4 * q);
    constexpr int DEPTH = 4;  // k steps of operands ahead
    v4i hf[DEPTH];
#pragma unroll
    for (int ks = 0; ks < DEPTH; ++ks) hf[ks] = hT[(rt * KS + ks) * 64 + lane];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int g = 0; g < 3; ++g) acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(Wf[g][ks], hf[ks % DEPTH], acc[g], 0, 0, 0);
      if (ks + DEPTH < KS) hf[ks % DEPTH] = hT[(rt * KS + ks + DEPTH) * 64 + lane];
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // the cell of a row tile: new state into h, its int8 form packed
  auto cell = [&](const v4i (&acc)[3], const short4 (&tx4)[3], int32_t (&h)[4]) {
    int32_t th[3][4], tx[3][4];
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      tx[g][0] = tx4[g].x; tx[g][1] = tx4[g].y; tx[g][2] = tx4[g].z; tx[g][3] = tx4[g].w;
    }
    if (pre) {
#pragma unroll
      for (int g = 0; g < 3; ++g)
#pragma unroll
        for (int c = 0; c < 4; ++c) th[g][c] = rescale_sat16_pre<2>(acc[g][c], ps[g]);
    } else {
#pragma unroll
      for (int g = 0; g < 3; ++g)
#pragma unroll
        for (int c = 0; c < 4; ++c) th[g][c] = rescale_sat16_pre<0>(acc[g][c], ps[g]);
    }
    int32_t x[8], v[8], xn[4], vn[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      x[c] = sat16(tx[0][c] + th[0][c]);
      x[4 + c] = sat16(tx[1][c] + th[1][c]);
    }
    gru_lookup<8>(lds, ls, x, v);
#pragma unroll
    for (int c = 0; c < 4; ++c) xn[c] = sat16(tx[2][c] + ((mul_i24(mirror_sigmoid(x[c], v[c]), th[2][c]) + 16384) >> 15));
    gru_lookup<4>(lds, lt, xn, vn);
    uint32_t pk = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int32_t u = mirror_sigmoid(x[4 + c], v[4 + c]);
      h[c] = cell_update32(cifg_input_gate(u), mirror_tanh(xn[c], vn[c]), u, h[c], 0);
      pk |= (uint32_t)(state_i8(h[c]) & 0xFF) << (8 * c);
    }
    return pk;
  };
  // byte 4 q of lane (c16, wave) of a piece: this lane's four cells
  const int mine = (wave * 16 + c16) * 16 + 4 * q;
  auto store_piece = [&](int t, int rt, uint32_t pk) {
    *reinterpret_cast<uint32_t *>(hx0 + (size_t)t * a.hx_step + (size_t)(rt * ks_n + member) * 1024 + mine) = pk;
  };
  auto fetch = [&](int t, int rt) {  // a quarter of the tile per wave
    const int8_t *src = hx0 + (size_t)t * a.hx_step + (size_t)rt * ks_n * 1024 + lane * 16;
    for (int m = m0; m < m1; ++m) dma16(src + (size_t)m * 1024, hT + (rt * KS + m) * 64);
  };
  auto raise = [&](int rt, int step) {
    if (tid == 0) __hip_atomic_store(flags + (rt * GS + member) * 16, (unsigned)step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto poll = [&](int rt, int step) {  // wave 0: all members have finished `step` steps of the row tile
    int budget = a.spin_limit;
    for (;;) {
      const unsigned f = __hip_atomic_load(flags + (rt * GS + (lane < GS ? lane : 0)) * 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__builtin_amdgcn_ballot_w64((int)(f - (unsigned)step) < 0 || a.never) == 0) break;
      if (gru_spent(a, budget)) {
        __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        flag[0] = 0;
        break;
      }
    }
  };
  auto output = [&](int t, int rt) {  // this workgroup's 64 columns: 16 cells of a row per lane of one wave
    const int row = row0 + rt * 16 + c16, n = member * 64 + 16 * q;
    if (row >= a.B) return;
    const size_t orow = (size_t)t * a.B + row;
    const v4i w = stage[rt * 64 + lane];
    if (a.h8) *reinterpret_cast<v4i *>(a.h8 + orow * a.Kp + n) = w;
    if (!a.y) return;
    int8_t *yd = a.y + orow * N + n;
    if (y_vec) {
      if (n < N) *reinterpret_cast<v4i *>(yd) = w;
    } else if (y_words) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (n + 4 * j < N) reinterpret_cast<int32_t *>(yd)[j] = w[j];
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (n + j < N) yd[j] = (int8_t)(w[j >> 2] >> (8 * (j & 3)));
    }
  };
  auto keep_piece = [&](int rt, uint32_t pk) {  // in LDS: for the output, and, where the group is this workgroup, as the state
    *reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(stage + rt * 64) + mine) = pk;
    if (GS == 1) *reinterpret_cast<uint32_t *>(lds + rt * KS * 1024 + mine) = pk;
  };

  if constexpr (RT == 1) {
    for (int t = 0; t < T; ++t) {
      short4 tx4[3];
      v4i acc[3];
      read_tx(t, 0, tx4);
      if (t + 1 < T) tx_request(t + 1);
      product(0, acc);
      // every wave is done with the tile before any wave fetches the next state into it
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      const uint32_t pk = cell(acc, tx4, hreg[0]);
      keep_piece(0, pk);
      if (GS == 1 || (t == T - 1 && T > 1)) {  // nobody else reads this state (see gru_quad_kernel)
        wait_vmem();
        __syncthreads();
      } else {
        store_piece(t, 0, pk);
        wait_vmem();
        __syncthreads();
        if (wave == 0) {
          raise(0, t + 1);
          for (int i = 0; i < a.sync_sleep; ++i) __builtin_amdgcn_s_sleep(1);
          poll(0, t + 1);
        }
        __syncthreads();
        asm volatile("" ::: "memory");
        fetch(t, 0);
        wait_vmem();
        __syncthreads();
        if (flag[0] == 0) return;
      }
      if (wave == 1) output(t, 0);
    }
  } else {
    // Two row tiles by turns: while the members exchange the state of one, they work on the other.  The flags of the other
    // tile were raised half a step ago when they are polled, its pieces arrive under the cell of this one.
    for (int t = 0; t < T; ++t) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        short4 tx4[3];
        v4i acc[3];
        read_tx(t, rt, tx4);
        if (rt == 0 && t + 1 < T) tx_request(t + 1);
        product(rt, acc);
        const int other_step = t - (rt == 0);  // the step whose state of the other tile comes in now
        const bool comes = GS > 1 && other_step >= 0 && other_step + 1 < T;
        if (comes && wave == 0) poll(1 - rt, other_step + 1);
        // (not __syncthreads: nothing waits for the stores of the output)
        asm volatile("s_waitcnt lgkmcnt(0)\n s_barrier" ::: "memory");
        if (comes) fetch(other_step, 1 - rt);
        const uint32_t pk = cell(acc, tx4, hreg[rt]);
        keep_piece(rt, pk);
        if (GS > 1 && t + 1 < T) store_piece(t, rt, pk);
        wait_vmem();
        __syncthreads();
        if (flag[0] == 0) return;
        if (GS > 1) raise(rt, t + 1);
        if (wave == 1) output(t, rt);
      }
    }
    if (GS > 1 && T == 1) {  // h16 is read by every member and written by each
      if (wave == 0) poll(1, 1);
      __syncthreads();
      if (flag[0] == 0) return;
    }
  }
  gru_placement_check(a);
  if (a.h16)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      int n1 = n0;
      asm volatile("" : "+v"(n1));
      const int row = row0 + rt * 16 + c16;
      if (row < a.B)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (n1 + c < N) a.h16[(size_t)row * N + n1 + c] = (int16_t)hreg[rt][c];
    }
}

typedef void (*gru_fn)(GruSeqArgs);
constexpr int kGruKS[] = {4, 8, 16, 24, 32};
template <int KS>
gru_fn gru_pick_ks(int rows) {
  return rows == 4 ? gru_quad_kernel<KS> : rows == 16 ? gru_rows_kernel<KS, 1> : gru_rows_kernel<KS, 2>;
}
int gru_ks(int Kp) {
  for (int k : kGruKS)
    if (Kp <= 64 * k) return k;
  return 0;
}
gru_fn gru_pick(int ks, int rows) {
  switch (ks) {
    case 4: return gru_pick_ks<4>(rows);
    case 8: return gru_pick_ks<8>(rows);
    case 16: return gru_pick_ks<16>(rows);
    case 24: return gru_pick_ks<24>(rows);
    case 32: return gru_pick_ks<32>(rows);
    default: return nullptr;
  }
}
size_t gru_lds_bytes(int ks, int rows, const LutWide (&lut)[2]) {
  size_t n = rows == 4 ? 8 * (size_t)(ks * 64 + 16) + 4096 + 16 : (size_t)(rows / 16) * (ks + 1) * 1024 + 2 * rows * 512 + 768 + 16;
  n = (n + 1023) & ~(size_t)1023;
  for (const LutWide &l : lut) n += (size_t)lut_wide_lds_bytes(l.dom, l.sh, l.tail != 0);
  return n;
}

}  // namespace

// The fewest rows whose groups fit one launch: the fewer rows a group has, the shorter its step (1024 cells: 2.2 us with 4
// rows, 2.9 with 16, 4.6 with 32).  32 is the most that keeps the tile of 2048 cells, the terms of two steps and the tables
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
  return hipLaunchKernel(reinterpret_cast<const void *>(gru_pick(ks, a.rows_pg)), dim3(8 * a.GS * ((a.groups + 7) / 8)), dim3(256), params, lds, s);
}

}  // namespace lstm_int

// Device code of the stacked recurrent kernel: up to 8 equal layers in one
// launch, layer l on XCD l, each layer one step behind the layer below it (the
// stack of Sec. 7 as a wavefront over layers and time).  The per-step
// arithmetic is rec_kernel's (Secs. 3.2.4-3.2.9); what differs:
//   * the W x term of an item (step t, row tile r) is computed here, when the
//     layer's input rows arrive, from weights streamed out of memory as MFMA
//     operands (R stays in registers for the whole launch);
//   * R h^{t-1} runs first and is kept as packed int16 terms, so that the only
//     work between the arrival of the input and the gate sums is W x;
//   * a layer's output rows are stored with agent-scope stores, which write
//     through the XCD's L2, and a flag per (layer, row tile) counts the
//     finished steps; the next layer polls it and reads the rows with loads
//     that bypass its own L2 (sc1).  With the flag every such line is written
//     once per launch and was never read before.  A launch of one item per layer
//     (ONE, below) reads the lines again and again while they are being
//     written, so there it is the loads alone, past the reader's L1 and L2,
//     that keep an older copy from being seen: a plain load of these rows could
//     go on finding the marks in that L2.
//   * the cell state lives in memory between the items of a row tile.
// A launch of one item per layer (ONE, the streaming call) hands m and the rows between the layers on in marked words: who needs
// them polls the words themselves.  8 layers of 2048 cells, 640 outputs, layer norm, 32 rows, one step, us: 111.6 with counters and flags,
// 105.9 with m in marked words, 103.0 with the rows too, 101.3 with what the first item needs asked for in the order of its use.
// What is left, by the timers of each layer's first workgroup: 27 us until layer 0 has its weights (19 the set-up launch, the start and
// what is loaded ahead of R h, 8 R and W, 10.5 MB through one XCD), 10 its step, then 9.4 a layer: W x 0.8, gate sums 0.6,
// statistics 1.4, layer norm to the cell 1.5, hidden 0.5, m and the projection 2.3, the rows to the next XCD 2.3.
// Included by the stack_inst_*.hip translation units.
#pragma once

#include <type_traits>

#include "lstm_int_math.h"
#include "persistent.h"
#include "rec_kernel.inc.h"  // group_sync, lut helpers, mirror_*, vector types

namespace lstm_int {

typedef short v2s __attribute__((ext_vector_type(2)));

struct StkPrm {  // per-layer constants in LDS, 320 bytes
  RescaleHi h[4], c[4], ln[4], x[4];
  RescaleHi m, p;
  int32_t zp_m, zp_h, m_c, glo;
  double inv_n;  // 1 / N
  int32_t pad[2];
};
static_assert(sizeof(StkPrm) == 320, "stack_lds_bytes assumes 320 bytes");

// sat16(rescale(.)) of two accumulators, packed low | high; PRE = operand treatment of the rescale
template <int PRE>
__device__ __forceinline__ int32_t stk_requant2(int32_t s0, int32_t s1, const RescaleHi &p) {
  const int32_t v0 = rescale_sat16_pre<PRE>(s0, p), v1 = rescale_sat16_pre<PRE>(s1, p);
  return (v0 & 0xFFFF) | (v1 << 16);
}

// Eight waves with one weight tile each, as in rec_kernel (four with two: 8 layers of 2048 cells, 640 outputs, layer norm, 32
// rows, one step 133.5 -> 120.6 us; 1024 cells, layer norm and peephole, 8 steps 365 -> 281).
// FL as in rec_kernel: bit 0 CIFG, bit 1 peephole, bit 2 layer norm, bit 3 "no projection".
// ONE: the launch has one item per layer (one step, one row tile).
template <int KS, int FL, bool ONE>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void stack_kernel(StackArgs sa) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const RecArgs &a = sa.c;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, b2 = lane >> 5;
  constexpr int WAVES = 8;  // one weight tile each, as in rec_kernel
  constexpr bool cifg = FL & 1, ph = FL & 2, ln = FL & 4;
  constexpr bool proj = !(FL & 8);
  const int GS = a.GS;

  // Placement as in rec_kernel: the XCD comes from the hardware register, the place on it from the
  // workgroup index; here the XCD is the layer.
  const int wg = blockIdx.x;
  const int xcc = (int)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7);
  const int slot = wg >> 3;
  int xcd = wg & 7;
  if (a.tickets) {
    xcd = xcc;
  } else if (xcc != xcd && tid == 0) {
    __hip_atomic_store(a.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  auto placement_check = [&]() {
    if (a.tickets && tid == 0) {
      const int xcc_now = (int)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7);
      const unsigned places = gridDim.x >> 3;  // at most 32
      const u64 mine = ((u64)1 << 32) + ((u64)1 << (wg >> 3));
      const u64 now =
          __hip_atomic_fetch_add(&a.tickets[xcc_now * 32], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine;
      const unsigned count = (unsigned)(now >> 32);
      const unsigned all = places >= 32 ? 0xFFFFFFFFu : (1u << places) - 1;
      if (count > places || (count == places && (unsigned)now != all))
        __hip_atomic_store(a.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };
  const int layer = xcd, member = slot;  // slot < GS: the launch has GS workgroups per XCD
  if (layer >= sa.L) {
    placement_check();
    return;
  }
  const StackLayer &sl = sa.layers[layer];
  const bool last_layer = layer == sa.L - 1;
  constexpr int items = 128;  // (gate, row) layer-norm rows of a row tile

  // per-layer buffers
  const int8_t *xin = layer == 0 ? sa.x : sa.out_base + (size_t)(layer - 1) * sa.out_stride;
  const int ldx = layer == 0 ? sa.ldx : a.Hpad;
  const bool x_bypass = layer > 0 || !sa.x_shared;  // rows written by another XCD during this launch
  int8_t *out = sa.out_base + (size_t)layer * sa.out_stride;
  const int8_t *h0 = sa.h0_base + (size_t)layer * a.B * a.Hpad;
  int8_t *mbuf = sa.mbuf_base + (size_t)layer * sa.mbuf_stride;
  int16_t *cbuf = sa.c_base + (size_t)layer * a.B * a.N;
  int8_t *yout = last_layer ? a.y : nullptr;
  int8_t *hfin = sa.h_final ? sa.h_final + (size_t)layer * a.B * a.H : nullptr;
  const int kx = sl.kx;

  // ---- LDS carve-up (stack_lds_bytes mirrors it): what has a fixed size first, at offsets known to the compiler
  constexpr int LS = KS * 32 + 16;  // tile row stride (h rows and x rows alike)
  uint8_t *p = lds;
  u64 *red = reinterpret_cast<u64 *>(p);                 p += (size_t)items * 8;
  LnRow2 *lnrow = reinterpret_cast<LnRow2 *>(p);         p += (size_t)items * sizeof(LnRow2);
  double *LdL = reinterpret_cast<double *>(p);           p += 4 * 64 * 8;
  double *bdL = reinterpret_cast<double *>(p);           p += 4 * 64 * 8;
  int16_t *PqL = reinterpret_cast<int16_t *>(p);         p += 4 * 64 * 2;
  int32_t *bhL = reinterpret_cast<int32_t *>(p);         p += 4 * 64 * 4;
  int32_t *bxL = reinterpret_cast<int32_t *>(p);         p += 8 * 32 * 4;  // folded input bias, tile row order
  int32_t *bpL = reinterpret_cast<int32_t *>(p);         p += 32 * 4;      // projection bias of the first output tile
  StkPrm *prm = reinterpret_cast<StkPrm *>(p);           p += sizeof(StkPrm);
  int *flag = reinterpret_cast<int *>(p);                p += 16;
  u64 *tickL = reinterpret_cast<u64 *>(p);               p += 12 * 8;  // phase timers
  LutLds *lutP = reinterpret_cast<LutLds *>(p);          p += 3 * sizeof(LutLds);
  int8_t *hT = reinterpret_cast<int8_t *>(p);
  v4i *pred = reinterpret_cast<v4i *>(p);  // projection partials [slot][4][64] reuse the tile between steps
  const bool four_slots = a.flags & kFourPredSlots;
  {
    const size_t tile_bytes = ((size_t)32 * LS + 1023) / 1024 * 1024;  // whole 1 KB chunks
    const size_t pred_bytes = proj ? (four_slots ? 4 : 8) * 4096 : 0;
    p += tile_bytes > pred_bytes ? tile_bytes : pred_bytes;
  }
  // the activation tables as in rec_kernel: prefixes of the wide form; the two gate tables are common to
  // the layers, the cell-format tanh is the layer's own (or the gate tanh's copy when the formats agree)
  const LutWide lw[3] = {a.lut[0], a.lut[1], sl.lutc};
  const bool share_tanh = lw[2].blob == lw[1].blob;
  const uint8_t *lutD[3];
  const uint8_t *lutB[3];
  const uint8_t *lutTl[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (i == 2 && share_tanh) {
      lutD[2] = lutD[1]; lutB[2] = lutB[1]; lutTl[2] = lutTl[1];
    } else {
      const int nb = ((((lw[i].dom >> lw[i].sh) * 2) + 1023) >> 10) << 10;
      lutD[i] = p;                            p += lw[i].dom;
      lutB[i] = p;                            p += nb;
      lutTl[i] = lw[i].tail ? p : nullptr;    p += lw[i].tail ? 3072 : 0;
    }
  }
  int8_t *WpL = reinterpret_cast<int8_t *>(p);
  const int WLS = a.npadp + 16;
  const int my_ptiles = proj ? (a.ptiles > member ? (a.ptiles - member + GS - 1) / GS : 0) : 0;

  // ---- one-time loads, in the order in which they are needed: the first item's rows of h -> LDS, the R slice -> registers,
  // tables and W_proj tiles -> LDS.  Loads return in order, so what is small and has to
  // go through a register first is asked for ahead of them.
  constexpr int TILE_KB = (32 * LS + 1023) / 1024;
  constexpr int NCH = (TILE_KB + WAVES - 1) / WAVES;  // chunks per wave
  // the tile of 32 rows starting at row0 of a [.., ld] buffer -> LDS; bytes of a row beyond `width`, the
  // row padding read offset 0 of the tile (they only ever meet zero weights or are
  // not used); BYPASS = the loads pass the L2 by (rows written by another XCD during this launch)
  auto tile_to_lds = [&](const int8_t *base, int ld, int width, int row0, auto bypass_tag) {
    constexpr int AUX = decltype(bypass_tag)::value ? 16 : 0;  // sc1
    const int8_t *tile = base + (size_t)row0 * ld;
    asm volatile("" : "+s"(tile));
    int l = lane;
    asm volatile("" : "+v"(l));  // the lane's offsets are computed here, not kept
#pragma unroll
    for (int j = 0; j < NCH; ++j) {
      if (WAVES * (j + 1) > TILE_KB && wave + WAVES * j >= TILE_KB) continue;  // uniform
      const int o = (wave + WAVES * j) * 1024 + l * 16;
      const int r = o / LS, c = o - r * LS, last = a.B - 1 - row0;
      const unsigned off = (r < 32 && c < width) ? (unsigned)((r < last ? r : last) * ld + c) : 0u;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(tile + off),
                                       (__attribute__((address_space(3))) void *)(hT + (wave + WAVES * j) * 1024), 16, 0, AUX);
    }
  };
  int16_t Lq = 0, Pq = 0;
  int32_t qb = 0, bh = 0, bx = 0, bp = 0;
  if (tid < 256) {
    const int g = tid >> 6, n = tid & 63;
    const size_t idx = (size_t)g * a.Ncp + member * 64 + n;
    if (ln) {
      Lq = sl.Lq4[idx];
      qb = sl.qb4[idx];
    }
    if (ph && g < 3) Pq = sl.Pq3[idx];
    bh = sl.bh4[idx];
    bx = sl.bx2[(size_t)member * 256 + tid];  // the workgroup's 8 tiles x 32 rows
  }
  if (my_ptiles > 0 && tid < 32) bp = sl.bp2[member * 32 + tid];
  tile_to_lds(h0, a.Hpad, a.Hpad, 0, std::false_type{});
  v4i Wf[KS];
  // 1 KB per wave load, all in flight together before the first is pinned to its place
  auto ask_operands = [&](const int4 *src, int n, auto &w) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) w[ks] = *reinterpret_cast<const v4i *>(src + (size_t)(ks < n ? ks : 0) * 64);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto pin_operands = [&](auto &w) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(w[ks]));
    __builtin_amdgcn_sched_barrier(0);
  };
  ask_operands(sl.R2 + (size_t)(member * WAVES + wave) * KS * 64 + lane, KS, Wf);
  
  {
    auto dma = [&](const void *src, const void *dst) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                       (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
    };
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      if (i == 2 && share_tanh) continue;
      const int nd = lw[i].dom >> 10;
      const int nb = (((lw[i].dom >> lw[i].sh) * 2) + 1023) >> 10;
      const int nt = lw[i].tail ? 3 : 0;
      for (int c = wave; c < nd + nb + nt; c += WAVES) {
        const int so = c < nd ? c * 1024 : (c < nd + nb ? kLutWideBaseOff + (c - nd) * 1024 : kLutWideTailOff + (c - nd - nb) * 1024);
        dma(lw[i].blob + so + lane * 16, lutD[i] + c * 1024);
      }
    }
    const int prow = a.prow;
    const int wp_rows = my_ptiles * prow;
    const int wp_chunks = (wp_rows * WLS + 1023) >> 10;
    for (int c = wave; c < wp_chunks; c += WAVES) {
      const int o = c * 1024 + lane * 16;
      const int r = o / WLS, col_b = o - r * WLS;
      const int8_t *src = sl.Wp2;
      if (r < wp_rows && col_b < a.npadp) {
        const int pt = r / prow;
        src = sl.Wp2 + ((size_t)(member + pt * GS) * 32 + (r - pt * prow)) * a.npadp + col_b;
      }
      dma(src, WpL + c * 1024);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  const int cell_w = wave * 8 + 4 * b2;  // + c, within the workgroup's 64 cells
  if (tid < 256) {
    LdL[tid] = ln ? ln_weight_scaled(Lq) : 0.0;
    bdL[tid] = ln ? ln_bias_scaled(qb) : 0.0;
    PqL[tid] = Pq;
    bhL[tid] = bh;
    bxL[tid] = bx;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)  // (indexed by the thread these would be loads that return behind the others)
    if (tid == i) {
      prm->h[i] = rescale_hi_prepare(sl.Mh[i], sl.rh[i]);
      prm->x[i] = rescale_hi_prepare(sl.Mx[i], sl.rx[i]);
      prm->c[i] = rescale_hi_prepare(i < 3 && ph ? sl.Mc[i < 3 ? i : 0] : 0, i < 3 && ph ? sl.rc[i < 3 ? i : 0] : 33);
      prm->ln[i] = rescale_hi_prepare(sl.Mln[i], ln ? sl.rln[i] : 33);
    }
#pragma unroll
  for (int i = 0; i < 3; ++i)  // (indexed by the thread these arrays would lie in scratch memory)
    if (tid == i) {
      LutLds d;
      d.dom = i == 2 && share_tanh ? lw[1].dom : lw[i].dom;  // a shared copy has the gate table's prefix
      d.sh = i == 2 && share_tanh ? lw[1].sh : lw[i].sh;
      d.offD = (int32_t)(lutD[i] - lds);
      d.offB = (int32_t)(lutB[i] - lds);
      d.offT = lutTl[i] ? (int32_t)(lutTl[i] - lds) : 0;
      d.pad[0] = d.pad[1] = d.pad[2] = 0;
      lutP[i] = d;
    }
  if (tid == 0) {
    prm->m = rescale_hi_prepare(sl.Mm, sl.rm);
    prm->p = rescale_hi_prepare(proj ? sl.Mp : 0, proj ? sl.rp : 33);
    prm->zp_m = sl.zp_m; prm->zp_h = sl.zp_h;
    prm->inv_n = 1.0 / (double)a.N;
    prm->m_c = sl.m_c; prm->glo = ln ? -32767 : -32768;
  }
  if (my_ptiles > 0 && tid < 32) bpL[tid] = bp;
  if (tid < items) red[tid] = 0;
  if (tid < 12) tickL[tid] = 0;
  if (tid == 0) {
    flag[0] = 1;
    flag[1] = 0;
  }
  pin_operands(Wf);  // the rows of h came ahead of them
  if (!ONE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_barrier();

  // optional phase timing (diagnostics): workgroup 0 of one layer, 100 MHz wall clock ticks per phase
  long long tick_last = 0;
  const bool timing = a.ticks && layer == sa.tick_layer && member == 0 && wave == 0;  // uniform
#define TICK(i)                                                                           \
  do {                                                                                    \
    if (timing) {                                                                         \
      asm volatile("" ::: "memory");                                                      \
      const long long now = (long long)wall_clock64();                                    \
      if (lane == 0)                                                                      \
        __hip_atomic_fetch_add(&tickL[i], (u64)(now - tick_last), __ATOMIC_RELAXED,       \
                               __HIP_MEMORY_SCOPE_WORKGROUP);                             \
      tick_last = now;                                                                    \
    }                                                                                     \
  } while (0)
  if (timing) tick_last = (long long)wall_clock64();

  unsigned epoch = 0;
  unsigned *counter = a.counters + layer * 64;
  u64 *accS = a.acc + (size_t)layer * kStatGroupWords;  // [set][round][S1|S2][item]
  // The layer's counter and statistics words were cleared by another kernel: a first access would fetch
  // them from memory in the middle of the first step.  Adding zero brings them into this XCD's L2 now,
  // while the layers below are still at work.
  if (tid < items) {
#pragma unroll
    for (int ss = 0; ss < 2; ++ss) {
      u64 *w = accS + ss * kStatSetWords;
      __hip_atomic_fetch_add(&w[0 * 256 + tid], (u64)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&w[1 * 256 + tid], (u64)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (ph) {
        __hip_atomic_fetch_add(&w[2 * 256 + tid], (u64)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_add(&w[3 * 256 + tid], (u64)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  if (tid == 0) __hip_atomic_fetch_add(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t prev1[2] = {0, 0};  // this thread's item, per round: the sums of the statistics words as last read
  u64 prev2[2] = {0, 0};
  const int g_first = cifg ? 1 : 0;
  const bool pre_ln = ln && (sl.rln[0] < 33 || sl.rln[1] < 33 || sl.rln[2] < 33 || sl.rln[3] < 33);
  const bool pre_m = sl.rm < 33;
  constexpr int32_t glo = ln ? -32767 : -32768;
  const int RTILES = sa.row_tiles;
  const int n_items = a.T * RTILES;
  const int pre_h = sl.pre_h, pre_x = sl.pre_x;

  // ONE: the rows of the layer below are polled themselves.  Its words of four outputs hold kMarkFree until they are stored; a
  // value that looks like that is believed when all workgroups that store rows have said, in a word each, that theirs are stored.
  auto poll_input = [&](auto count, int tid) {
    constexpr int U = decltype(count)::value;
    const int per_row = 2 * kx;
    const uint32_t per_piece = (1u << 20) / (uint32_t)per_row + 1;  // c / per_row = c per_piece / 2^20: c < 2048, per_row <= 64
    const int sayers = proj ? (a.ptiles < GS ? a.ptiles : GS) : GS, lane = tid & 63;
    unsigned at[U], to[U];
    v4i w[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int c = k * 512 + tid < 64 * kx ? k * 512 + tid : tid;
      const int r = (int)((uint32_t)c * per_piece >> 20), pc = c - r * per_row;
      at[k] = (unsigned)((r < a.B ? r : a.B - 1) * ldx + pc * 16);
      to[k] = (unsigned)(r * LS + pc * 16);
    }
    int budget = a.spin_limit;
    bool all_said = false;
    for (;;) {
      poll_pairs(reinterpret_cast<const u64 *>(xin), at, w);
      bool open = a.extra_arrivals != 0;  // tests: rows that never come
#pragma unroll
      for (int k = 0; k < U; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) open |= (uint32_t)w[k][i] == kMarkFree;
      if (all_said || __builtin_amdgcn_ballot_w64(open) == 0) break;
      --budget;
      if ((budget & 7) == 0) {
        if (budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
          __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          flag[0] = 0;
          break;
        }
        const unsigned said =
            lane < sayers ? __hip_atomic_load(sa.flags + (layer - 1) * 32 + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 1u;
        all_said = a.extra_arrivals == 0 && __builtin_amdgcn_ballot_w64(said == 0) == 0;
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (k * 512 + tid < 64 * kx) *reinterpret_cast<v4i *>(hT + to[k]) = w[k];
  };

  // ONE: this wave's k steps of m in marked words, as in rec_kernel
  auto poll_m = [&](const int8_t *mrow, unsigned moff, int kmine, v4i (&mv)[8]) {
    unsigned at[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) at[k] = moff + (k < kmine ? k : 0) * 1024;
    int budget = a.spin_limit;
    uint32_t least;
    for (;;) {
      poll_marked(mrow, at, mv);
      least = 0xFFFFFFFFu;
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
          const uint32_t d = (uint32_t)mv[k][i] ^ kMarkFree;
          least = least < d ? least : d;
        }
      if (a.extra_arrivals) least = 0;  // tests: words that nobody writes
      if (__builtin_amdgcn_ballot_w64(least == 0) == 0) break;
      --budget;
      if ((budget & 15) == 0 && (budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
        __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        flag[0] = 0;
        break;
      }
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(least == 1) != 0, 0)) {
      const int8_t *esc = sa.m_escape + (size_t)layer * sa.mbuf_stride + (mrow - mbuf);
#pragma unroll
      for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int i = 0; i < 4; i += 2)
          if ((uint32_t)mv[k][i] == kMarkEscape)
            mv[k][i] = (int)__hip_atomic_load(reinterpret_cast<const uint32_t *>(esc + at[k] + 4 * i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };

  const bool tails = lw[0].tail | lw[1].tail | lw[2].tail;  // some table's LDS copy ends before its flat part
  // this lane's operand row of W_proj; rows beyond a tile's prow outputs re-read row 0: their results are never stored
  const int wp_lane = (col < a.prow ? col : 0) * WLS + (b2 << 4);
  int32_t creg[4] = {0, 0, 0, 0};
  const int tid0 = tid;
  for (int it = 0; it < n_items; ++it) {
    // addresses of a lane are computed anew for every item (see rec_kernel)
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, col = lane & 31, b2 = lane >> 5, cell_w = wave * 8 + 4 * b2;
    const int t = it / RTILES, rtile = it - t * RTILES;
    const int row0 = rtile * 32;
    const int row = row0 + col;

    // ---- cell state of this lane's 4 cells: in registers from step to step when the batch is one row
    // tile, in memory between the items of a row tile otherwise
    if (t == 0 || RTILES > 1) {
      const int n0 = member * 64 + cell_w;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        creg[c] = ((t > 0 || sa.c_given) && row < a.B && n0 + c < a.N) ? cbuf[(size_t)row * a.N + n0 + c] : 0;
    }

    // ---- h^{t-1} rows of the tile -> LDS; R h on the MFMA; kept as packed int16 terms
    if (!ONE && it > 0) {  // the first item's rows are there
      const int8_t *hp = t == 0 ? h0 : out + (size_t)(t - 1) * a.B * a.Hpad;
      tile_to_lds(hp, a.Hpad, a.Hpad, row0, std::false_type{});
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
    TICK(0);
    // The first part of this wave's slice of W (one tile of kx fragments of 1 KB, contiguous) is asked for
    // ahead of its use, one word per 128-byte line, so that it is on its way into the L2 while R h runs and
    // the input is waited for.  Not all of it: a layer's W can be larger than the XCD's L2, and the last
    // lines would push the first out again before they are used (measured on the 8-layer benchmark stack:
    // about half of W ahead is best, all of it is as slow as none).
    constexpr int NPF = (KS * 8 + 63) / 64;
    unsigned pf[NPF];
    {
      const int8_t *w0 = sl.W2f + ((size_t)(member * WAVES + wave) * kx) * 1024;
#pragma unroll
      for (int i = 0; i < NPF; ++i) {
        const int line = lane + 64 * i;
        pf[i] = (line < sa.prefetch_lines && !ONE) ? *reinterpret_cast<const unsigned *>(w0 + (size_t)line * 128) : 0u;
      }
    }
    int32_t thp[8];  // [(4 gate + c) / 2]: low half = even index
    {
      v16i acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = bhL[(v >> 2) * 64 + cell_w + (v & 3)];
      constexpr int DEPTH = 4;
      v4i hf[DEPTH];
      const int8_t *hbase = hT + (size_t)col * LS + (b2 << 4);
#pragma unroll
      for (int ks = 0; ks < DEPTH && ks < KS; ++ks) hf[ks] = *reinterpret_cast<const v4i *>(hbase + ks * 32);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(Wf[ks], hf[ks % DEPTH], acc, 0, 0, 0);
        if (ks + DEPTH < KS) hf[ks % DEPTH] = *reinterpret_cast<const v4i *>(hbase + (ks + DEPTH) * 32);
        __builtin_amdgcn_sched_barrier(0);
      }
      auto pack = [&](auto pre_tag) {
        constexpr int PRE = decltype(pre_tag)::value;
#pragma unroll
        for (int j = 0; j < 8; ++j) thp[j] = stk_requant2<PRE>(acc[2 * j], acc[2 * j + 1], prm->h[(2 * j) >> 2]);
      };
      if (pre_h == 0)
        pack(std::integral_constant<int, 0>{});
      else if (pre_h == 1)
        pack(std::integral_constant<int, 1>{});
      else
        pack(std::integral_constant<int, 2>{});
    }
    // A launch of one item per layer (one step, one row tile -- the streaming call) has no further use for
    // R: W takes its place in the registers while the layers below are still at work, and W x below
    // runs from registers instead of waiting for memory.
    constexpr bool w_resident = ONE;
    if constexpr (w_resident) {  // (beside R, in registers of its own, W spills 12 to 240 bytes a lane: 136 us for the call below instead of 101)
      ask_operands(reinterpret_cast<const int4 *>(sl.W2f + ((size_t)(member * WAVES + wave) * kx) * 1024) + lane, kx, Wf);
      pin_operands(Wf);
    }
    TICK(1);

    // ---- W x^t: weights streamed from memory as MFMA operands, DW k steps ahead
    constexpr int DW = 6;
    v4i wq[DW];
    const int8_t *wbase = sl.W2f + ((size_t)(member * WAVES + wave) * kx) * 1024 + (lane << 4);
    auto wload = [&](int ks) -> v4i { return *reinterpret_cast<const v4i *>(wbase + (size_t)ks * 1024); };
#pragma unroll
    for (int ks = 0; ks < DW && ks < KS; ++ks)
      if (ks < kx && !w_resident) wq[ks] = wload(ks);
    // The input rows: wait until the layer below has finished step t of this row tile.  ONE: until one of its workgroups is
    // at the end of its step; what they hand over is polled itself then.
    if (layer > 0) {
      if (tid == 0) {
        const unsigned *f = ONE ? sa.near_end + (layer - 1) * 32 : sa.flags + ((size_t)(layer - 1) * RTILES + rtile) * 32;
        const unsigned want = (unsigned)(t + 1);
        int budget = a.spin_limit;
        for (;;) {
          const unsigned v = __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if ((int)(v - want) >= 0) break;
          if (--budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            flag[0] = 0;
            break;
          }
          for (int i = 0; i < sa.flag_sleep; ++i) __builtin_amdgcn_s_sleep(1);
        }
      }
    }
    __syncthreads();  // also: every wave has read its h fragments, the tile can be overwritten
    if (flag[0] == 0) return;
    TICK(2);
    if (ONE && layer > 0) {
      const int mine = (64 * kx - wave * 64 + 511) >> 9;  // 16-byte pieces of the tile for a thread of this wave
      if (mine >= 4)
        poll_input(std::integral_constant<int, 4>{}, tid);
      else if (mine == 3)
        poll_input(std::integral_constant<int, 3>{}, tid);
      else if (mine == 2)
        poll_input(std::integral_constant<int, 2>{}, tid);
      else if (mine == 1)
        poll_input(std::integral_constant<int, 1>{}, tid);
    } else {
      const int8_t *xp = xin + (size_t)t * a.B * ldx;
      if (x_bypass)
        tile_to_lds(xp, ldx, kx * 32, row0, std::true_type{});
      else
        tile_to_lds(xp, ldx, kx * 32, row0, std::false_type{});
      // the x chunks are the youngest NCH loads of this wave; the weight loads ahead of them are done then too
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
      for (int i = 0; i < NPF; ++i) asm volatile("" ::"v"(pf[i]));  // the prefetched words themselves are not used
    }
    if (ONE) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // tables and W_proj tiles, of waves that polled nothing too
    __syncthreads();
    if (ONE && flag[0] == 0) return;
    TICK(3);
    v16i acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = bxL[wave * 32 + (v >> 2) * 8 + 4 * b2 + (v & 3)];
    {
      constexpr int DEPTH = 4;
      v4i xf[DEPTH];
      const int8_t *xbase = hT + (size_t)col * LS + (b2 << 4);
#pragma unroll
      for (int ks = 0; ks < DEPTH && ks < KS; ++ks) xf[ks] = *reinterpret_cast<const v4i *>(xbase + ks * 32);
      __builtin_amdgcn_sched_barrier(0);
      if (w_resident) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          if (ks < kx) {  // uniform
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(Wf[ks], xf[ks % DEPTH], acc, 0, 0, 0);
            if (ks + DEPTH < KS) xf[ks % DEPTH] = *reinterpret_cast<const v4i *>(xbase + (ks + DEPTH) * 32);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          if (ks < kx) {  // uniform
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wq[ks % DW], xf[ks % DEPTH], acc, 0, 0, 0);
            if (ks + DW < KS && ks + DW < kx) wq[ks % DW] = wload(ks + DW);
            if (ks + DEPTH < KS) xf[ks % DEPTH] = *reinterpret_cast<const v4i *>(xbase + (ks + DEPTH) * 32);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }

    TICK(4);
    // ---- gate sums (Secs. 3.2.4/3.2.5) and layer-norm partial statistics
    auto gate_sums = [&](auto pre_tag) {
      constexpr int PRE = decltype(pre_tag)::value;
      int32_t s1[4] = {0, 0, 0, 0};
      uint32_t s2[4] = {0, 0, 0, 0};  // four squares of 16-bit values fit 32 bits
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const RescaleHi pg = prm->x[g];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int idx = g * 4 + c;
          const int32_t tx = rescale_sat16_pre<PRE>(acc[idx], pg);
          const int32_t w = thp[idx >> 1];
          const int32_t th = (idx & 1) ? (w >> 16) : (int32_t)(int16_t)(w & 0xFFFF);
          int32_t v = tx + th;
          if (ph && g < 2) v += rescale_sat16_pre(mul_i24(PqL[g * 64 + cell_w + c], creg[c]), prm->c[g]);
          if (!(ph && g == 3)) v = clamp_i32(v, glo, 32767);
          acc[idx] = v;
          s1[g] += v;
          s2[g] += (uint32_t)v * (uint32_t)v;
        }
      }
      if (ln) {
#pragma unroll
        for (int g = 0; g < (ph ? 3 : 4); ++g) {
          const int64_t pk = ((int64_t)(u64)s2[g] << 24) + s1[g];
          __hip_atomic_fetch_add(&red[g * 32 + col], (u64)pk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    };
    if (pre_x == 0)
      gate_sums(std::integral_constant<int, 0>{});
    else if (pre_x == 1)
      gate_sums(std::integral_constant<int, 1>{});
    else
      gate_sums(std::integral_constant<int, 2>{});

    // statistics exchange among the layer's workgroups: rec_kernel's words (never reset, the top byte
    // counts the adds); `it` counts the exchanges of this launch
    constexpr u64 kValMask = ((u64)1 << 56) - 1;
    auto publish_stats = [&](int round, int g_lo, int g_hi) {
      __syncthreads();
      if (tid < items) {
        const int g = (tid >> 5) & 3;
        if (g >= g_lo && g <= g_hi) {
          const int64_t pk = (int64_t)red[tid];
          red[tid] = 0;
          const int64_t v1 = ((pk + (1 << 23)) & 0xFFFFFF) - (1 << 23);
          const int64_t v2 = (pk - v1) >> 24;
          u64 *mine = accS + (stat_two_sets(GS) ? (member & 1) : 0) * kStatSetWords;  // this workgroup's set of words
          __hip_atomic_fetch_add(&mine[(round * 2 + 0) * 256 + tid], ((u64)1 << 56) + (u64)(v1 + (1 << 22)),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_fetch_add(&mine[(round * 2 + 1) * 256 + tid], ((u64)1 << 56) + (u64)v2, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    };
    auto collect_stats = [&](int round, int g_lo, int g_hi) -> bool {
      if (tid < items) {
        const int g = (tid >> 5) & 3;
        if (g >= g_lo && g <= g_hi) {
          // two sets: set 0 holds the adds of the even members, set 1 those of the odd ones
          const bool two = stat_two_sets(GS);
          const unsigned n0 = two ? ((unsigned)GS + 1) >> 1 : (unsigned)GS, n1 = two ? (unsigned)GS >> 1 : 0u;
          const u64 expect0 = (u64)((n0 * (unsigned)(it + 1)) & 0xFFu), expect1 = (u64)((n1 * (unsigned)(it + 1)) & 0xFFu);
          u64 c1[2], c2[2];
          int budget = a.spin_limit;
          for (int i = 0; i < a.stats_first_sleep; ++i) __builtin_amdgcn_s_sleep(1);
          for (;;) {
            c1[0] = __hip_atomic_load(&accS[(round * 2 + 0) * 256 + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            c2[0] = __hip_atomic_load(&accS[(round * 2 + 1) * 256 + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            c1[1] = c2[1] = 0;  // one set: the second set's words are never added to, nor read
            if (two) {
              c1[1] = __hip_atomic_load(&accS[kStatSetWords + (round * 2 + 0) * 256 + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              c2[1] = __hip_atomic_load(&accS[kStatSetWords + (round * 2 + 1) * 256 + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if ((c1[0] >> 56) == expect0 && (c2[0] >> 56) == expect0 && (c1[1] >> 56) == expect1 && (c2[1] >> 56) == expect1) break;
            if (--budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
              __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              *flag = 0;
              break;
            }
            for (int i = 0; i < a.stats_sleep; ++i) __builtin_amdgcn_s_sleep(1);
          }
          // the sets' value fields together, less those of the step before; a step adds less than 2^29 and 2^42
          const uint32_t now1 = (uint32_t)c1[0] + (uint32_t)c1[1];
          const u64 now2 = (c2[0] + c2[1]) & kValMask;
          const int64_t S1 = (int64_t)(now1 - prev1[round]) - (int64_t)GS * (1 << 22);
          const int64_t S2 = (int64_t)((now2 - prev2[round]) & kValMask);
          prev1[round] = now1;
          prev2[round] = now2;
          int n = a.N;
          asm volatile("" : "+s"(n));  // its conversions to double are made here, not kept
          lnrow[tid] = ln_row2(S1, S2, n, prm->inv_n);
        }
      }
      __syncthreads();
      return *flag != 0;
    };
    TICK(5);
    if (ONE && !proj && !last_layer && member == 0 && tid == 0)
      __hip_atomic_store(sa.near_end + layer * 32, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ln) {
      publish_stats(0, g_first, ph ? 2 : 3);
      if (!collect_stats(0, g_first, ph ? 2 : 3)) return;
    }
    TICK(6);

    // ---- layer norm, sigma/tanh, cell update (Secs. 3.2.6, 3.2.1, 3.2.9, 3.2.7)
    constexpr int LNB = ONE ? 2 : 1;  // gates per batch of reads: with the operands of W x on their way there is room for one
    auto normalize = [&](int gmask, const LnRow2 (&lr)[4], int32_t (&xv)[4][4], bool narrow, auto sat_tag) {
      constexpr bool SAT = decltype(sat_tag)::value;  // false: the lookup that follows clamps the magnitude anyway
      if (ln) {
#pragma unroll
        for (int gp = 0; gp < 4; gp += LNB) {  // LNB gates per batch of reads: 8 LNB doubles in flight
          if (!(gmask >> gp & ((1 << LNB) - 1))) continue;
          double wL[LNB][4], wb[LNB][4];
          RescaleHi pl[LNB];
#pragma unroll
          for (int g = gp; g < gp + LNB; ++g)
            if (gmask >> g & 1) {
              pl[g - gp] = prm->ln[g];
#pragma unroll
              for (int c = 0; c < 4; ++c) {
                wL[g - gp][c] = LdL[g * 64 + cell_w + c];
                wb[g - gp][c] = bdL[g * 64 + cell_w + c];
              }
            }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int g = gp; g < gp + LNB; ++g)
            if (gmask >> g & 1)
#pragma unroll
              for (int c = 0; c < 4; ++c)
                xv[g][c] = narrow ? ln_second_stage_narrow(acc[g * 4 + c], lr[g], wL[g - gp][c], wb[g - gp][c])
                                  : ln_second_stage(acc[g * 4 + c], lr[g], wL[g - gp][c], wb[g - gp][c]);
          if (pre_ln) {  // some second-stage shift is below 33 (uniform; rare)
#pragma unroll
            for (int g = gp; g < gp + LNB; ++g)
              if (gmask >> g & 1)
#pragma unroll
                for (int c = 0; c < 4; ++c) xv[g][c] = rescale_preshift(xv[g][c], pl[g - gp]);
          }
#pragma unroll
          for (int g = gp; g < gp + LNB; ++g)
            if (gmask >> g & 1)
#pragma unroll
              for (int c = 0; c < 4; ++c) xv[g][c] = SAT ? rescale_sat16_pre<0>(xv[g][c], pl[g - gp]) : rescale_hi_pre(xv[g][c], pl[g - gp]);
        }
      } else {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if (gmask >> g & 1)
#pragma unroll
            for (int c = 0; c < 4; ++c) xv[g][c] = acc[g * 4 + c];
      }
    };
    // table values of |xv[g][c]| for the gates of gmask; tb[g] = which table (0 sigma, 1 tanh, 2 cell tanh)
    auto lookup = [&](int gmask, const int32_t (&xv)[4][4], const int (&tb)[4], int32_t (&tv)[4][4], auto tails_tag) {
      constexpr bool TAILS = decltype(tails_tag)::value;
      int32_t mag[4][4];
      uint32_t base[4][4], delta[4][4];
      int32_t top[3] = {0, 0, 0};  // largest |x| looked up in each table
      // the tables' places and sizes come from LDS (the same words for every lane)
      LutLds lp[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        bool used = false;
#pragma unroll
        for (int g = 0; g < 4; ++g) used = used || ((gmask >> g & 1) && tb[g] == i);
        if (used) lp[i] = lutP[i];
      }
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (gmask >> g & 1) {
          const int dom = lp[tb[g]].dom, sh = lp[tb[g]].sh;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            mag[g][c] = abs_masked(xv[g][c]);  // at most 2^15
            if (TAILS) top[tb[g]] = top[tb[g]] > mag[g][c] ? top[tb[g]] : mag[g][c];
            const int32_t ai = mag[g][c] < dom ? mag[g][c] : dom - 1;
            base[g][c] = *reinterpret_cast<const uint16_t *>(lds + lp[tb[g]].offB + 2 * (ai >> sh));
            delta[g][c] = lds[lp[tb[g]].offD + ai];
          }
        }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (gmask >> g & 1)
#pragma unroll
          for (int c = 0; c < 4; ++c) tv[g][c] = (int32_t)(base[g][c] + delta[g][c]);
      if (!TAILS) return;
      bool over = false;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        bool used = false;
#pragma unroll
        for (int g = 0; g < 4; ++g) used = used || ((gmask >> g & 1) && tb[g] == i);
        if (used) over |= top[i] >= lp[i].dom;
      }
      if (__builtin_amdgcn_ballot_w64(over) != 0) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if ((gmask >> g & 1) && lp[tb[g]].offT) {
            const int dom = lp[tb[g]].dom;
            const bool og = mag[g][0] >= dom || mag[g][1] >= dom || mag[g][2] >= dom || mag[g][3] >= dom;
            if (__builtin_amdgcn_ballot_w64(og) != 0) {
#pragma unroll
              for (int c = 0; c < 4; ++c)
                if (mag[g][c] >= dom) tv[g][c] = lut_wide_tail(lds + lp[tb[g]].offT, mag[g][c]);
            }
          }
      }
    };
    const int gate_tb[4] = {0, 0, 1, 0};
    constexpr int gates_now = (cifg ? 0 : 1) | 2 | 4 | (ph ? 0 : 8);
    int32_t xo[4];
    const int32_t m_c = prm->m_c;
    {
      LnRow2 lr[4];
      bool narrow = false;  // uniform: every row of this wave has sigma >= 2^12 (see rec_kernel)
      if (ln) {
        bool wide = false;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          lr[g] = lnrow[g * 32 + col];
          if (gates_now >> g & 1) wide |= !ln_row_is_narrow(lr[g]);
        }
        narrow = __builtin_amdgcn_ballot_w64(wide) == 0;
      }
      int32_t xv[4][4], tv[4][4];
      if ((!ln || narrow) && !tails) {
        normalize(gates_now, lr, xv, true, std::false_type{});
        lookup(gates_now, xv, gate_tb, tv, std::false_type{});
      } else {
        asm volatile("");  // keeps what both forms begin with from being computed ahead of them, for all gates at once
        if (narrow) {
          normalize(gates_now, lr, xv, true, std::true_type{});
        } else {
          asm volatile("");
          normalize(gates_now, lr, xv, false, std::true_type{});
        }
        lookup(gates_now & 3, xv, gate_tb, tv, std::true_type{});  // two gates' reads at a time: the rarer form, and the larger
        lookup(gates_now & 12, xv, gate_tb, tv, std::true_type{});
      }
      int32_t s1 = 0;
      int64_t s2 = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        xo[c] = ph ? 0 : mirror_sigmoid_masked(xv[3][c], tv[3][c]);
        const int32_t f = mirror_sigmoid_masked(xv[1][c], tv[1][c]);
        const int32_t i = cifg ? cifg_input_gate(f) : mirror_sigmoid_masked(xv[0][c], tv[0][c]);
        const int32_t cnew = cell_update32(i, mirror_tanh_masked(xv[2][c], tv[2][c]), f, creg[c], m_c);
        creg[c] = cnew;
        if (ph) {  // finish the o gate sum with P_o . c^t (eq. 5)
          int32_t v = acc[12 + c] + rescale_sat16_pre(mul_i24(PqL[2 * 64 + cell_w + c], cnew), prm->c[2]);
          v = clamp_i32(v, glo, 32767);
          acc[12 + c] = v;
          s1 += v;
          s2 += (int64_t)v * v;
        }
      }
      if (ph && ln) {
        const int64_t pk = (s2 << 24) + s1;
        __hip_atomic_fetch_add(&red[3 * 32 + col], (u64)pk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    // the new cell state goes back to memory: read again by this thread at the tile's next step, or, after
    // the last step, the state the caller gets back
    if (RTILES > 1 || t == a.T - 1) {
      const int n0 = member * 64 + cell_w;
      if (row < a.B && n0 < a.N)
#pragma unroll
        for (int c = 0; c < 4; ++c) cbuf[(size_t)row * a.N + n0 + c] = (int16_t)creg[c];
    }
    TICK(7);
    if (ph && ln) {
      publish_stats(1, 3, 3);
      if (!collect_stats(1, 3, 3)) return;
    }

    // ---- hidden state (Sec. 3.2.7)
    int32_t tc[4];
    {
      const int hid_tb[4] = {2, 0, 0, 0};  // c^t, then the o gate sums
      LnRow2 lr[4];
      if (ph && ln) lr[3] = lnrow[3 * 32 + col];
      int32_t xv[4][4], tv[4][4], ov[4][4];
#pragma unroll
      for (int c = 0; c < 4; ++c) xv[0][c] = creg[c];
      if (ph) {
        normalize(8, lr, ov, false, std::true_type{});
#pragma unroll
        for (int c = 0; c < 4; ++c) xv[1][c] = ov[3][c];
      }
      if (tails) {
        asm volatile("");
        lookup(ph ? 3 : 1, xv, hid_tb, tv, std::true_type{});
      } else {
        lookup(ph ? 3 : 1, xv, hid_tb, tv, std::false_type{});
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        tc[c] = mirror_tanh_masked(xv[0][c], tv[0][c]);
        if (ph) xo[c] = mirror_sigmoid_masked(xv[1][c], tv[1][c]);
      }
    }
    // Without a projection m is the layer output h: it goes to [T, B, Hpad] with stores that write through
    // the L2 (the next layer's XCD reads it).  With one it goes to the exchange buffer of this XCD.
    int8_t *mdst = proj ? mbuf + (size_t)t * a.Bp * a.npadp : out + (size_t)t * a.B * a.Hpad;
    const RescaleHi pm = prm->m;
    const int32_t zp_m = prm->zp_m;
    const bool final_step = t == a.T - 1;
    {
      const int n0 = member * 64 + cell_w;
      uint32_t pk = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        int32_t om = mul_i24(xo[c], tc[c]);
        if (pre_m) om = rescale_preshift(om, pm);
        const int32_t mq = sat8(rescale_sat16_pre<0>(om, pm) + zp_m);
        pk |= (uint32_t)(mq & 0xFF) << (8 * c);
      }
      if (ONE && proj) {  // marked words as in rec_kernel, rows beyond the batch too
        const auto both = __builtin_amdgcn_permlane32_swap(pk, pk, false, false);
        uint32_t lo = both[0];
        if (b2 == 0) {
          const unsigned off = (member * 2 + (wave >> 2)) * 1024 + col * 32 + (wave & 3) * 8;
          if (__builtin_expect((lo ^ kMarkFree) < 2, 0)) {
            *reinterpret_cast<uint32_t *>(sa.m_escape + (size_t)layer * sa.mbuf_stride + off) = lo;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lo = kMarkEscape;
          }
          *reinterpret_cast<v2i *>(mbuf + off) = v2i{(int)lo, (int)both[1]};
        }
      } else if (row < a.B && n0 < a.N) {
        if (proj) {
          const size_t off = (((size_t)(row >> 5) * (a.npadp >> 5) + (n0 >> 5)) * 32 + (row & 31)) * 32 + (n0 & 31);
          *reinterpret_cast<uint32_t *>(mdst + off) = pk;
        } else {
          __hip_atomic_store(reinterpret_cast<uint32_t *>(mdst + (size_t)row * a.Hpad + n0), pk, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
          if (yout)
            __builtin_nontemporal_store(pk, reinterpret_cast<uint32_t *>(yout + ((size_t)t * a.B + row) * a.H + n0));
          if (final_step && hfin) *reinterpret_cast<uint32_t *>(hfin + (size_t)row * a.H + n0) = pk;
        }
      }
    }
    TICK(8);
    if (ONE && proj && !last_layer && member == 0 && tid == 0)
      __hip_atomic_store(sa.near_end + layer * 32, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (ONE && proj && !ln) __syncthreads();  // every wave is past W x: the partial sums may lie in the tile
    if (!ONE && !group_sync(counter, epoch, GS + a.extra_arrivals, a.status, a.spin_limit, a.sync_sleep, a.poll_sleep, flag)) return;
    TICK(9);

    // ---- projection (Sec. 3.2.8)
    if (proj) {
      const int ksteps = a.npadp >> 5;     // 32-wide k steps, a multiple of 4, at most 64 (N <= 2048)
      const int per_wave = (ksteps + 7) >> 3;
      const int kfirst = wave * per_wave;  // the last waves may have fewer, or none
      const int kend = ONE ? 2 * GS : ksteps;  // ONE: k steps that somebody writes
      const int kmine = kend - kfirst < per_wave ? kend - kfirst : per_wave;  // uniform
      for (int pt = 0; pt < my_ptiles; ++pt) {
        const int ptile = member + pt * GS;
        const int8_t *wrow = WpL + wp_lane + pt * a.prow * WLS + kfirst * 32;
        const int8_t *mrow = mbuf + (size_t)t * a.Bp * a.npadp + ((size_t)(row0 >> 5) * ksteps + kfirst) * 1024;
        const unsigned moff = col * 32 + b2 * 16;
        v4i mv[8];
        v16i pacc;
#pragma unroll
        for (int v = 0; v < 16; ++v) pacc[v] = 0;
        if (ONE && kmine > 0) poll_m(mrow, moff, kmine, mv);
        if (kmine == 8) {  // straight, as in rec_kernel (8 layers of 2048 cells, 32 rows, one step 110.6 -> 107.7 us)
          if (!ONE)
#pragma unroll
            for (int k = 0; k < 8; ++k) mv[k] = *reinterpret_cast<const v4i *>(mrow + moff + k * 1024);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int k = 0; k < 8; ++k)
            pacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i *>(wrow + k * 32), mv[k], pacc, 0, 0, 0);
        } else {
          if (!ONE)
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (k < kmine) mv[k] = *reinterpret_cast<const v4i *>(mrow + moff + k * 1024);
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (k < kmine)
              pacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i *>(wrow + k * 32), mv[k], pacc, 0, 0, 0);
        }
        // partial sums through LDS and two outputs per thread, as in rec_kernel
        const int own = ((wave & (four_slots ? 3 : 7)) << 8) + lane;
        if (!four_slots || wave >= 4)
#pragma unroll
          for (int q = 0; q < 4; ++q) pred[own + q * 64] = v4i{pacc[4 * q], pacc[4 * q + 1], pacc[4 * q + 2], pacc[4 * q + 3]};
        __syncthreads();
        if (four_slots) {
          if (wave < 4)
#pragma unroll
            for (int q = 0; q < 4; ++q) pred[own + q * 64] += v4i{pacc[4 * q], pacc[4 * q + 1], pacc[4 * q + 2], pacc[4 * q + 3]};
          __syncthreads();
        }
        if (4 * wave < a.prow) {
          const int pl = 4 * wave + 2 * b2;
          const v2i *mine = reinterpret_cast<const v2i *>(pred) + (wave << 6) + 2 * col + b2;
          v2i sum = (mine[0] + mine[512]) + (mine[1024] + mine[1536]);
          if (!four_slots) sum += (mine[2048] + mine[2560]) + (mine[3072] + mine[3584]);
          const RescaleHi pp = prm->p;
          const int32_t zp_h = prm->zp_h;
          const int p0 = ptile * a.prow + pl;
          uint32_t hq[2];
#pragma unroll
          for (int c = 0; c < 2; ++c)
            hq[c] = (uint32_t)(sat8(rescale_sat16_pre(sum[c] + (pt == 0 ? bpL[pl + c] : sl.bp2[ptile * 32 + pl + c]), pp) + zp_h) & 0xFF);
          const size_t orow0 = (size_t)t * a.B + row0;
          int8_t *od = out + orow0 * a.Hpad + ptile * a.prow + (unsigned)(col * a.Hpad + pl);
          // an output past H falls into the padding of the row (and only ever meets zero weights)
          if (ONE) {  // whole words, which the layer above polls
            const uint32_t pk = hq[0] | hq[1] << 8;
            const auto both = __builtin_amdgcn_permlane32_swap(pk, pk, false, false);
            if (b2 == 0 && row < a.B && p0 < a.H)
              __hip_atomic_store(reinterpret_cast<uint32_t *>(od), both[0] | both[1] << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          if (row < a.B && p0 < a.H) {
            if (!ONE) __hip_atomic_store(reinterpret_cast<uint16_t *>(od), (uint16_t)(hq[0] | hq[1] << 8), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (yout) {
              int8_t *yd = yout + orow0 * a.H + ptile * a.prow + (unsigned)(col * a.H + pl);
              yd[0] = (int8_t)hq[0];
              if (p0 + 1 < a.H) yd[1] = (int8_t)hq[1];
            }
            if (final_step && hfin) {
              int8_t *hd = hfin + (size_t)row * a.H + p0;
              hd[0] = (int8_t)hq[0];
              if (p0 + 1 < a.H) hd[1] = (int8_t)hq[1];
            }
          }
        }
        // the last tile's partial sums are overwritten behind the group barrier only, or not at all
        if (pt + 1 < my_ptiles) __syncthreads();
      }
      TICK(10);
      if (!ONE && !group_sync(counter, epoch, GS + a.extra_arrivals, a.status, a.spin_limit, my_ptiles == 0 ? a.idle_sleep : 0,
                              my_ptiles == 0 ? a.idle_poll_sleep : a.poll_sleep, flag))
        return;
      TICK(11);
    }
    // The stores of step t are acknowledged, those of the whole layer (the barrier above), or, ONE, of this workgroup: tell
    // the layer above
    if (ONE) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
    }
    if (!last_layer && (ONE || member == 0) && tid == 0)
      __hip_atomic_store(sa.flags + ((size_t)layer * RTILES + rtile) * 32 + member, (unsigned)(t + 1), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }
#undef TICK
  if (timing && lane == 0)
    for (int i = 0; i < 12; ++i) a.ticks[i] += (long long)tickL[i];
  placement_check();
}

typedef void (*stack_fn)(StackArgs);

}  // namespace lstm_int

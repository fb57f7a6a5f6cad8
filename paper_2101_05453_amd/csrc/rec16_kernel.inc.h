// Persistent recurrent kernel for small batches: groups of 16 batch rows on
// the 16x16x64 int8 MFMA (rec_kernel.inc.h has the design; this is the same
// step with half the rows per workgroup, so that 128 rows already fill the
// chip and a workgroup's arithmetic per step is half as long).  FL: bit 0 CIFG,
// bit 1 peephole, bit 2 layer norm; the projection is a runtime flag.
//
// Eight waves, two to a block of 16 cells.  Lane (r = lane % 16, q = lane / 16)
// of wave w = 2 b + s owns batch row r of the group and cells 16 b + 4 q + 2 s + c,
// c = 0, 1, of the workgroup's 64, all four gates: weight tile j of the block
// holds, in row 4 q' + gate, cell 16 b + 4 q' + j, so that result value `gate` of
// the wave's tile c in that lane is (cell 4 q + 2 s + c, gate).  The W x terms are
// read in the layout the input GEMM writes for the 32-row kernel.
//
// The hidden state travels as (value, tag) byte pairs, the tag being the step (kTaggedState, quad_kernel.inc.h has more on it):
// 16 bytes a thread hold eight cells, and who needs them polls them, up to four loads a thread.  Through the layer output, the
// group's counter and a load of the tile behind it -> this, 200 steps, us:
//   1024 cells, 128 rows  788 -> 606, layer norm 1127 -> 908       512 cells, 200 rows  653 -> 510, layer norm 971 -> 774
//   two directions of 512 cells, 100 rows, 100 steps 364 -> 271    512 cells, 256 outputs, layer norm, 200 rows 1382 -> 1158
//   2048 cells, 640 outputs, 128 rows 1168 -> 999, layer norm 1592 -> 1396, and peephole 1868 -> 1653; 160 outputs, layer norm 1577 -> 1314
// With a projection m goes in marked words then (below).  It went through the exchange buffer and the group's counter before (every
// wave's stores acknowledged, one add per workgroup, polls, a load of the tile); 100 steps, us: 2048 cells, 640 outputs, 128 rows 504 ->
// 451, layer norm 726 -> 667, and peephole 849 -> 788; 160 outputs, layer norm 682 -> 617; 1088 cells, 320 outputs, layer norm, 100
// rows 659 -> 598; 512 cells, 256 outputs, layer norm, 200 rows 588 -> 544.  A pause ahead of the first poll of m only adds to the step (4 x
// 64 clocks: 0.1 us), and so do pauses of the workgroups without outputs between their polls of the state, from 8 x 64 clocks on.
// The counter remains where one workgroup is the group, and where the words of all groups find no room.  Either way is a form of its
// own (FORM): with both in one kernel, chosen by a test in the step loop, the registers that each keeps for itself spilled (12 to
// 80 bytes a lane at 2048 cells with layer norm, three times the scalar ones everywhere), and the same calls took 632, 950, 533, 847,
// 277, 1253, 1158, 1544, 1792 and 1958 us, the ones through the counter up to 25 % longer than alone.
//
// What bounds it: the exchanges of a step (two, one without a projection, and one
// per round of statistics, 0.6 to 1.2 us each) and the instructions between them.
// Two waves per SIMD issue those in less time than one of twice the work: 128 rows
// of 2048 cells, projection to 640: 6.3 -> 5.9 us a step, with layer norm 8.3 -> 8.1,
// and peephole 9.4 -> 9.2; 512 cells, 200 rows 3.1 -> 2.9, with layer norm 4.8 -> 4.6
// (before the tagged words).  Machine LICM off, which the deepest k needed with both ways in one kernel, makes it 1 to 2 % slower.
#pragma once

#include "rec_kernel.inc.h"

namespace lstm_int {

// 100 MHz wall clock ticks per phase, summed in LDS by thread 0 of workgroup 0
#define TICK(i)                                                                           \
  do {                                                                                    \
    if (timing) {                                                                         \
      asm volatile("" ::: "memory");                                                      \
      const long long now = (long long)wall_clock64();                                    \
      __hip_atomic_fetch_add(&tickL[i], (u64)(now - tick_last), __ATOMIC_RELAXED,         \
                             __HIP_MEMORY_SCOPE_WORKGROUP);                               \
      tick_last = now;                                                                    \
    }                                                                                     \
  } while (0)

__device__ __forceinline__ const RecArgs &rec16_args(const RecArgs &a, int) { return a; }
__device__ __forceinline__ const RecDirArgs &rec16_args(const RecArgs2 &a, int i) { return a.d[i]; }
__device__ __forceinline__ int rec16_ldy(const RecArgs &a) { return a.H; }
__device__ __forceinline__ int rec16_ldy(const RecDirArgs &a) { return a.ldy; }
__device__ __forceinline__ int rec16_rev(const RecArgs &) { return 0; }
__device__ __forceinline__ int rec16_rev(const RecDirArgs &a) { return a.rev; }

// PAIR: the launch runs two layers of one shape side by side, each possibly backward in time (RecArgs2).
// FORM: 0 = the state through the counter; 1, 2 = in tagged words, without and with a projection; 3 = as 2, and the statistics in a word
// of each member (rec16_form).  A form of its own for that too: as a test in the step loop it cost the others 1 to 5 %.
template <int KS16, int FL, bool PAIR, int FORM>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void rec16_kernel(
    std::conditional_t<PAIR, RecArgs2, RecArgs> args) {
  constexpr bool cifg = FL & 1, ph = FL & 2, ln = FL & 4;
  constexpr int TAG = FORM == 3 ? 2 : FORM;
  constexpr bool member_words = FORM == 3;
  const long long t_start = (long long)wall_clock64();
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x;
  int lane = tid & 63;
  const int wave = KS16 > 10 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  int r = lane & 15, q = lane >> 4;
  constexpr int g_first = cifg ? 1 : 0;
  const auto &a0 = rec16_args(args, 0);
  const int GS = a0.GS;

  // placement, as in rec_kernel
  const int wg = blockIdx.x;
  const int xcc = (int)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7);
  const int slot = wg >> 3;
  // both layers of the launch depend on where its workgroups are
  auto misplaced = [&]() {
    __hip_atomic_store(a0.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (PAIR) __hip_atomic_store(other_status<RecArgs2>(), 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  int xcd = wg & 7;
  if (a0.tickets) {
    xcd = xcc;
  } else if (xcc != xcd && GS > 1 && tid == 0) {
    misplaced();
  }
  auto placement_check = [&]() {
    if (a0.tickets && tid == 0) {
      const int xcc_now = (int)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7);
      const unsigned places = gridDim.x >> 3;  // at most 32
      const u64 mine = ((u64)1 << 32) + ((u64)1 << (wg >> 3));
      const u64 now =
          __hip_atomic_fetch_add(&a0.tickets[xcc_now * 32], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine;
      const unsigned count = (unsigned)(now >> 32);
      const unsigned all = places >= 32 ? 0xFFFFFFFFu : (1u << places) - 1;
      if (count > places || (count == places && (unsigned)now != all)) misplaced();
    }
  };
  const int gl = xcd + 8 * (slot / GS), member = slot % GS;  // group of the launch
  if (gl >= a0.groups + (PAIR ? rec16_args(args, 1).groups : 0)) {
    placement_check();
    return;
  }
  const int which = PAIR && gl >= a0.groups ? 1 : 0;
  const auto &a = rec16_args(args, which);
  const int group = gl - (which ? a0.groups : 0);
  const bool proj = TAG == 0 ? (a.flags & 8) != 0 : TAG == 2;
  const int ldy = rec16_ldy(a);
  // time of step t
  auto time_of = [&](int t) { return rec16_rev(a) ? a.T - 1 - t : t; };
  constexpr int items = 64;                    // (gate, row) layer-norm rows of the group
  const int row0 = a.batch0 + group * 16;      // first batch row of the group
  constexpr int CPL = 2;                       // cells of a lane: whatever runs over them counts to this
  int cellw = (wave >> 1) * 16 + 4 * q + CPL * (wave & 1);  // + c, within the workgroup's 64 cells

  // ---- LDS carve-up (rec16_lds_bytes mirrors it)
  constexpr int LS = KS16 * 64 + 16;  // h tile row stride: LS / 4 = 4 * odd (mod 64), reads are conflict-free
  constexpr int TILE_KB = (16 * LS + 1023) / 1024;
  // m or h of a step leaves through LDS, by one wave in stores of 16 bytes a lane, which are acknowledged 0.25 us before those
  // of two bytes a lane from all waves.  Behind a second round of statistics the barrier that takes costs more: 2048 cells
  // with peephole and layer norm 9.2 -> 9.5 us a step (marked words come in whole pieces of eight cells, and no other barrier follows).
  constexpr bool GATHER = !(ph && ln) || TAG == 2;
  uint8_t *p = lds;
  int8_t *hT = reinterpret_cast<int8_t *>(p);
  // hidden state of the step on its way out, where the loads past the h tile go, which nobody reads: 16-byte pieces of row r
  // at r * 64, exchanged by r / 4 so that rows in the same banks differ.  With neither layer norm nor a projection two of them by
  // turns: no barrier lies between the barrier behind which wave 1 reads it once more (store_output) and the next hidden state.
  constexpr int mflip = TAG == 1 && !ln ? 1024 : 0;
  // In marked words (below) wave 0 reads m there while other waves may have their partial sums of the projection already: with layer
  // norm, whose barriers lie between R h and m, it is where wave 0's own sums go, else where the statistics would be.  Whoever has a
  // word of the step's hidden state knows that m has been read.
  constexpr int kPredBytes = 8 * 2 * 64 * 16, kTileBytes = (TILE_KB + 1) * 1024 + mflip;  // one spare chunk for the loads past the tile
  constexpr int kScratch = TAG == 2 && kTileBytes < kPredBytes ? kPredBytes : kTileBytes;
  static_assert(sizeof(LnRow2) * items >= 1024);
  int8_t *const mS0 = reinterpret_cast<int8_t *>(lds) + (TAG != 2 ? TILE_KB * 1024 : ln ? 0 : kScratch + items * 8);
  auto mS_of = [&](int t) { return mS0 + (t & 1) * mflip; };
  auto piece_at = [](int row, int piece) { return row * 64 + ((piece ^ (row >> 2)) << 4); };
  v4i *pred = reinterpret_cast<v4i *>(p);  // projection partials [8 waves][2 halves][64 lanes] reuse the h tile between steps
  {
    const int pred_bytes = proj ? kPredBytes : 0;
    p += kTileBytes > pred_bytes ? kTileBytes : pred_bytes;
  }
  u64 *red = reinterpret_cast<u64 *>(p);                 p += (size_t)items * 8;  // [item] sums
  LnRow2 *lnrow = reinterpret_cast<LnRow2 *>(p);         p += (size_t)items * sizeof(LnRow2);
  double *LdL = reinterpret_cast<double *>(p);           p += 4 * 64 * 8;
  double *bdL = reinterpret_cast<double *>(p);           p += 4 * 64 * 8;
  int32_t *bhL = reinterpret_cast<int32_t *>(p);         p += 4 * 64 * 4;
  int16_t *PqL = reinterpret_cast<int16_t *>(p);         p += 4 * 64 * 2;  // 3 used
  PrmLds *prm = reinterpret_cast<PrmLds *>(p);           p += sizeof(PrmLds);
  int *flag = reinterpret_cast<int *>(p);                p += 16;
  u64 *tickL = reinterpret_cast<u64 *>(p);               p += 16 * 8;  // phase timers
  LutLds *lutP = reinterpret_cast<LutLds *>(p);          p += 3 * sizeof(LutLds);
  // the activation tables as in rec_kernel: prefixes of the wide form, chosen by the launch
  const bool share_tanh = a.lut[2].blob == a.lut[1].blob;
  const uint8_t *lutD[3];
  const uint8_t *lutB[3];
  const uint8_t *lutTl[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (i == 2 && share_tanh) {
      lutD[2] = lutD[1]; lutB[2] = lutB[1]; lutTl[2] = lutTl[1];
    } else {
      const int nb = ((((a.lut[i].dom >> a.lut[i].sh) * 2) + 1023) >> 10) << 10;
      lutD[i] = p;                               p += a.lut[i].dom;
      lutB[i] = p;                               p += nb;
      lutTl[i] = a.lut[i].tail ? p : nullptr;    p += a.lut[i].tail ? 3072 : 0;
    }
  }
  int8_t *WpL = reinterpret_cast<int8_t *>(p);
  const int WLS = a.npadp + 16;  // W_proj tile row stride in LDS
  const int my_ptiles = proj ? (a.ptiles > member ? (a.ptiles - member + GS - 1) / GS : 0) : 0;

  // ---- one-time loads: R slice -> registers, per-cell parameters, tables and W_proj tiles -> LDS
  // the loads into LDS go first: they need no registers and are in flight while the R slice arrives
  {
    auto dma = [&](const void *src, const void *dst) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                       (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
    };
    for (int i = 0; i < (share_tanh ? 2 : 3); ++i) {
      const int nd = a.lut[i].dom >> 10;
      const int nb = (((a.lut[i].dom >> a.lut[i].sh) * 2) + 1023) >> 10;
      const int nt = a.lut[i].tail ? 3 : 0;
      for (int c = wave; c < nd + nb + nt; c += 8) {
        const int so = c < nd ? c * 1024 : (c < nd + nb ? kLutWideBaseOff + (c - nd) * 1024 : kLutWideTailOff + (c - nd - nb) * 1024);
        dma(a.lut[i].blob + so + lane * 16, lutD[i] + c * 1024);
      }
    }
    if (tid < 3) {
      LutLds d;
      d.dom = a.lut[tid].dom; d.sh = a.lut[tid].sh;
      d.offD = (int32_t)(lutD[tid] - lds);
      d.offB = (int32_t)(lutB[tid] - lds);
      d.offT = lutTl[tid] ? (int32_t)(lutTl[tid] - lds) : 0;
      d.pad[0] = d.pad[1] = d.pad[2] = 0;
      lutP[tid] = d;
    }
    const int wp_rows = my_ptiles * 32;
    const int wp_chunks = (wp_rows * WLS + 1023) >> 10;
    for (int c = wave; c < wp_chunks; c += 8) {
      const int o = c * 1024 + lane * 16;
      const int rr = o / WLS, col_b = o - rr * WLS;
      const int8_t *src = a.Wp2;
      if (rr < wp_rows && col_b < a.npadp) {
        const int pt = rr >> 5;
        src = a.Wp2 + ((size_t)(member + pt * GS) * 32 + (rr & 31)) * a.npadp + col_b;
      }
      dma(src, WpL + c * 1024);
    }
  }
  v4i Wf[CPL][KS16];
  {
    const int4 *src = a.R2h + ((size_t)(member * 4 + (wave >> 1)) * 4 + CPL * (wave & 1)) * KS16 * 64 + lane;
    // all loads of the slice are issued before the first value is pinned (a pin waits for its load);
    // at the deepest k the staging registers do not hold both tiles
    constexpr int TB = KS16 <= 10 ? CPL : 1;
#pragma unroll
    for (int j0 = 0; j0 < CPL; j0 += TB) {
      int4 w[TB][KS16];
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) w[j][ks] = src[(size_t)((j0 + j) * KS16 + ks) * 64];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
          Wf[j0 + j][ks] = v4i{w[j][ks].x, w[j][ks].y, w[j][ks].z, w[j][ks].w};
          asm volatile("" : "+a"(Wf[j0 + j][ks]));  // resident in accumulation registers for the whole launch
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (tid < 256) {
    const int g = tid >> 6, n = tid & 63;  // 4 gates x 64 cells
    const size_t idx = (size_t)g * a.Ncp + member * 64 + n;
    LdL[tid] = ln_weight_scaled(a.Lq4[idx]);
    bdL[tid] = ln_bias_scaled(a.qb4[idx]);
    bhL[tid] = a.bh4[idx];
    PqL[tid] = (ph && g < 3) ? a.Pq3[idx] : 0;
  }
  if (tid < 4) {
    prm->h[tid] = rescale_hi_prepare(a.Mh[tid], a.rh[tid]);
    prm->c[tid] = rescale_hi_prepare(tid < 3 && ph ? a.Mc[tid] : 0, tid < 3 && ph ? a.rc[tid] : 33);
    prm->ln[tid] = rescale_hi_prepare(a.Mln[tid], a.rln[tid]);
  }
  if (tid == 0) {
    prm->m = rescale_hi_prepare(a.Mm, a.rm);
    prm->p = rescale_hi_prepare(proj ? a.Mp : 0, proj ? a.rp : 33);
    prm->zp_m = a.zp_m; prm->zp_h = a.zp_h;
    prm->m_c = a.m_c; prm->glo = -32767;
  }
  for (int i = tid; i < 16 * LS / 16; i += 512) reinterpret_cast<int4 *>(hT)[i] = int4{0, 0, 0, 0};

  // cell state of this lane's cells of its row, kept in registers
  int row = row0 + r;
  int n0 = member * 64 + cellw;
  int32_t creg[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c)
    creg[c] = (a.c_in && row < a.B && n0 + c < a.N) ? a.c_in[(size_t)row * a.N + n0 + c] : 0;

  // h tile staging: wave instruction (wave + 8 j) fills bytes [1024 c, 1024 (c + 1)) of the tile
  constexpr int NCH = (TILE_KB + 7) / 8;
  int hsrc[NCH];
#pragma unroll
  for (int j = 0; j < NCH; ++j) {
    const int o = (wave + 8 * j) * 1024 + lane * 16;
    const int rr = o / LS, c = o - rr * LS;
    int rw = row0 + rr;
    rw = rw < a.B ? rw : a.B - 1;
    hsrc[j] = (rr < 16 && c < a.Hpad) ? rw * a.Hpad + c : 0;
  }
  auto load_tile = [&](const int8_t *hp) {
#pragma unroll
    for (int j = 0; j < NCH; ++j)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void *)(hp + hsrc[j]),
          (__attribute__((address_space(3))) void *)(lds + (wave + 8 * j < TILE_KB ? wave + 8 * j : TILE_KB) * 1024),
          16, 0, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };

  // projection: thread (ct = tid / 64 < 2, lane) finishes outputs 16 ct + 4 q + 0..3 of row r
  int32_t bpr[4] = {0, 0, 0, 0};
  if (my_ptiles > 0 && tid < 128) {
    const int4 b4 = *reinterpret_cast<const int4 *>(a.bp2 + member * 32 + 16 * wave + 4 * q);
    bpr[0] = b4.x; bpr[1] = b4.y; bpr[2] = b4.z; bpr[3] = b4.w;
  }
  if (tid == 0) {
    flag[0] = 1;
    flag[1] = 0;
  }
  if (tid < 16) tickL[tid] = 0;
  if (tid < items) red[tid] = 0;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // tables and W_proj tiles are in LDS
  __syncthreads();

  unsigned epoch = 0;
  unsigned *counter = a.counters + gl * 64;
  // one set of words: two sets (as in rec_kernel) made this kernel 2-3 % slower, at 8 and at 32 workgroups per group
  constexpr bool tagged = TAG != 0;
  const int Hr = tagged_row(a.H);                    // cells of a row of the exchange
  // statistics: [round][S1|S2][item], item < 64, or [step % 2][round][item][member]
  constexpr int stat_words = member_words ? kMemberStatWords : kStatGroupWords;
  u64 *accS = a.acc + (size_t)gl * (stat_words + (tagged ? tagged_group_words(a.H, 16) : 0));
  u64 *const xh = accS + stat_words;                 // [2 slots][16 rows][Hr] (value, tag)
  const unsigned never = a.extra_arrivals ? 0x80u : 0;  // tests: a tag nobody stores in so few steps
  int64_t prevS[2][2] = {{0, 0}, {0, 0}};       // this thread's item, per round: S1, S2
  const double inv_n = 1.0 / (double)a.N;
  const bool pre_ln = a.rln[0] < 33 || a.rln[1] < 33 || a.rln[2] < 33 || a.rln[3] < 33;
  const bool pre_m = a.rm < 33;
  constexpr u64 kValMask = ((u64)1 << 56) - 1;

  // optional phase timing of workgroup 0 (diagnostics), phases numbered as in rec_kernel
  long long tick_last = 0;
  const bool timing = a.ticks && wg == 0 && tid == 0;
  if (timing) {
    tick_last = t_start;
    __hip_atomic_store(&a.ticks[15], t_start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  TICK(10);  // everything before the first step

  // this lane's W x terms of step t, a pair of cells of each gate in a word, read in the layout of the 32-row kernel:
  // cell tile of 8 = 2 (wave / 2) + q / 2, lane there = row % 32 + 32 * (q % 2), whose two pieces hold gates 0, 1 and 2, 3
  // of four cells
  int32_t txn[4];
  auto tx_request = [&](int t) {
    if (PAIR) t = time_of(t < a.T ? t : a.T - 1);
    size_t rb = ((size_t)t * a.Bp + row0) >> 5;
    const size_t rbmax = ((size_t)a.T * a.Bp) >> 5;
    rb = rb < rbmax ? rb : rbmax - 1;
    const int32_t *src = reinterpret_cast<const int32_t *>(
        a.tx2 + ((rb * (size_t)(GS * 8) + member * 8 + (wave >> 1) * 2 + (q >> 1)) * 2) * 64 + ((row0 + r) & 31) + 32 * (q & 1)) + (wave & 1);
    // read once: streaming loads keep the W x terms from displacing the exchange buffers in L2
#pragma unroll
    for (int g = 0; g < 4; ++g) txn[g] = __builtin_nontemporal_load(src + (g >> 1) * 256 + (g & 1) * 2);
  };
  tx_request(0);
  if (tagged) load_tile(a.h0);

  // The state of a step in words of (value, tag) pairs, the tag being the step: a thread polls the pieces of eight cells it
  // needs until all carry the tag, U of them at a time, and puts them into the tile.  No acknowledgement, no counter, no load
  // after the barrier.
  const int row_pieces = Hr >> 3;
  const uint32_t per_piece = (1u << 20) / (uint32_t)row_pieces + 1;  // c / row_pieces = c per_piece / 2^20: c < 16 row_pieces, row_pieces <= 128
  auto poll_state = [&](auto count, int t) {
    constexpr int U = decltype(count)::value;
    const uint32_t want = (((unsigned)t + 1) & 0xFF ^ never) * 0x01000100u;
    const u64 *src = xh + (size_t)(t & 1) * Hr * 4;
    unsigned at[U];
    v4i w[U];
#pragma unroll
    for (int k = 0; k < U; ++k) at[k] = k * 512 + tid < 16 * row_pieces ? (unsigned)(k * 512 + tid) * 16 : 0;
    int budget = a.spin_limit;
    for (;;) {
      poll_pairs(src, at, w);
      uint32_t off = 0;
#pragma unroll
      for (int k = 0; k < U; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) off |= (uint32_t)w[k][i] ^ want;
      if (__builtin_amdgcn_ballot_w64((off & 0xFF00FF00u) != 0) == 0) break;
      --budget;
      if ((budget & 15) == 0 && (budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
        __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        flag[0] = 0;
        break;
      }
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int c = k * 512 + tid;
      if (c < 16 * row_pieces) {
        const int rr = (int)((uint32_t)c * per_piece >> 20);
        *reinterpret_cast<v2i *>(hT + rr * LS + 8 * (c - rr * row_pieces)) =
            v2i{(int)__builtin_amdgcn_perm((uint32_t)w[k][1], (uint32_t)w[k][0], 0x06040200u),
                (int)__builtin_amdgcn_perm((uint32_t)w[k][3], (uint32_t)w[k][2], 0x06040200u)};
      }
    }
  };
  // m in marked words (TAG == 2), as in rec_kernel: 64 bits of eight cells whose low half is kMarkFree are not written yet; four slots
  // of [row / 16][k step of 64 cells = member][row % 16][64 cells] that take turns, and one for what looks like a mark.
  auto m_word = [&](int t) -> int8_t * {  // wave 0: the 16 cells of a row that this lane stores
    return a.mbuf + (size_t)(t & 3) * a.Bp * a.npadp + (((size_t)(row0 >> 4) * (a.npadp >> 6) + member) << 10) + lane * 16;
  };
  // Tagged state: the layer output of step t, which nobody waits for, behind the polls of the next step
  uint32_t hkeep = 0;
  auto store_output = [&](int t) {
    if (proj) {
      const int p0 = member * 32 + 16 * wave + 4 * q;
      if (my_ptiles > 0 && wave < 2 && row < a.B && p0 < a.H) {
        const size_t orow = (size_t)time_of(t) * a.B + row;
        int8_t *od = a.out + orow * a.Hpad + p0;
        if (p0 + 3 < a.H) {
          *reinterpret_cast<uint32_t *>(od) = hkeep;
        } else {
          for (int c = 0; c < 4 && p0 + c < a.H; ++c) od[c] = (int8_t)(hkeep >> (8 * c));
        }
        if (a.y) {
          int8_t *yd = a.y + orow * ldy + p0;
          for (int c = 0; c < 4 && p0 + c < a.H; ++c) yd[c] = (int8_t)(hkeep >> (8 * c));
        }
      }
    } else if (GATHER && wave == 1) {
      const int srow = row0 + (lane >> 2), n = member * 64 + 16 * (lane & 3);
      const v4i piece = *reinterpret_cast<const v4i *>(mS_of(t) + piece_at(lane >> 2, lane & 3));
      if (srow < a.B && n < a.N) {
        const size_t orow = (size_t)time_of(t) * a.B + srow;
        *reinterpret_cast<v4i *>(a.out + orow * a.Hpad + n) = piece;
        if (a.y) {  // N a multiple of four, y of four bytes
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (n + 4 * k < a.N) __builtin_nontemporal_store(piece[k], reinterpret_cast<int32_t *>(a.y + orow * ldy + n + 4 * k));
        }
      }
    }
  };

  for (int t = 0; t < a.T; ++t) {
    if (KS16 > 10) {  // half of the registers are weights: what follows from the lane is worked out in every step
      asm volatile("" : "+v"(lane));
      r = lane & 15;
      q = lane >> 4;
      cellw = (wave >> 1) * 16 + 4 * q + 2 * (wave & 1);
      row = row0 + r;
      n0 = member * 64 + cellw;
    }
    // ---- h^{t-1} rows of the group -> LDS
    if (tagged) {
      // pieces of this wave: a wave without any does not poll, its loads would cost as much as the others'
      // 32 KB a poll: a first one too early delays the arrivals (1024 cells, 120 rows, 60 steps 196 -> 189 us, layer norm 291 -> 285)
      if (TAG == 1 && KS16 > 10 && GATHER && t > 0) __builtin_amdgcn_s_sleep(3);
      const int mine = t > 0 ? (16 * row_pieces - wave * 64 + 511) >> 9 : 0;
      if (mine >= 4)
        poll_state(std::integral_constant<int, 4>{}, t - 1);
      else if (mine == 3)
        poll_state(std::integral_constant<int, 3>{}, t - 1);
      else if (mine == 2)
        poll_state(std::integral_constant<int, 2>{}, t - 1);
      else if (mine == 1)
        poll_state(std::integral_constant<int, 1>{}, t - 1);
    } else {
      load_tile(t == 0 ? a.h0 : a.out + (size_t)time_of(t - 1) * a.B * a.Hpad);
    }
    __syncthreads();
    if (tagged && t > 0) {
      if (flag[0] == 0) return;
      store_output(t - 1);
      // everyone's h of step t - 1 is here, so everyone has read m of that step: the words that this lane wrote are marked as not
      // written, for step t + 3
      if (TAG == 2 && t + 3 < a.T && wave == 0) *reinterpret_cast<v4i *>(m_word(t - 1)) = v4i{} + (int)kMarkFree;
    }
    // the W x terms of this step were requested one step ahead (they come from HBM)
    const int32_t txw[4] = {txn[0], txn[1], txn[2], txn[3]};
    TICK(0);

    // ---- R h on the MFMA: acc[j][gate] for the lane's cell j; each tile's k loop runs to its end
    // before the next tile starts (dependent 16x16x64 MFMAs issue back to back, rotating
    // accumulators do not)
    v4i acc[CPL];
    RescaleHi ph4[4];  // the R h rescale constants, read here so that the MFMAs cover the LDS round trip
#pragma unroll
    for (int g = 0; g < 4; ++g) ph4[g] = prm->h[g];
    {
      constexpr int KC = KS16 <= 10 ? KS16 : KS16 / 2;  // k steps at a time: the deepest k leaves no registers for all
      const int8_t *hbase = hT + (size_t)r * LS + (q << 4);
#pragma unroll
      for (int j = 0; j < CPL; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) acc[j][g] = bhL[g * 64 + cellw + j];
#pragma unroll
      for (int k0 = 0; k0 < KS16; k0 += KC) {
        v4i hf[KC];
#pragma unroll
        for (int ks = 0; ks < KC; ++ks) hf[ks] = *reinterpret_cast<const v4i *>(hbase + (k0 + ks) * 64);
#pragma unroll
        for (int j = 0; j < CPL; ++j)
#pragma unroll
          for (int ks = 0; ks < KC; ++ks)
            acc[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(Wf[j][k0 + ks], hf[ks], acc[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }

    TICK(1);

    // ---- gate sums (Secs. 3.2.4/3.2.5) and layer-norm partial statistics.
    // With a peephole the o gate keeps tx + th here and is finished after c^t.
    constexpr int32_t glo = ln ? -32767 : -32768;  // layer norm takes symmetric gate sums
    int32_t gs[4][CPL];  // [gate][cell]
    auto gate_sums = [&](auto pre_tag) {
      constexpr int PRE = decltype(pre_tag)::value;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const RescaleHi pg = ph4[g];
        int32_t s1 = 0;
        uint32_t s2 = 0;  // squares of 16-bit values
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const int32_t th = rescale_sat16_pre<PRE>(acc[c][g], pg);
          const int32_t tx = c ? (txw[g] >> 16) : (int32_t)(int16_t)(txw[g] & 0xFFFF);
          int32_t v = tx + th;
          if (ph && g < 2) v += rescale_sat16_pre(mul_i24(PqL[g * 64 + cellw + c], creg[c]), prm->c[g]);
          if (!(ph && g == 3)) v = clamp_i32(v, glo, 32767);
          gs[g][c] = v;
          s1 += v;
          s2 += (uint32_t)v * (uint32_t)v;
        }
        if (ln && !(ph && g == 3)) {
          // the 32 lanes of a row (4 per wave) add into one LDS word: no cross-lane traffic, no wait
          const int64_t pk = ((int64_t)(u64)s2 << 24) + s1;
          __hip_atomic_fetch_add(&red[g * 16 + r], (u64)pk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    };
    if (a.pre_h == 0)
      gate_sums(std::integral_constant<int, 0>{});
    else if (a.pre_h == 1)
      gate_sums(std::integral_constant<int, 1>{});
    else
      gate_sums(std::integral_constant<int, 2>{});
    // Statistics over the group's workgroups; item = 16 gate + row: as in rec_kernel (words that are never reset, the top byte counts
    // the adds), or (FORM 3) a word of each member per item, its sum of squares, its sum and a tag of six bits.  A wave polls those of
    // eight items, two members per lane: no add waits for another at the L2, and nothing has to be subtracted.  128 rows, 640 outputs,
    // layer norm, 100 steps, adds -> words: 2048 cells 667 -> 640 us, with a peephole 781 -> 762.  In small groups the adds are ahead: 1088 cells,
    // 320 outputs, 60 steps 347 against 354, 1024 cells without a projection 470 against 484, 512 cells, 256 rows 402 against 420.  (Two slots by
    // turns: who stores step t + 2 has all words of step t + 1, whose writers had those of step t.)
    auto publish_stats = [&](int round, int g_lo, int g_hi) {
      __syncthreads();
      if (tid < items) {
        const int g = tid >> 4;
        if (g >= g_lo && g <= g_hi) {
          const int64_t pk = (int64_t)red[tid];
          red[tid] = 0;  // the next adds to this word come after the next barrier
          const int64_t v1 = ((pk + (1 << 23)) & 0xFFFFFF) - (1 << 23);
          const int64_t v2 = (pk - v1) >> 24;
          if (member_words)
            __hip_atomic_store(&accS[(((t & 1) * 2 + round) * 64 + tid) * 32 + member],
                               (u64)(v1 + (1 << 21)) | (u64)v2 << 22 | (u64)((t + 1) & 63) << 58, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          else {
            __hip_atomic_fetch_add(&accS[(round * 2 + 0) * 256 + tid], ((u64)1 << 56) + (u64)(v1 + (1 << 22)),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(&accS[(round * 2 + 1) * 256 + tid], ((u64)1 << 56) + (u64)v2, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
    };
    auto poll_stats = [&](int round) {
      int l = lane;
      asm volatile("" : "+v"(l));
      const int sub = l & 15, it = l >> 4;  // members 2 sub, 2 sub + 1 of items 8 wave + it and, in the second load, + 4
      const uint32_t want = (((unsigned)t + 1) << 26) ^ (never << 24);
      const uint32_t m0 = 2 * sub < GS ? 0xFC000000u : 0, m1 = 2 * sub + 1 < GS ? 0xFC000000u : 0;
      unsigned at[2];
      v4i w[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) at[k] = ((((t & 1) * 2 + round) * 64 + wave * 8 + it + 4 * k) * 16 + sub) * 16;
      int budget = a.spin_limit;
      for (int i = 0; i < a.stats_first_sleep; ++i) __builtin_amdgcn_s_sleep(1);
      for (;;) {
        poll_pairs(accS, at, w);
        uint32_t off = 0;
#pragma unroll
        for (int k = 0; k < 2; ++k) off |= (((uint32_t)w[k][1] ^ want) & m0) | (((uint32_t)w[k][3] ^ want) & m1);
        if (__builtin_amdgcn_ballot_w64(off != 0) == 0) break;
        --budget;
        if ((budget & 15) == 0 && (budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
          __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          *flag = 0;
          break;
        }
        for (int i = 0; i < a.stats_sleep; ++i) __builtin_amdgcn_s_sleep(1);
      }
      // the sum, and the sum of squares in 20 and 16 bits; words of members that are not there are zero
      uint32_t s[2][3];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint32_t lo0 = (uint32_t)w[k][0], hi0 = (uint32_t)w[k][1], lo1 = (uint32_t)w[k][2], hi1 = (uint32_t)w[k][3];
        s[k][0] = (lo0 & 0x3FFFFFu) + (lo1 & 0x3FFFFFu);
        s[k][1] = (__builtin_amdgcn_alignbit(hi0, lo0, 22) & 0xFFFFFu) + (__builtin_amdgcn_alignbit(hi1, lo1, 22) & 0xFFFFFu);
        s[k][2] = ((hi0 >> 10) & 0xFFFFu) + ((hi1 >> 10) & 0xFFFFu);
      }
      auto add_lanes = [&](auto ctrl) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int i = 0; i < 3; ++i)
            s[k][i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)s[k][i], decltype(ctrl)::value, 0xF, 0xF, false);
      };
      add_lanes(std::integral_constant<int, 0xB1>{});   // lane ^ 1
      add_lanes(std::integral_constant<int, 0x4E>{});   // lane ^ 2
      add_lanes(std::integral_constant<int, 0x141>{});  // the other four of eight
      add_lanes(std::integral_constant<int, 0x140>{});  // the other eight of sixteen
      const int k = sub >> 3;
      const uint32_t sum = k ? s[1][0] : s[0][0], lo = k ? s[1][1] : s[0][1], hi = k ? s[1][2] : s[0][2];
      if ((sub & 7) == 0)
        lnrow[wave * 8 + it + 4 * k] = ln_row2((int64_t)sum - (int64_t)GS * (1 << 21), (int64_t)lo + ((int64_t)hi << 20), a.N, inv_n);
    };
    // false: a wait gave up (status word raised), every thread leaves the kernel
    auto collect_stats = [&](int round, int g_lo, int g_hi) -> bool {
      if (member_words) {
        if ((wave >> 1) >= g_lo && (wave >> 1) <= g_hi) poll_stats(round);
      } else if (tid < items) {
        const int g = tid >> 4;
        if (g >= g_lo && g <= g_hi) {
          const u64 expect = (u64)(((unsigned)GS * (unsigned)(t + 1)) & 0xFFu);
          u64 c1, c2;
          int budget = a.spin_limit;
          for (int i = 0; i < a.stats_first_sleep; ++i) __builtin_amdgcn_s_sleep(1);
          for (;;) {
            c1 = __hip_atomic_load(&accS[(round * 2 + 0) * 256 + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            c2 = __hip_atomic_load(&accS[(round * 2 + 1) * 256 + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((c1 >> 56) == expect && (c2 >> 56) == expect) break;
            if (--budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
              __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              *flag = 0;
              break;
            }
            for (int i = 0; i < a.stats_sleep; ++i) __builtin_amdgcn_s_sleep(1);
          }
          c1 &= kValMask;
          c2 &= kValMask;
          const int64_t S1 = (int64_t)((c1 - (u64)prevS[round][0]) & kValMask) - (int64_t)GS * (1 << 22);
          const int64_t S2 = (int64_t)((c2 - (u64)prevS[round][1]) & kValMask);
          prevS[round][0] = (int64_t)c1;
          prevS[round][1] = (int64_t)c2;
          lnrow[tid] = ln_row2(S1, S2, a.N, inv_n);
        }
      }
      __syncthreads();
      return *flag != 0;
    };
    TICK(2);
    if (ln) {
      publish_stats(0, g_first, ph ? 2 : 3);
      TICK(3);
      if (!collect_stats(0, g_first, ph ? 2 : 3)) return;
      TICK(4);
    }
    // past the last step: the last block again, unused.  Not ahead of the statistics, whose wait takes 0.5 us longer beside
    // loads from memory.
    tx_request(t + 1);

    // ---- layer norm, sigma/tanh, cell update (Secs. 3.2.6, 3.2.1, 3.2.9, 3.2.7); LDS reads in batches
    // gates of `gmask` (bit g): gate sums -> layer norm -> xv[g][c]
    auto normalize = [&](int gmask, int32_t (&xv)[4][CPL]) {
      if (ln) {
        LnRow2 lr[4];
        bool wide = false;
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if (gmask >> g & 1) {
            lr[g] = lnrow[g * 16 + r];
            wide |= !ln_row_is_narrow(lr[g]);
          }
        // uniform: every row of this wave has sigma >= 2^12, and the second stage needs no int32 clamp
        const bool narrow = __builtin_amdgcn_ballot_w64(wide) == 0;
        auto second_stage = [&](auto narrow_tag) {
#pragma unroll
        for (int gp = 0; gp < 4; gp += 2) {
          if (!(gmask >> gp & 3)) continue;
          double wL[2][CPL], wb[2][CPL];
          RescaleHi pl[2];
#pragma unroll
          for (int g = gp; g < gp + 2; ++g)
            if (gmask >> g & 1) {
              pl[g - gp] = prm->ln[g];
#pragma unroll
              for (int c = 0; c < CPL; ++c) {
                wL[g - gp][c] = LdL[g * 64 + cellw + c];
                wb[g - gp][c] = bdL[g * 64 + cellw + c];
              }
            }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int g = gp; g < gp + 2; ++g)
            if (gmask >> g & 1)
#pragma unroll
              for (int c = 0; c < CPL; ++c) {
                int32_t v = decltype(narrow_tag)::value ? ln_second_stage_narrow(gs[g][c], lr[g], wL[g - gp][c], wb[g - gp][c])
                                                        : ln_second_stage(gs[g][c], lr[g], wL[g - gp][c], wb[g - gp][c]);
                if (pre_ln) v = rescale_preshift(v, pl[g - gp]);
                xv[g][c] = rescale_sat16_pre<0>(v, pl[g - gp]);
              }
        }
        };
        if (narrow)
          second_stage(std::true_type{});
        else
          second_stage(std::false_type{});
      } else {
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if (gmask >> g & 1)
#pragma unroll
            for (int c = 0; c < CPL; ++c) xv[g][c] = gs[g][c];
      }
    };
    // table values of |x[g][c]| for the gates of gmask; tb[g] = which table (0 sigma, 1 tanh, 2 cell tanh);
    // see rec_kernel's lookup
    auto lookup = [&](int gmask, const int32_t (&x)[4][CPL], const int (&tb)[4], int32_t (&out)[4][CPL]) {
      int32_t mag[4][CPL];
      uint32_t base[4][CPL], delta[4][CPL];
      int32_t top[3] = {0, 0, 0};  // largest |x| looked up in each table
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
          for (int c = 0; c < CPL; ++c) {
            mag[g][c] = abs_masked(x[g][c]);
            top[tb[g]] = top[tb[g]] > mag[g][c] ? top[tb[g]] : mag[g][c];
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
          for (int c = 0; c < CPL; ++c) out[g][c] = (int32_t)(base[g][c] + delta[g][c]);
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
            const bool og = mag[g][0] >= dom || mag[g][1] >= dom;
            if (__builtin_amdgcn_ballot_w64(og) != 0) {
#pragma unroll
              for (int c = 0; c < CPL; ++c)
                if (mag[g][c] >= dom) out[g][c] = lut_wide_tail(lds + lp[tb[g]].offT, mag[g][c]);
            }
          }
      }
    };
    constexpr int gates_now = (cifg ? 0 : 1) | 2 | 4 | (ph ? 0 : 8);  // with a peephole the o gate waits for c^t
    int32_t xv[4][CPL], tv[4][CPL];
    normalize(gates_now, xv);
    {
      const int gate_tb[4] = {0, 0, 1, 0};
      lookup(gates_now, xv, gate_tb, tv);
    }
    const int32_t m_c = prm->m_c;
    int32_t xo[CPL];
    int32_t cx[4][CPL];  // slot 0: the new cell state, for its tanh; slot 3: the o gate with a peephole
    {
      int32_t s1 = 0;
      uint32_t s2 = 0;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int32_t fg = mirror_sigmoid_masked(xv[1][c], tv[1][c]);
        const int32_t ig = cifg ? cifg_input_gate(fg) : mirror_sigmoid_masked(xv[0][c], tv[0][c]);
        const int32_t zg = mirror_tanh_masked(xv[2][c], tv[2][c]);
        xo[c] = ph ? 0 : mirror_sigmoid_masked(xv[3][c], tv[3][c]);
        creg[c] = cell_update32(ig, zg, fg, creg[c], m_c);
        cx[0][c] = creg[c];
        if (ph) {  // finish the o gate sum with P_o . c^t (eq. 5)
          int32_t v = gs[3][c] + rescale_sat16_pre(mul_i24(PqL[2 * 64 + cellw + c], creg[c]), prm->c[2]);
          v = clamp_i32(v, glo, 32767);
          gs[3][c] = v;
          s1 += v;
          s2 += (uint32_t)v * (uint32_t)v;
        }
      }
      if (ph && ln) {
        const int64_t pk = ((int64_t)(u64)s2 << 24) + s1;
        __hip_atomic_fetch_add(&red[3 * 16 + r], (u64)pk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    TICK(5);
    // ---- hidden state (Sec. 3.2.7): tanh of the new cell state in its own format (Sec. 3.2.2), and
    // with a peephole the layer norm and sigma of the o gate; the tanh does not wait for the o gate's
    // statistics, so it runs while they travel
    int32_t tcv[4][CPL];
    const int hid_tb[4] = {2, 2, 2, 0};
    if (ph && ln) {
      publish_stats(1, 3, 3);
      lookup(1, cx, hid_tb, tcv);
      if (!collect_stats(1, 3, 3)) return;
    } else {
      lookup(1, cx, hid_tb, tcv);
    }
    if (ph) {
      int32_t ov[4][CPL];
      normalize(8, ov);
#pragma unroll
      for (int c = 0; c < CPL; ++c) cx[3][c] = ov[3][c];
      lookup(8, cx, hid_tb, tcv);
#pragma unroll
      for (int c = 0; c < CPL; ++c) xo[c] = mirror_sigmoid_masked(cx[3][c], tcv[3][c]);
    }
    {
      const RescaleHi pm = prm->m;
      const int32_t zp_m = prm->zp_m;
      uint32_t pk = 0;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        int32_t om = mul_i24(xo[c], mirror_tanh_masked(cx[0][c], tcv[0][c]));
        if (pre_m) om = rescale_preshift(om, pm);
        const int32_t mq = sat8(rescale_sat16_pre<0>(om, pm) + zp_m);
        pk |= (uint32_t)(mq & 0xFF) << (8 * c);
      }
      if constexpr (GATHER) {
        *reinterpret_cast<uint16_t *>(mS_of(t) + piece_at(r, cellw >> 4) + (cellw & 15)) = (uint16_t)pk;
      } else {
        if (tagged && !proj && n0 < Hr) {
          const uint32_t tag = ((unsigned)t + 1) & 0xFF;
          *reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(xh + (size_t)(t & 1) * Hr * 4) + (r * Hr + n0) * 2) =
              __builtin_amdgcn_perm(pk, tag, 0x00050004u);
        }
        if (row < a.B && n0 < a.N) {
          if (proj) {
            // exchange buffer [t][row / 16][k step of 64 cells = member][row % 16][64 cells]: a wave's
            // load of one projection k step is one contiguous KB
            int8_t *mdst = a.mbuf + (size_t)t * a.Bp * a.npadp +
                           ((((size_t)(row >> 4) * (a.npadp >> 6) + member) * 16 + (row & 15)) << 6) + cellw;
            *reinterpret_cast<uint16_t *>(mdst) = (uint16_t)pk;
          } else {
            const size_t orow = (size_t)time_of(t) * a.B + row;
            *reinterpret_cast<uint16_t *>(a.out + orow * a.Hpad + n0) = (uint16_t)pk;
            if (a.y) __builtin_nontemporal_store((uint16_t)pk, reinterpret_cast<uint16_t *>(a.y + orow * ldy + n0));
          }
        }
      }
    }
    if constexpr (GATHER) {
      __syncthreads();
      if (wave == 0) {
        // the group's rows of these 64 cells in one store of 16 bytes a lane; cells past the last are written too, they
        // meet zero weights
        const int srow = row0 + (lane >> 2), n = member * 64 + 16 * (lane & 3);
        const v4i piece = *reinterpret_cast<const v4i *>(mS_of(t) + piece_at(lane >> 2, lane & 3));
        if (tagged && !proj) {
          const uint32_t tag = ((unsigned)t + 1) & 0xFF;
          uint8_t *dst = reinterpret_cast<uint8_t *>(xh + (size_t)(t & 1) * Hr * 4) + ((lane >> 2) * Hr + n) * 2;
#pragma unroll
          for (int k = 0; k < 2; ++k)
            if (n + 8 * k < Hr) {
              v4i w;
#pragma unroll
              for (int i = 0; i < 4; ++i) w[i] = (int)__builtin_amdgcn_perm((uint32_t)piece[2 * k + (i >> 1)], tag, i & 1 ? 0x00070006u : 0x00050004u);
              *reinterpret_cast<v4i *>(dst + 16 * k) = w;
            }
        } else if (TAG == 2) {  // rows beyond the batch too: their words are polled with the others
          int8_t *const to = m_word(t);
          v4i w = piece;
          if (__builtin_expect(((uint32_t)w[0] ^ kMarkFree) < 2 || ((uint32_t)w[2] ^ kMarkFree) < 2, 0)) {
            *reinterpret_cast<v4i *>(to + (size_t)(4 - (t & 3)) * a.Bp * a.npadp) = w;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (((uint32_t)w[0] ^ kMarkFree) < 2) w[0] = (int)kMarkEscape;
            if (((uint32_t)w[2] ^ kMarkFree) < 2) w[2] = (int)kMarkEscape;
          }
          *reinterpret_cast<v4i *>(to) = w;
        } else if (srow < a.B && n < a.N) {
          if (proj) {  // the same exchange buffer
            *reinterpret_cast<v4i *>(a.mbuf + (size_t)t * a.Bp * a.npadp +
                                     (((size_t)(srow >> 4) * (a.npadp >> 6) + member) << 10) + lane * 16) = piece;
          } else {
            const size_t orow = (size_t)time_of(t) * a.B + srow;
            *reinterpret_cast<v4i *>(a.out + orow * a.Hpad + n) = piece;
            if (a.y) {  // N a multiple of four, y of four bytes
#pragma unroll
              for (int k = 0; k < 4; ++k)
                if (n + 4 * k < a.N) __builtin_nontemporal_store(piece[k], reinterpret_cast<int32_t *>(a.y + orow * ldy + n + 4 * k));
            }
          }
        }
      }
    }
    TICK(6);
    if (!tagged && !group_sync(counter, epoch, GS + a.extra_arrivals, a.status, a.spin_limit, a.sync_sleep, a.poll_sleep, flag)) return;
    TICK(7);

    // ---- projection (Sec. 3.2.8): tile pt of 32 outputs as two 16-wide halves, K = N split over the waves
    if (proj) {
      const int ksteps = TAG == 2 ? GS : a.npadp >> 6;  // marked words: k steps that somebody writes
      const int per_wave = (ksteps + 7) >> 3;
      const RescaleHi pp = prm->p;
      const int32_t zp_h = prm->zp_h;
      auto poll_m = [&](int t, v4i (&mv)[4]) {  // the wave's k steps; steps past the end: the last one again
        const int8_t *base = a.mbuf + (size_t)(t & 3) * a.Bp * a.npadp + (((size_t)(row0 >> 4) * (a.npadp >> 6)) << 10);
        unsigned at[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          int kk = wave * per_wave + (k < per_wave ? k : per_wave - 1);
          kk = kk < ksteps ? kk : ksteps - 1;
          at[k] = (unsigned)(kk * 1024 + r * 64 + q * 16);
        }
        int budget = a.spin_limit;
        uint32_t least;
        for (;;) {
          poll_pairs(reinterpret_cast<const u64 *>(base), at, mv);
          least = 0xFFFFFFFFu;
#pragma unroll
          for (int k = 0; k < 4; ++k)
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
          const int8_t *esc = base + (size_t)(4 - (t & 3)) * a.Bp * a.npadp;
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < 4; i += 2)
              if ((uint32_t)mv[k][i] == kMarkEscape)
                mv[k][i] = (int)__hip_atomic_load(reinterpret_cast<const uint32_t *>(esc + at[k] + 4 * i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      };
      for (int pt = 0; pt < my_ptiles; ++pt) {
        const int ptile = member + pt * GS;
        v4i pacc[2] = {v4i{0, 0, 0, 0}, v4i{0, 0, 0, 0}};
        const int8_t *mbase = a.mbuf + (size_t)t * a.Bp * a.npadp + (((size_t)(row0 >> 4) * (a.npadp >> 6) * 16 + r) << 6) + (q << 4);
        const int8_t *wbase = WpL + ((size_t)pt * 32 + r) * WLS + (q << 4);
        // all loads of the wave's k steps first (at most 4: N <= 2048); steps past the end re-read the
        // last one against zero weights
        v4i mv[4];
        if constexpr (TAG == 2) {
          poll_m(t, mv);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            int kk = wave * per_wave + (k < per_wave ? k : per_wave - 1);
            kk = kk < ksteps ? kk : ksteps - 1;
            mv[k] = *reinterpret_cast<const v4i *>(mbase + (size_t)kk * 1024);
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          int kk = wave * per_wave + (k < per_wave ? k : per_wave - 1);
          const bool real = k < per_wave && kk < ksteps;
          kk = kk < ksteps ? kk : ksteps - 1;
          const v4i mf = mv[k];
#pragma unroll
          for (int ct = 0; ct < 2; ++ct) {
            v4i wf = *reinterpret_cast<const v4i *>(wbase + (size_t)ct * 16 * WLS + kk * 64);
            if (!real) wf = v4i{0, 0, 0, 0};
            pacc[ct] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wf, mf, pacc[ct], 0, 0, 0);
          }
        }
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) pred[(wave * 2 + ct) * 64 + lane] = pacc[ct];
        __syncthreads();
        if (tid < 128) {
          const int ct = wave;  // threads 0..127: waves 0 and 1
          const int p0 = ptile * 32 + ct * 16 + 4 * q;
          v4i sum = pred[ct * 64 + lane];
#pragma unroll
          for (int w = 1; w < 8; ++w) sum += pred[(w * 2 + ct) * 64 + lane];
          uint32_t pk = 0;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int32_t s = sum[v] + (pt == 0 ? bpr[v] : a.bp2[p0 + v]);
            const int32_t hq = sat8(rescale_sat16_pre(s, pp) + zp_h);
            pk |= (uint32_t)(hq & 0xFF) << (8 * v);
          }
          if (tagged && p0 < Hr) {
            const uint32_t tag = ((unsigned)t + 1) & 0xFF;
            *reinterpret_cast<v2i *>(reinterpret_cast<uint8_t *>(xh + (size_t)(t & 1) * Hr * 4) + (r * Hr + p0) * 2) =
                v2i{(int)__builtin_amdgcn_perm(pk, tag, 0x00050004u), (int)__builtin_amdgcn_perm(pk, tag, 0x00070006u)};
          }
          if (tagged && pt == 0) {
            hkeep = pk;
          } else if (row < a.B && p0 < a.H) {
            const size_t orow = (size_t)time_of(t) * a.B + row;
            int8_t *od = a.out + orow * a.Hpad + p0;
            if (p0 + 3 < a.H) {
              *reinterpret_cast<uint32_t *>(od) = pk;
            } else {
              for (int c = 0; c < 4 && p0 + c < a.H; ++c) od[c] = (int8_t)(pk >> (8 * c));
            }
            if (a.y) {
              int8_t *yd = a.y + orow * ldy + p0;
              for (int c = 0; c < 4 && p0 + c < a.H; ++c) yd[c] = (int8_t)(pk >> (8 * c));
            }
          }
        }
        __syncthreads();
      }
      TICK(8);
      // Tagged: workgroups without outputs poll the state at once and without a pause.  Late for the next step they hold up its
      // statistics and its m: with the counter's first pause of 64 2048 cells, 640 outputs, layer norm, 40 steps of 40 rows take 381 us,
      // and pauses of 12 between the polls 368, with none 285.
      if (!tagged && !group_sync(counter, epoch, GS + a.extra_arrivals, a.status, a.spin_limit, my_ptiles == 0 ? a.idle_sleep : 0,
                                 my_ptiles == 0 ? a.idle_poll_sleep : a.poll_sleep, flag))
        return;
      TICK(9);
    }
  }
  if (tagged) store_output(a.T - 1);
  if (timing)
    for (int i = 0; i < 11; ++i) a.ticks[i] += (long long)tickL[i];
  if (a.ticks && tid == 0) {
    // spread of the workgroups' lifetimes against workgroup 0's start (maxima over all launches)
    const long long t0 = __hip_atomic_load(&a.ticks[15], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const long long t_end = (long long)wall_clock64();
    if (wg == 0) a.ticks[11] += t_end - t_start;
    __hip_atomic_fetch_max(&a.ticks[12], t_start - t0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_max(&a.ticks[13], t_end - t0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_max(&a.ticks[14], t0 - t_start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  placement_check();
  if (a.c_out && row < a.B && n0 < a.N) {
    int n1 = n0;
    asm volatile("" : "+v"(n1));  // computed here: shared with the prologue it would hold registers through the loop
#pragma unroll
    for (int c = 0; c < CPL; ++c)
      if (n1 + c < a.N) a.c_out[(size_t)row * a.N + n1 + c] = (int16_t)creg[c];
  }
}

#undef TICK

typedef void (*rec16_pair_fn)(RecArgs2);

// kernel for (flags & 7) at k depth KS16
template <int KS16, bool PAIR, int FORM, class Fn>
Fn rec16_pick_tag(int fl) {
  switch (fl & 7) {
    case 0: return rec16_kernel<KS16, 0, PAIR, FORM>;
    case 1: return rec16_kernel<KS16, 1, PAIR, FORM>;
    case 2: return rec16_kernel<KS16, 2, PAIR, FORM>;
    case 3: return rec16_kernel<KS16, 3, PAIR, FORM>;
    case 4: return rec16_kernel<KS16, 4, PAIR, FORM>;
    case 5: return rec16_kernel<KS16, 5, PAIR, FORM>;
    case 6: return rec16_kernel<KS16, 6, PAIR, FORM>;
    default: return rec16_kernel<KS16, 7, PAIR, FORM>;
  }
}
template <int KS16, bool PAIR = false, class Fn = rec_fn>
Fn rec16_pick_ks(int fl, int tag) {
  if (tag == 3) {  // layer norm
    if constexpr (KS16 <= 10 && !PAIR) switch (fl) {
        case 4: return rec16_kernel<KS16, 4, PAIR, 3>;
        case 5: return rec16_kernel<KS16, 5, PAIR, 3>;
        case 6: return rec16_kernel<KS16, 6, PAIR, 3>;
        case 7: return rec16_kernel<KS16, 7, PAIR, 3>;
      }
    return nullptr;
  }
  if (tag == 0) return rec16_pick_tag<KS16, PAIR, 0, Fn>(fl);
  return tag == 1 ? rec16_pick_tag<KS16, PAIR, 1, Fn>(fl) : rec16_pick_tag<KS16, PAIR, 2, Fn>(fl);
}

}  // namespace lstm_int

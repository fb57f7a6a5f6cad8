// The GRU's recurrent kernel for groups of 16 or 32 rows (gru_seq.hip has the design), in a file of its own: the two machine
// passes that build.py switches off for it cost gru_quad_kernel 1 to 3 %.
#include "gru_kernel.inc.h"

namespace lstm_int {

namespace {

// ---------------------------------------------------------------------------------------------------------------------
// Two waves per SIMD issue the cell's instructions in less than half of the time that one of twice the work takes (an
// instruction every 2.2 to 4.3 clocks against every 5), but the registers hold the weights once: so the waves are four blocks
// of 16 cells times two halves of the depth, and behind the product a wave hands the sums of two of a lane's four cells to the
// wave of the other half, through 12 KB of LDS and a barrier that is there anyway.  Four waves of the whole depth and four
// cells a lane -> these, 250 steps (us):
//    1024 cells, 128 rows  765 -> 732    2048 cells, 128 rows  1080 -> 1063    333 cells, 333 rows  808 -> 770
//    1024 cells, 512 rows 1370 -> 1264   2048 cells, 256 rows  1574 -> 1502    512 cells, 256 rows  693 -> 680
// Chains of four products of a gate instead of the gates in turn: 1 to 10 % slower; weights in accumulation registers: the same.
template <int KS, int RT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void gru_rows_kernel(GruSeqArgs a) {
  constexpr int R = 16 * RT;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x;
  int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int KW = KS / 2;                      // k steps of a wave
  const int blk = wave & 3, kh = wave >> 2;       // block of 16 cells; half of the depth
  int c16 = lane & 15, q = lane >> 4;
  const int GS = a.GS, N = a.N, T = a.T, ks_n = a.Kp >> 6;  // ks_n = GS
  const GruPlace pl = gru_place(a);
  const int member = pl.member;
  if (pl.group >= a.groups) {
    gru_placement_check(a);
    return;
  }
  const int row0 = a.batch0 + pl.group * R;

  // ---- LDS: the h tile [row tile][k step][64 lanes][16 B], the W x terms of the turns to come, biases, the flag, the tables
  v4i *hT = reinterpret_cast<v4i *>(lds);
  uint8_t *txL = lds + RT * KS * 1024;
  int32_t *bhL = reinterpret_cast<int32_t *>(txL + kGruTxSlots(RT) * kGruTxBytes);  // [3][64]
  v4i *stage = reinterpret_cast<v4i *>(bhL + 192);           // [row tile][64 lanes]: this workgroup's piece of the new state
  v2i *ex = reinterpret_cast<v2i *>(stage + RT * 64);        // [wave][gate][64 lanes]: sums for the wave of the other half
  int *flag = reinterpret_cast<int *>(ex + 8 * 3 * 64);
  int off = (RT * KS * 1024 + kGruTxSlots(RT) * kGruTxBytes + 768 + RT * 1024 + kGruExchange + 16 + 1023) & ~1023;
  const GruLut ls = gru_lut_place(a.lut[0], off), lt = gru_lut_place(a.lut[1], off);
  gru_lut_load<8>(a.lut[0], ls, lds, wave, lane);
  gru_lut_load<8>(a.lut[1], lt, lds, wave, lane);
  if (tid < 192) bhL[tid] = a.bh[(tid >> 6) * 64 * GS + member * 64 + (tid & 63)];

  // W x terms of a row tile's step, turn u = RT t + rt, -> LDS slot u % kGruTxSlots, by waves 2 to 7: the polls of wave 0 and
  // the stores of wave 1 would wait behind them.
  // Tile order: piece ((tile 2 + half) 2 + quad) 16 + row; row-major: piece (row 3 + gate) 8 + j
  const int8_t *tx_src;  // of the first step
  size_t tx_step;
  if (a.tx2) {
    tx_src = reinterpret_cast<const int8_t *>(a.tx2 + ((size_t)(row0 >> 5) * a.tiles + member * 8) * 128);
    tx_step = (size_t)(a.Bp >> 5) * a.tiles * 2048;
  } else {
    tx_src = reinterpret_cast<const int8_t *>(a.tx + (size_t)row0 * 3 * a.Nt);
    tx_step = (size_t)a.B * 3 * a.Nt * 2;
  }
  auto tx_request = [&](int t, int rt) {
    const int8_t *src = tx_src + (size_t)t * tx_step;
    uint8_t *dst = txL + (RT * t + rt) % kGruTxSlots(RT) * kGruTxBytes;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int pc = (wave - 2 + 6 * i) * 64 + lane;
      if (wave < 2 || wave - 2 + 6 * i >= 8) continue;
      unsigned o;
      bool has = true;
      if (a.tx2) {
        const int rr = pc & 15, quad = (pc >> 4) & 1, half = (pc >> 5) & 1, tile = pc >> 6;
        o = (unsigned)(tile * 128 + half * 64 + 32 * quad + ((row0 + 16 * rt) & 31) + rr) * 16;
      } else {
        const int rr = pc / 24, g = (pc >> 3) % 3, n = member * 64 + (pc & 7) * 8, row = 16 * rt + rr;
        o = (unsigned)(((row0 + row < a.B ? row : a.B - 1 - row0) * 3 + g) * a.Nt + n) * 2;
        has = rr < 16 && n < a.Nt;
      }
      if (has) dma16(src + o, dst + (wave - 2 + 6 * i) * 1024);
    }
  };
  // byte offset of a lane's two terms of a gate
  auto tx_at = [&](int g) {
    return a.tx2 ? ((((blk * 2 + (q >> 1)) * 2 + ((g + 1) >> 1)) * 2 + (q & 1)) * 16 + c16) * 16 + ((g + 1) & 1) * 8 + 4 * kh
                 : ((c16 * 3 + g) * 64 + blk * 16 + 4 * q + 2 * kh) * 2;
  };
  tx_request(0, 0);
  if (RT == 2) tx_request(0, 1);

  v4i Wf[3][KW];
  gru_load_weights<KW, 0>(a, member, blk, kh * KW, lane, Wf);
  RescaleHi ps[3];
  bool pre = false;
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    ps[g] = rescale_hi_prepare(a.Mh[g], a.rh[g]);
    pre |= a.rh[g] < 33;
  }
  // what follows from the lane is worked out in every step where the weights leave no registers for it
  auto lane_anew = [&]() {
    if (RT == 1 || KS <= 16) return;
    asm volatile("" : "+v"(lane));
    c16 = lane & 15;
    q = lane >> 4;
  };
  const int n0 = member * 64 + blk * 16 + 4 * q + 2 * kh;  // this lane's two cells
  int32_t hreg[RT][2];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int row = row0 + rt * 16 + c16 < a.B ? row0 + rt * 16 + c16 : a.B - 1;
#pragma unroll
    for (int c = 0; c < 2; ++c) hreg[rt][c] = !a.zero_state && n0 + c < N ? a.h16[(size_t)row * N + n0 + c] : 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) asm volatile("" : "+v"(hreg[rt][c]));  // wait here, not at the first use in the loop
  }
  // the tile before step 0: 16 cells of a row per piece
  {
    const bool vec = (N & 7) == 0 && (reinterpret_cast<uintptr_t>(a.h16) & 15) == 0;
    for (int i = tid; i < RT * KS * 64; i += 512) {
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
  const int per = (GS + 7) >> 3, m0 = wave * per < GS ? wave * per : GS, m1 = m0 + per < GS ? m0 + per : GS;  // members whose pieces this wave fetches
  // group's part of a step of the exchange buffer, in rows of 16: tiles of ks_n KB
  int8_t *const hx0 = a.hx + (size_t)(a.batch0 / 16 + pl.group * RT) * ks_n * 1024;
  wait_vmem();
  __syncthreads();

  // The terms of a step.  (Read in an asm: behind an ordinary read of memory that transfers fill, the compiler waits for
  // every operation on global memory before it, here the stores of the output of the step before.)
  auto read_tx = [&](int t, int rt, int32_t (&tx2)[3]) {
    const unsigned at = (unsigned)(RT * KS * 1024 + (RT * t + rt) % kGruTxSlots(RT) * kGruTxBytes);
    asm volatile("ds_read_b32 %0, %3\n ds_read_b32 %1, %4\n ds_read_b32 %2, %5\n s_waitcnt lgkmcnt(0)"
                 : "=&v"(tx2[0]), "=&v"(tx2[1]), "=&v"(tx2[2])
                 : "v"(at + tx_at(0)), "v"(at + tx_at(1)), "v"(at + tx_at(2))
                 : "memory");
  };
  // R h over this half of the depth; the sums of two of the block's four cells a lane go to the wave of the other half.
  // `between` runs half way through.
  auto product = [&](int rt, v4i (&acc)[3], auto between) {
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      acc[g] = *reinterpret_cast<const v4i *>(bhL + g * 64 + blk * 16 + 4 * q);
      if (kh) acc[g] = v4i{0, 0, 0, 0};
    }
    constexpr int DEPTH = KW < 4 || (KW > 12 && RT == 1) ? 2 : 4;  // k steps of operands ahead
    const v4i *tile = hT + (rt * KS + kh * KW) * 64 + lane;
    v4i hf[DEPTH];
#pragma unroll
    for (int ks = 0; ks < DEPTH; ++ks) hf[ks] = tile[ks * 64];
#pragma unroll
    for (int ks = 0; ks < KW; ++ks) {
#pragma unroll
      for (int g = 0; g < 3; ++g) acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(Wf[g][ks], hf[ks % DEPTH], acc[g], 0, 0, 0);
      if (ks + DEPTH < KW) hf[ks % DEPTH] = tile[(ks + DEPTH) * 64];
      __builtin_amdgcn_sched_barrier(0);
      if (ks == KW / 4) between();
    }
#pragma unroll
    for (int g = 0; g < 3; ++g) ex[(wave * 3 + g) * 64 + lane] = kh ? v2i{acc[g][0], acc[g][1]} : v2i{acc[g][2], acc[g][3]};
  };
  // the cell of a row tile, behind the barrier that follows the product: new state into h, its int8 form packed
  auto cell = [&](const v4i (&acc)[3], const int32_t (&tx2)[3], int32_t (&h)[2]) {
    int32_t s[3][2], th[3][2], tx[3][2];
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      const v2i o = ex[((wave ^ 4) * 3 + g) * 64 + lane];
      s[g][0] = (kh ? acc[g][2] : acc[g][0]) + o[0];
      s[g][1] = (kh ? acc[g][3] : acc[g][1]) + o[1];
      tx[g][0] = (int32_t)(int16_t)(tx2[g] & 0xFFFF);
      tx[g][1] = tx2[g] >> 16;
    }
    if (pre) {
#pragma unroll
      for (int g = 0; g < 3; ++g)
#pragma unroll
        for (int c = 0; c < 2; ++c) th[g][c] = rescale_sat16_pre<2>(s[g][c], ps[g]);
    } else {
#pragma unroll
      for (int g = 0; g < 3; ++g)
#pragma unroll
        for (int c = 0; c < 2; ++c) th[g][c] = rescale_sat16_pre<0>(s[g][c], ps[g]);
    }
    int32_t x[4], v[4], xn[2], vn[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      x[c] = sat16(tx[0][c] + th[0][c]);
      x[2 + c] = sat16(tx[1][c] + th[1][c]);
    }
    gru_lookup<4>(lds, ls, x, v);
#pragma unroll
    for (int c = 0; c < 2; ++c) xn[c] = sat16(tx[2][c] + ((mul_i24(mirror_sigmoid(x[c], v[c]), th[2][c]) + 16384) >> 15));
    gru_lookup<2>(lds, lt, xn, vn);
    uint32_t pk = 0;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int32_t u = mirror_sigmoid(x[2 + c], v[2 + c]);
      h[c] = cell_update32(cifg_input_gate(u), mirror_tanh(xn[c], vn[c]), u, h[c], 0);
      pk |= (uint32_t)(state_i8(h[c]) & 0xFF) << (8 * c);
    }
    return pk;
  };
  // a piece: bytes 4 q + 2 kh of lane (c16, blk) are this lane's two cells
  auto mine = [&]() { return (blk * 16 + c16) * 16 + 4 * q + 2 * kh; };
  // Groups of 16 rows: the state travels in marked words, as m does in rec_kernel.  Who needs a piece fetches it until no 64 bits of it
  // hold kMarkFree, and what looks like a mark leaves through an escape slot.  Slots by turns, an escape slot for the even steps and
  // one for the odd: who stores step t + 2 has seen step t + 1 of all others, who had step t of everyone before they made that.
  auto slot_of = [&](int slot) { return hx0 + (size_t)slot * a.hx_step; };
  auto store_marked = [&](int t) {  // by one wave, from LDS, in whole words
    v4i w = stage[lane];
    const unsigned at = member * 1024 + lane * 16;
    const bool lo = ((uint32_t)w[0] ^ kMarkFree) < 2, hi = ((uint32_t)w[2] ^ kMarkFree) < 2;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(lo || hi) != 0, 0)) {
      int8_t *const esc = slot_of(kGruSlots + (t & 1)) + at;
      if (lo) *reinterpret_cast<int *>(esc) = w[0];
      if (hi) *reinterpret_cast<int *>(esc + 8) = w[2];
      wait_vmem();
      if (lo) w[0] = (int)kMarkEscape;
      if (hi) w[2] = (int)kMarkEscape;
    }
    *reinterpret_cast<v4i *>(slot_of(t & (kGruSlots - 1)) + at) = w;
  };
  // By the wave that stores the pieces, when the group's state of step t + 1 is here: then everyone has read this one, whose words
  // are marked for step t + 4.  (The next piece leaves behind a wait for this store, and step t + 4 is looked for behind that piece.)
  auto mark_piece = [&](int t) {
    *reinterpret_cast<v4i *>(slot_of(t & (kGruSlots - 1)) + (unsigned)(member * 1024 + lane * 16)) = v4i{} + (int)kMarkFree;
  };
  auto fetch_marked = [&](int t) {  // an eighth of the tile per wave, until every word is there
    const int8_t *src = slot_of(t & (kGruSlots - 1)) + lane * 16;
    v4i *const tile = hT + m0 * 64 + lane;
    int budget = a.spin_limit;
    uint32_t least;
    for (;;) {
#pragma unroll
      for (int i = 0; i < (KS + 7) / 8; ++i)
        if (m0 + i < m1) dma16_agent(src + (size_t)(m0 + i) * 1024, hT + (m0 + i) * 64);
      wait_vmem();
      least = 0xFFFFFFFFu;
#pragma unroll
      for (int i = 0; i < (KS + 7) / 8; ++i)
        if (m0 + i < m1) {
          const v4i w = tile[i * 64];
          const uint32_t d0 = (uint32_t)w[0] ^ kMarkFree, d1 = (uint32_t)w[2] ^ kMarkFree, d = d0 < d1 ? d0 : d1;
          least = least < d ? least : d;
        }
      if (a.never) least = 0;
      if (__builtin_amdgcn_ballot_w64(least == 0) == 0) break;
      if (gru_spent(a, budget)) {
        __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        flag[0] = 0;
        return;
      }
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(least == 1) != 0, 0)) {
      const int8_t *esc = slot_of(kGruSlots + (t & 1)) + lane * 16;
      for (int m = m0; m < m1; ++m)
#pragma unroll
        for (int k = 0; k < 4; k += 2) {
          int *const w = reinterpret_cast<int *>(tile + (m - m0) * 64) + k;
          if ((uint32_t)*w == kMarkEscape)
            *w = __hip_atomic_load(reinterpret_cast<const int *>(esc + (size_t)m * 1024 + 4 * k), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
  };
  auto store_piece = [&](int t, int rt) {  // by one wave, from LDS: stores of 16 bytes a lane are acknowledged sooner than two-byte ones of all waves
    *reinterpret_cast<v4i *>(hx0 + (size_t)t * a.hx_step + (size_t)(rt * ks_n + member) * 1024 + lane * 16) = stage[rt * 64 + lane];
  };
  auto fetch = [&](int t, int rt) {  // an eighth of the tile per wave
    const int8_t *src = hx0 + (size_t)t * a.hx_step + (size_t)rt * ks_n * 1024 + lane * 16;
    for (int m = m0; m < m1; ++m) dma16(src + (size_t)m * 1024, hT + (rt * KS + m) * 64);
  };
  auto raise = [&](int rt, int step) {
    if (lane == 0) __hip_atomic_store(flags + (rt * GS + member) * 16, (unsigned)step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
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
    *reinterpret_cast<uint16_t *>(reinterpret_cast<uint8_t *>(stage + rt * 64) + mine()) = (uint16_t)pk;
    if (GS == 1) *reinterpret_cast<uint16_t *>(lds + rt * KS * 1024 + mine()) = (uint16_t)pk;
  };

  if constexpr (RT == 1) {
    for (int t = 0; t < T; ++t) {
      lane_anew();
      int32_t tx2[3];
      v4i acc[3];
      if (t + 1 < T) tx_request(t + 1, 0);
      product(0, acc, []() {});
      read_tx(t, 0, tx2);
      // every wave is done with the tile before any wave fetches the next state into it, and the sums are in LDS
      lds_barrier();
      const uint32_t pk = cell(acc, tx2, hreg[0]);
      keep_piece(0, pk);
      if (GS == 1 || (t == T - 1 && T > 1)) {  // nobody else reads this state (see gru_quad_kernel)
        wait_vmem();
        __syncthreads();
      } else {
        lds_barrier();
        if (wave == 0) store_marked(t);
        for (int i = 0; i < a.sync_sleep; ++i) __builtin_amdgcn_s_sleep(1);  // a first look too early costs the arrivals
        fetch_marked(t);
        lds_barrier();
        if (flag[0] == 0) return;
        if (wave == 0 && t > 0 && t + kGruSlots < T) mark_piece(t - 1);
      }
      if (wave == 1) output(t, 0);
    }
  } else {
    // Two row tiles by turns: while the members exchange the state of one, they work on the other.  Wave 1 stores a tile's
    // piece when its turn ends and raises the flag half way through the product of the next turn, when the store has been
    // acknowledged; at the end of that product the others' flags are polled, and their pieces arrive under the cell.
    for (int t = 0; t < T; ++t) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        lane_anew();
        int32_t tx2[3];
        v4i acc[3];
        if (t + 1 < T) tx_request(t + 1, rt);
        const int other_step = t - (rt == 0);  // the step whose state of the other tile comes in now
        const bool comes = GS > 1 && other_step >= 0 && other_step + 1 < T;
        product(rt, acc, [&]() {
          if (wave == 1 && comes) {
            wait_vmem();
            raise(1 - rt, other_step + 1);
          }
        });
        read_tx(t, rt, tx2);
        if (comes && wave == 0) poll(1 - rt, other_step + 1);
        lds_barrier();  // (not __syncthreads: nothing waits for the stores of the output)
        if (comes) fetch(other_step, 1 - rt);
        const uint32_t pk = cell(acc, tx2, hreg[rt]);
        keep_piece(rt, pk);
        wait_vmem();
        __syncthreads();
        if (flag[0] == 0) return;
        if (wave == 1 && GS > 1 && t + 1 < T) store_piece(t, rt);
        if (wave == 2) output(t, rt);
      }
    }
    if (GS > 1 && T == 1) {  // h16 is read by every member and written by each
      if (wave == 0) {
        raise(1, 1);
        poll(1, 1);
      }
      __syncthreads();
      if (flag[0] == 0) return;
    }
  }
  gru_placement_check(a);
  if (a.h16)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int n1 = member * 64 + blk * 16 + 4 * q + 2 * kh;
      const int row = row0 + rt * 16 + c16;
      if (row < a.B)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          if (n1 + c < N) a.h16[(size_t)row * N + n1 + c] = (int16_t)hreg[rt][c];
    }
}

template <int KS>
gru_fn rows_pick_ks(int rows) {
  return rows == 16 ? gru_rows_kernel<KS, 1> : gru_rows_kernel<KS, 2>;
}

}  // namespace

gru_fn gru_rows_pick(int ks, int rows) {
  switch (ks) {
    case 4: return rows_pick_ks<4>(rows);
    case 8: return rows_pick_ks<8>(rows);
    case 16: return rows_pick_ks<16>(rows);
    case 24: return rows_pick_ks<24>(rows);
    case 32: return rows_pick_ks<32>(rows);
    default: return nullptr;
  }
}

}  // namespace lstm_int

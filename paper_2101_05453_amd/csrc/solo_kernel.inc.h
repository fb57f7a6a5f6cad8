// Recurrent kernel for layers of up to 256 cells: ONE workgroup runs all T steps
// of 4 batch rows.  In rec_kernel and rec16_kernel the cells of a row are
// spread over workgroups that meet two or three times per step in the L2, about
// 1.1 us each, and a wave's step is bound by the instructions of its 16 rows x 16
// cells (about 700 at four cells per lane, one issued every 4-5 clocks).  Here a
// row's cells are all in one workgroup -- h, m and the layer-norm sums pass
// through LDS, no workgroup depends on another: any batch, no residency
// requirement, no placement check -- and a lane has ONE cell of one row: a
// quarter of the instructions, for which the chip has the compute units (4 rows
// per workgroup: 1024 rows before the second round of workgroups).
// Measured: solo_inst.hip.
//
// The 16x16x64 MFMA with the batch rows as its first operand (result rows) and
// the 16 cells of one gate as its second: lane (c = lane % 16, q = lane / 16)
// ends with gate g of cell c for result rows 4 q + i, and batch row q is put in
// result row 4 q: value 0 of every lane is used (the other three quarters of the
// matrix work are spare).  The weights are rec16_kernel's, gathered once into that
// order; the W x terms are read in the layout the input GEMM writes for the 32-row
// kernel.
//
// A wave takes one block of 16 cells; WAVES * 16 cells bound the layer.  With 16 waves (129 to 256 cells) a lane has 128
// registers, 64 of them weights: rescale constants are read from the arguments where they are used, layer-norm parameters
// from LDS, and a layer-norm step works out lane numbers and addresses anew.  Eight waves of two blocks each have the
// registers, and half as many waves to fill the gaps: 256 cells, 32 rows, a step without / with layer norm / and peephole
// 1.85, 4.0, 4.9 us, with 16 waves 1.55, 3.1, 3.6.
//
// Four and eight waves have the registers, and are the faster for keeping things in them: with the 16-wave form's economies
// (LEAN) in their code 60 steps of 16 rows with peephole and layer norm took, without -> with, 39 cells 144 -> 152 us, 64 cells
// 137 -> 145, 128 cells 155 -> 167.  Whether there is a projection is compiled in for them (39 cells, plain 60 -> 56 us, 128
// cells 62 -> 57; the masks of mirror_*_masked instead of selects 57 -> 56 and 60 -> 57).  The 16-wave form looks the
// projection up: compiled in, the plain forms and peephole or layer norm alone gain up to 3 %, 203 cells with both lose 4 %.
#pragma once

#include "rec_kernel.inc.h"

namespace lstm_int {

// The LDS of a launch, from the front (solo_lds_bytes mirrors it): two h tiles, the m tile, statistics, tables, W_proj.
template <int WAVES, int KS16, int FL>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES / 4, WAVES / 4))) void solo_kernel(RecArgs2 args) {
  constexpr bool cifg = FL & 1, ph = FL & 2, ln = FL & 4;
  constexpr int NT = 64 * WAVES, NC = 16 * WAVES, RG = 4;  // threads; cells and batch rows of the workgroup
  constexpr bool LN_LDS = ln && WAVES > 8;  // layer-norm parameters in LDS
  constexpr bool LEAN = WAVES == 16;
  constexpr bool ROW_ADDR = !LEAN && cifg && ph && ln;  // outputs addressed by their row, not within the step's rows
  constexpr int LS = KS16 * 64 + 16;           // row stride of the h and m tiles
  constexpr int g_first = cifg ? 1 : 0;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x;
  int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int c16 = lane & 15, q = lane >> 4;
  const int which = (int)blockIdx.x >= args.d[0].groups ? 1 : 0;
  const RecDirArgs &a = args.d[which];
  const int row0 = ((int)blockIdx.x - (which ? args.d[0].groups : 0)) * RG;
  const bool proj = LEAN ? a.flags & 8 : FL & 8;
  const int ldy = a.ldy;

  uint8_t *p = lds;
  int8_t *hT = reinterpret_cast<int8_t *>(p);       p += 2 * RG * LS;
  int8_t *mT = reinterpret_cast<int8_t *>(p);       p += RG * LS;
  u64 *red = reinterpret_cast<u64 *>(p);            p += 16 * 8;  // [gate][row] sums
  LnRow2 *lnrow = reinterpret_cast<LnRow2 *>(p);    p += 16 * sizeof(LnRow2);  // [gate][row]
  int *flag = reinterpret_cast<int *>(p);           p += 16;  // 1: every row has sigma >= 2^12
  double *LdL = reinterpret_cast<double *>(p);      p += LN_LDS ? 4 * NC * 8 : 0;
  double *bdL = reinterpret_cast<double *>(p);      p += LN_LDS ? 4 * NC * 8 : 0;
  p = lds + (((size_t)(p - lds) + 1023) & ~(size_t)1023);
  const bool share_tanh = a.lut[2].blob == a.lut[1].blob;
  int offD[3], offB[3], offT[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (i == 2 && share_tanh) {
      offD[2] = offD[1]; offB[2] = offB[1]; offT[2] = offT[1];
    } else {
      const int nb = ((((a.lut[i].dom >> a.lut[i].sh) * 2) + 1023) >> 10) << 10;
      offD[i] = (int)(p - lds);                            p += a.lut[i].dom;
      offB[i] = (int)(p - lds);                            p += nb;
      offT[i] = a.lut[i].tail ? (int)(p - lds) : 0;        p += a.lut[i].tail ? 3072 : 0;
    }
  }
  int8_t *WpL = reinterpret_cast<int8_t *>(p);  // [round_up(H, 16)][LS]

  // ---- once: tables and W_proj -> LDS, R -> registers, per-cell parameters -> registers
  {
    auto dma = [&](const void *src, const void *dst) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                       (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
    };
    for (int i = 0; i < (share_tanh ? 2 : 3); ++i) {
      const int nd = a.lut[i].dom >> 10;
      const int nb = (((a.lut[i].dom >> a.lut[i].sh) * 2) + 1023) >> 10;
      const int nt = a.lut[i].tail ? 3 : 0;
      for (int c = wave; c < nd + nb + nt; c += WAVES) {
        const int so = c < nd ? c * 1024 : (c < nd + nb ? kLutWideBaseOff + (c - nd) * 1024 : kLutWideTailOff + (c - nd - nb) * 1024);
        dma(a.lut[i].blob + so + lane * 16, lds + offD[i] + c * 1024);
      }
    }
    if (proj) {  // output rows of npadp >= N bytes each
      const int rows = (a.H + 15) & ~15, pieces = KS16 * 4;
      for (int i = tid; i < rows * pieces; i += NT) {
        const int row = i / pieces, o = (i - row * pieces) * 16;
        int4 v = {0, 0, 0, 0};
        if (o < a.npadp) v = *reinterpret_cast<const int4 *>(a.Wp2 + (size_t)row * a.npadp + o);
        *reinterpret_cast<int4 *>(WpL + row * LS + o) = v;
      }
    }
  }
  const bool real = wave < (a.Ncp >> 4);  // the layer has this block of 16 cells (cells past N are zero weights)
  v4i Wf[4][KS16];        // [gate]: lane (c16, q) holds bytes 16 q.. of each 64-deep k step of cell c16's row
  int32_t bh[4], Pq[3];
  double wL[4], wb[4];    // not with LN_LDS
  {
    const int cb = real ? wave : 0;
    // rec16_kernel's tile j holds, in row 4 q' + g, gate g of cell 4 q' + j
    const int4 *src = a.R2h + (size_t)(cb * 4 + (c16 & 3)) * a.ks16 * 64 + 4 * (c16 >> 2) + 16 * q;
    int4 w[4][KS16];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int ks = 0; ks < KS16; ++ks) w[g][ks] = real ? src[(size_t)ks * 64 + g] : int4{0, 0, 0, 0};
    const size_t n = cb * 16 + c16;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      bh[g] = real ? a.bh4[(size_t)g * a.Ncp + n] : 0;
      if (g < 3) Pq[g] = ph && real ? a.Pq3[(size_t)g * a.Ncp + n] : 0;
      wL[g] = ln && real ? ln_weight_scaled(a.Lq4[(size_t)g * a.Ncp + n]) : 0.0;
      wb[g] = ln && real ? ln_bias_scaled(a.qb4[(size_t)g * a.Ncp + n]) : 0.0;
      if (LN_LDS && q == 0) {
        LdL[g * NC + wave * 16 + c16] = wL[g];
        bdL[g * NC + wave * 16 + c16] = wb[g];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int ks = 0; ks < KS16; ++ks) {
        Wf[g][ks] = v4i{w[g][ks].x, w[g][ks].y, w[g][ks].z, w[g][ks].w};
        asm volatile("" : "+a"(Wf[g][ks]));
      }
    __builtin_amdgcn_sched_barrier(0);
  }
  // rescale constants: kept, or with 16 waves (128 registers a lane, half of them weights) read again from the arguments
  // where they are used
  RescaleHi ps_[4], pc_[3], pl_[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    ps_[g] = rescale_hi_prepare(a.Mh[g], a.rh[g]);
    pl_[g] = rescale_hi_prepare(a.Mln[g], ln ? a.rln[g] : 33);
    if (g < 3) pc_[g] = rescale_hi_prepare(ph ? a.Mc[g] : 0, ph ? a.rc[g] : 33);
  }
  typedef const __attribute__((address_space(4))) RecArgs2 *KernArgs;
  auto fresh = [&] {
    KernArgs k = (KernArgs)__builtin_amdgcn_kernarg_segment_ptr();
    if constexpr (LEAN) asm volatile("" : "+s"(k));
    return k;
  };
  auto ps = [&](KernArgs k, int g) { return LEAN ? rescale_hi_prepare(k->d[which].Mh[g], k->d[which].rh[g]) : ps_[g]; };
  auto pl = [&](KernArgs k, int g) { return LEAN ? rescale_hi_prepare(k->d[which].Mln[g], k->d[which].rln[g]) : pl_[g]; };
  auto pc = [&](KernArgs k, int j) { return LEAN ? rescale_hi_prepare(k->d[which].Mc[j], k->d[which].rc[j]) : pc_[j]; };
  if (tid < 16) red[tid] = 0;
  // the h tile before step 0; the other tile and m start as zeros (bytes past a row's real ones only meet zero weights)
  for (int i = tid; i < 3 * RG * LS / 4; i += NT) {
    const int o = 4 * i, rr = o / LS, c = o - rr * LS;
    const int row = row0 + rr < a.B ? row0 + rr : a.B - 1;
    reinterpret_cast<int32_t *>(hT)[i] = rr < RG && c < a.Hpad ? *reinterpret_cast<const int32_t *>(a.h0 + (size_t)row * a.Hpad + c) : 0;
  }
  // rows past the batch repeat the last one and are not stored
  bool row_ok = row0 + q < a.B;
  int row = row_ok ? row0 + q : a.B - 1;
  const int own = wave * 16 + c16;  // this lane's cell, and its output of the projection
  int32_t creg = (a.c_in && own < a.N) ? a.c_in[(size_t)row * a.N + own] : 0;
  const double inv_n = 1.0 / (double)a.N;
  const bool pre_ln = ln && (a.rln[0] < 33 || a.rln[1] < 33 || a.rln[2] < 33 || a.rln[3] < 33);
  const bool pre_m = a.rm < 33;
  const int T = a.T, pre_h = a.pre_h, rev = a.rev, N = a.N, H = a.H, B = a.B;
  const RescaleHi pm_ = rescale_hi_prepare(a.Mm, a.rm), pp_ = rescale_hi_prepare(proj ? a.Mp : 0, proj ? a.rp : 33);
  const int dom[3] = {a.lut[0].dom, a.lut[1].dom, a.lut[2].dom}, sh[3] = {a.lut[0].sh, a.lut[1].sh, a.lut[2].sh};
  const int32_t zp_m = a.zp_m, zp_h = a.zp_h, m_c = a.m_c;
  const int32_t bp = proj && own < H ? a.bp2[own] : 0;

  // W x terms: value (gate, cell) of row b is the int16 [2-gate half][lane][4 (gate % 2) + cell % 4] of the row's block;
  // two steps on their way (they come from memory, and a step is shorter than that)
  constexpr int AHEAD = 2;
  int32_t txq[AHEAD][4];
  const size_t tx_step = (size_t)(a.Bp >> 5) * (a.Ncp >> 3) * 1024;  // int16 values of one step
  const int16_t *const tx_base = reinterpret_cast<const int16_t *>(a.tx2) +
                                 ((size_t)(row >> 5) * (a.Ncp >> 3) + wave * 2 + (c16 >> 3)) * 1024 +
                                 ((row & 31) + 32 * ((c16 >> 2) & 1)) * 8 + (c16 & 3);
  auto tx_request = [&](int t, int32_t (&dst)[4]) {
    t = t < T ? t : T - 1;
    if (rev) t = T - 1 - t;
    const int16_t *src = tx_base + (size_t)t * tx_step;
#pragma unroll
    for (int g = g_first; g < 4; ++g)  // a block the layer does not have: its gate sums are 0, as for padded cells
      dst[g] = real ? src[(g >> 1) * 512 + (g & 1) * 4] : 0;
  };
#pragma unroll
  for (int s = 0; s < AHEAD; ++s) tx_request(s, txq[s]);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // The sums of v and of v^2 over the cells of a row into red[gate][row], S2 in the bits above S1.  Squares are at most
  // 2^30: the four of a quad of lanes fit 32 bits, and the four quads of a row add into the word (LDS atomics, four lanes
  // to a word; folding the quads in the lanes first, S2 as two halves, takes 0.1 to 0.2 us a step more at 256 cells).
  auto rot = [](int32_t x, auto ctrl) { return x + __builtin_amdgcn_mov_dpp(x, decltype(ctrl)::value, 0xF, 0xF, true); };
  auto add_stats = [&](int g, int32_t v) {
    using Q1 = std::integral_constant<int, 0xB1>;   // quad_perm [1,0,3,2]
    using Q2 = std::integral_constant<int, 0x4E>;   // quad_perm [2,3,0,1]
    const int32_t s1 = rot(rot(v, Q1{}), Q2{});
    const uint32_t s2 = (uint32_t)rot(rot((int32_t)((uint32_t)v * (uint32_t)v), Q1{}), Q2{});
    if ((lane & 3) == 0)
      __hip_atomic_fetch_add(&red[g * 4 + q], ((u64)s2 << 24) + (u64)(int64_t)s1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // gates g_lo..g_hi: one wave turns the sums into (mean, sigma) form
  auto statistics = [&](int g_lo, int g_hi) {
    __syncthreads();
    if (LEAN ? wave == 0 : tid < 64) {
      int item = lane;  // (gate, row)
      if constexpr (LEAN) asm volatile("" : "+v"(item));  // worked out here, not kept through the step
      const bool first16 = item < 16;
      item &= 15;
      const bool here = first16 && (item >> 2) >= g_lo && (item >> 2) <= g_hi;
      const int64_t pk = (int64_t)red[item];
      const int64_t S1 = ((pk + (1 << 23)) & 0xFFFFFF) - (1 << 23);  // 256 values of at most 32767: below 2^23
      const LnRow2 lr = ln_row2(S1, (pk - S1) >> 24, N, inv_n);
      const bool narrow = __builtin_amdgcn_ballot_w64(here && !ln_row_is_narrow(lr)) == 0;
      if (here) {
        u64 zero = 0;
        if constexpr (LEAN) asm volatile("" : "+v"(zero));  // made here: as a constant of the loop it takes two registers
        red[item] = zero;  // the next adds come after the barrier below
        lnrow[item] = lr;
      }
      if (lane == 0) flag[0] = narrow;
    }
    __syncthreads();
  };
  // layer norm of K gate sums
  auto normalize = [&](auto count, const int *gates, int32_t *v) {
    constexpr int K = decltype(count)::value;
    LnRow2 lr[K];
    double cL[K], cb[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int g = gates[k];
      lr[k] = lnrow[g * 4 + q];
      cL[k] = LN_LDS ? LdL[g * NC + wave * 16 + c16] : wL[g];
      cb[k] = LN_LDS ? bdL[g * NC + wave * 16 + c16] : wb[g];
    }
    const bool narrow = __builtin_amdgcn_readfirstlane(flag[0]) != 0;
    const KernArgs ka = fresh();
    __builtin_amdgcn_sched_barrier(0);
    if (narrow) {
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = ln_second_stage_narrow(v[k], lr[k], cL[k], cb[k]);
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = ln_second_stage(v[k], lr[k], cL[k], cb[k]);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const RescaleHi pg = pl(ka, gates[k]);
      if (pre_ln) v[k] = rescale_preshift(v[k], pg);
      v[k] = rescale_sat16_pre<0>(v[k], pg);
    }
  };
  // table values of |x| (table tb: 0 sigma, 1 tanh, 2 cell tanh) for K values at once; see rec_kernel's lookup
  auto lookup = [&](auto count, const int32_t *x, const int *tb, int32_t *out) {
    constexpr int K = decltype(count)::value;
    int32_t mag[K];
    uint32_t base[K], delta[K];
    bool over = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      mag[k] = abs_i32(x[k]);
      over |= mag[k] >= dom[tb[k]];
      const int32_t ai = mag[k] < dom[tb[k]] ? mag[k] : dom[tb[k]] - 1;
      base[k] = *reinterpret_cast<const uint16_t *>(lds + offB[tb[k]] + 2 * (ai >> sh[tb[k]]));
      delta[k] = lds[offD[tb[k]] + ai];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = (int32_t)(base[k] + delta[k]);
    if (__builtin_amdgcn_ballot_w64(over) != 0) {
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (offT[tb[k]] && mag[k] >= dom[tb[k]]) out[k] = lut_wide_tail(lds + offT[tb[k]], mag[k]);
    }
  };
  constexpr int32_t glo = ln ? -32767 : -32768;
  // first operand of the MFMA: result row 4 q is row q of the group; the other result rows read it too, and nobody uses
  // what comes of them

  for (int t = 0; t < T; ++t) {
    if (LEAN && ln) {  // what follows from the lane is worked out in every step, not kept in registers that are not there
      asm volatile("" : "+v"(lane));
      c16 = lane & 15;
      q = lane >> 4;
      row_ok = row0 + q < B;
      row = row_ok ? row0 + q : B - 1;
    }
    const int8_t *hcur = hT + (t & 1) * RG * LS;
    int8_t *hnext = hT + ((t + 1) & 1) * RG * LS;
    // this step's rows of the outputs; a lane's place in them fits 32 bits (at most 2048 rows)
    const size_t orow0 = (size_t)(rev ? T - 1 - t : t) * a.B;
    int8_t *const out_t = a.out + orow0 * a.Hpad, *const y_t = a.y ? a.y + orow0 * ldy : nullptr;
    int32_t gs[4];
    {
      v4i hf[KS16];
#pragma unroll
      for (int ks = 0; ks < KS16; ++ks) hf[ks] = *reinterpret_cast<const v4i *>(hcur + (c16 >> 2) * LS + (q << 4) + ks * 64);
      v4i acc[4];
#pragma unroll
      for (int g = g_first; g < 4; ++g) {
        acc[g] = v4i{LEAN ? 0 : bh[g], 0, 0, 0};  // with 16 waves four registers too many to keep from step to step
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(hf[ks], Wf[g][ks], acc[g], 0, 0, 0);
      }
      // gate sums (Secs. 3.2.4/3.2.5); with a peephole the o gate is finished after c^t
      const KernArgs ka = fresh();
      auto gate_sums = [&](auto pre_tag) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          if (g < g_first) continue;
          int32_t v = txq[0][g] + rescale_sat16_pre<decltype(pre_tag)::value>(acc[g][0] + (LEAN ? bh[g] : 0), ps(ka, g));
          if (ph && g < 2) v += rescale_sat16_pre(mul_i24(Pq[g < 3 ? g : 0], creg), pc(ka, g < 3 ? g : 0));
          if (!(ph && g == 3)) v = clamp_i32(v, glo, 32767);
          gs[g] = v;
        }
      };
      if (pre_h == 0)
        gate_sums(std::integral_constant<int, 0>{});
      else if (pre_h == 1)
        gate_sums(std::integral_constant<int, 1>{});
      else
        gate_sums(std::integral_constant<int, 2>{});
      if (ln) {
#pragma unroll
        for (int g = g_first; g < (ph ? 3 : 4); ++g) add_stats(g, gs[g]);
      }
    }
    // the terms of the next step are taken over here, ahead of this step's stores: a wait for them further down would
    // wait for those stores too (the counter drains in order), 0.28 us
#pragma unroll
    for (int s = 0; s + 1 < AHEAD; ++s)
#pragma unroll
      for (int g = g_first; g < 4; ++g) {
        txq[s][g] = txq[s + 1][g];
        asm volatile("" : "+v"(txq[s][g]));
      }
    tx_request(t + AHEAD, txq[AHEAD - 1]);
    if (ln) statistics(g_first, ph ? 2 : 3);

    // layer norm, sigma / tanh, cell update (Secs. 3.2.6, 3.2.1, 3.2.9, 3.2.7)
    int32_t xo;
    {
      // f, z, then o unless a peephole keeps it for later, then i unless it is coupled
      constexpr int KG = 4 - (ph ? 1 : 0) - (cifg ? 1 : 0);
      const int gates[4] = {1, 2, ph ? 0 : 3, 0}, tb[4] = {0, 1, 0, 0};
      int32_t x[4], tv[4];
#pragma unroll
      for (int k = 0; k < KG; ++k) x[k] = gs[gates[k]];
      if (ln && !LEAN) normalize(std::integral_constant<int, KG>{}, gates, x);
      if (ln && LEAN) {  // two at a time
        normalize(std::integral_constant<int, KG / 2>{}, gates, x);
        normalize(std::integral_constant<int, KG - KG / 2>{}, gates + KG / 2, x + KG / 2);
      }
      lookup(std::integral_constant<int, KG>{}, x, tb, tv);
      const int32_t fg = mirror_sigmoid_masked(x[0], tv[0]);
      const int32_t ig = cifg ? cifg_input_gate(fg) : mirror_sigmoid_masked(x[KG - 1], tv[KG - 1]);
      xo = ph ? 0 : mirror_sigmoid_masked(x[2], tv[2]);
      creg = cell_update32(ig, mirror_tanh_masked(x[1], tv[1]), fg, creg, m_c);
      if (ph) {  // finish the o gate sum with P_o . c^t (eq. 5)
        gs[3] = clamp_i32(gs[3] + rescale_sat16_pre(mul_i24(Pq[2], creg), pc(fresh(), 2)), glo, 32767);
        if (ln) add_stats(3, gs[3]);
      }
    }
    if (ph && ln) statistics(3, 3);

    // hidden state (Sec. 3.2.7)
    {
      const int cell = wave * 16 + c16;
      const int tb[2] = {2, 0}, gates[1] = {3};
      int32_t x[2] = {creg, gs[3]}, tv[2];
      if (ph && ln) normalize(std::integral_constant<int, 1>{}, gates, x + 1);
      lookup(std::integral_constant<int, ph ? 2 : 1>{}, x, tb, tv);
      const int32_t o = ph ? mirror_sigmoid_masked(x[1], tv[1]) : xo;
      int32_t om = mul_i24(o, mirror_tanh_masked(x[0], tv[0]));
      const KernArgs ka = fresh();
      const RescaleHi pm = LEAN ? rescale_hi_prepare(ka->d[which].Mm, ka->d[which].rm) : pm_;
      if (pre_m) om = rescale_preshift(om, pm);
      const int8_t mq = (int8_t)sat8(rescale_sat16_pre<0>(om, pm) + zp_m);
      if (proj) {
        mT[q * LS + cell] = mq;
      } else {
        hnext[q * LS + cell] = mq;
        if (row_ok && cell < N) {
          if constexpr (ROW_ADDR) {
            const size_t orow = orow0 + row;
            a.out[orow * a.Hpad + cell] = mq;
            if (a.y) a.y[orow * ldy + cell] = mq;
          } else {
            out_t[(uint32_t)row * (uint32_t)a.Hpad + (uint32_t)cell] = mq;
            if (y_t) y_t[(uint32_t)row * (uint32_t)ldy + (uint32_t)cell] = mq;
          }
        }
      }
    }
    // projection (Sec. 3.2.8): tiles of 16 outputs over the waves, the whole depth in one wave
    if (proj) {
      __syncthreads();
      v4i mf[KS16];
      const KernArgs ka = fresh();
      const RescaleHi pp = LEAN ? rescale_hi_prepare(ka->d[which].Mp, ka->d[which].rp) : pp_;
#pragma unroll
      for (int ks = 0; ks < KS16; ++ks) mf[ks] = *reinterpret_cast<const v4i *>(mT + (c16 >> 2) * LS + (q << 4) + ks * 64);
      const int p0 = wave * 16;
      if (p0 < H) {
        v4i pacc = v4i{LEAN ? 0 : bp, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks)
          pacc = __builtin_amdgcn_mfma_i32_16x16x64_i8(
              mf[ks], *reinterpret_cast<const v4i *>(WpL + (p0 + c16) * LS + (q << 4) + ks * 64), pacc, 0, 0, 0);
        const int8_t hq = (int8_t)sat8(rescale_sat16_pre(pacc[0] + (LEAN ? bp : 0), pp) + zp_h);
        hnext[q * LS + p0 + c16] = hq;
        if (row_ok && p0 + c16 < H) {
          if constexpr (ROW_ADDR) {
            const size_t orow = orow0 + row;
            a.out[orow * a.Hpad + p0 + c16] = hq;
            if (a.y) a.y[orow * ldy + p0 + c16] = hq;
          } else {
            out_t[(uint32_t)row * (uint32_t)a.Hpad + (uint32_t)(p0 + c16)] = hq;
            if (y_t) y_t[(uint32_t)row * (uint32_t)ldy + (uint32_t)(p0 + c16)] = hq;
          }
        }
      }
    }
    __syncthreads();  // the next h tile is complete
  }
  if (a.c_out && row_ok) {
    if (own < N) a.c_out[(size_t)row * N + own] = (int16_t)creg;
  }
}

typedef void (*solo_fn)(RecArgs2);

// kernel for (flags & 15); with 16 waves the projection is looked up in the run
template <int WAVES, int KS16>
solo_fn solo_pick_size(int fl) {
  constexpr int P = WAVES == 16 ? 0 : 8;
  switch (fl & (7 | P)) {
    case 0: return solo_kernel<WAVES, KS16, 0>;
    case 1: return solo_kernel<WAVES, KS16, 1>;
    case 2: return solo_kernel<WAVES, KS16, 2>;
    case 3: return solo_kernel<WAVES, KS16, 3>;
    case 4: return solo_kernel<WAVES, KS16, 4>;
    case 5: return solo_kernel<WAVES, KS16, 5>;
    case 6: return solo_kernel<WAVES, KS16, 6>;
    case 7: return solo_kernel<WAVES, KS16, 7>;
    case 8: return solo_kernel<WAVES, KS16, P>;
    case 9: return solo_kernel<WAVES, KS16, P | 1>;
    case 10: return solo_kernel<WAVES, KS16, P | 2>;
    case 11: return solo_kernel<WAVES, KS16, P | 3>;
    case 12: return solo_kernel<WAVES, KS16, P | 4>;
    case 13: return solo_kernel<WAVES, KS16, P | 5>;
    case 14: return solo_kernel<WAVES, KS16, P | 6>;
    default: return solo_kernel<WAVES, KS16, P | 7>;
  }
}

}  // namespace lstm_int

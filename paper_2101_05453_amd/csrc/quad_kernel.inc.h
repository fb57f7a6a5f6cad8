// Recurrent kernel for small batches of layers with more than 256 cells: groups
// of FOUR batch rows, the cells of a group spread over the workgroups of an XCD
// as in rec16_kernel (64 each), a lane with one cell of one row as in
// solo_kernel.  Against rec16_kernel (16 rows per group, four cells per lane) a
// wave issues a quarter of the instructions per step, and the exchanges carry so
// little -- 2 KB of h, 16 words of statistics per workgroup -- that the data can be
// its own signal:
//
//  * h and m travel as (value, tag) byte pairs, four cells to a 64-bit word, the
//    tag being the step: a reader polls the very words it needs and is done when
//    all carry the step's tag -- no acknowledged stores, no counter, no second
//    trip for the data.  (One exchange among 8 workgroups: 0.9 us instead of 1.08
//    with stores, counter and a tile load; the tile of 16 rows x 1024 cells that
//    rec16_kernel moves is too large for tags to pay.)
//  * Layer norm: a workgroup stores its (sum q, sum q^2), 60 bits with a 4-bit tag
//    in one word per (gate, row), and its first wave polls the words of all
//    members, adds them up and turns them into (mean, sigma).
//
// Words are single-copy atomic at 64 bits, so a tag vouches for its values.  Two
// slots alternate: a workgroup stores step t + 2 only after it has read step t + 1
// of all others, who stored that after they had read all of step t.
// A word is stored at workgroup scope and polled at agent scope.  What makes the
// two meet is the placement, not the scopes: the L1 writes through, so the store is
// in the L2 of the group's XCD, and a load of agent scope goes past the L1 to that
// L2.  A group spread over two XCDs would never see its words (the waits end, and
// the placement check says why).  An agent-scope store goes on through the L2 to
// memory: 512 cells, layer norm, 16 rows, 100 steps 304 -> 383 us.
// A wave's memory operations return in order, so nothing slow may be ahead of a
// poll: the W x terms (from memory, asked for two steps ahead) go to LDS by waves 2
// and 3, the layer output is stored by wave 1, each right after the step's last
// exchange; the statistics are polled by wave 0.
//
// The h and m words are polled 16 bytes per load (poll_pairs): what a poll costs is
// its loads.
//
// What bounds it: the chain of a step -- one exchange (two with a projection; and
// one per round of statistics), 0.8 to 1.3 us each -- and the ~150 to 250
// instructions a wave issues between them.  Time per step at batch 16 (250 against
// 50 steps), rec16_kernel -> this kernel with 8 bytes per load -> now (us):
//                            no layer norm          layer norm            and peephole
//   320 cells              3.31 -> 1.53 -> 1.44   4.73 -> 2.81 -> 2.66   6.06 -> 3.92 -> 3.72
//   512 cells              3.31 -> 1.58 -> 1.46   4.72 -> 2.85 -> 2.69   5.97 -> 3.96 -> 3.73
//   1024 cells             3.92 -> 2.03 -> 1.80   5.52 -> 3.59 -> 3.25   6.94 -> 4.88 -> 4.46
//   1024, 256 outputs      5.40 -> 2.99 -> 2.71   6.92 -> 4.46 -> 4.14   8.36 -> 5.76 -> 5.35
//   2048, 640 outputs      5.82 -> 4.38 -> 3.82   7.76 -> 6.20 -> 5.54   8.96 -> 7.70 -> 6.95
// (the first column with the input matmul's share in it)
#pragma once

#include "rec_kernel.inc.h"

namespace lstm_int {

template <int KS16, int FL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void quad_kernel(RecArgs2 args) {
  constexpr bool cifg = FL & 1, ph = FL & 2, ln = FL & 4;
  constexpr int RG = 4;
  constexpr int LS = KS16 * 64 + 16;  // row stride of the h tiles
  constexpr int g_first = cifg ? 1 : 0;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, q = lane >> 4;
  const RecArgs &a0 = args.d[0];
  const int GS = a0.GS;

  // placement, as in rec_kernel
  const int wg = blockIdx.x;
  const int xcc = (int)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7);
  const int slot = wg >> 3;
  // both layers of the launch depend on where its workgroups are
  auto misplaced = [&]() {
    __hip_atomic_store(a0.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int *other = other_status<RecArgs2>();
    if (other) __hip_atomic_store(other, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  int xcd = wg & 7;
  if (a0.tickets) {
    xcd = xcc;
  } else if (xcc != xcd && tid == 0) {
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
  if (gl >= a0.groups + args.d[1].groups) {
    placement_check();
    return;
  }
  const int which = gl >= a0.groups ? 1 : 0;
  const RecDirArgs &a = args.d[which];
  const int row0 = a.batch0 + (gl - (which ? a0.groups : 0)) * RG;
  const bool proj = a.flags & 8;
  const int ldy = a.ldy;

  // ---- LDS carve-up (quad_lds_bytes mirrors it)
  const int MLS = ((a.N + 63) & ~63) + 16;  // row stride of the m tile and of W_proj
  uint8_t *p = lds;
  int8_t *hT = reinterpret_cast<int8_t *>(p);       p += 2 * RG * LS;
  int8_t *mT = reinterpret_cast<int8_t *>(p);       p += proj ? RG * MLS : 0;
  int16_t *txL = reinterpret_cast<int16_t *>(p);    p += 2 * 2048;  // W x terms of two steps
  u64 *red = reinterpret_cast<u64 *>(p);            p += 16 * 8;              // [gate][row] sums of the workgroup
  LnRow2 *lnrow = reinterpret_cast<LnRow2 *>(p);    p += 16 * sizeof(LnRow2);  // [gate][row]
  int *flag = reinterpret_cast<int *>(p);           p += 16;  // [0] 0: a wait gave up; [1] 1: every row has sigma >= 2^12
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
  int8_t *WpL = reinterpret_cast<int8_t *>(p);  // [my tiles][16 rows][MLS]
  const int N = a.N, H = a.H, T = a.T;
  // projection: tile ti of 16 outputs belongs to wave ti / GS of member ti % GS
  const int tiles = proj ? (H + 15) >> 4 : 0;
  const int my_tiles = tiles > member ? (tiles - member + GS - 1) / GS : 0;
  const int p0 = (member + wave * GS) * 16;  // first output of this wave's tile
  const bool has_tile = wave < my_tiles;

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
      for (int c = wave; c < nd + nb + nt; c += 4) {
        const int so = c < nd ? c * 1024 : (c < nd + nb ? kLutWideBaseOff + (c - nd) * 1024 : kLutWideTailOff + (c - nd - nb) * 1024);
        dma(a.lut[i].blob + so + lane * 16, lds + offD[i] + c * 1024);
      }
    }
    const int pieces = (MLS - 16) >> 4;
    for (int i = tid; i < my_tiles * 16 * pieces; i += 256) {
      const int rr = i / pieces, o = (i - rr * pieces) * 16;
      *reinterpret_cast<int4 *>(WpL + rr * MLS + o) =
          *reinterpret_cast<const int4 *>(a.Wp2 + (size_t)((member + (rr >> 4) * GS) * 16 + (rr & 15)) * a.npadp + o);
    }
  }
  v4i Wf[4][KS16];  // [gate]: lane (c16, q) holds bytes 16 q.. of each 64-deep k step of cell c16's row
  int32_t bh[4], Pq[3];
  double wL[4], wb[4];
  {
    // rec16_kernel's tile j holds, in row 4 q' + g, gate g of cell 4 q' + j
    const int4 *src = a.R2h + (size_t)((member * 4 + wave) * 4 + (c16 & 3)) * a.ks16 * 64 + 4 * (c16 >> 2) + 16 * q;
    constexpr int GB = KS16 <= 10 ? 4 : 2;  // gates whose loads are in flight together
#pragma unroll
    for (int g0 = 0; g0 < 4; g0 += GB) {
      int4 w[GB][KS16];
#pragma unroll
      for (int g = 0; g < GB; ++g)
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) w[g][ks] = ks < a.ks16 ? src[(size_t)ks * 64 + g0 + g] : int4{0, 0, 0, 0};
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < GB; ++g)
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) {
          Wf[g0 + g][ks] = v4i{w[g][ks].x, w[g][ks].y, w[g][ks].z, w[g][ks].w};
          asm volatile("" : "+a"(Wf[g0 + g][ks]));
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    const size_t n = (size_t)member * 64 + wave * 16 + c16;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      bh[g] = a.bh4[(size_t)g * a.Ncp + n];
      if (g < 3) Pq[g] = ph ? a.Pq3[(size_t)g * a.Ncp + n] : 0;
      wL[g] = ln ? ln_weight_scaled(a.Lq4[(size_t)g * a.Ncp + n]) : 0.0;
      wb[g] = ln ? ln_bias_scaled(a.qb4[(size_t)g * a.Ncp + n]) : 0.0;
    }
  }
  RescaleHi ps[4], pc[3], pl[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    ps[g] = rescale_hi_prepare(a.Mh[g], a.rh[g]);
    pl[g] = rescale_hi_prepare(a.Mln[g], ln ? a.rln[g] : 33);
    if (g < 3) pc[g] = rescale_hi_prepare(ph ? a.Mc[g] : 0, ph ? a.rc[g] : 33);
  }
  // The constants of the step in vector registers, of which there are plenty: as scalars they do not fit, and every use of
  // one that was spilled to a lane of a vector register is an instruction.
  auto in_vgpr = [](int32_t v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  auto rescale_in_vgpr = [&](RescaleHi v) { return RescaleHi{in_vgpr(v.M), in_vgpr(v.add), in_vgpr(v.sh), in_vgpr(v.k)}; };
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    ps[g] = rescale_in_vgpr(ps[g]);
    if (ln) pl[g] = rescale_in_vgpr(pl[g]);
    if (ph && g < 3) pc[g] = rescale_in_vgpr(pc[g]);
  }
  // the h tile before step 0; the other tile and m start as zeros (bytes past a row's real ones only meet zero weights)
  for (int i = tid; i < 2 * RG * LS / 4; i += 256) {
    const int o = 4 * i, rr = o / LS, c = o - rr * LS;
    const int rw = row0 + rr < a.B ? row0 + rr : a.B - 1;
    reinterpret_cast<int32_t *>(hT)[i] = rr < RG && c < a.Hpad ? *reinterpret_cast<const int32_t *>(a.h0 + (size_t)rw * a.Hpad + c) : 0;
  }
  if (proj)
    for (int i = tid; i < RG * MLS / 4; i += 256) reinterpret_cast<int32_t *>(mT)[i] = 0;
  if (tid < 16) red[tid] = 0;
  if (tid == 0) flag[0] = 1;
  const bool row_ok = row0 + q < a.B;
  const int row = row_ok ? row0 + q : a.B - 1;  // rows past the batch repeat the last one and are not stored
  const int cell = member * 64 + wave * 16 + c16;
  int32_t creg = (a.c_in && cell < N) ? a.c_in[(size_t)row * N + cell] : 0;
  const double inv_n = 1.0 / (double)N;
  const bool pre_ln = ln && (a.rln[0] < 33 || a.rln[1] < 33 || a.rln[2] < 33 || a.rln[3] < 33);
  const bool pre_m = a.rm < 33;
  const int pre_h = a.pre_h, rev = a.rev;
  const RescaleHi pm = rescale_in_vgpr(rescale_hi_prepare(a.Mm, a.rm));
  const RescaleHi pp = rescale_in_vgpr(rescale_hi_prepare(proj ? a.Mp : 0, proj ? a.rp : 33));
  int dom[3], sh[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    dom[i] = in_vgpr(a.lut[i].dom);
    sh[i] = in_vgpr(a.lut[i].sh);
    offD[i] = in_vgpr(offD[i]);
    offB[i] = in_vgpr(offB[i]);
  }
  const int32_t zp_m = a.zp_m, zp_h = a.zp_h, m_c = a.m_c;
  const int32_t bp = has_tile && p0 + c16 < H ? a.bp2[p0 + c16] : 0;

  // exchange words of this group: [2 slots][h of the group | m of the group | statistics round 0 | round 1]
  u64 *const xw = a.acc + (size_t)gl * GS * 2 * kQuadWgWords;
  const int slot_words = GS * kQuadWgWords;
  const int h_row_words = proj ? tiles * 4 : GS * 16, m_row_words = GS * 16;  // words of four cells per row
  u64 *const xh = xw, *const xm = xw + GS * 64, *const xs = xw + GS * 128;  // kQuadWgWords = 64 + 64 + 2 * 16
  const unsigned never = a.extra_arrivals ? 0x80u : 0;  // tests: a tag nobody stores in so few steps

  // W x terms of a step -> LDS, waves 2 and 3: piece p = ((tile 2 + half) 2 + quad) 4 + row holds gates 2 half, 2 half + 1 of
  // the four cells 4 quad.. of the tile of 8, as the input GEMM writes them for the 32-row kernel
  auto tx_request = [&](int t) {
    if (wave < 2) return;
    t = t < T ? t : T - 1;
    int8_t *dst = reinterpret_cast<int8_t *>(txL) + (t & 1) * 2048 + (wave - 2) * 1024;
    if (rev) t = T - 1 - t;
    const int pc2 = (wave - 2) * 64 + lane, rr = pc2 & 3, quad = (pc2 >> 2) & 1, half = (pc2 >> 3) & 1, tile = pc2 >> 4;
    const int4 *src = a.tx2 + ((((size_t)t * a.Bp + row0) >> 5) * (size_t)(GS * 8) + member * 8 + tile) * 128 + half * 64 +
                      ((row0 + rr) & 31) + 32 * quad;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
  };
  tx_request(0);
  if (T > 1) tx_request(1);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // a wait that gave up: every thread leaves the kernel at the next barrier
  auto give_up = [&]() {
    __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    flag[0] = 0;
  };
  auto spent = [&](int &budget) {
    --budget;
    return (budget & 15) == 0 && (budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0);
  };
  // (value, tag) words of `row_words` per row, a multiple of four, -> an LDS tile; a thread polls its words, two per load and U
  // loads per round, until all carry the tag
  auto poll_tile = [&](auto count, const u64 *src, int row_words, unsigned tag, int8_t *dst, int ld) {
    constexpr int U = decltype(count)::value;
    const uint32_t want = (tag & 0xFF) * 0x01000100u;
    const int half = row_words >> 1, pairs = 4 * half;
    for (int base = 0; base < pairs; base += 256 * U) {
      unsigned at[U];
      v4i w[U];
#pragma unroll
      for (int k = 0; k < U; ++k) at[k] = base + k * 256 + tid < pairs ? (unsigned)(base + k * 256 + tid) * 16 : 0;
      int budget = a.spin_limit;
      for (;;) {
        poll_pairs(src, at, w);
        uint32_t off = 0;
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
          for (int i = 0; i < 4; ++i) off |= (uint32_t)w[k][i] ^ want;
        if (__builtin_amdgcn_ballot_w64((off & 0xFF00FF00u) != 0) == 0) break;
        if (spent(budget)) {
          give_up();
          break;
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int c = base + k * 256 + tid;
        if (c < pairs) {
          const int rr = (c >= half) + (c >= 2 * half) + (c >= 3 * half);
          *reinterpret_cast<v2i *>(dst + rr * ld + 8 * (c - rr * half)) =
              v2i{(int)__builtin_amdgcn_perm((uint32_t)w[k][1], (uint32_t)w[k][0], 0x06040200u),
                  (int)__builtin_amdgcn_perm((uint32_t)w[k][3], (uint32_t)w[k][2], 0x06040200u)};
        }
      }
    }
  };
  // this lane's int8 value of the step -> the group: the four cells of a quad of lanes make a word
  auto publish = [&](u64 *dst, int32_t value, unsigned tag) {
    const int32_t b = (value & 0xFF) | (int32_t)((tag & 0xFF) << 8);
    const int32_t w = b | (__builtin_amdgcn_mov_dpp(b, 0xB1, 0xF, 0xF, true) << 16);  // lanes 0, 2 of a quad: cells (0, 1), (2, 3)
    const int32_t w2 = __builtin_amdgcn_mov_dpp(w, 0x4E, 0xF, 0xF, true);              // lane 0: the word of lane 2
    if ((lane & 3) == 0)
      __hip_atomic_store(dst, (u64)(uint32_t)w | (u64)(uint32_t)w2 << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // Statistics of a gate: the sums over the four cells of a quad of lanes (their squares, at most 2^30, fit 32 bits) go
  // into the workgroup's word of (gate, row), S2 in the bits above S1
  auto rot = [](int32_t x, auto ctrl) { return x + __builtin_amdgcn_mov_dpp(x, decltype(ctrl)::value, 0xF, 0xF, true); };
  auto add_stats = [&](int g, int32_t v) {
    using Q1 = std::integral_constant<int, 0xB1>;  // quad_perm [1,0,3,2]
    using Q2 = std::integral_constant<int, 0x4E>;  // quad_perm [2,3,0,1]
    const int32_t s1 = rot(rot(v, Q1{}), Q2{});
    const uint32_t s2 = (uint32_t)rot(rot((int32_t)((uint32_t)v * (uint32_t)v), Q1{}), Q2{});
    if ((lane & 3) == 0)
      __hip_atomic_fetch_add(&red[g * 4 + q], ((u64)s2 << 24) + (u64)(int64_t)s1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // x + the other half of the wave's / the neighbouring row of lanes' x
  auto add_far = [](int64_t x) {
    auto step = [](int64_t v, auto swap) {
      const auto lo = swap((uint32_t)v), hi = swap((uint32_t)(v >> 32));
      return (int64_t)(((u64)hi[0] << 32) | lo[0]) + (int64_t)(((u64)hi[1] << 32) | lo[1]);
    };
    x = step(x, [](uint32_t v) { return __builtin_amdgcn_permlane16_swap(v, v, false, false); });
    return step(x, [](uint32_t v) { return __builtin_amdgcn_permlane32_swap(v, v, false, false); });
  };
  // Wave 0: the workgroup's sums -> the group, tag | S2 (36 bits) | S1 + 2^22 (24 bits); the words of all members, a
  // quarter of them (U) in each quarter of the wave -> (mean, sigma) of the gates g_lo..g_hi.  (Words of the single waves
  // instead, without the workgroup barrier before, were four times as many to poll and 0.1 to 0.6 us slower.)
  auto collect_members = [&](auto count, int round, int g_lo, int g_hi, int t) {
    constexpr int U = decltype(count)::value;
    const int item = c16;  // (gate, row)
    const bool here = (item >> 2) >= g_lo && (item >> 2) <= g_hi;
    u64 *const words = xs + (size_t)(t & 1) * slot_words + round * GS * 16 + item;
    if (q == 0 && here) {
      const int64_t pk = (int64_t)red[item];
      red[item] = 0;  // the next adds come after the barrier below
      const int64_t S1 = ((pk + (1 << 23)) & 0xFFFFFF) - (1 << 23);
      __hip_atomic_store(words + member * 16, ((u64)((t + 1) & 15) << 60) | ((u64)((pk - S1) >> 24) << 24) | (u64)(S1 + (1 << 22)),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    const unsigned tag = ((unsigned)(t + 1) & 15) ^ (never ? 8u : 0);
    u64 v[U];
    int budget = a.spin_limit;
    for (;;) {
      unsigned off = 0;
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int mb = q + 4 * k;
        v[k] = __hip_atomic_load(words + (mb < GS ? mb : q < GS ? q : 0) * 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int k = 0; k < U; ++k) off |= ((unsigned)(v[k] >> 32) >> 28) ^ tag;
      if (__builtin_amdgcn_ballot_w64(here && off != 0) == 0) break;
      if (spent(budget)) {
        give_up();
        break;
      }
    }
    int64_t s1 = 0, s2 = 0;
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (q + 4 * k < GS) {
        s1 += (int64_t)((uint32_t)v[k] & 0xFFFFFF) - (1 << 22);
        s2 += (int64_t)((v[k] >> 24) & 0xFFFFFFFFFull);
      }
    const LnRow2 lr = ln_row2(add_far(s1), add_far(s2), N, inv_n);
    const bool narrow = __builtin_amdgcn_ballot_w64(here && !ln_row_is_narrow(lr)) == 0;
    if (here && q == 0) lnrow[item] = lr;
    if (lane == 0) flag[1] = narrow;
  };
  auto collect_stats = [&](int round, int g_lo, int g_hi, int t) -> bool {
    __syncthreads();
    if (wave == 0) {
      if (GS <= 8)
        collect_members(std::integral_constant<int, 2>{}, round, g_lo, g_hi, t);
      else if (GS <= 16)
        collect_members(std::integral_constant<int, 4>{}, round, g_lo, g_hi, t);
      else
        collect_members(std::integral_constant<int, 8>{}, round, g_lo, g_hi, t);
    }
    __syncthreads();
    return flag[0] != 0;
  };
  // layer norm of K gate sums
  auto normalize = [&](auto count, const int *gates, int32_t *v) {
    constexpr int K = decltype(count)::value;
    LnRow2 lr[K];
#pragma unroll
    for (int k = 0; k < K; ++k) lr[k] = lnrow[gates[k] * 4 + q];
    const bool narrow = __builtin_amdgcn_readfirstlane(flag[1]) != 0;
    __builtin_amdgcn_sched_barrier(0);
    if (narrow) {
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = ln_second_stage_narrow(v[k], lr[k], wL[gates[k]], wb[gates[k]]);
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) v[k] = ln_second_stage(v[k], lr[k], wL[gates[k]], wb[gates[k]]);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (pre_ln) v[k] = rescale_preshift(v[k], pl[gates[k]]);
      v[k] = rescale_sat16_pre<0>(v[k], pl[gates[k]]);
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
  const int arow = c16 >> 2;

  for (int t = 0; t < T; ++t) {
    const int8_t *hcur = hT + (t & 1) * RG * LS;
    int8_t *hnext = hT + ((t + 1) & 1) * RG * LS;
    const unsigned tag = (unsigned)(t + 1);
    int32_t gs[4];
    {
      v4i hf[KS16];
#pragma unroll
      for (int ks = 0; ks < KS16; ++ks) hf[ks] = *reinterpret_cast<const v4i *>(hcur + arow * LS + (q << 4) + ks * 64);
      int32_t tx[4];
#pragma unroll
      for (int g = g_first; g < 4; ++g) {
        const int piece = (((wave * 2 + (c16 >> 3)) * 2 + (g >> 1)) * 2 + ((c16 >> 2) & 1)) * 4 + q;
        tx[g] = txL[(t & 1) * 1024 + piece * 8 + (g & 1) * 4 + (c16 & 3)];
      }
      v4i acc[4];
#pragma unroll
      for (int g = g_first; g < 4; ++g) {
        acc[g] = v4i{bh[g], 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS16; ++ks) acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(hf[ks], Wf[g][ks], acc[g], 0, 0, 0);
      }
      // gate sums (Secs. 3.2.4/3.2.5); with a peephole the o gate is finished after c^t
      auto gate_sums = [&](auto pre_tag) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          if (g < g_first) continue;
          int32_t v = tx[g] + rescale_sat16_pre<decltype(pre_tag)::value>(acc[g][0], ps[g]);
          if (ph && g < 2) v += rescale_sat16_pre(mul_i24(Pq[g < 3 ? g : 0], creg), pc[g < 3 ? g : 0]);
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
    }
    if (ln) {
#pragma unroll
      for (int g = g_first; g < (ph ? 3 : 4); ++g) add_stats(g, gs[g]);
      if (!collect_stats(0, g_first, ph ? 2 : 3, t)) return;
    }

    // layer norm, sigma / tanh, cell update (Secs. 3.2.6, 3.2.1, 3.2.9, 3.2.7): f, z, then o unless a peephole keeps it for
    // later, then i unless it is coupled
    int32_t xo;
    {
      constexpr int KG = 4 - (ph ? 1 : 0) - (cifg ? 1 : 0);
      const int gates[4] = {1, 2, ph ? 0 : 3, 0}, tb[4] = {0, 1, 0, 0};
      int32_t x[4], tv[4];
#pragma unroll
      for (int k = 0; k < KG; ++k) x[k] = gs[gates[k]];
      if (ln) normalize(std::integral_constant<int, KG>{}, gates, x);
      lookup(std::integral_constant<int, KG>{}, x, tb, tv);
      const int32_t fg = mirror_sigmoid(x[0], tv[0]);
      const int32_t ig = cifg ? cifg_input_gate(fg) : mirror_sigmoid(x[KG - 1], tv[KG - 1]);
      xo = ph ? 0 : mirror_sigmoid(x[2], tv[2]);
      creg = cell_update32(ig, mirror_tanh(x[1], tv[1]), fg, creg, m_c);
    }
    if (ph) {  // finish the o gate sum with P_o . c^t (eq. 5)
      gs[3] = clamp_i32(gs[3] + rescale_sat16_pre(mul_i24(Pq[2], creg), pc[2]), glo, 32767);
      if (ln) {
        add_stats(3, gs[3]);
        if (!collect_stats(1, 3, 3, t)) return;
      }
    }
    // hidden state (Sec. 3.2.7)
    {
      const int tb[2] = {2, 0}, gates[1] = {3};
      int32_t x[2] = {creg, gs[3]}, tv[2];
      if (ph && ln) normalize(std::integral_constant<int, 1>{}, gates, x + 1);
      lookup(std::integral_constant<int, ph ? 2 : 1>{}, x, tb, tv);
      const int32_t o = ph ? mirror_sigmoid(x[1], tv[1]) : xo;
      int32_t om = mul_i24(o, mirror_tanh(x[0], tv[0]));
      if (pre_m) om = rescale_preshift(om, pm);
      const int32_t mq = sat8(rescale_sat16_pre<0>(om, pm) + zp_m);
      publish((proj ? xm : xh) + (size_t)(t & 1) * slot_words + q * m_row_words + member * 16 + wave * 4 + (c16 >> 2), mq, tag);
    }
    // projection (Sec. 3.2.8): a tile of 16 outputs per wave, the whole depth in one wave
    if (proj && my_tiles > 0) {
      if (GS <= 16)
        poll_tile(std::integral_constant<int, 2>{}, xm + (size_t)(t & 1) * slot_words, m_row_words, tag ^ never, mT, MLS);
      else
        poll_tile(std::integral_constant<int, 4>{}, xm + (size_t)(t & 1) * slot_words, m_row_words, tag ^ never, mT, MLS);
      __syncthreads();
      if (flag[0] == 0) return;
      if (has_tile) {
        v4i pacc = v4i{bp, 0, 0, 0};
        const int8_t *ma = mT + arow * MLS + (q << 4), *wp = WpL + (wave * 16 + c16) * MLS + (q << 4);
        for (int ks = 0; ks < GS; ks += 4) {  // four steps' operands in flight together
          v4i mf[4], wf[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int kk = ks + k < GS ? ks + k : GS - 1;
            mf[k] = *reinterpret_cast<const v4i *>(ma + kk * 64);
            wf[k] = *reinterpret_cast<const v4i *>(wp + kk * 64);
          }
#pragma unroll
          for (int k = 0; k < 4; ++k)
            pacc = __builtin_amdgcn_mfma_i32_16x16x64_i8(ks + k < GS ? mf[k] : v4i{0, 0, 0, 0}, wf[k], pacc, 0, 0, 0);
        }
        const int32_t hq = sat8(rescale_sat16_pre(pacc[0], pp) + zp_h);
        publish(xh + (size_t)(t & 1) * slot_words + q * h_row_words + (p0 >> 2) + (c16 >> 2), hq, tag);
      }
    }
    // a wave without words (narrow projections) does not poll: its loads of some word or other cost as much as the others'
    if (!proj || wave * 64 < 2 * h_row_words)
      poll_tile(std::integral_constant<int, KS16 <= 8 ? 1 : 2>{}, xh + (size_t)(t & 1) * slot_words, h_row_words, tag ^ never, hnext, LS);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the W x terms asked for a step ago are in LDS (a wave may have had nothing to poll)
    __syncthreads();
    if (flag[0] == 0) return;
    tx_request(t + 2 < T ? t + 2 : t);  // (past the end: the buffer of step t again, with what it holds)
    if (wave == 1) {  // this workgroup's share of the output columns, four at a time
      const int quads = (H + 3) >> 2, share = (quads + GS - 1) / GS;  // at most 16 per row
      const int rr = lane >> 4, c = member * share + c16;
      if (c16 < share && c < quads && row0 + rr < a.B) {
        const size_t orow = (size_t)(rev ? T - 1 - t : t) * a.B + row0 + rr;
        const uint32_t v = *reinterpret_cast<const uint32_t *>(hnext + rr * LS + 4 * c);
        *reinterpret_cast<uint32_t *>(a.out + orow * a.Hpad + 4 * c) = v;
        if (a.y) {
          int8_t *yd = a.y + orow * ldy + 4 * c;
          if ((ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(a.y) & 3) == 0 && 4 * c + 3 < H)
            *reinterpret_cast<uint32_t *>(yd) = v;
          else
            for (int k = 0; k < 4 && 4 * c + k < H; ++k) yd[k] = (int8_t)(v >> (8 * k));
        }
      }
    }
  }
  placement_check();
  if (a.c_out && row_ok && cell < N) a.c_out[(size_t)row * N + cell] = (int16_t)creg;
}

typedef void (*quad_fn)(RecArgs2);

// kernel for (flags & 7)
template <int KS16>
quad_fn quad_pick_ks(int fl) {
  switch (fl & 7) {
    case 0: return quad_kernel<KS16, 0>;
    case 1: return quad_kernel<KS16, 1>;
    case 2: return quad_kernel<KS16, 2>;
    case 3: return quad_kernel<KS16, 3>;
    case 4: return quad_kernel<KS16, 4>;
    case 5: return quad_kernel<KS16, 5>;
    case 6: return quad_kernel<KS16, 6>;
    default: return quad_kernel<KS16, 7>;
  }
}

}  // namespace lstm_int

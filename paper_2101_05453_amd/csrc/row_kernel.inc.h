// Recurrent kernel for layers of up to 256 cells and small batches: ONE workgroup runs all T steps of ONE batch row, and the
// four gates of a cell are worked on by four lanes at once.
//
// solo_kernel, which takes these layers at larger batches, has four rows per workgroup and a lane per (row, cell), which works
// through its four gates one after the other.  A step there is a chain of 130 to 330 instructions of a wave, three quarters of
// them the same for each gate.  A small batch leaves most of the chip idle in that form (37 rows are 10 workgroups); with a
// row per workgroup the same number of waves has a lane per (gate, cell) and issues about half of the instructions per step.
// The 16x16x64 MFMA gets the row's h as every row of its first operand, so that each of the four groups of 16 lanes holds the
// sums of all four gates for the wave's 16 cells; lane (c = lane % 16, q = lane / 16) keeps gate q of cell c through rescale,
// layer norm and table, with the gate's constants in vector registers.  Three lane swaps (v_permlane16_swap,
// v_permlane32_swap) then give every lane all four gates of its cell, and the cell update runs in the four lanes alike.  With
// coupled gates, group 0 repeats the f gate.
//
// Everything else is as in solo_kernel: h, m and the layer-norm sums pass through LDS, no workgroup waits for another, but in a launch
// of several layers (kRowStack) for the layer below.
//
// What bounds it: the chain of a step, 64 cells 0.5 us (product 0.1, two table lookups 0.1 each, the arithmetic between them one
// dependent instruction per 8 clocks), layer norm 0.45 us more; with 16 waves (129 to 256 cells, 1.1 us) the issue of four waves a
// SIMD and 64 matrix instructions of 16 rows for one.  What had to go: every wait for global memory inside a step (lds_add_u64,
// lds_barrier; the W x terms eight or 16 steps ahead; with them 64 cells take 77 instead of 62 us for 100 steps), and, with 16
// waves and 128 registers a lane, every spilled register, whose reload returns behind those terms (203 cells, peephole and layer
// norm 382 -> 269 us).  Measured: row_inst.hip.
#pragma once

#include "rec_kernel.inc.h"
#include "row_stack_plan.h"

namespace lstm_int {

// Steps whose W x terms are on their way.  A wave waits until at most so many of its memory operations are open, two stores per
// step among them: a term has at least five steps of 0.4 us, with 16 waves two of 1.2 us, to come from memory.
constexpr int row_ahead(int waves) { return waves == 16 ? 8 : 16; }
// Most steps whose W x terms a launch computes itself, all of them ahead of its first step, and bytes of LDS for a wave's terms:
// those of all steps then, and otherwise of the steps on their way, however many steps the launch has.
constexpr int row_input_steps(int waves) { return waves == 16 ? 16 : 64; }
__host__ __device__ constexpr int row_terms_bytes(int waves, int T, bool own) {
  return (own && T > row_ahead(waves) ? T : row_ahead(waves)) * 128;
}

// Where a wave's W x terms come from
constexpr int kRowTerms = 0;  // tx2, a ring of the steps on their way
constexpr int kRowOwn = 1;    // computed here, all steps ahead of the first
constexpr int kRowStack = 2;  // a launch of several layers: computed here, a piece of the sequence at a time, as soon as the layer
                              // below has it; or, with tx2, its terms a piece ahead

// The LDS of a launch, from the front (row_lds_bytes mirrors it): h twice, m, sums, statistics, W x terms, tables.
// KS16: k steps of R h, as the outputs ask for: with 16 waves (129 to 256 cells) two to four (each that is not there saves 16 of 64 products
// a wave and 16 of its 128 registers: layers of 129 to 192 cells 0.93 of the time with four, up to 128 outputs of wider ones 0.85)
// FL: bit 0 coupled gates, bit 1 peephole, bit 2 layer norm, bit 3 projection.  MODE: kRow...
// kRowStack: several layers in one launch, a workgroup per (layer, row).  Rows never interact, so a layer's workgroup waits for one
// other alone, that of the same row in the layer below, and for nobody above it; a row's workgroups take its layers in the order in
// which they start, from the bottom, so that whoever is waited for has started (row_stack_plan.h).
template <int WAVES, int KS16, int FL, int MODE>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES == 4 ? 2 : WAVES / 4, WAVES == 4 ? 2 : WAVES / 4)))
void row_kernel(std::conditional_t<MODE == kRowStack, RowStackArgs, RowArgs> all) {
  constexpr bool OWN = MODE == kRowOwn, STACK = MODE == kRowStack;
  constexpr bool cifg = FL & 1, ph = FL & 2, ln = FL & 4, proj = FL & 8;
  constexpr int NC = 16 * WAVES;  // cells and outputs of the workgroup at most
  constexpr int KSP = NC / 64;    // k steps of the projection (KS16: of R h)
  const int waves = (int)(blockDim.x >> 6), NT = (int)blockDim.x;  // as many as the layer has blocks of 16 cells or outputs
  // Statistics to (mean, sigma) form, a chain of 60 dependent instructions: up to two waves a SIMD every wave does it for
  // itself, which costs no more than one wave and saves a barrier; with four it would take the SIMD twice as long
  constexpr bool STATS_BY_ALL = WAVES <= 8;
  constexpr bool LEAN = WAVES == 16;  // 128 registers a lane, 64 of them recurrent weights
  constexpr int AHEAD = row_ahead(WAVES);
  constexpr int LS = NC + 16;         // row stride of W_proj in LDS (LEAN)
  constexpr int g_first = cifg ? 1 : 0;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, q = lane >> 4;
  const int gq = cifg && q == 0 ? 1 : q;  // this lane's gate
  // the layer of the launch this workgroup works on, and its row (written out: through functions that return references the
  // kernels of one layer take two registers more, which 16 waves with peephole and layer norm do not have)
  int which, row = (int)blockIdx.x;
  if constexpr (STACK) {
    const RowStackPlace place = row_stack_place((int)blockIdx.x, all.rec.d[0].B, all.dirs);
    int *const order = reinterpret_cast<int *>(lds + 3 * NC + 16 * 8 + 4 * sizeof(LnRow2)) + 2;  // (behind `flag`, not written again)
    if (tid == 0)
      *order = __hip_atomic_fetch_add(all.in[0].done + place.chain * kRowFlagWords + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    // (in scalar registers again: the compiler carries what the branch above has read in vector ones, and the arguments with it)
    which = __builtin_amdgcn_readfirstlane(row_stack_link(*order, place.dir, all.dirs));
    row = __builtin_amdgcn_readfirstlane(place.row);
  } else {
    which = (int)blockIdx.x >= all.rec.d[0].groups ? 1 : 0;
    row -= which ? all.rec.d[0].groups : 0;
  }
  const auto &a = all.rec.d[which];
  const RowInput &in = all.in[which];
  const int T = a.T, N = a.N, H = a.H, rev = a.rev, ldy = a.ldy;

  uint8_t *p = lds;
  int8_t *hT = reinterpret_cast<int8_t *>(p);     p += 2 * NC;
  int8_t *mT = reinterpret_cast<int8_t *>(p);     p += NC;
  u64 *red = reinterpret_cast<u64 *>(p);          p += 16 * 8;  // [step % 2][round][gate] sums
  LnRow2 *lnrow = reinterpret_cast<LnRow2 *>(p);  p += 4 * sizeof(LnRow2);
  int *flag = reinterpret_cast<int *>(p);         p += 64;  // 1: every gate's sigma >= 2^12
  v4i *tables = reinterpret_cast<v4i *>(p);       p += 128;  // LEAN: [gates, second lookups][lane group]
  p = lds + (((size_t)(p - lds) + 1023) & ~(size_t)1023);
  // W x terms: [step % AHEAD][wave][8 pieces of 16 bytes], or, computed here, [step][wave][gate][16 cells]; of several layers
  // [wave][step of the piece] of either kind, of two pieces by turns with tx2
  const int piece = STACK ? in.piece : 0;
  const bool from_tx = STACK && in.x == nullptr;
  uint8_t *const txL = p + wave * (STACK ? in.term_steps * 128 : 128);
  p += WAVES * (STACK ? in.term_steps * 128 : row_terms_bytes(WAVES, T, OWN));
  int8_t *const xT = reinterpret_cast<int8_t *>(p);  // several layers: x of a piece as MFMA operands, [k step][lane][16 bytes]
  p += STACK ? in.x_bytes : 0;
  double *const lnL = reinterpret_cast<double *>(p) + tid * 2;  // LEAN: layer-norm weight and bias of the lane's gate and cell
  p += ln && LEAN ? 64 * WAVES * 16 : 0;
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
  int8_t *const WpL = reinterpret_cast<int8_t *>(p);  // [round_up(H, 16)][LS]

  // ---- once: tables -> LDS, weights and per-cell parameters -> registers
  auto dma = [&](const void *src, const void *dst) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                     (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
  };
  for (int i = 0; i < (share_tanh ? 2 : 3); ++i) {
    const int nd = a.lut[i].dom >> 10;
    const int nb = (((a.lut[i].dom >> a.lut[i].sh) * 2) + 1023) >> 10;
    const int nt = a.lut[i].tail ? 3 : 0;
    for (int c = wave; c < nd + nb + nt; c += waves) {
      const int so = c < nd ? c * 1024 : (c < nd + nb ? kLutWideBaseOff + (c - nd) * 1024 : kLutWideTailOff + (c - nd - nb) * 1024);
      dma(a.lut[i].blob + so + lane * 16, lds + offD[i] + c * 1024);
    }
  }
  const bool real = wave < (a.Ncp >> 4);  // the layer has this block of 16 cells (cells past N are zero weights)
  // W x of up to 16 steps t0 .. tn - 1 of the row: the steps are the rows of the MFMA's first operand (step t0 + lane % 16), the second is the
  // input GEMM's operand of two tiles of eight cells, gathered; a lane ends with cell c16 in steps 4 q + v.
  constexpr int TERM_STRIDE = STACK ? 128 : WAVES * 128;  // LDS bytes from a step's terms to the next one's
  auto input_row = [&](int t0, int tn) {
    const int t = t0 + c16 < tn ? t0 + c16 : tn - 1;
    return in.x + ((size_t)(rev ? T - 1 - t : t) * a.B + row) * in.ldx + (q << 4);
  };
  auto input_weights = [&]() { return in.W2f + ((size_t)(wave * 2 + (c16 >> 3)) * 2 * in.kx + (q >> 1)) * 1024 + ((c16 & 7) + 32 * (q & 1)) * 16; };
  auto input_terms = [&](int t0, int tn, uint8_t *dst) {
    const int8_t *xr = STACK ? xT + lane * 16 : input_row(t0, tn);
    const int8_t *wr = input_weights();
    const int32_t *br = in.bx2 + (wave * 2 + (c16 >> 3)) * 32 + (c16 & 7);
    // With 16 waves the pieces of a sequence are worked out beside the recurrent weights, one gate at a time
    constexpr int GATES = STACK && LEAN ? 1 : 4, U = STACK && LEAN ? 2 : 4;  // U: k steps whose operands are on their way together
#pragma unroll
    for (int g0 = GATES == 4 ? 0 : g_first; g0 < 4; g0 += GATES) {
      const int g_from = GATES == 4 ? g_first : g0, g_end = g0 + GATES;
      v4i acc[GATES];
#pragma unroll
      for (int g = g_from; g < g_end; ++g) {
        const int32_t b = br[8 * g];
        acc[g - g0] = v4i{b, b, b, b};
      }
      for (int k0 = 0; k0 < in.kx; k0 += U) {
        v4i xf[U], wf[U][GATES];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int ks = k0 + u < in.kx ? k0 + u : in.kx - 1;
          if (!STACK) {
            xf[u] = v4i{0, 0, 0, 0};
            if (ks * 64 + (q << 4) < in.cols && k0 + u < in.kx) xf[u] = *reinterpret_cast<const v4i *>(xr + ks * 64);
          }
#pragma unroll
          for (int g = g_from; g < g_end; ++g) wf[u][g - g0] = *reinterpret_cast<const v4i *>(wr + (size_t)ks * 2048 + g * 128);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (STACK) {
            xf[u] = *reinterpret_cast<const v4i *>(xr + (k0 + u < in.kx ? k0 + u : in.kx - 1) * 1024);
            if (k0 + u >= in.kx) xf[u] = v4i{0, 0, 0, 0};
          }
#pragma unroll
          for (int g = g_from; g < g_end; ++g) acc[g - g0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xf[u], wf[u][g - g0], acc[g - g0], 0, 0, 0);
        }
      }
      if (__builtin_expect(in.pre, 0)) {
#pragma unroll
        for (int g = g_from; g < g_end; ++g)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[g - g0][v] = rescale_preshift(acc[g - g0][v], in.rs[g]);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int t = t0 + 4 * q + v;  // steps past the last one go to a place nobody reads
        uint8_t *const to = t < tn ? dst + (OWN ? t : 4 * q + v) * TERM_STRIDE + c16 * 2 : reinterpret_cast<uint8_t *>(flag) - g_from * 32 + 4;
#pragma unroll
        for (int g = g_from; g < g_end; ++g)
          *reinterpret_cast<int16_t *>(to + (t < tn ? g : g_from) * 32) = (int16_t)rescale_sat16_pre<0>(acc[g - g0][v], in.rs[g]);
      }
    }
  };
  // (with LEAN ahead of the recurrent weights, which take the registers)
  if (OWN && real)
    for (int t0 = 0; t0 < T; t0 += 16) input_terms(t0, T, txL);
  v4i Wf[4][KS16];  // [gate]: lane (c16, q) holds bytes 16 q.. of each 64-deep k step of cell c16's row
  v4i Wp[proj && !LEAN ? KSP : 1];  // W_proj: the same of output 16 wave + c16
  const size_t n = (real ? wave : 0) * 16 + c16;
  {
    // rec16_kernel's tile j holds, in row 4 q' + g, gate g of cell 4 q' + j
    const int4 *src = a.R2h + (size_t)((real ? wave : 0) * 4 + (c16 & 3)) * a.ks16 * 64 + 4 * (c16 >> 2) + 16 * q;
    int4 w[4][KS16], wp[KSP];
#pragma unroll
    for (int g = g_first; g < 4; ++g)
#pragma unroll
      for (int ks = 0; ks < KS16; ++ks) w[g][ks] = real ? src[(size_t)ks * 64 + g] : int4{0, 0, 0, 0};
    if (proj && LEAN) {  // output rows of npadp >= N bytes each
      const int rows = (H + 15) & ~15, pieces = KSP * 4;
      for (int i = tid; i < rows * pieces; i += NT) {
        const int o = i / pieces, k = (i - o * pieces) * 16;
        int4 v = {0, 0, 0, 0};
        if (k < a.npadp) v = *reinterpret_cast<const int4 *>(a.Wp2 + (size_t)o * a.npadp + k);
        *reinterpret_cast<int4 *>(WpL + o * LS + k) = v;
      }
    }
    if (proj && !LEAN) {
      const int o = wave * 16 + c16;
#pragma unroll
      for (int ks = 0; ks < KSP; ++ks) {
        const int k = ks * 64 + q * 16;
        wp[ks] = int4{0, 0, 0, 0};
        if (o < H && k < a.npadp) wp[ks] = *reinterpret_cast<const int4 *>(a.Wp2 + (size_t)o * a.npadp + k);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = g_first; g < 4; ++g)
#pragma unroll
      for (int ks = 0; ks < KS16; ++ks) {
        Wf[g][ks] = v4i{w[g][ks].x, w[g][ks].y, w[g][ks].z, w[g][ks].w};
        asm volatile("" : "+v"(Wf[g][ks]));
      }
    if (proj && !LEAN)
#pragma unroll
      for (int ks = 0; ks < KSP; ++ks) {
        Wp[ks] = v4i{wp[ks].x, wp[ks].y, wp[ks].z, wp[ks].w};
        asm volatile("" : "+v"(Wp[ks]));
      }
    __builtin_amdgcn_sched_barrier(0);
  }
  auto of_gate = [&](int32_t v0, int32_t v1, int32_t v2, int32_t v3) {  // the lane's own of four values
    const int32_t lo = q & 1 ? v1 : (cifg ? v1 : v0), hi = q & 1 ? v3 : v2;
    return q & 2 ? hi : lo;
  };
  // A rescale in the high-word form (lstm_int_math.h) with the lane's gate's constants; with LEAN one register less and an
  // instruction more: floor((hi + 2^(s-1)) / 2^s) = floor((floor(hi / 2^(s-1)) + 1) / 2).  Shifts below 33 shift the operand up
  // first (and clamp it, which changes nothing where it is not needed): rare, in a branch of its own that looks the shift up.
  struct Rescale {
    int32_t M, add, sh;
  };
  auto rescale_of_gate = [&](const int32_t *M, const int32_t *r) {
    const RescaleHi v = rescale_hi_prepare(of_gate(M[0], M[1], M[2], M[3]), of_gate(r[0], r[1], r[2], r[3]));
    return LEAN ? Rescale{v.M, 0, v.sh - 1} : Rescale{v.M, v.add, v.sh};
  };
  auto rescaled16 = [&](int32_t v, const Rescale &c, bool low_shifts, auto shift_of) {
    if (__builtin_expect(low_shifts, 0)) {
      asm volatile("" : "+v"(v));  // a branch, not both ways and a select
      const int32_t r = shift_of();
      v = rescale_preshift(v, RescaleHi{0, 0, 0, r < 33 ? 33 - r : 0});
    }
    const int32_t hi = __mulhi(v, c.M);
    return sat16(LEAN ? ((hi >> c.sh) + 1) >> 1 : (hi + c.add) >> c.sh);
  };
  const Rescale ps = rescale_of_gate(a.Mh, a.rh);
  const Rescale pl = ln ? rescale_of_gate(a.Mln, a.rln) : Rescale{0, 0, 0};
  // peephole: i and f look at the old state, o at the new one (z has no weight: a product of 0)
  const int32_t Mc[4] = {a.Mc[0], a.Mc[1], a.Mc[1], a.Mc[2]}, rc[4] = {a.rc[0], a.rc[1], a.rc[1], a.rc[2]};
  const Rescale pc = ph ? rescale_of_gate(Mc, rc) : Rescale{0, 0, 0};
  const int32_t Pold = ph && real && gq < 2 ? a.Pq3[(size_t)gq * a.Ncp + n] : 0;
  const int32_t Pnew = ph && real && q == 3 ? a.Pq3[(size_t)2 * a.Ncp + n] : 0;
  const int32_t bh = real ? a.bh4[(size_t)gq * a.Ncp + n] : 0;
  const double wL = ln && real ? ln_weight_scaled(a.Lq4[(size_t)gq * a.Ncp + n]) : 0.0;
  const double wb = ln && real ? ln_bias_scaled(a.qb4[(size_t)gq * a.Ncp + n]) : 0.0;
  if (ln && LEAN) {
    lnL[0] = wL;
    lnL[1] = wb;
  }
  // tables of the gates and of the second lookups (the o gate with a peephole, else tanh of the cell state): last entry, bases,
  // block shift, deltas
  auto table = [&](int i) { return v4i{a.lut[i].dom - 1, offB[i], a.lut[i].sh, offD[i]}; };
  auto choose = [](bool first, const v4i &x, const v4i &y) {
    return v4i{first ? x[0] : y[0], first ? x[1] : y[1], first ? x[2] : y[2], first ? x[3] : y[3]};
  };
  const v4i gate_table = choose(q == 2, table(1), table(0)), late_table = choose(ph && q == 3, table(0), table(2));
  if (LEAN && wave == 0 && c16 == 0) {
    tables[q] = gate_table;
    tables[4 + q] = late_table;
  }

  if (tid < 16) red[tid] = 0;
  // h before step 0; the other half and m start as zeros (bytes past the real ones only meet zero weights)
  for (int i = tid; i < 3 * NC; i += NT) {
    int8_t v = 0;
    if (i < H) v = MODE == kRowTerms ? a.h0[(size_t)row * a.Hpad + i] : in.h_src ? in.h_src[(size_t)row * H + i] : (int8_t)a.zp_h;
    hT[i] = v;
  }
  const int cell = wave * 16 + c16;  // this lane's cell, and its output of the projection
  int32_t creg = (a.c_in && cell < N) ? a.c_in[(size_t)row * N + cell] : 0;
  double inv_n = 1.0 / (double)N;
  if (STACK)  // in scalar registers, where it is not spilled: a reload would wait for the stores of the output
    inv_n = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(inv_n)), __builtin_amdgcn_readfirstlane(__double2loint(inv_n)));
  const bool pre_ln = ln && (a.rln[0] < 33 || a.rln[1] < 33 || a.rln[2] < 33 || a.rln[3] < 33);
  const bool pre_m = a.rm < 33, pre_p = proj && a.rp < 33;
  const bool pre_h = a.pre_h != 0;
  const bool pre_c = ph && ((!cifg && a.rc[0] < 33) || a.rc[1] < 33 || a.rc[2] < 33);
  const RescaleHi pm = rescale_hi_prepare(a.Mm, a.rm), pp = rescale_hi_prepare(proj ? a.Mp : 0, proj ? a.rp : 33);
  const int32_t zp_m = a.zp_m, zp_h = a.zp_h, m_c = a.m_c;
  const int32_t bp = proj && cell < H ? a.bp2[cell] : 0;

  // W x terms of a step, as the input GEMM writes them for the 32-row kernel: value (gate, cell) of row b is the int16
  // [cell tile of 8][gate / 2][b % 32 + 32 * (cell / 4 % 2)][4 (gate % 2) + cell % 4] of the row's block.  The wave's 16 cells
  // are eight pieces of 16 bytes, fetched by lanes 0 to 7 straight into LDS.
  const size_t tx_step = (size_t)(a.Bp >> 5) * (a.Ncp >> 3) * 1024;  // int16 values of one step
  const int16_t *const tx_base = reinterpret_cast<const int16_t *>(a.tx2) +
                                 ((size_t)(row >> 5) * (a.Ncp >> 3) + (real ? wave : 0) * 2 + ((lane >> 2) & 1)) * 1024 +
                                 ((lane >> 1) & 1) * 512 + ((row & 31) + 32 * (lane & 1)) * 8;
  const int16_t *tx_src = tx_base + (rev ? (size_t)(T - 1) * tx_step : 0);
  const long long tx_ahead = rev ? -(long long)tx_step : (long long)tx_step;
  auto tx_request = [&](int t) {  // steps in their order; past the end the last one again, into places nobody reads any more
    if (lane < 8) dma(tx_src, txL + (t & (AHEAD - 1)) * WAVES * 128);
    tx_src += t + 1 < T ? tx_ahead : 0;
  };
  const int tx_at = OWN || (STACK && !from_tx) ? gq * 32 + c16 * 2 : ((c16 >> 3) * 4 + (gq >> 1) * 2 + ((c16 >> 2) & 1)) * 16 + ((gq & 1) * 4 + (c16 & 3)) * 2;
  // several layers: the terms of steps t0 .. tn - 1 (at most 16), eight steps per load of the wave
  auto piece_request = [&](int t0, int tn, uint8_t *dst) {
    for (int s = 0; t0 + s < tn; s += 8) {
      const int t = t0 + s + (lane >> 3), l8 = lane & 7;
      const int16_t *src = reinterpret_cast<const int16_t *>(a.tx2) + (size_t)(rev ? T - 1 - t : t) * tx_step +
                           ((size_t)(row >> 5) * (a.Ncp >> 3) + (real ? wave : 0) * 2 + (l8 >> 2)) * 1024 + ((l8 >> 1) & 1) * 512 +
                           ((row & 31) + 32 * (l8 & 1)) * 8;
      if (t < tn) dma(src, dst + s * 128);
    }
  };
  if (MODE == kRowTerms)
    for (int s = 0; s < AHEAD && s < T; ++s) tx_request(s);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // The sums of v and of v^2 over the cells into the gate's word, S2 in the bits above S1: the squares of the four cells of a
  // quad of lanes (at most 2^30 each) fit 32 bits, the quads add into the word
  auto rot = [](int32_t x, auto ctrl) { return x + __builtin_amdgcn_mov_dpp(x, decltype(ctrl)::value, 0xF, 0xF, true); };
  auto add_stats = [&](u64 *word, int32_t v, bool mine) {
    using Q1 = std::integral_constant<int, 0xB1>;  // quad_perm [1,0,3,2]
    using Q2 = std::integral_constant<int, 0x4E>;  // quad_perm [2,3,0,1]
    const int32_t s1 = rot(rot(v, Q1{}), Q2{});
    const uint32_t s2 = (uint32_t)rot(rot((int32_t)((uint32_t)v * (uint32_t)v), Q1{}), Q2{});
    if ((lane & 3) == 0 && mine) lds_add_u64(word, ((u64)s2 << 24) + (u64)(int64_t)s1);
  };
  auto row_of = [&](const u64 *word) {
    const int64_t pk = (int64_t)*word;
    const int32_t S1 = (int32_t)((uint32_t)pk << 8) >> 8;  // 256 values of at most 32767: below 2^23
    return ln_row2(S1, (pk - S1) >> 24, N, inv_n);
  };
  auto peephole = [&](int32_t weight, int32_t c) {
    return rescaled16(mul_i24(weight, c), pc, pre_c, [&] { return of_gate(a.rc[0], a.rc[1], a.rc[1], a.rc[2]); });
  };
  // layer norm of the lane's gate sum; `here`: lanes whose result is used
  auto normalize = [&](const u64 *word, int32_t v, bool here) {
    lds_barrier();  // the sums are complete
    LnRow2 lr;
    bool narrow;
    double cL = wL, cb = wb;
    if constexpr (STATS_BY_ALL) {
      lr = row_of(word);
      narrow = __builtin_amdgcn_ballot_w64(here && !ln_row_is_narrow(lr)) == 0;
    } else {
      if (wave == 0) {
        lr = row_of(word);
        narrow = __builtin_amdgcn_ballot_w64(here && !ln_row_is_narrow(lr)) == 0;
        if (c16 == 0) lnrow[q] = lr;
        if (lane == 0) flag[0] = narrow;
      }
      lds_barrier();
      lr = lnrow[q];
      cL = lnL[0];
      cb = lnL[1];
      narrow = __builtin_amdgcn_readfirstlane(flag[0]) != 0;
    }
    if (__builtin_expect(narrow, 1)) {
      v = ln_second_stage_narrow(v, lr, cL, cb);
    } else {
      asm volatile("" : "+v"(v));
      v = ln_second_stage(v, lr, cL, cb);
    }
    return rescaled16(v, pl, pre_ln, [&] { return of_gate(a.rln[0], a.rln[1], a.rln[2], a.rln[3]); });
  };
  // sigma (table 0) or tanh (1 gate, 2 cell) of x: the value for |x| from the lane's table (see rec_kernel's lookup), mirrored
  // as mirror_sigmoid and mirror_tanh do.  With LEAN the table's place is read from LDS, not kept in registers.
  auto activation = [&](int32_t x, int which_tables, bool tanh_lane, auto tail_of) {
    const v4i tb = LEAN ? tables[which_tables * 4 + q] : which_tables ? late_table : gate_table;
    const int32_t mag = abs_i32(x);
    const int32_t ai = mag < tb[0] ? mag : tb[0];
    const uint32_t base = *reinterpret_cast<const uint16_t *>(lds + tb[1] + 2 * (ai >> tb[2]));
    const uint32_t delta = lds[tb[3] + ai];
    int32_t v = (int32_t)(base + delta);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(mag > tb[0]) != 0, 0)) {
      const int tail = tail_of();
      if (tail && mag > tb[0]) v = lut_wide_tail(lds + tail, mag);
    }
    const int32_t s = sign_mask(x);
    v = (v ^ s) + (s & (tanh_lane ? 1 : 32769));  // ~v + 32769 = 32768 - v, ~v + 1 = -v
    return v > 32767 ? 32767 : v;
  };
  constexpr int32_t glo = ln ? -32767 : -32768;
  // the outputs of this lane's cell, moved on by a step at a time
  int8_t *out = a.out + ((size_t)(rev ? T - 1 : 0) * a.B + row) * a.Hpad, *y = (a.y ? a.y : a.out) + ((size_t)(rev ? T - 1 : 0) * a.B + row) * ldy;
  const long long out_step = rev ? -(long long)a.B * a.Hpad : (long long)a.B * a.Hpad, y_step = rev ? -(long long)a.B * ldy : (long long)a.B * ldy;
  const bool writes = q == 0 && cell < H, has_y = a.y != nullptr;

  // several layers: the terms of the step, the first step of the next piece, its half of the terms' LDS
  const uint8_t *tx_now = txL + tx_at;
  int next = 0, half = 0;
  bool gave_up = false;
  if constexpr (STACK) {
    if (from_tx) {
      piece_request(0, piece < T ? piece : T, txL);
    } else if (in.ready && real) {
      // while the layer below is on its way: the input weights into the L2
      const int8_t *wr = input_weights();
      for (int ks = 0; ks < in.kx; ++ks) {
        int32_t w[4];
#pragma unroll
        for (int g = g_first; g < 4; ++g) w[g] = *reinterpret_cast<const int32_t *>(wr + (size_t)ks * 2048 + g * 128);
#pragma unroll
        for (int g = g_first; g < 4; ++g) asm volatile("" ::"v"(w[g]));
      }
    }
  }

  for (int t = 0; t < T; ++t) {
    bool publish = false;
    if constexpr (STACK) {
      if (t == next) {
        publish = t > 0 && in.done;
        next = t + piece < T ? t + piece : T;
        if (from_tx) {
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this piece has landed; the next one is asked for
          if (next < T) piece_request(next, next + piece < T ? next + piece : T, txL + (half ^ 1) * piece * 128);
        } else {
          // x of the piece into LDS, a k step by a wave, past the L1 and the L2: another workgroup of the launch may have written it, on
          // another XCD.  (Every wave for itself, out of the product's loop, came to 1.5 us a piece more with 16 waves.)
          if (wave < in.kx) {
            if (in.ready && !gave_up) {
              const int *const flag = in.ready + row * kRowFlagWords;
              int budget = in.spin_limit;
              while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < next + in.never) {
                __builtin_amdgcn_s_sleep(1);
                if (--budget < 0) {  // the outputs are not valid; every later wait is skipped
                  gave_up = true;
                  if (lane == 0) __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                  break;
                }
              }
            }
            const int8_t *xr = input_row(t, next);
            for (int ks = wave; ks < in.kx; ks += waves) {
              // bytes that may not be read meet zero weights
              const int8_t *from = ks * 64 + (q << 4) < in.cols ? xr + ks * 64 : xr - (q << 4);
              __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from,
                                               (__attribute__((address_space(3))) void *)(xT + ks * 1024), 16, 0, 16 /* sc1 */);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          }
          lds_barrier();
          if (real) input_terms(t, next, txL);
        }
        tx_now = txL + (from_tx ? half * piece * 128 : 0) + tx_at;
        half ^= 1;
      }
    }
    const int8_t *hcur = hT + (t & 1) * NC;
    int8_t *hnext = hT + ((t + 1) & 1) * NC;
    u64 *const sums = red + (t & 1) * 8;
    v4i hf[KS16];
#pragma unroll
    for (int ks = 0; ks < KS16; ++ks) hf[ks] = *reinterpret_cast<const v4i *>(hcur + (q << 4) + ks * 64);
    // the terms of this step: the loads of the steps ahead are younger (and stores among them make the wait stricter)
    if (MODE == kRowTerms) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(AHEAD - 1) : "memory");
    const int32_t tx = *reinterpret_cast<const int16_t *>(STACK ? tx_now : txL + (OWN ? t : t & (AHEAD - 1)) * WAVES * 128 + tx_at);
    if (STACK) tx_now += 128;
    if (ln && tid < 8) red[((t + 1) & 1) * 8 + tid] = 0;  // read in the step before, added to in the next one
    int32_t acc[4];
#pragma unroll
    for (int g = g_first; g < 4; ++g) {
      v4i c = v4i{0, 0, 0, 0};
#pragma unroll
      for (int ks = 0; ks < KS16; ++ks) c = __builtin_amdgcn_mfma_i32_16x16x64_i8(hf[ks], Wf[g][ks], c, 0, 0, 0);
      acc[g] = c[0];
    }
    // gate sum (Secs. 3.2.4/3.2.5); with a peephole the o gate is finished after c^t
    int32_t s = of_gate(cifg ? 0 : acc[0], acc[1], acc[2], acc[3]) + bh;
    int32_t v = rescaled16(s, ps, pre_h, [&] { return of_gate(a.rh[0], a.rh[1], a.rh[2], a.rh[3]); }) + ((proj || STACK) && !real ? 0 : tx);
    if (ph) v += peephole(Pold, creg);
    const int32_t open = v;
    v = clamp_i32(v, glo, 32767);
    if (ln) add_stats(sums + q, v, true);
    asm volatile("" ::"v"(v));  // the term has been read: its place takes the one of a later step
    if (MODE == kRowTerms) tx_request(t + AHEAD);
    // layer norm, sigma / tanh (Secs. 3.2.6, 3.2.1)
    if (ln) v = normalize(sums + q, v, !(ph && q == 3));
    const int32_t act = activation(v, 0, q == 2, [&] { return q == 2 ? offT[1] : offT[0]; });
    // all four gates of the cell in each of its lanes
    const auto r16 = __builtin_amdgcn_permlane16_swap((uint32_t)act, (uint32_t)act, false, false);
    const auto even = __builtin_amdgcn_permlane32_swap(r16[0], r16[0], false, false);
    const auto odd = __builtin_amdgcn_permlane32_swap(r16[1], r16[1], false, false);
    const int32_t fg = (int32_t)odd[0], zg = (int32_t)even[1];
    const int32_t ig = cifg ? cifg_input_gate(fg) : (int32_t)even[0];
    int32_t og = (int32_t)odd[1];
    // cell update and hidden state (Secs. 3.2.9, 3.2.7)
    creg = cell_update32(ig, zg, fg, creg, m_c);
    int32_t tc;
    if constexpr (ph) {  // finish the o gate with P_o . c^t (eq. 5); its lanes look sigma up, the others tanh of the cell
      int32_t vo = clamp_i32(open + peephole(Pnew, creg), glo, 32767);
      if (ln) {
        add_stats(sums + 4, vo, q == 3);
        vo = normalize(sums + 4, vo, q == 3);
      }
      const int32_t late = activation(q == 3 ? vo : creg, 1, q != 3, [&] { return q == 3 ? offT[0] : offT[2]; });
      const auto l16 = __builtin_amdgcn_permlane16_swap((uint32_t)late, (uint32_t)late, false, false);
      tc = (int32_t)__builtin_amdgcn_permlane32_swap(l16[0], l16[0], false, false)[0];
      og = (int32_t)__builtin_amdgcn_permlane32_swap(l16[1], l16[1], false, false)[1];
    } else {
      tc = activation(creg, 1, true, [&] { return offT[2]; });
    }
    int32_t om = mul_i24(og, tc);
    if (__builtin_expect(pre_m, 0)) {
      asm volatile("" : "+v"(om));
      om = rescale_preshift(om, pm);
    }
    int8_t hq = (int8_t)sat8(rescale_sat16_pre<0>(om, pm) + zp_m);
    if (proj) {  // Sec. 3.2.8: 16 outputs per wave, the whole depth
      if (q == 0) mT[cell] = hq;
      lds_barrier();
      if (!LEAN || wave * 16 < H) {
        v4i pacc = v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KSP; ++ks)
          pacc = __builtin_amdgcn_mfma_i32_16x16x64_i8(*reinterpret_cast<const v4i *>(mT + (q << 4) + ks * 64),
                                                       LEAN ? *reinterpret_cast<const v4i *>(WpL + cell * LS + (q << 4) + ks * 64) : Wp[LEAN ? 0 : ks],
                                                       pacc, 0, 0, 0);
        int32_t sum = pacc[0] + bp;
        if (__builtin_expect(pre_p, 0)) {
          asm volatile("" : "+v"(sum));
          sum = rescale_preshift(sum, pp);
        }
        hq = (int8_t)sat8(rescale_sat16_pre<0>(sum, pp) + zp_h);
      }
    }
    if (q == 0) hnext[cell] = hq;
    if (STACK && publish) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the steps before this one have left
    lds_barrier();  // the next h is complete
    if (STACK && publish && tid == 0) __hip_atomic_store(in.done + row * kRowFlagWords, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (writes) {
      if (!STACK)
        out[cell] = hq;
      else if (in.done)  // for the layer above, through the L2
        __hip_atomic_store(out + cell, hq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else if (!has_y)
        out[cell] = hq;
      if (has_y) y[cell] = hq;
    }
    out += out_step;
    y += y_step;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing is on its way into LDS when the workgroup gives it back
  if (STACK && in.done) {
    __syncthreads();
    if (tid == 0) __hip_atomic_store(in.done + row * kRowFlagWords, T, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (MODE != kRowTerms && in.h_dst)
    for (int i = tid; i < H; i += NT) in.h_dst[(size_t)row * H + i] = hT[(T & 1) * NC + i];
  if (a.c_out && q == 0 && cell < N) a.c_out[(size_t)row * N + cell] = (int16_t)creg;
}

typedef void (*row_fn)(RowArgs);
typedef void (*row_stack_fn)(RowStackArgs);

// kernel for fl of FL to 15
template <int WAVES, int KS16, int MODE, int FL>
auto row_pick_size(int fl) -> decltype(&row_kernel<WAVES, KS16, 15, MODE>) {
  if constexpr (FL < 15) {
    return fl == FL ? row_kernel<WAVES, KS16, FL, MODE> : row_pick_size<WAVES, KS16, MODE, FL + 1>(fl);
  } else {
    return row_kernel<WAVES, KS16, 15, MODE>;
  }
}

}  // namespace lstm_int

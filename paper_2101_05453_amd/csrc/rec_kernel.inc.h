// Device code of the persistent recurrent kernel (see persistent.hip for the
// design).  Included by the rec_inst_*.hip translation units, which
// instantiate it for their k depth.
#pragma once

#include <type_traits>

#include "lstm_int_math.h"
#include "persistent.h"

namespace lstm_int {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned long long u64;

// ---------------------------------------------------------------------------
// Recurrent kernel
// ---------------------------------------------------------------------------

// Barrier among the GS workgroups of a group.  Every wave first waits for its
// own stores (vmcnt(0)); thread 0 then adds one to the group's counter and
// polls it, pausing poll_sleep x 64 clocks between polls: the polls of all the
// group's workgroups go to one L2 channel, the one that also serves the
// arrivals, and polling at full rate delays those (measured: every poller
// added made the barrier slower).  Gives up after spin_limit polls (or when
// another workgroup gave up), raising the status word so that every workgroup
// leaves the kernel; lds_flag[0] is then 0 for good.
__device__ __forceinline__ bool group_sync(unsigned *counter, unsigned &epoch, int GS, int *status,
                                           int spin_limit, int first_sleep, int poll_sleep, int *lds_flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (GS == 1) return true;
  epoch += (unsigned)GS;
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // a workgroup that knows the others have work left before they arrive keeps off the counter meanwhile
    for (int i = 0; i < first_sleep; ++i) __builtin_amdgcn_s_sleep(1);
    int budget = spin_limit;
    for (;;) {
      const unsigned c = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((int)(c - epoch) >= 0) break;
      // the status word (another workgroup gave up) is looked at every 16th poll: each look is one more request
      // in the polling thread's queue (measured: 0.3 % of the step)
      --budget;
      if ((budget & 15) == 0 &&
          (budget <= 0 || __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
        __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lds_flag[0] = 0;
        break;
      }
      for (int i = 0; i < poll_sleep; ++i) __builtin_amdgcn_s_sleep(1);
    }
  }
  __syncthreads();
  return lds_flag[0] != 0;
}

// Eight loads of 16 bytes per lane at agent scope (past the L1): w[k] = the 16 bytes at base + at[k]
__device__ __forceinline__ void poll_marked(const int8_t *base, const unsigned (&at)[8], v4i (&w)[8]) {
  asm volatile("global_load_dwordx4 %0, %8, %16 sc1\n\tglobal_load_dwordx4 %1, %9, %16 sc1\n\t"
               "global_load_dwordx4 %2, %10, %16 sc1\n\tglobal_load_dwordx4 %3, %11, %16 sc1\n\t"
               "global_load_dwordx4 %4, %12, %16 sc1\n\tglobal_load_dwordx4 %5, %13, %16 sc1\n\t"
               "global_load_dwordx4 %6, %14, %16 sc1\n\tglobal_load_dwordx4 %7, %15, %16 sc1\n\ts_waitcnt vmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
               : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]), "v"(at[6]), "v"(at[7]), "s"(base)
               : "memory");
}

// The status word of the second layer of a launch of two (RecArgs2, the kernel's only argument), NULL if there is none.
// Read from the argument segment where it is needed, at the end of a launch: as a use of the argument it stayed in a pair of
// scalar registers through the step loop, and the four-row kernel took 3.4 % longer (512 cells, layer norm, 16 rows).
template <class Args>
__device__ __forceinline__ int *other_status() {
  typedef const __attribute__((address_space(4))) uint8_t *arg_ptr;
  arg_ptr p = (arg_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(int *const __attribute__((address_space(4))) *)(p + offsetof(Args, d) + sizeof(((Args *)0)->d[0]) +
                                                           offsetof(RecArgs, status));
}

// Adds into a word of LDS, in an asm with no result.  Ahead of an LDS atomic the compiler waits for every operation on global
// memory that is on its way, because one of them may be a transfer into LDS (and does so whether or not the kernel has waited
// for those): here the terms of later steps and the stores of the output, a round trip to memory in the middle of a step.
// The compiler does not know that LDS has work to do either: a lds_barrier has to come before what reads the word.
__device__ __forceinline__ void lds_add_u64(u64 *word, u64 v) {
  asm volatile("ds_add_u64 %0, %1" ::"v"((uint32_t)(uintptr_t)(__attribute__((address_space(3))) u64 *)word), "v"(v) : "memory");
}
// A barrier of the workgroup that waits for LDS only.  __syncthreads waits for every load and store of the wave besides.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A poll of (value, tag) byte pairs, 16 bytes per lane, at agent scope (past the L1): w[k] = the 16 bytes at base + at[k].  A load
// of that width may be torn, and a pair vouches for its own value only: that is enough where every pair's tag is looked at.
// What a poll costs is its loads: with 8 bytes per lane, twice as many of them, an exchange takes 0.1 us (512 cells) to
// 0.4 us (2048 cells, 640 outputs) longer.
__device__ __forceinline__ void poll_pairs(const u64 *base, const unsigned (&at)[1], v4i (&w)[1]) {
  asm volatile("global_load_dwordx4 %0, %1, %2 sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(w[0]) : "v"(at[0]), "s"(base) : "memory");
}
__device__ __forceinline__ void poll_pairs(const u64 *base, const unsigned (&at)[2], v4i (&w)[2]) {
  asm volatile("global_load_dwordx4 %0, %2, %4 sc1\n\tglobal_load_dwordx4 %1, %3, %4 sc1\n\ts_waitcnt vmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1])
               : "v"(at[0]), "v"(at[1]), "s"(base)
               : "memory");
}
__device__ __forceinline__ void poll_pairs(const u64 *base, const unsigned (&at)[3], v4i (&w)[3]) {
  asm volatile("global_load_dwordx4 %0, %3, %6 sc1\n\tglobal_load_dwordx4 %1, %4, %6 sc1\n\t"
               "global_load_dwordx4 %2, %5, %6 sc1\n\ts_waitcnt vmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2])
               : "v"(at[0]), "v"(at[1]), "v"(at[2]), "s"(base)
               : "memory");
}
__device__ __forceinline__ void poll_pairs(const u64 *base, const unsigned (&at)[4], v4i (&w)[4]) {
  asm volatile("global_load_dwordx4 %0, %4, %8 sc1\n\tglobal_load_dwordx4 %1, %5, %8 sc1\n\t"
               "global_load_dwordx4 %2, %6, %8 sc1\n\tglobal_load_dwordx4 %3, %7, %8 sc1\n\ts_waitcnt vmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
               : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "s"(base)
               : "memory");
}

__device__ __forceinline__ void poll_pairs(const u64 *base, const unsigned (&at)[5], v4i (&w)[5]) {
  asm volatile("global_load_dwordx4 %0, %5, %10 sc1\n\tglobal_load_dwordx4 %1, %6, %10 sc1\n\t"
               "global_load_dwordx4 %2, %7, %10 sc1\n\tglobal_load_dwordx4 %3, %8, %10 sc1\n\t"
               "global_load_dwordx4 %4, %9, %10 sc1\n\ts_waitcnt vmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4])
               : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "s"(base)
               : "memory");
}

// Per-layer constants, kept in LDS and read where they are used: as kernel
// arguments they would all be live in scalar registers across the time loop.
struct PrmLds {  // 256 bytes (kPrmLdsBytes in persistent.hip)
  RescaleHi h[4], c[4], ln[4];  // R h terms, peephole terms, layer-norm second stage
  RescaleHi m, p;               // hidden state, projection
  int32_t zp_m, zp_h, m_c, glo;
  double inv_n;  // 1 / N
  int32_t pad[2];
};

static_assert(sizeof(PrmLds) == 256, "rec_lds_bytes assumes 256 bytes");

// Where rec_kernel keeps a table in LDS (byte offsets from the start of the dynamic LDS), for the same
// reason in LDS itself: offD = deltas, offB = bases, offT = tail part (0 = none kept).
struct LutLds {
  int32_t dom, sh, offD, offB, offT, pad[3];
};
static_assert(sizeof(LutLds) == 32, "rec_lds_bytes assumes 3 x 32 bytes");

__device__ __forceinline__ int32_t abs_i32(int32_t v) { return v < 0 ? -v : v; }
// table value t = tab[|x|] -> sigma(x), tanh(x) (Sec. 3.2.1 output clamp)
__device__ __forceinline__ int32_t mirror_sigmoid(int32_t x, int32_t t) {
  return x < 0 ? 32768 - t : (t > 32767 ? 32767 : t);
}
__device__ __forceinline__ int32_t mirror_tanh(int32_t x, int32_t t) {
  return x < 0 ? -t : (t > 32767 ? 32767 : t);
}
// The same for a kernel with two or more waves per SIMD, which then issues an add, a shift or a logical operation every 2.2
// clocks and a comparison, a select, a maximum or a three-operand instruction every 4.3 (one wave alone: every 5 clocks,
// whatever it is): signs are handled by masks.  (The compiler would make the comparisons of these again if it knew what
// the mask is.)
__device__ __forceinline__ int32_t sign_mask(int32_t v) {
  int32_t s = v >> 31;
  asm("" : "+v"(s));
  return s;
}
__device__ __forceinline__ int32_t abs_masked(int32_t v) {
  const int32_t s = sign_mask(v);
  return (v ^ s) - s;
}
// sigma of Q3.12 stays below 32767 (32757 at the largest x): its output clamp never acts
__device__ __forceinline__ int32_t mirror_sigmoid_masked(int32_t x, int32_t t) {
  const int32_t s = sign_mask(x);
  return (t ^ s) + (s & 32769);  // x < 0: ~t + 32769 = 32768 - t
}
__device__ __forceinline__ int32_t mirror_tanh_masked(int32_t x, int32_t t) {
  const int32_t s = sign_mask(x), v = (t ^ s) - s;
  return v > 32767 ? 32767 : v;
}

// Eight waves, two per SIMD, each with one weight tile (8 cells, 4 gates, all of k).  The arithmetic of a step is bound by
// the issue of its instructions, and one wave alone issues one every 5 clocks whatever it is; four waves with two tiles each
// took 1220 us where this form takes 1063 (two layers of 1024 cells, coupled gates, layer norm, 1024 rows, 32 steps) and 5590
// where it takes 5380 (eight layers of 2048 cells, 640 outputs, layer norm, 256 rows, 64 steps).  A wave has half of the
// registers then, and a register spilled to scratch memory is read back behind the W x terms on their way from HBM (the
// first build of this form, with 32 such registers, took 5900): hence the lane addresses computed anew in every step, the
// LDS arrays of fixed size at known offsets, and the two machine passes switched off for these files (build.py).
// FL: bit 0 CIFG, bit 1 peephole, bit 2 layer norm, bit 3 "no projection" (compile
// time, so that the code carries no tests of them); with bit 3 clear the
// projection is a runtime flag.  SP: the recurrent weights are in the 2:4
// compressed form (persistent.h) and R h runs on the sparse MFMA.  TAG: how the
// hidden state travels, 0 through the group's counter, 1 in tagged words
// (kTaggedState), 2 in marked words (kMarkedState, no projection): forms of
// their own, as in rec16_kernel.
template <int KS, int RT, int FL, bool SP = false, int TAG = 0>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void rec_kernel(RecArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const long long t_start = (long long)wall_clock64();
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, b2 = lane >> 5;
  constexpr int WAVES = 8;  // one weight tile each
  constexpr bool cifg = FL & 1, ph = FL & 2, ln = FL & 4;
  // bit 3: the layer is known to have no projection (measured: dropping the projection code from
  // those kernels gains 1.7 % at C5, while fixing the flag to "on" at compile time loses 5 % at C4)
  const bool proj = !(FL & 8) && (a.flags & 8);
  const int GS = a.GS;

  // Placement: the workgroups of a group share one XCD (one L2).  XCC_ID register (id 20), bits 3:0,
  // is the XCD this workgroup runs on.
  const int wg = blockIdx.x;
  const int xcc = (int)(__builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)) & 7);
  const int slot = wg >> 3;
  int xcd = wg & 7;
  if (a.tickets) {
    // Plain launch: the dispatcher deals workgroups out to the XCDs in turn, but starts wherever the
    // kernel before stopped: workgroup w runs on XCD (w + r) % 8 with an r nobody knows beforehand.
    // Each block of 8 consecutive workgroups still covers every XCD once, so (the XCD read from the
    // hardware, w / 8) names a place exactly once -- if the dealing was strict, which every
    // workgroup helps to check when it is done (end of the kernel).
    xcd = xcc;
  } else if (xcc != xcd && GS > 1 && tid == 0) {
    // cooperative launch: workgroup w runs on XCD w % 8
    __hip_atomic_store(a.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // Placement check of a plain launch, made by every workgroup when it is done (not at the start, so
  // that nothing waits for it): one 64-bit word per XCD, low half a sum of 2^(w / 8), high half a count
  // of workgroups.  The workgroup that completes its XCD's count finds every place taken once (the sum
  // is then all ones), or raises the status word; so does one that finds the count exceeded -- and an
  // XCD that got too few leaves another with too many.  (The register is read again: kept from the
  // start it would occupy a register across the time loop.)
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
  const int group = xcd + 8 * (slot / GS), member = slot % GS;
  if (group >= a.groups) {  // no rows for this workgroup
    placement_check();
    return;
  }
  constexpr int rows_pg = 32 * RT;
  constexpr int items = RT * 128;  // (rt, gate, row) layer-norm rows of the group
  const int row0 = a.batch0 + group * rows_pg;  // first batch row of the group

  // ---- LDS carve-up (rec_lds_bytes mirrors it): what has a fixed size first, at offsets known to the compiler
  constexpr int LS = KS * 32 + 16;  // h tile row stride
  constexpr bool MARK = TAG == 2;
  static_assert(TAG != 1 || (RT == 1 && !SP && KS <= 20));  // rec_tagged is the host's side of this
  static_assert(!MARK || (RT == 1 && (FL & 8) && !SP && KS == 32));  // rec_marked
  uint8_t *p = lds;
  u64 *red = reinterpret_cast<u64 *>(p);                 p += (size_t)items * 8;
  LnRow2 *lnrow = reinterpret_cast<LnRow2 *>(p);         p += (size_t)items * sizeof(LnRow2);
  double *LdL = reinterpret_cast<double *>(p);           p += 4 * 64 * 8;  // layer-norm weights / 2^10 as doubles
  double *bdL = reinterpret_cast<double *>(p);           p += 4 * 64 * 8;  // layer-norm biases / 2^10 + 2^-11 as doubles
  int16_t *PqL = reinterpret_cast<int16_t *>(p);         p += 4 * 64 * 2;  // 3 used
  int32_t *bhL = reinterpret_cast<int32_t *>(p);         p += 4 * 64 * 4;
  int32_t *bpL = reinterpret_cast<int32_t *>(p);         p += 32 * 4;
  PrmLds *prm = reinterpret_cast<PrmLds *>(p);           p += sizeof(PrmLds);
  int *flag = reinterpret_cast<int *>(p);                p += 16;
  u64 *tickL = reinterpret_cast<u64 *>(p);               p += 16 * 8;  // phase timers
  LutLds *lutP = reinterpret_cast<LutLds *>(p);          p += 3 * sizeof(LutLds);
  int8_t *hT = reinterpret_cast<int8_t *>(p);
  v4i *pred = reinterpret_cast<v4i *>(p);  // projection partials [slot][4][64] reuse the h tile between steps
  const bool four_slots = a.flags & kFourPredSlots;
  {
    const size_t tile_bytes = ((size_t)rows_pg * LS + 1023) / 1024 * 1024;  // whole 1 KB chunks
    const size_t pred_bytes = proj ? (four_slots ? 4 : 8) * 4096 : 0;
    p += tile_bytes > pred_bytes ? tile_bytes : pred_bytes;
  }
  // compressed sigma / tanh tables (wide form, lstm_int_math.h): deltas of the first dom entries, their
  // bases, and the tail part where one is kept; the cell-format tanh shares the gate one if equal
  const bool share_tanh = a.lut[2].blob == a.lut[1].blob;
  const uint8_t *lutD[3];   // deltas
  const uint16_t *lutB[3];  // bases
  const uint8_t *lutTl[3];  // tail part, or NULL
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (i == 2 && share_tanh) {
      lutD[2] = lutD[1]; lutB[2] = lutB[1]; lutTl[2] = lutTl[1];
    } else {
      const int nb = ((((a.lut[i].dom >> a.lut[i].sh) * 2) + 1023) >> 10) << 10;
      lutD[i] = p;                                        p += a.lut[i].dom;
      lutB[i] = reinterpret_cast<const uint16_t *>(p);    p += nb;
      lutTl[i] = a.lut[i].tail ? p : nullptr;             p += a.lut[i].tail ? 3072 : 0;
    }
  }
  int8_t *WpL = reinterpret_cast<int8_t *>(p);
  const int WLS = a.npadp + 16;  // W_proj tile row stride in LDS
  const int my_ptiles = proj ? (a.ptiles > member ? (a.ptiles - member + GS - 1) / GS : 0) : 0;

  // ---- one-time loads: R slice and its biases -> registers, other per-cell
  // parameters, the tables and the W_proj tiles -> LDS
  constexpr int KW = SP ? KS / 2 : KS;  // weight operands per tile: 64-deep k steps in the sparse form
  static_assert(!SP || KS % 2 == 0, "the sparse form takes k in steps of 64");
  v4i Wf[KW];
  int Wi[SP ? KW : 1];  // sparse form: the index word of each operand
  {
    const int4 *src = a.R2 + (size_t)(member * WAVES + wave) * KW * 64 + lane;
    const int *isrc = reinterpret_cast<const int *>(a.R2 + (size_t)GS * WAVES * KW * 64) +
                      (size_t)(member * WAVES + wave) * KW * 64 + lane;
    // all loads are in flight together before the first is pinned to its place
    int4 w[KW];
    int wi[KW];
#pragma unroll
    for (int ks = 0; ks < KW; ++ks) {
      w[ks] = src[(size_t)ks * 64];
      if (SP) wi[ks] = isrc[(size_t)ks * 64];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KW; ++ks) {
      Wf[ks] = v4i{w[ks].x, w[ks].y, w[ks].z, w[ks].w};
      asm volatile("" : "+v"(Wf[ks]));  // resident in registers for the whole launch
      if (SP) {
        Wi[ks] = wi[ks];
        asm volatile("" : "+v"(Wi[ks]));  // the index operand is read from an ordinary vector register
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  const int cell_w = wave * 8 + 4 * b2;  // + c, within the workgroup's 64 cells
  if (tid < 256) {
    const int g = tid >> 6, n = tid & 63;  // 256 threads = 4 gates x 64 cells
    const size_t idx = (size_t)g * a.Ncp + member * 64 + n;
    LdL[tid] = ln ? ln_weight_scaled(a.Lq4[idx]) : 0.0;
    bdL[tid] = ln ? ln_bias_scaled(a.qb4[idx]) : 0.0;
    PqL[tid] = (ph && g < 3) ? a.Pq3[idx] : 0;
    bhL[tid] = a.bh4[idx];  // folded recurrent bias, the accumulators' initial value each step
  }
  if (tid < 4) {
    prm->h[tid] = rescale_hi_prepare(a.Mh[tid], a.rh[tid]);
    prm->c[tid] = rescale_hi_prepare(tid < 3 && ph ? a.Mc[tid] : 0, tid < 3 && ph ? a.rc[tid] : 33);
    prm->ln[tid] = rescale_hi_prepare(a.Mln[tid], ln ? a.rln[tid] : 33);
  }
  if (tid < 3) {
    LutLds d;
    d.dom = a.lut[tid].dom; d.sh = a.lut[tid].sh;
    d.offD = (int32_t)(lutD[tid] - lds);
    d.offB = (int32_t)(reinterpret_cast<const uint8_t *>(lutB[tid]) - lds);
    d.offT = lutTl[tid] ? (int32_t)(lutTl[tid] - lds) : 0;
    d.pad[0] = d.pad[1] = d.pad[2] = 0;
    lutP[tid] = d;
  }
  if (tid == 0) {
    prm->m = rescale_hi_prepare(a.Mm, a.rm);
    prm->p = rescale_hi_prepare(proj ? a.Mp : 0, proj ? a.rp : 33);
    prm->zp_m = a.zp_m; prm->zp_h = a.zp_h;
    prm->inv_n = 1.0 / (double)a.N;
    prm->m_c = a.m_c; prm->glo = ln ? -32767 : -32768;
  }
  for (int i = tid; i < rows_pg * LS / 16; i += 64 * WAVES) reinterpret_cast<int4 *>(hT)[i] = int4{0, 0, 0, 0};
  // tables and W_proj tiles: global -> LDS loads, all in flight together
  {
    auto dma = [&](const void *src, const void *dst) {
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                       (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
    };
    // per table: dom / 1024 chunks of deltas, then the chunks of bases, then the 3 chunks of the tail part,
    // which sit in this order in LDS and at fixed offsets in the wide blob
    for (int i = 0; i < (share_tanh ? 2 : 3); ++i) {
      const int nd = a.lut[i].dom >> 10;
      const int nb = (((a.lut[i].dom >> a.lut[i].sh) * 2) + 1023) >> 10;
      const int nt = a.lut[i].tail ? 3 : 0;
      for (int c = wave; c < nd + nb + nt; c += WAVES) {
        const int so = c < nd ? c * 1024 : (c < nd + nb ? kLutWideBaseOff + (c - nd) * 1024 : kLutWideTailOff + (c - nd - nb) * 1024);
        dma(a.lut[i].blob + so + lane * 16, lutD[i] + c * 1024);
      }
    }
    // the workgroup's tiles pt = 0.. are rows [prow pt, prow pt + prow) of one [rows][WLS] block in LDS (only
    // the prow output rows a tile really has are kept); bytes of the row padding and past the last row read
    // the start of the weights
    const int prow = a.prow;
    const int wp_rows = my_ptiles * prow;
    const int wp_chunks = (wp_rows * WLS + 1023) >> 10;
    for (int c = wave; c < wp_chunks; c += WAVES) {
      const int o = c * 1024 + lane * 16;
      const int r = o / WLS, col_b = o - r * WLS;
      const int8_t *src = a.Wp2;
      if (r < wp_rows && col_b < a.npadp) {
        const int pt = r / prow;
        src = a.Wp2 + ((size_t)(member + pt * GS) * 32 + (r - pt * prow)) * a.npadp + col_b;
      }
      dma(src, WpL + c * 1024);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }

  // cell state of this lane's 4 cells x RT row tiles, kept in registers
  int32_t creg[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int row = row0 + rt * 32 + col;
    const int n0 = member * 64 + cell_w;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      creg[rt][c] = (a.c_in && row < a.B && n0 + c < a.N) ? a.c_in[(size_t)row * a.N + n0 + c] : 0;
  }

  // h tile staging by global -> LDS loads (no registers in between): wave
  // instruction c = wave + 8 j fills bytes [1024 c, 1024 (c + 1)) of the tile,
  // lane l its 16 bytes at 16 l; the lane's source is wherever that byte range
  // falls in the padded [row][LS] tile (pad bytes and the tail read offset 0
  // and hold garbage that only ever meets zero weights)
  constexpr int TILE_KB = (rows_pg * LS + 1023) / 1024;
  constexpr int NCH = (TILE_KB + WAVES - 1) / WAVES;  // chunks per wave
  unsigned hsrc[NCH];
  constexpr bool HSRC_KEPT = !TAG && !(RT > 1 && KS > 20);  // two tiles at the longest k have no registers for it
  auto h_source = [&](int j, int lane) {
    const int o = (wave + WAVES * j) * 1024 + lane * 16;
    const int r = o / LS, c = o - r * LS;
    int row = row0 + r;
    row = row < a.B ? row : a.B - 1;
    return (r < rows_pg && c < a.Hpad) ? (unsigned)(row * a.Hpad + c) : 0u;
  };
  if (HSRC_KEPT)
#pragma unroll
    for (int j = 0; j < NCH; ++j) hsrc[j] = h_source(j, lane);

  if (my_ptiles > 0 && tid < 32) bpL[tid] = a.bp2[member * 32 + tid];  // the first tile's projection bias

  if (tid < 16) tickL[tid] = 0;
  if (tid < items) red[tid] = 0;
  if (tid == 0) {
    flag[0] = 1;
    flag[1] = 0;
  }
  __syncthreads();  // LDS contents above are in place before the first step

  unsigned epoch = 0;
  unsigned *counter = a.counters + group * 64;
  // The hidden state in tagged words as in rec16_kernel, where a group has one row tile and at most 640 outputs (five loads of 16
  // bytes a thread and poll; two tiles or 1024 outputs would be eight and more); of a projection one tile of them per workgroup.
  // Counter -> words, 64 steps (us): 2048 cells, 640 outputs, 256 rows 553 -> 526, layer norm 685 -> 631, and peephole 794 -> 739; 160
  // outputs, layer norm 688 -> 551; 1024 cells, 512 outputs, 512 rows, layer norm 640 -> 581; 512 cells, 1024 rows, layer norm 460 -> 449;
  // 320 cells, 1400 rows 345 -> 314.  (Both ways in one kernel, with the counter's pauses for the workgroups without outputs: 539, 641,
  // 756, 574, 594, 458 and 319, and 2 to 5 % on the calls through the counter.)
  const int Hr = FL & 8 ? tagged_row(a.H) : a.H;  // outputs of a projection are whole pieces
  u64 *accS = a.acc + (size_t)group * (kStatGroupWords + (TAG == 1 ? tagged_group_words(a.H, 32) : 0));  // [set][round][S1|S2][item]
  u64 *const xh = accS + kStatGroupWords;  // [2 slots][32 rows][Hr] (value, tag)
  uint32_t prev1[2] = {0, 0};  // this thread's item, per round: the sums of the statistics words as last read
  u64 prev2[2] = {0, 0};
  const int g_first = cifg ? 1 : 0;
  // uniform: some shift of the layer norm's second stage / of the hidden state's rescale is below 33
  const bool pre_ln = ln && (a.rln[0] < 33 || a.rln[1] < 33 || a.rln[2] < 33 || a.rln[3] < 33);
  const bool pre_m = a.rm < 33;

  // optional phase timing of workgroup 0 (diagnostics): 100 MHz wall clock
  // ticks per phase, summed in LDS (an add that returns nothing, so the timer
  // waits for no memory) and written out after the last step
  long long tick_last = 0;
  const bool timing = a.ticks && wg == 0 && wave == 0;  // uniform
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
  if (timing) {
    tick_last = t_start;
    if (lane == 0) __hip_atomic_store(&a.ticks[15], t_start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  TICK(10);  // everything before the first step

  // the two 16-byte W x pieces of row tile rt for step t
  auto tx_ptr = [&](int t, int rt) -> const int4 * {
    size_t rb = ((size_t)t * a.Bp + row0 + rt * 32) >> 5;
    const size_t rbmax = ((size_t)a.T * a.Bp) >> 5;
    rb = rb < rbmax ? rb : rbmax - 1;
    return a.tx2 + ((rb * (size_t)(GS * 8) + member * 8 + wave) * 2) * 64 + lane;
  };

  // The W x terms of a step come from memory, not from a cache: those of step t + 1 are asked for when step t has its
  // row statistics (or its gate sums, without a layer norm), under the cell's arithmetic and ahead of the stores of m.
  // (Two row tiles have no registers for that: they ask when the h tile is in LDS, and R h of both covers most of it.)
  int4 txv[RT][2];
  auto load_tx = [&](int t) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int4 *src = tx_ptr(t, rt);  // clamped to the last row block: step T reads step T - 1's again
      // read once: a streaming load keeps the W x terms from displacing the exchange buffers in L2
      const v4i t0 = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(src));
      const v4i t1 = __builtin_nontemporal_load(reinterpret_cast<const v4i *>(src + 64));
      txv[rt][0] = int4{t0.x, t0.y, t0.z, t0.w};
      txv[rt][1] = int4{t1.x, t1.y, t1.z, t1.w};
    }
  };
  if (RT == 1 && a.T > 0) load_tx(0);

  // as in rec16_kernel
  const unsigned never = a.extra_arrivals ? 0x80u : 0;  // tests: a tag nobody stores in so few steps
  const int row_pieces = Hr >> 3;
  const uint32_t per_piece = TAG == 1 ? 0xFFFFFFFFu / (uint32_t)row_pieces + 1 : 0;  // c / row_pieces = high word of c per_piece, c < 2^12, two pieces or more
  auto poll_state = [&](auto count, int t, int tid) {
    constexpr int U = decltype(count)::value;
    const uint32_t want = (((unsigned)t + 1) & 0xFF ^ never) * 0x01000100u;
    const u64 *src = xh + (size_t)(t & 1) * Hr * 8;
    unsigned at[U];
    v4i w[U];
#pragma unroll
    for (int k = 0; k < U; ++k) at[k] = k * 512 + tid < 32 * row_pieces ? (unsigned)(k * 512 + tid) * 16 : 0;
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
      // a workgroup without outputs has nothing to do meanwhile, and its polls delay the others' loads of m
      if (!(FL & 8) && my_ptiles == 0) __builtin_amdgcn_s_sleep(2);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int c = k * 512 + tid;
      if (c < 32 * row_pieces) {
        const int rr = (int)__umulhi((uint32_t)c, per_piece);
        *reinterpret_cast<v2i *>(hT + rr * LS + 8 * (c - rr * row_pieces)) =
            v2i{(int)__builtin_amdgcn_perm((uint32_t)w[k][1], (uint32_t)w[k][0], 0x06040200u),
                (int)__builtin_amdgcn_perm((uint32_t)w[k][3], (uint32_t)w[k][2], 0x06040200u)};
      }
    }
  };
  uint32_t hkeep = 0;  // this thread's outputs of the step, four, or two of a projection
  auto store_output = [&](int t, int lane) {
    if (FL & 8) {
      const int col = lane & 31, cell_w = wave * 8 + 4 * (lane >> 5);
      if (row0 + col < a.B && member * 64 + cell_w < a.N) {
        const size_t orow0 = (size_t)t * a.B + row0;
        *reinterpret_cast<uint32_t *>(a.out + orow0 * a.Hpad + member * 64 + (unsigned)(col * a.Hpad + cell_w)) = hkeep;
        if (a.y) __builtin_nontemporal_store(hkeep, reinterpret_cast<uint32_t *>(a.y + orow0 * a.H + member * 64 + (unsigned)(col * a.H + cell_w)));
      }
      return;
    }
    const int col = lane & 31, pl = 4 * wave + 2 * (lane >> 5), p0 = member * a.prow + pl;
    if (my_ptiles > 0 && 4 * wave < a.prow && row0 + col < a.B && p0 < a.H) {
      const size_t orow0 = (size_t)t * a.B + row0;
      *reinterpret_cast<uint16_t *>(a.out + orow0 * a.Hpad + member * a.prow + (unsigned)(col * a.Hpad + pl)) = (uint16_t)hkeep;
      if (a.y) {
        int8_t *yd = a.y + orow0 * a.H + member * a.prow + (unsigned)(col * a.H + pl);
        yd[0] = (int8_t)hkeep;
        if (p0 + 1 < a.H) yd[1] = (int8_t)(hkeep >> 8);
      }
    }
  };

  // m in marked words (TAG and a projection): who needs m polls the words that hold it, eight cells of a row in 64 bits, in one of four
  // slots that take turns.  A word that is not written yet holds kMarkFree in its low half; a value that looks like that, or like
  // kMarkEscape, leaves in the escape slot, and kMarkEscape says so.  What a word holds is the operand of the product, so that
  // nothing is unpacked, and there is no store to wait for, no counter and no second trip for the data.
  auto m_word = [&](int t, int lane) -> int8_t * {  // of lane and lane ^ 32: cells 8 wave .. 8 wave + 7 of row lane % 32
    int8_t *slot = a.mbuf + (size_t)(t & 3) * a.Bp * a.npadp + ((size_t)(row0 >> 5) * (a.npadp >> 5) + member * 2 + (wave >> 2)) * 1024;
    return slot + (unsigned)((lane & 31) * 32 + (wave & 3) * 8);
  };
  // The hidden state in marked words (MARK), half of the bytes of pairs, so that the longest k goes without the counter too.  The h
  // tile is in the order of the exchange, [k step][32 rows][32 cells], and a wave's eighth of it goes global -> LDS until no word is
  // marked as not written.  Two escape slots: who stores step t + 2 has seen step t + 1 of all others, who had read step t before
  // they made that.  1024 cells, 400 rows, 60 steps, layer norm, counter -> this 485 -> 439 us, without it 331 -> 329; 500 rows,
  // peephole and layer norm 549 -> 535; 700 cells, 300 rows, layer norm 437 -> 391.  Two row tiles, twice the bytes, keep the counter: 1024
  // cells, 1024 rows, layer norm 843 -> 981, coupled gates too 728 -> 857 -- a look takes more than 1 us then, workgroups that need a second one come late to the
  // statistics, and neither a first pause nor looking at a word per writer first made up for that.
  const size_t hslot = MARK ? (size_t)a.Bp * GS * 64 : 0;
  constexpr int HCH = KS / WAVES;  // pieces of 1 KB for a wave
  auto h_word = [&](int slot, int lane) -> int8_t * {  // as m_word
    return a.mbuf + slot * hslot + (size_t)((row0 >> 5) * 2 * GS + member * 2 + (wave >> 2)) * 1024 + (unsigned)((lane & 31) * 32 + (wave & 3) * 8);
  };
  auto fetch_state = [&](int t, int lane) {
    int8_t *const tile = hT + lane * 16;
    auto has = [&](int j) { return wave + WAVES * j < 2 * GS; };
    auto from = [&](int j) { return (unsigned)(((row0 >> 5) * 2 * GS + wave + WAVES * j) * 1024 + lane * 16); };
    const int8_t *src = a.mbuf + (t & 3) * hslot;
    asm volatile("" : "+s"(src));
    int budget = a.spin_limit;
    uint32_t least;
    for (int i = 0; i < a.sync_sleep; ++i) __builtin_amdgcn_s_sleep(1);
    for (;;) {
#pragma unroll
      for (int j = 0; j < HCH; ++j)
        if (has(j))
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + from(j)),
                                           (__attribute__((address_space(3))) void *)(hT + (wave + WAVES * j) * 1024), 16, 0, 16 /* sc1 */);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      least = 0xFFFFFFFFu;
#pragma unroll
      for (int j = 0; j < HCH; ++j)
        if (has(j)) {
          const v4i w = *reinterpret_cast<const v4i *>(tile + (wave + WAVES * j) * 1024);
          const uint32_t d0 = (uint32_t)w[0] ^ kMarkFree, d1 = (uint32_t)w[2] ^ kMarkFree, d = d0 < d1 ? d0 : d1;
          least = least < d ? least : d;
        }
      if (a.extra_arrivals) least = 0;  // tests: words that nobody writes
      if (__builtin_amdgcn_ballot_w64(least == 0) == 0) break;
      --budget;
      if ((budget & 15) == 0 && (budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
        __hip_atomic_store(a.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        flag[0] = 0;
        return;
      }
    }
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(least == 1) != 0, 0)) {
      const int8_t *esc = a.mbuf + (4 + (t & 1)) * hslot;
      for (int j = 0; j < HCH; ++j)
        if (has(j))
          for (int i = 0; i < 4; i += 2) {
            int *const w = reinterpret_cast<int *>(tile + (wave + WAVES * j) * 1024) + i;
            if ((uint32_t)*w == kMarkEscape)
              *w = __hip_atomic_load(reinterpret_cast<const int *>(esc + from(j) + 4 * i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
    }
  };
  const int tid0 = tid;
  const bool tails = a.lut[0].tail | a.lut[1].tail | a.lut[2].tail;  // some table's LDS copy ends before its flat part
  // this lane's operand row of W_proj; rows beyond a tile's prow outputs re-read row 0: their results are never stored
  const int wp_lane = (col < a.prow ? col : 0) * WLS + (b2 << 4);
  if (MARK) {  // h before the first step, in the order of the exchange
#pragma unroll
    for (int j = 0; j < HCH; ++j) {
      const int c = wave + WAVES * j, k = c * 32 + (lane & 1) * 16;
      int row = row0 + (lane >> 1);
      row = row < a.B ? row : a.B - 1;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(a.h0 + (k < a.Hpad ? (unsigned)(row * a.Hpad + k) : 0u)),
                                       (__attribute__((address_space(3))) void *)(hT + c * 1024), 16, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  if (TAG == 1) {  // h before the first step
#pragma unroll
    for (int j = 0; j < NCH; ++j)
      if (WAVES * (j + 1) <= TILE_KB || wave + WAVES * j < TILE_KB)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(a.h0 + h_source(j, lane)),
                                         (__attribute__((address_space(3))) void *)(hT + (wave + WAVES * j) * 1024), 16, 0, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  for (int t = 0; t < a.T; ++t) {
    // Addresses of a lane are computed anew in every step: kept from before the loop they would cost registers that the
    // compiler then finds in scratch memory, whose loads return behind the W x terms on their way from HBM.
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, col = lane & 31, b2 = lane >> 5, cell_w = wave * 8 + 4 * b2;
    // ---- h^{t-1} rows of the group -> LDS
    if (MARK) {
      if (t > 0) fetch_state(t - 1, lane);
    } else if (TAG) {
      const int mine = t > 0 ? (4 * Hr - wave * 64 + 511) >> 9 : 0;  // pieces of eight cells for a thread of this wave, 32 rows of Hr / 8
      if (mine >= 5)
        poll_state(std::integral_constant<int, 5>{}, t - 1, tid);
      else if (mine == 4)
        poll_state(std::integral_constant<int, 4>{}, t - 1, tid);
      else if (mine == 3)
        poll_state(std::integral_constant<int, 3>{}, t - 1, tid);
      else if (mine == 2)
        poll_state(std::integral_constant<int, 2>{}, t - 1, tid);
      else if (mine == 1)
        poll_state(std::integral_constant<int, 1>{}, t - 1, tid);
    } else {
      const int8_t *hp = t == 0 ? a.h0 : a.out + (size_t)(t - 1) * a.B * a.Hpad;
      asm volatile("" : "+s"(hp));  // one scalar base: not a pointer per lane for each of the two
#pragma unroll
      for (int j = 0; j < NCH; ++j)
        if (WAVES * (j + 1) <= TILE_KB || wave + WAVES * j < TILE_KB) {
          unsigned o = HSRC_KEPT ? hsrc[j] : h_source(j, lane);
          asm volatile("" : "+v"(o));  // widened here, not kept widened
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(hp + o),
                                           (__attribute__((address_space(3))) void *)(hT + (wave + WAVES * j) * 1024), 16, 0, 0);
        }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    if (TAG && t > 0) {
      if (flag[0] == 0) return;
      store_output(t - 1, lane);
      // everyone's h of step t - 1 is here, so everyone has read h of the step before: this lane's words of that are marked as not
      // written, for step t + 2
      if (MARK && t > 1 && t + 3 < a.T && b2 == 0)
        *reinterpret_cast<uint32_t *>(h_word((t - 2) & 3, lane)) = kMarkFree;
      // everyone's h of step t - 1 is here, so everyone has read m of that step: this lane's word of it is marked as not written, for
      // step t + 3
      if (proj && t + 3 < a.T && b2 == 0) *reinterpret_cast<uint32_t *>(m_word(t - 1, lane)) = kMarkFree;
    }
    if (RT > 1) load_tx(t);
    TICK(0);

    // ---- R h on the MFMA: acc[rt][4*gate + c]
    v16i acc[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[rt][v] = bhL[(v >> 2) * 64 + cell_w + (v & 3)];
    if constexpr (SP) {
      constexpr int DEPTH = 2;  // 64-deep h fragments in flight ahead of the MFMAs
      v8i hf[RT][DEPTH];
      const int8_t *hbase = hT + (size_t)col * LS + (b2 << 5);
      auto frag = [&](int rt, int kq) {
        const v4i lo = *reinterpret_cast<const v4i *>(hbase + (size_t)rt * 32 * LS + kq * 64);
        const v4i hi = *reinterpret_cast<const v4i *>(hbase + (size_t)rt * 32 * LS + kq * 64 + 16);
        return v8i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      };
#pragma unroll
      for (int kq = 0; kq < DEPTH && kq < KW; ++kq)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) hf[rt][kq] = frag(rt, kq);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kq = 0; kq < KW; ++kq) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          acc[rt] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(Wf[kq], hf[rt][kq % DEPTH], acc[rt], Wi[kq], 0, 0);
          if (kq + DEPTH < KW) hf[rt][kq % DEPTH] = frag(rt, kq + DEPTH);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      constexpr int DEPTH = RT == 1 ? 4 : 2;  // h fragments in flight ahead of the MFMAs
      v4i hf[RT][DEPTH];
      constexpr int HROW = MARK ? 32 : LS, HSTEP = MARK ? 1024 : 32, HTILE = MARK ? KS * 1024 : 32 * LS;
      const int8_t *hbase = hT + (size_t)col * HROW + (b2 << 4);
#pragma unroll
      for (int ks = 0; ks < DEPTH && ks < KS; ++ks)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          hf[rt][ks] = *reinterpret_cast<const v4i *>(hbase + (size_t)rt * HTILE + ks * HSTEP);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          acc[rt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(Wf[ks], hf[rt][ks % DEPTH], acc[rt], 0, 0, 0);  // acc starts from the folded bias
          if (ks + DEPTH < KS)
            hf[rt][ks % DEPTH] = *reinterpret_cast<const v4i *>(hbase + (size_t)rt * HTILE + (ks + DEPTH) * HSTEP);
        }
        // keep the LDS reads DEPTH iterations ahead of their MFMAs: without
        // this the instruction scheduler sinks each read next to its use
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    TICK(1);

    // ---- gate sums (Secs. 3.2.4/3.2.5) and layer-norm partial statistics.
    // With a peephole the o gate keeps tx + th here and is finished after c^t.
    constexpr int32_t glo = ln ? -32767 : -32768;  // layer norm takes symmetric gate sums
    auto gate_sums = [&](auto pre_tag) {
      constexpr int PRE = decltype(pre_tag)::value;  // operand treatment of the R h rescale (RecArgs::pre_h)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if (RT > 1) __builtin_amdgcn_sched_barrier(0);  // the row tiles one after the other: both at once do not fit the registers
        int32_t s1[4] = {0, 0, 0, 0};
        uint32_t s2[4] = {0, 0, 0, 0};  // four squares of 16-bit values fit 32 bits
        const int32_t txw[8] = {txv[rt][0].x, txv[rt][0].y, txv[rt][0].z, txv[rt][0].w,
                                txv[rt][1].x, txv[rt][1].y, txv[rt][1].z, txv[rt][1].w};
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const RescaleHi pg = prm->h[g];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int idx = g * 4 + c;
            const int32_t th = rescale_sat16_pre<PRE>(acc[rt][idx], pg);
            const int32_t w = txw[idx >> 1];
            const int32_t tx = (idx & 1) ? (w >> 16) : (int32_t)(int16_t)(w & 0xFFFF);
            int32_t v = tx + th;
            if (ph && g < 2) v += rescale_sat16_pre(mul_i24(PqL[g * 64 + cell_w + c], creg[rt][c]), prm->c[g]);
            if (!(ph && g == 3)) v = clamp_i32(v, glo, 32767);
            acc[rt][idx] = v;
            s1[g] += v;
            s2[g] += (uint32_t)v * (uint32_t)v;
          }
        }
        if (ln) {
#pragma unroll
          for (int g = 0; g < (ph ? 3 : 4); ++g) {  // with a peephole the o gate follows after c^t
            // the 16 lanes of a row (2 per wave) add into one LDS word: no cross-lane traffic, no wait
            const int64_t pk = ((int64_t)(u64)s2[g] << 24) + s1[g];
            __hip_atomic_fetch_add(&red[(rt * 4 + g) * 32 + col], (u64)pk, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
      }
    };
    if (a.pre_h == 0)
      gate_sums(std::integral_constant<int, 0>{});
    else if (a.pre_h == 1)
      gate_sums(std::integral_constant<int, 1>{});
    else
      gate_sums(std::integral_constant<int, 2>{});

    // Layer-norm statistics of a row are summed over the group's workgroups by
    // atomic adds into two 64-bit words per (row, gate), which are never reset:
    // the reader subtracts what it read the step before.  The top byte of each
    // word counts the adds, so the words themselves tell when every workgroup of
    // the group has contributed and no separate barrier is needed.  Value field
    // (56 bits): S1 + 2^22 >= 0 per add, at most 2^23; S2 at most 2^36 per add;
    // with at most 32 adds per step the fields hold more than 2^14 steps.
    constexpr u64 kValMask = ((u64)1 << 56) - 1;
    auto publish_stats = [&](int round, int g_lo, int g_hi) {
      __syncthreads();
      if (tid < items) {
        const int g = (tid >> 5) & 3;
        if (g >= g_lo && g <= g_hi) {
          const int64_t pk = (int64_t)red[tid];
          red[tid] = 0;  // the next adds to this word come after the next barrier
          const int64_t v1 = ((pk + (1 << 23)) & 0xFFFFFF) - (1 << 23);  // signed low 24 bits
          const int64_t v2 = (pk - v1) >> 24;
          u64 *mine = accS + (stat_two_sets(GS) ? (member & 1) : 0) * kStatSetWords;  // this workgroup's set of words
          __hip_atomic_fetch_add(&mine[(round * 2 + 0) * 256 + tid], ((u64)1 << 56) + (u64)(v1 + (1 << 22)),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_fetch_add(&mine[(round * 2 + 1) * 256 + tid], ((u64)1 << 56) + (u64)v2, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    };
    // false: a wait gave up (status word raised), every thread leaves the kernel
    auto collect_stats = [&](int round, int g_lo, int g_hi) -> bool {
      if (tid < items) {
        const int g = (tid >> 5) & 3;
        if (g >= g_lo && g <= g_hi) {
          // two sets: set 0 holds the adds of the even members, set 1 those of the odd ones
          const bool two = stat_two_sets(GS);
          const unsigned n0 = two ? ((unsigned)GS + 1) >> 1 : (unsigned)GS, n1 = two ? (unsigned)GS >> 1 : 0u;
          const u64 expect0 = (u64)((n0 * (unsigned)(t + 1)) & 0xFFu), expect1 = (u64)((n1 * (unsigned)(t + 1)) & 0xFFu);
          u64 c1[2], c2[2];
          int budget = a.spin_limit;
          // the adds of the other workgroups need this long to land; a poll before that only delays them
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
            --budget;
            if ((budget & 15) == 0 &&
                (budget <= 0 || __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
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
    TICK(2);
    if (ln) {
      publish_stats(0, g_first, ph ? 2 : 3);
      TICK(3);
      if (!collect_stats(0, g_first, ph ? 2 : 3)) return;
      TICK(4);
    }
    if (RT == 1) load_tx(t + 1);

    // ---- layer norm, sigma/tanh, cell update (Secs. 3.2.6, 3.2.1, 3.2.9, 3.2.7),
    // in batches of one weight tile (up to 4 gates x 4 cells of a row).  Every
    // LDS read of a batch is issued before the first use of any of them: the
    // scheduling barriers keep the compiler from sinking each read next to its
    // use, which exposes one LDS round trip per element (measured: more than
    // half of this phase).
    // gates of `gmask` (bit g) of row tile rt: gate sums -> layer norm -> xv[g][c]
    constexpr int LNB = RT == 1 ? 2 : 1;
    auto normalize = [&](int rt, int gmask, const LnRow2 (&lr)[4], int32_t (&xv)[4][4], bool narrow, auto sat_tag) {
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
                xv[g][c] = narrow ? ln_second_stage_narrow(acc[rt][g * 4 + c], lr[g], wL[g - gp][c], wb[g - gp][c])
                                  : ln_second_stage(acc[rt][g * 4 + c], lr[g], wL[g - gp][c], wb[g - gp][c]);
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
            for (int c = 0; c < 4; ++c) xv[g][c] = acc[rt][g * 4 + c];
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
      // A value at or beyond the prefix kept in LDS takes its table value from the tail part (a table kept
      // without one is flat from there on, and the clamped index was the lookup).  How often that happens is
      // the launch's choice of prefix: with 16384 entries (|x| < 4 in Q3.12) about one layer-norm output in a
      // thousand, i.e. some lane of most batches -- and the step then waits for the slowest of the group's
      // 256 waves; with 24576 entries it is one in a million.  The tests narrow down from the batch to the
      // gate to the cell.
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
    constexpr int gates_now = (cifg ? 0 : 1) | 2 | 4 | (ph ? 0 : 8);  // with a peephole the o gate waits for c^t
    const int32_t m_c = prm->m_c;
    int32_t xo[RT][4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      if (RT > 1) __builtin_amdgcn_sched_barrier(0);
      LnRow2 lr[4];
      bool narrow = false;  // uniform: every row of this wave has sigma >= 2^12, the second stage stays within int32
      if (ln) {
        bool wide = false;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          lr[g] = lnrow[(rt * 4 + g) * 32 + col];
          if (gates_now >> g & 1) wide |= !ln_row_is_narrow(lr[g]);
        }
        narrow = __builtin_amdgcn_ballot_w64(wide) == 0;
      }
      int32_t xv[4][4], tv[4][4];
      if constexpr (RT > 1 && KS > 20) {
        // two tiles at the longest k: two gates at a time, which leaves the registers for the other tile's gate sums
        auto two_gates = [&](int gmask) {
          if ((!ln || narrow) && !tails) {
            normalize(rt, gmask, lr, xv, true, std::false_type{});
            lookup(gmask, xv, gate_tb, tv, std::false_type{});
          } else {
            asm volatile("");
            if (narrow) {
              normalize(rt, gmask, lr, xv, true, std::true_type{});
            } else {
              asm volatile("");
              normalize(rt, gmask, lr, xv, false, std::true_type{});
            }
            lookup(gmask, xv, gate_tb, tv, std::true_type{});
          }
        };
        two_gates(gates_now & 3);
        __builtin_amdgcn_sched_barrier(0);
        two_gates(gates_now & 12);
      } else if ((!ln || narrow) && !tails) {
        normalize(rt, gates_now, lr, xv, true, std::false_type{});
        lookup(gates_now, xv, gate_tb, tv, std::false_type{});
      } else {
        asm volatile("");  // keeps what both forms begin with from being computed ahead of them, for all gates at once
        if (narrow) {
          normalize(rt, gates_now, lr, xv, true, std::true_type{});
        } else {
          asm volatile("");
          normalize(rt, gates_now, lr, xv, false, std::true_type{});
        }
        lookup(gates_now, xv, gate_tb, tv, std::true_type{});
      }
      int32_t s1 = 0;
      int64_t s2 = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        xo[rt][c] = ph ? 0 : mirror_sigmoid_masked(xv[3][c], tv[3][c]);
        const int32_t f = mirror_sigmoid_masked(xv[1][c], tv[1][c]);
        const int32_t i = cifg ? cifg_input_gate(f) : mirror_sigmoid_masked(xv[0][c], tv[0][c]);
        const int32_t cnew = cell_update32(i, mirror_tanh_masked(xv[2][c], tv[2][c]), f, creg[rt][c], m_c);
        creg[rt][c] = cnew;
        if (ph) {  // finish the o gate sum with P_o . c^t (eq. 5)
          int32_t v = acc[rt][12 + c] + rescale_sat16_pre(mul_i24(PqL[2 * 64 + cell_w + c], cnew), prm->c[2]);
          v = clamp_i32(v, glo, 32767);
          acc[rt][12 + c] = v;
          s1 += v;
          s2 += (int64_t)v * v;
        }
      }
      if (ph && ln) {
        const int64_t pk = (s2 << 24) + s1;
        __hip_atomic_fetch_add(&red[(rt * 4 + 3) * 32 + col], (u64)pk, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
    TICK(5);
    if (ph) {
      if (ln) {
        publish_stats(1, 3, 3);
        if (!collect_stats(1, 3, 3)) return;
      }
    }

    // ---- hidden state (Sec. 3.2.7); m is int8.  tanh of the new cell state in its
    // own format (Sec. 3.2.2), and with a peephole the layer norm and sigma of the o gate
    int32_t tc[RT][4];
    {
      const int hid_tb[4] = {2, 0, 0, 0};  // c^t, then the o gate sums
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if (RT > 1) __builtin_amdgcn_sched_barrier(0);
        LnRow2 lr[4];
        if (ph && ln) lr[3] = lnrow[(rt * 4 + 3) * 32 + col];
        int32_t xv[4][4], tv[4][4], ov[4][4];
#pragma unroll
        for (int c = 0; c < 4; ++c) xv[0][c] = creg[rt][c];
        if (ph) {
          normalize(rt, 8, lr, ov, false, std::true_type{});
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
          tc[rt][c] = mirror_tanh_masked(xv[0][c], tv[0][c]);
          if (ph) xo[rt][c] = mirror_sigmoid_masked(xv[1][c], tv[1][c]);
        }
      }
    }
    // Without a projection m is h and goes to the layer output [T, B, Hpad].  With one it goes to the
    // exchange buffer in the order the projection reads it: [t][row tile][k step][row % 32][32 cells],
    // so that a wave's load of one k step is one contiguous KB of whole cache lines.
    int8_t *mdst = proj ? a.mbuf + (size_t)t * a.Bp * a.npadp : a.out + (size_t)t * a.B * a.Hpad;
    const RescaleHi pm = prm->m;
    const int32_t zp_m = prm->zp_m;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int row = row0 + rt * 32 + col;
      const int n0 = member * 64 + cell_w;
      uint32_t pk = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        // sat8 of the sum is unchanged by the 16-bit clamp before it: |zp| <= 128
        int32_t om = mul_i24(xo[rt][c], tc[rt][c]);  // below 2^30 in magnitude
        if (pre_m) om = rescale_preshift(om, pm);
        const int32_t mq = sat8(rescale_sat16_pre<0>(om, pm) + zp_m);
        pk |= (uint32_t)(mq & 0xFF) << (8 * c);
      }
      if (MARK) {  // rows beyond the batch and cells beyond the layer's too
        hkeep = pk;
        const auto both = __builtin_amdgcn_permlane32_swap(pk, pk, false, false);
        uint32_t lo = both[0];
        if (b2 == 0 && t + 1 < a.T) {  // nobody else reads the last one
          if (__builtin_expect((lo ^ kMarkFree) < 2, 0)) {
            *reinterpret_cast<uint32_t *>(h_word(4 + (t & 1), lane)) = lo;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lo = kMarkEscape;
          }
          *reinterpret_cast<v2i *>(h_word(t & 3, lane)) = v2i{(int)lo, (int)both[1]};
        }
      } else if (TAG && (FL & 8)) {  // rows beyond the batch and cells up to whole pieces too
        hkeep = pk;
        const uint32_t tag = ((unsigned)t + 1) & 0xFF;
        if (n0 < Hr)
          *reinterpret_cast<v2i *>(reinterpret_cast<uint8_t *>(xh + (size_t)(t & 1) * Hr * 8) + (unsigned)(col * Hr + n0) * 2) =
              v2i{(int)__builtin_amdgcn_perm(pk, tag, 0x00050004u), (int)__builtin_amdgcn_perm(pk, tag, 0x00070006u)};
      } else if (TAG) {  // rows beyond the batch too: their words are polled with the others
        const auto both = __builtin_amdgcn_permlane32_swap(pk, pk, false, false);
        uint32_t lo = both[0];
        if (b2 == 0) {
          int8_t *const to = m_word(t, lane);
          if (__builtin_expect((lo ^ kMarkFree) < 2, 0)) {
            *reinterpret_cast<uint32_t *>(to + (size_t)(4 - (t & 3)) * a.Bp * a.npadp) = lo;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            lo = kMarkEscape;
          }
          *reinterpret_cast<v2i *>(to) = v2i{(int)lo, (int)both[1]};
        }
      } else if (row < a.B && n0 < a.N) {  // cells past N fill padding of the row (and only ever meet zero weights)
        // scalar bases, 32-bit offsets of the lane: pointers of the lane's own would be held through the loop
        int8_t *mb = mdst + (proj ? ((size_t)((row0 >> 5) + rt) * (a.npadp >> 5) + member * 2 + (wave >> 2)) * 1024
                                  : (size_t)(row0 + rt * 32) * a.Hpad + member * 64);
        *reinterpret_cast<uint32_t *>(mb + (unsigned)(proj ? col * 32 + (wave & 3) * 8 + 4 * b2 : col * a.Hpad + cell_w)) = pk;
        if (!proj && a.y) {
          int8_t *yb = a.y + ((size_t)t * a.B + row0 + rt * 32) * a.H + member * 64;  // H = N, a multiple of 4 (y is NULL otherwise)
          __builtin_nontemporal_store(pk, reinterpret_cast<uint32_t *>(yb + (unsigned)(col * a.H + cell_w)));  // not read again here
        }
      }
    }
    TICK(6);
    if (TAG) {
      if (!ln) __syncthreads();  // every wave is past R h: the h tile may be filled again, with h or with partial sums
    } else {
      if (!group_sync(counter, epoch, GS + a.extra_arrivals, a.status, a.spin_limit, a.sync_sleep, a.poll_sleep, flag)) return;
    }
    TICK(7);

    // ---- projection (Sec. 3.2.8): tile pt of 32 outputs, K = N split over the eight waves
    if (proj) {
      const int ksteps = a.npadp >> 5;     // 32-wide k steps, a multiple of 4, at most 64 (N <= 2048)
      const int per_wave = (ksteps + 7) >> 3;
      const int kfirst = wave * per_wave;  // the last waves may have fewer, or none
      const int kend = TAG ? 2 * GS : ksteps;  // TAG: k steps that somebody writes
      for (int pt = 0; pt < my_ptiles; ++pt) {
        const int ptile = member + pt * GS;
        const int8_t *wrow = WpL + wp_lane + pt * a.prow * WLS + kfirst * 32;
        const int kmine = kend - kfirst < per_wave ? kend - kfirst : per_wave;  // uniform
        // A wave with all eight steps (from 1793 cells on all waves but perhaps the last) runs them straight.  Two layers, projection
        // to 640, layer norm, 256 rows, 32 steps, with the tests -> this: 2048 cells 735 -> 713 us, 1984 752 -> 715, 1856 736 -> 707
        v4i mv[8];
        auto poll_m = [&]() {
          const int8_t *mrow = a.mbuf + (size_t)(t & 3) * a.Bp * a.npadp + ((size_t)(row0 >> 5) * ksteps + kfirst) * 1024;
          const unsigned moff = col * 32 + b2 * 16;
          unsigned at[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) at[k] = moff + (k < kmine ? k : 0) * 1024;
          int budget = a.spin_limit;
          uint32_t least;
          for (int i = 0; i < a.sync_sleep; ++i) __builtin_amdgcn_s_sleep(1);
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
            const int8_t *esc = mrow + (size_t)(4 - (t & 3)) * a.Bp * a.npadp;
#pragma unroll
            for (int k = 0; k < 8; ++k)
#pragma unroll
              for (int i = 0; i < 4; i += 2)
                if ((uint32_t)mv[k][i] == kMarkEscape)
                  mv[k][i] = (int)__hip_atomic_load(reinterpret_cast<const uint32_t *>(esc + at[k] + 4 * i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        };
        auto load_m = [&](int rt) {
          // rows of the tile beyond the batch were never written; their results are not stored either
          const int8_t *mrow = a.mbuf + (size_t)t * a.Bp * a.npadp + ((size_t)((row0 >> 5) + rt) * ksteps + kfirst) * 1024;
          const unsigned moff = col * 32 + b2 * 16;
          if (kmine == 8) {  // no test ahead of each load, all of them on their way before the first product
#pragma unroll
            for (int k = 0; k < 8; ++k) mv[k] = *reinterpret_cast<const v4i *>(mrow + moff + k * 1024);
            __builtin_amdgcn_sched_barrier(0);
          } else {
#pragma unroll
            for (int k = 0; k < 8; ++k)
              if (k < kmine) mv[k] = *reinterpret_cast<const v4i *>(mrow + moff + k * 1024);
          }
        };
        // a row tile that starts beyond the batch (second tile of a ragged last group) has no rows in the exchange buffer
        // at all; the test is uniform over the workgroup, so the barriers below stay matched
        auto has_rows = [&](int rt) { return rt == 0 || (rt < RT && row0 + rt * 32 < a.B); };
        if (TAG) {
          if (kmine > 0) poll_m();
        } else {
          load_m(0);
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          if (!has_rows(rt)) continue;
          v16i pacc;
#pragma unroll
          for (int v = 0; v < 16; ++v) pacc[v] = 0;
          if (kmine == 8) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
              pacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i *>(wrow + k * 32), mv[k], pacc, 0, 0, 0);
          } else {
#pragma unroll
            for (int k = 0; k < 8; ++k)
              if (k < kmine)
                pacc = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i *>(wrow + k * 32), mv[k], pacc, 0, 0, 0);
          }
          if (has_rows(rt + 1)) load_m(rt + 1);  // on their way while this tile's sums are added up
          // result v of a lane: output 8 (v / 4) + 4 (lane / 32) + v % 4 of row lane % 32.  Eight partial sums in LDS, or
          // four where a layer's W_proj leaves no room for them: two waves then share a slot, one after the other
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
          if (4 * wave < a.prow) {  // a thread finishes the outputs pl, pl + 1 of row `col`; prow is a multiple of 4
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
              hq[c] = (uint32_t)(sat8(rescale_sat16_pre(sum[c] + (pt == 0 ? bpL[pl + c] : a.bp2[ptile * 32 + pl + c]), pp) + zp_h) & 0xFF);
            if (TAG) {  // rows beyond the batch too
              hkeep = hq[0] | hq[1] << 8;
              const uint32_t tag = ((unsigned)t + 1) & 0xFF;
              if (p0 < a.H)
                *reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(xh + (size_t)(t & 1) * Hr * 8) + (unsigned)(col * Hr + p0) * 2) =
                    __builtin_amdgcn_perm(hkeep, tag, 0x00050004u);
            } else if (row0 + rt * 32 + col < a.B && p0 < a.H) {
              const size_t orow0 = (size_t)t * a.B + row0 + rt * 32;
              int8_t *od = a.out + orow0 * a.Hpad + ptile * a.prow + (unsigned)(col * a.Hpad + pl);
              // outputs past H fall into the padding of the row (and only ever meet zero weights)
              *reinterpret_cast<uint16_t *>(od) = (uint16_t)(hq[0] | hq[1] << 8);
              if (a.y) {
                int8_t *yd = a.y + orow0 * a.H + ptile * a.prow + (unsigned)(col * a.H + pl);
                yd[0] = (int8_t)hq[0];
                if (p0 + 1 < a.H) yd[1] = (int8_t)hq[1];
              }
            }
          }
          // the last tile's partial sums are overwritten behind the group barrier only
          if (pt + 1 < my_ptiles || rt + 1 < RT || TAG) __syncthreads();
        }
      }
      TICK(8);
      // (TAG: without outputs a workgroup goes on to its polls at once, as in rec16_kernel; 1088 cells, 160 outputs, layer norm, 250 rows,
      // 40 steps with a first pause of 64 and 12 between polls 0.98 of the counter's time, with 0 and 2 0.88, with no pause 0.88, but at
      // 1792 cells, 640 outputs 0.922, 0.929 and 0.939)
      if (!TAG && !group_sync(counter, epoch, GS + a.extra_arrivals, a.status, a.spin_limit, my_ptiles == 0 ? a.idle_sleep : 0,
                              my_ptiles == 0 ? a.idle_poll_sleep : a.poll_sleep, flag))
        return;
      TICK(9);
    }
  }
#undef TICK
  if (TAG) store_output(a.T - 1, lane);
  if (timing && lane == 0)
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
  if (a.c_out) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int row = row0 + rt * 32 + col;
      int n0 = member * 64 + cell_w;
      asm volatile("" : "+v"(n0));  // computed here: shared with the prologue it would hold six registers through the loop
      if (row < a.B && n0 < a.N)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (n0 + c < a.N) a.c_out[(size_t)row * a.N + n0 + c] = (int16_t)creg[rt][c];
    }
  }
}


typedef void (*rec_fn)(RecArgs);

// sparse-weight kernel for the flags at k depth KS (one row tile per group)
template <int KS>
rec_fn rec_pick_sparse_ks(int fl) {
#define LSTM_REC_CASE(F) \
  if (fl == F) return rec_kernel<KS, 1, F, true>;
  LSTM_REC_CASE(0) LSTM_REC_CASE(1) LSTM_REC_CASE(2) LSTM_REC_CASE(3)
  LSTM_REC_CASE(4) LSTM_REC_CASE(5) LSTM_REC_CASE(6) LSTM_REC_CASE(7)
  LSTM_REC_CASE(8) LSTM_REC_CASE(9) LSTM_REC_CASE(10) LSTM_REC_CASE(11)
  LSTM_REC_CASE(12) LSTM_REC_CASE(13) LSTM_REC_CASE(14) LSTM_REC_CASE(15)
#undef LSTM_REC_CASE
  return nullptr;
}

// kernel for (rt, flags & 7) at k depth KS; tag as in rec_kernel
template <int KS>
rec_fn rec_pick_ks(int rt, int fl, int tag) {
#define LSTM_REC_CASE(R, F) \
  if (rt == R && fl == F) return rec_kernel<KS, R, F>;
#define LSTM_REC_TAG(F) \
  if (rt == 1 && fl == F) return rec_kernel<KS, 1, F, false, 1>;
#define LSTM_REC_MARK(F) \
  if (rt == 1 && fl == F) return rec_kernel<KS, 1, F, false, 2>;
  if (tag == 2) {
    if constexpr (KS == 32) {
      LSTM_REC_MARK(8) LSTM_REC_MARK(9) LSTM_REC_MARK(10) LSTM_REC_MARK(11)
      LSTM_REC_MARK(12) LSTM_REC_MARK(13) LSTM_REC_MARK(14) LSTM_REC_MARK(15)
    }
    return nullptr;
  }
  if constexpr (KS <= 20) {
    if (tag) {
      LSTM_REC_TAG(0) LSTM_REC_TAG(1) LSTM_REC_TAG(2) LSTM_REC_TAG(3)
      LSTM_REC_TAG(4) LSTM_REC_TAG(5) LSTM_REC_TAG(6) LSTM_REC_TAG(7)
      LSTM_REC_TAG(8) LSTM_REC_TAG(9) LSTM_REC_TAG(10) LSTM_REC_TAG(11)
      LSTM_REC_TAG(12) LSTM_REC_TAG(13) LSTM_REC_TAG(14) LSTM_REC_TAG(15)
    }
  }
  if (tag) return nullptr;
  LSTM_REC_CASE(1, 0) LSTM_REC_CASE(1, 1) LSTM_REC_CASE(1, 2) LSTM_REC_CASE(1, 3)
  LSTM_REC_CASE(1, 4) LSTM_REC_CASE(1, 5) LSTM_REC_CASE(1, 6) LSTM_REC_CASE(1, 7)
  LSTM_REC_CASE(1, 8) LSTM_REC_CASE(1, 9) LSTM_REC_CASE(1, 10) LSTM_REC_CASE(1, 11)
  LSTM_REC_CASE(1, 12) LSTM_REC_CASE(1, 13) LSTM_REC_CASE(1, 14) LSTM_REC_CASE(1, 15)
  if constexpr (KS < 32) {
    LSTM_REC_CASE(2, 0) LSTM_REC_CASE(2, 1) LSTM_REC_CASE(2, 2) LSTM_REC_CASE(2, 3)
    LSTM_REC_CASE(2, 4) LSTM_REC_CASE(2, 5) LSTM_REC_CASE(2, 6) LSTM_REC_CASE(2, 7)
  }
  LSTM_REC_CASE(2, 8) LSTM_REC_CASE(2, 9) LSTM_REC_CASE(2, 10) LSTM_REC_CASE(2, 11)
  LSTM_REC_CASE(2, 12) LSTM_REC_CASE(2, 13) LSTM_REC_CASE(2, 14) LSTM_REC_CASE(2, 15)
#undef LSTM_REC_MARK
#undef LSTM_REC_TAG
#undef LSTM_REC_CASE
  return nullptr;
}

}  // namespace lstm_int

// What gru_quad_kernel (gru_seq.hip) and gru_rows_kernel (gru_rows.hip) have in common: tables in LDS, the place of a
// workgroup, weights into registers.
#pragma once

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

__device__ __forceinline__ void dma16_agent(const void *src, void *dst) {  // past the L1
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                   (__attribute__((address_space(3))) void *)dst, 16, 0, 16 /* sc1 */);
}

// All of this wave's vector memory operations are done.  (The builtin, not an asm: the compiler then knows it too, and adds
// no wait of its own before reads of the LDS that the transfers above filled.)
__device__ __forceinline__ void wait_vmem() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  asm volatile("" ::: "memory");
}

// gru_rows_kernel: W x terms of 16 rows and a step, and how many of them are kept: of the turn at hand, and of those to come
constexpr int kGruTxBytes = 8192;
__host__ __device__ constexpr int kGruTxSlots(int row_tiles) { return row_tiles + 1; }
constexpr int kGruExchange = 8 * 3 * 64 * 8;  // gru_rows_kernel: sums on their way between the halves of the depth

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
template <int WAVES>
__device__ __forceinline__ void gru_lut_load(const LutWide &w, const GruLut &l, uint8_t *lds, int wave, int lane) {
  const int nd = w.dom >> 10, nb = (((w.dom >> w.sh) * 2) + 1023) >> 10, nt = w.tail ? 3 : 0;
  for (int c = wave; c < nd + nb + nt; c += WAVES) {
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

// recurrent weights of block `blk` of 16 cells, KW k steps from k0 on -> registers (the first ACC
// operands: accumulation registers); k steps past the layer's zero
template <int KW, int ACC>
__device__ __forceinline__ void gru_load_weights(const GruSeqArgs &a, int member, int blk, int k0, int lane, v4i (&Wf)[3][KW]) {
  const int ks_n = a.Kp >> 6;
  const v4i *src = reinterpret_cast<const v4i *>(a.R16) + (size_t)(member * 4 + blk) * 3 * ks_n * 64 + lane;
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    v4i w[KW];  // a gate's loads in flight together
#pragma unroll
    for (int ks = 0; ks < KW; ++ks) w[ks] = k0 + ks < ks_n ? src[((size_t)g * ks_n + k0 + ks) * 64] : v4i{0, 0, 0, 0};
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KW; ++ks) {
      Wf[g][ks] = w[ks];
      if (g * KW + ks < ACC)
        asm volatile("" : "+a"(Wf[g][ks]));
      else
        asm volatile("" : "+v"(Wf[g][ks]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

typedef void (*gru_fn)(GruSeqArgs);

}  // namespace

// gru_rows.hip: the kernel for groups of 16 or 32 rows at k depth ks
void (*gru_rows_pick(int ks, int rows))(GruSeqArgs);

}  // namespace lstm_int

// Input matmul of the GRU's and the SRU's wide layers for gfx950 (MI355X): the input terms of all T B rows of a layer,
//   out[m][g N + n] = sat16(rescale(x[m] . W[g N + n] + bias)),
// for input depths beyond 1024, rows of int16 as the general matmul writes them.
//
// The weights stay in registers, as in in_gemm.hip: a workgroup owns 128 columns (four tiles of 32) over the whole depth and
// streams over blocks of 32 rows, so that only the activations travel.  A tile of 32 columns is 64 KB at a depth of 2048 and
// a wave has room for 64 KB of weights.  With one whole tile per wave every operand read from LDS would feed one MFMA, and the
// four waves would read 256 KB per block; instead the four waves are two halves of the depth times two pairs of tiles: an
// operand feeds two MFMAs, and a wave hands half of its sums (one tile) to the wave with the other half of the depth, through
// 16 KB of LDS, and finishes the other tile itself.
//
// x goes global -> LDS in stages of 32 rows x 8 k steps of either half (16 KB), a ring of two blocks of them, so that a stage
// is asked for nearly two blocks (2 us) ahead: 112 KB in flight per compute unit.  A stage's rows are not padded; the 16-byte
// piece p of row r lies at position p ^ (r % 16), which leaves the operand reads (lane = row % 32) free of bank conflicts,
// and the lane of a global -> LDS load fetches the piece that belongs at its place.
//
// The results leave through 8 KB of LDS.  Written straight from the lanes that hold them, a store covered 32 bytes of each of
// 32 rows: 200 us for 16384 x 6144 x 2048 (168 without stores); four rows of 256 bytes at a time: 187.
//
// Under the MFMAs every instruction must find an issue slot: 64 clocks per k step, for one wave on its SIMD.  Hence the stores
// whose bounds the buffer descriptor checks (a branch around them gathered the requantization of four pieces in one lump of 40
// instructions), the requantization spread over two stages at S = 4, waits for the LDS writes alone, and descriptors made from
// 32-bit row counts, one per block, between MFMAs (32 scalar instructions in front of a block's second MFMA before): 187 -> 180.
//
// 16384 x 6144 x 2048: 180 us = 2.29 POP/s (the general matmul on the same box: 238), 8192 rows 91 (118), 2048 rows 29.5 (39),
// 256 rows 12 (15).  The chip runs it at 1.9 to 1.95 GHz, what its power leaves for MFMAs with stores, as in in_gemm.hip; called
// back to back for long it takes 10 % more.  Operands read eight k steps ahead instead of four, streaming stores: no difference.
#include <cstring>
#include <type_traits>

#include "lstm_int_math.h"
#include "persistent.h"

namespace lstm_int {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef short v2s __attribute__((ext_vector_type(2)));

namespace {

// Loads through a buffer descriptor are bounded: what lies at or beyond base + bytes reads as zero.
#if defined(__HIP_DEVICE_COMPILE__)
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const int8_t *base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t *>(base), 0, bytes, 0x00020000);  // raw, stride 0
}
__device__ __forceinline__ void rsrc_store16(rsrc_t r, v4i v, unsigned offset) {  // nothing where it lies beyond the end
  __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)offset, 0, 0);
}
__device__ __forceinline__ void rsrc_load_lds16(rsrc_t r, uint8_t *dst, unsigned offset) {  // lane l: 16 bytes to dst + 16 l
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16, (int)offset, 0, 0, 0);
}
#else
typedef int rsrc_t;
__device__ rsrc_t make_rsrc(const int8_t *, int) { return 0; }
__device__ void rsrc_store16(rsrc_t, v4i, unsigned) {}
__device__ void rsrc_load_lds16(rsrc_t, uint8_t *, unsigned) {}
#endif

constexpr int kStage = 16384;     // bytes of a stage
constexpr int kExchange = 16384;  // partial sums: 4 KB per wave
constexpr int kOutTile = 8192;    // results: 32 rows x 128 columns

// S: stages per block; a half of the depth is 8 S k steps of 32.  PRE: operand treatment of the rescale (DeepGemmArgs::pre).
template <int S, int PRE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void deep_gemm_kernel(DeepGemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  constexpr int KH = 8 * S, R = 2 * S;  // k steps of a half; stages in the ring
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 31, b2 = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kh = wave >> 1, pair = wave & 1;
  // Consecutive workgroups go to the eight XCDs in turn, each with an L2 of its own: XCD id % 8 gets a run of (column block,
  // part of the rows) pairs.  The part runs fastest: an XCD then fetches an eighth of the weights (2048 x 6144: the prologue
  // is 8 us shorter than the other way round, 200 against 208 us for 16384 rows), and all rows.  With up to 8 column blocks
  // (2 MB of weights) the column block runs fastest: an XCD fetches an eighth of the rows (2048 x 1024: 50 -> 38 us).
  const int share = (a.cbs * a.parts + 7) >> 3;
  const int idx = (blockIdx.x & 7) * share + (blockIdx.x >> 3);
  if ((int)(blockIdx.x >> 3) >= share || idx >= a.cbs * a.parts) return;
  const int cb = a.by_rows ? idx % a.cbs : idx / a.parts, part = a.by_rows ? idx / a.cbs : idx % a.parts;
  const int nrb = (a.M + 31) >> 5;
  const int rb0 = (int)((long long)nrb * part / a.parts), rb1 = (int)((long long)nrb * (part + 1) / a.parts);
  if (rb0 >= rb1) return;  // the whole workgroup

  // ---- loads of a stage: wave instruction j fills rows 2 c and 2 c + 1 of the stage, c = 4 wave + j; a row is 16 pieces of
  // either half.  Pieces beyond the row's depth read what follows in memory (or nothing, at the end) and meet zero weights.
  unsigned voff[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int r = 2 * (4 * wave + j) + b2, p = col ^ (r & 15);
    voff[j] = (unsigned)(r * a.lda + (p >= 16 ? KH * 32 - 256 : 0) + p * 16);
  }
  auto block_rsrc = [&](int rb) {
    const int b = rb < rb1 ? rb : rb1 - 1;  // past the end: the last block again, into stages nobody reads
    const int rows = a.M - 1 - b * 32;  // a block's loads reach at most 4 KB past its rows, rows of over 1 KB
    return make_rsrc(a.A + (long long)b * 32 * a.lda, (int)((unsigned)(rows < 63 ? rows : 63) * a.lda + a.kpad));
  };
  auto load_piece = [&](rsrc_t r, int slot, int s, int j) {
    rsrc_load_lds16(r, lds + slot * kStage + (4 * wave + j) * 1024, voff[j] + s * 256);
  };
  // the first stages are requested before anything else: their latency covers the weight loads
  {
    const rsrc_t r0 = block_rsrc(rb0), r1 = block_rsrc(rb0 + 1);
#pragma unroll
    for (int q = 0; q < R - 1; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) load_piece(q < S ? r0 : r1, q, q < S ? q : q - S, j);
  }

  // ---- this wave's weights: tile 0 the one it finishes, tile 1 the one whose sums it hands over
  v4i Wf[2][KH];
#pragma unroll
  for (int tl = 0; tl < 2; ++tl) {
    const int tile = cb * 4 + pair * 2 + (tl ^ kh);
    const int4 *src = a.Wd + ((size_t)tile * 2 + kh) * KH * 64 + lane;
    int4 w[KH];
#pragma unroll
    for (int ks = 0; ks < KH; ++ks) w[ks] = src[ks * 64];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KH; ++ks) {
      Wf[tl][ks] = v4i{w[ks].x, w[ks].y, w[ks].z, w[ks].w};
      asm volatile("" : "+a"(Wf[tl][ks]));  // resident in accumulation registers for the whole launch
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  const int tile = cb * 4 + pair * 2 + kh;
  // the lane's 16 results are two pieces of 8 columns of row col: packed columns 32 tile + 16 p + 8 b2 .. + 7, so that a
  // store covers 32 bytes of a row; a piece lies in one gate, the same for the whole wave
  v16i bias;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int4 b = *reinterpret_cast<const int4 *>(a.bias + tile * 32 + 16 * (q >> 1) + 8 * b2 + 4 * (q & 1));
    bias[4 * q] = b.x; bias[4 * q + 1] = b.y; bias[4 * q + 2] = b.z; bias[4 * q + 3] = b.w;
  }
  RescaleHi rs[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int gate = (tile * 32 + 16 * p) / a.Np;
    rs[p] = a.rs[gate < 3 ? gate : 3];
  }
  // Results leave through LDS, rows of 256 bytes, piece q of row r at q ^ (r % 16): a store covers four whole rows (half rows
  // where a gate ends in the block) instead of 32 bytes of 32 rows.
  unsigned ooff[2];
  {
    const int pc = cb * 128 + (lane & 15) * 8, gate = pc / a.Np, n0 = pc - gate * a.Np;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      ooff[i] = gate < a.G && n0 < a.N ? ((unsigned)(8 * wave + 4 * i + (lane >> 4)) * a.ldc + gate * a.N + n0) * 2 : 0x80000000u;
  }
  uint8_t *ot = lds + R * kStage + kExchange;
  auto out_rsrc = [&](int rb) {  // block rb of the output; beyond the last row, or ahead of the first block, nothing is stored
    const int rows = a.M - rb * 32;
    return make_rsrc(reinterpret_cast<const int8_t *>(a.out + (long long)rb * 32 * a.ldc), rb < rb0 ? 0 : (rows < 32 ? rows : 32) * a.ldc * 2);
  };

  // operand addresses within a stage
  const int x0 = col * 512 + kh * 256 + ((b2 ^ (col & 15)) << 4);
  uint8_t *ex = lds + R * kStage;

  auto requant = [&](int32_t s0, int32_t s1, const RescaleHi &r) {
    if (PRE == 2) {
      s0 = rescale_preshift(s0, r);
      s1 = rescale_preshift(s1, r);
    }
    if (PRE == 1) {
      s0 <<= r.k;
      s1 <<= r.k;
    }
    const v2s pk = __builtin_amdgcn_cvt_pk_i16((__mulhi(s0, r.M) + r.add) >> r.sh, (__mulhi(s1, r.M) + r.add) >> r.sh);
    return __builtin_bit_cast(int32_t, pk);  // both halves saturated
  };
  int32_t word[4];
  auto piece_pair = [&](const v16i &v, int p) {  // results 2 p, 2 p + 1; four make a 16-byte piece
    word[p & 3] = requant(v[2 * p], v[2 * p + 1], rs[p >> 2]);
    if ((p & 3) == 3)
      *reinterpret_cast<v4i *>(ot + col * 256 + (((pair * 2 + kh) * 4 + 2 * (p >> 2) + b2) ^ (col & 15)) * 16) =
          v4i{word[0], word[1], word[2], word[3]};
  };
  auto store_rows = [&](int i, rsrc_t r) {
    const int row = 8 * wave + 4 * i + (lane >> 4);
    rsrc_store16(r, *reinterpret_cast<const v4i *>(ot + row * 256 + ((lane & 15) ^ (row & 15)) * 16), ooff[i]);
  };

  constexpr int DEPTH = 4;
  v4i xf[DEPTH];
  auto operand = [&](int slot, int k) { return *reinterpret_cast<const v4i *>(lds + slot * kStage + (x0 ^ (k << 5))); };
  v16i other;  // the partner's sums of this wave's tile
  rsrc_t rx = block_rsrc(rb0 + 1), ro = out_rsrc(rb0 - 1);  // the block whose stages are being asked for, the one being stored
  // Stage s of block rb (ring position P S + s): 16 MFMAs; under them the loads of the stage 2 S - 1 later, into the place of
  // the stage just done, and, in the first three stages, what the block before still needs: its sums handed over (s = 0), the
  // partner's read (s = 1, behind a barrier that waits for the LDS writes), requantization into LDS (s = 2)
  // (S = 4: s = 2 and 3), and in the next block's first stage the stores of the rows.
  // At the top of a stage the loads of the next one are complete: 4 (R - 3) are younger (stores among them only make the wait
  // stricter), and past the barrier that holds for every wave, so operands are read ahead across the stage's end.
  auto stage = [&](auto p_tag, auto s_tag, auto have_tag, int rb, v16i (&acc)[2], v16i (&prev)[2]) {
    constexpr int P = decltype(p_tag)::value, s = decltype(s_tag)::value;
    constexpr bool HAVE = decltype(have_tag)::value;
    constexpr int slot = P * S + s, next = (slot + 1) % R, target = (slot + R - 1) % R;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * (R - 3)) : "memory");
    // this wave's LDS writes of the stage before are done; the operand reads after them may be under way
    if (HAVE && s == 0) asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(S > 3 ? 1 : 0) : "memory");
    if (HAVE && s == 1) asm volatile("s_waitcnt lgkmcnt(4)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < 8; ++k) {
#pragma unroll
      for (int tl = 0; tl < 2; ++tl) {
        if (s == 0 && k == 0) {
          v16i c0 = bias;
          if (tl == 1)
#pragma unroll
            for (int v = 0; v < 16; ++v) c0[v] = 0;
          acc[tl] = __builtin_amdgcn_mfma_i32_32x32x32_i8(Wf[tl][0], xf[0], c0, 0, 0, 0);
        } else {
          acc[tl] = __builtin_amdgcn_mfma_i32_32x32x32_i8(Wf[tl][s * 8 + k], xf[k % DEPTH], acc[tl], 0, 0, 0);
        }
      }
      xf[k % DEPTH] = k + DEPTH < 8 ? operand(slot, k + DEPTH) : operand(next, k + DEPTH - 8);
      if (k % 2 == 0) load_piece(rx, target, s == 0 ? S - 1 : s - 1, k / 2);
      if (HAVE && s == 0 && k < 4)
        *reinterpret_cast<v4i *>(ex + wave * 4096 + k * 1024 + lane * 16) =
            v4i{prev[1][4 * k], prev[1][4 * k + 1], prev[1][4 * k + 2], prev[1][4 * k + 3]};
      if (HAVE && s == 1 && k < 4) {
        const v4i o = *reinterpret_cast<const v4i *>(ex + (wave ^ 2) * 4096 + k * 1024 + lane * 16);
#pragma unroll
        for (int c = 0; c < 4; ++c) other[4 * k + c] = o[c];
      }
      if (HAVE && s == 1 && k >= 4)
#pragma unroll
        for (int c = 0; c < 4; ++c) prev[0][4 * (k - 4) + c] += other[4 * (k - 4) + c];
      if (HAVE && s == 2 && S == 3) piece_pair(prev[0], k);
      if (HAVE && s >= 2 && S > 3 && k % 2 == 0) piece_pair(prev[0], 4 * (s - 2) + k / 2);
      if (HAVE && s == 0 && k == 3) ro = out_rsrc(rb - 2);
      if (HAVE && s == 0 && k >= 4 && k % 2 == 0) store_rows(k / 2 - 2, ro);
      if (s == 0 && k == 7) rx = block_rsrc(rb + 2);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto block = [&](auto p_tag, auto have_tag, int rb, v16i (&acc)[2], v16i (&prev)[2]) {
    stage(p_tag, std::integral_constant<int, 0>{}, have_tag, rb, acc, prev);
    stage(p_tag, std::integral_constant<int, 1>{}, have_tag, rb, acc, prev);
    stage(p_tag, std::integral_constant<int, 2>{}, have_tag, rb, acc, prev);
    if constexpr (S > 3) stage(p_tag, std::integral_constant<int, 3>{}, have_tag, rb, acc, prev);
    asm volatile("" : "+v"(acc[0]), "+v"(acc[1]));
  };
  const std::integral_constant<int, 0> p0{};
  const std::integral_constant<int, 1> p1{};
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * (R - 2)) : "memory");  // stage 0
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int k = 0; k < DEPTH; ++k) xf[k] = operand(0, k);
  v16i accA[2], accB[2];
  block(p0, std::false_type{}, rb0, accA, accB);
  int rb = rb0 + 1;
  for (; rb + 1 < rb1; rb += 2) {
    block(p1, std::true_type{}, rb, accB, accA);
    block(p0, std::true_type{}, rb + 1, accA, accB);
  }
  // the last block's sums, after the last even block (accA) or one more odd one (accB)
  auto finish = [&](v16i (&last)[2]) {
    __syncthreads();
    const rsrc_t rp = out_rsrc(rb1 - 2);  // the rows of the block before
    store_rows(0, rp);
    store_rows(1, rp);
    __syncthreads();  // the last readers of the exchange area and of the rows are done
#pragma unroll
    for (int k = 0; k < 4; ++k)
      *reinterpret_cast<v4i *>(ex + wave * 4096 + k * 1024 + lane * 16) =
          v4i{last[1][4 * k], last[1][4 * k + 1], last[1][4 * k + 2], last[1][4 * k + 3]};
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const v4i o = *reinterpret_cast<const v4i *>(ex + (wave ^ 2) * 4096 + k * 1024 + lane * 16);
#pragma unroll
      for (int c = 0; c < 4; ++c) last[0][4 * k + c] += o[c];
    }
#pragma unroll
    for (int p = 0; p < 8; ++p) piece_pair(last[0], p);
    __syncthreads();
    const rsrc_t ro = out_rsrc(rb1 - 1);
    store_rows(0, ro);
    store_rows(1, ro);
  };
  if (rb < rb1) {
    block(p1, std::true_type{}, rb, accB, accA);
    finish(accB);
  } else {
    finish(accA);
  }
}

template <int S>
constexpr unsigned lds_bytes_s() {
  return 2u * S * kStage + kExchange + kOutTile;
}

template <int S>
hipError_t init_s() {
  const void *fn[] = {reinterpret_cast<const void *>(deep_gemm_kernel<S, 0>), reinterpret_cast<const void *>(deep_gemm_kernel<S, 1>),
                      reinterpret_cast<const void *>(deep_gemm_kernel<S, 2>)};
  for (const void *f : fn) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes_s<S>());
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int S>
void launch_s(hipStream_t s, const DeepGemmArgs &a, int grid) {
  if (a.pre == 0)
    hipLaunchKernelGGL((deep_gemm_kernel<S, 0>), dim3(grid), dim3(256), lds_bytes_s<S>(), s, a);
  else if (a.pre == 1)
    hipLaunchKernelGGL((deep_gemm_kernel<S, 1>), dim3(grid), dim3(256), lds_bytes_s<S>(), s, a);
  else
    hipLaunchKernelGGL((deep_gemm_kernel<S, 2>), dim3(grid), dim3(256), lds_bytes_s<S>(), s, a);
}

}  // namespace

hipError_t deep_gemm_init() {
  hipError_t e = init_s<3>();
  if (e == hipSuccess) e = init_s<4>();
  return e;
}

DeepWeights deep_weights(int kpad, int G, int N) {
  DeepWeights w;
  if (kpad <= 1024 || kpad > 2048 || N % 8 != 0) return w;
  w.stages = kpad <= 1536 ? 3 : 4;
  w.Np = (N + 15) / 16 * 16;
  w.cbs = (G * w.Np + 127) / 128;
  return w;
}

void deep_pack(const DeepWeights &w, int G, int N, int kpad, const int8_t *W, const int32_t *bias, int8_t *Wd, int32_t *bd) {
  const int KH = 8 * w.stages;
  for (int g = 0; g < G; ++g)
    for (int n = 0; n < N; ++n) {
      const int pc = g * w.Np + n, tile = pc / 32, c = pc % 32;
      // the operand row whose result the lane half (c / 8) % 2 finds in its register v
      const int v = c / 16 * 8 + c % 8, rho = 8 * (v / 4) + 4 * (c / 8 % 2) + v % 4;
      const int8_t *src = W + (size_t)(g * N + n) * kpad;
      for (int k = 0; k < kpad; k += 16) {
        const int ks = k / 32, kh = ks / KH;
        std::memcpy(Wd + ((((size_t)tile * 2 + kh) * KH + ks - kh * KH) * 64 + rho + (k & 16) * 2) * 16, src + k, 16);
      }
      bd[pc] = bias[g * N + n];
    }
}

bool deep_gemm_supported(const DeepGemmArgs &a, const int32_t *r) {
  if (!a.Wd || a.lda % 16 != 0 || a.ldc % 8 != 0 || ((reinterpret_cast<uintptr_t>(a.A) | reinterpret_cast<uintptr_t>(a.out)) & 15)) return false;
  if (32ll * a.lda + 4096 >= (1ll << 31) || 64ll * a.ldc + 65536 >= (1ll << 31)) return false;  // 32-bit offsets within a block
  for (int g = 0; g < a.G; ++g)
    if (r[g] < 3 || r[g] > 62) return false;
  return true;
}

void launch_deep_gemm(hipStream_t s, const DeepGemmArgs &a0, const DeepWeights &w, int num_cus) {
  if (a0.M <= 0) return;
  DeepGemmArgs a = a0;
  a.Np = w.Np;
  a.cbs = w.cbs;
  const int nrb = (a.M + 31) / 32;
  a.parts = num_cus / a.cbs;
  if (a.parts < 1) a.parts = 1;
  if (a.parts > nrb) a.parts = nrb;
  a.by_rows = a.cbs <= 8;
  const int grid = 8 * ((a.cbs * a.parts + 7) / 8);
  if (w.stages == 3)
    launch_s<3>(s, a, grid);
  else
    launch_s<4>(s, a, grid);
}

}  // namespace lstm_int

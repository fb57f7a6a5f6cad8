// Host side of the stacked recurrent kernel (stack_kernel.inc.h): eligibility,
// LDS budget, launch, and the kernel that sets a stack launch up.
#include "persistent.h"

#include "lstm_int_math.h"

namespace lstm_int {

typedef void (*stack_fn)(StackArgs);
stack_fn stack_pick_8(int fl, bool one);   // stack_inst_8.hip
stack_fn stack_pick_20(int fl, bool one);  // stack_inst_20.hip
stack_fn stack_pick_32(int fl, bool one);  // stack_inst_32.hip

static const int kStackKS[] = {8, 20, 32};

// one = the variant for launches of one item per layer (one step, one row tile)
static stack_fn pick(int ks, int fl, bool one) {
  if (ks == 8) return stack_pick_8(fl, one);
  if (ks == 20) return stack_pick_20(fl, one);
  if (ks == 32) return stack_pick_32(fl, one);
  return nullptr;
}

bool stack_supported(int N, int H, int flags, int ipad0, int L, int T, int B, int *ks) {
  if (L < 1 || L > 8 || T < 1 || B < 1) return false;
  // whole words of four cells: tests of single cells in the stores of c, h and y made a one-step call 3 % slower
  if (N % 4 != 0 || N > 2048) return false;
  if (!(flags & 8) && H != N) return false;
  const int hpad = (H + 127) / 128 * 128;
  int k = 0;
  for (int cand : kStackKS)
    if (!k && cand * 32 >= hpad) k = cand;
  if (!k) return false;
  // the input rows of every layer go through the same LDS tile as the h rows
  const int ipad = (H + 63) / 64 * 64;  // layers above the first read the layer below
  if (ipad0 > k * 32 || ipad0 % 64 != 0 || (L > 1 && ipad > k * 32)) return false;
  // the statistics words of the kernel count up over the launch
  const int64_t items = (int64_t)T * ((B + 31) / 32);
  if (items > (1 << 14)) return false;
  *ks = k;
  return true;
}

size_t stack_lds_bytes(const StackArgs &sa) {
  const RecArgs &a = sa.c;
  const int items = 128;
  const bool proj = a.flags & 8;
  size_t tile = ((size_t)32 * (a.ks * 32 + 16) + 1023) / 1024 * 1024;
  const size_t pred = proj ? (size_t)(a.flags & kFourPredSlots ? 4 : 8) * 4096 : 0;
  if (tile < pred) tile = pred;
  size_t n = tile + (size_t)items * 8 + (size_t)items * sizeof(LnRow2) + 2 * 4 * 64 * 8 + 4 * 64 * 2 + 4 * 64 * 4 +
             8 * 32 * 4 + 32 * 4 + 320 /* StkPrm */ + 16 + 12 * 8 + 3 * 32 /* LutLds */;
  for (int i = 0; i < 2; ++i) n += (size_t)lut_wide_lds_bytes(a.lut[i].dom, a.lut[i].sh, a.lut[i].tail != 0);
  n += (size_t)sa.lutc_lds_bytes;  // the largest cell-format copy among the layers
  if (proj) {
    const int per_cu = (a.ptiles + a.GS - 1) / a.GS;
    n += ((size_t)per_cu * a.prow * (a.npadp + 16) + 1023) / 1024 * 1024;
  }
  return n;
}

hipError_t stack_init() {
  for (int ks : kStackKS)
    for (int fl = 0; fl < 32; ++fl) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick(ks, fl & 15, fl >= 16)),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

// Everything a stack launch needs in place: the initial h of every layer ([B, Hpad], given rows or the
// layer's zero point, padding bytes 0), the zeroed synchronization words and flags, and the marks of words not stored yet.
__global__ void stack_init_kernel(StackInit w) {
  const long long gtid = blockIdx.x * (long long)blockDim.x + threadIdx.x, gthreads = (long long)gridDim.x * blockDim.x;
  for (long long i = gtid; i < w.sync_vec; i += gthreads) w.sync[i] = int4{0, 0, 0, 0};
  for (long long i = gtid; i < w.mark_vec; i += gthreads) w.mark[i] = int4{(int)kMarkFree, (int)kMarkFree, (int)kMarkFree, (int)kMarkFree};
  // words of four cells; 32-bit indices, whose division is a tenth of a 64-bit one
  const unsigned row_words = (unsigned)w.ld_h0 / 4, rows = (unsigned)w.rows, total = (unsigned)w.L * rows * row_words;
  for (unsigned i = (unsigned)gtid; i < total; i += (unsigned)gthreads) {
    const unsigned row = i / row_words, l = row / rows, word = i - row * row_words;
    const int col = (int)word * 4;
    uint32_t v = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (col + c < w.cols) v |= (uint32_t)(uint8_t)(w.h_src ? w.h_src[(size_t)row * w.cols + col + c] : (int8_t)w.zp[l]) << (8 * c);
    reinterpret_cast<uint32_t *>(w.h0)[i] = v;
    if (w.mark_out && l + 1 < (unsigned)w.L)
      w.mark_out[(size_t)l * (w.mark_out_stride / 4) + (i - l * rows * row_words)] = col < w.cols ? kMarkFree : 0u;
  }
}

void launch_stack_init(hipStream_t s, const StackInit &w) {
  const long long words = (long long)w.rows * w.ld_h0 / 4 * w.L;  // below 2^31: stack_supported holds the rows below 2^19
  long long most = w.sync_vec > words ? w.sync_vec : words;
  if (w.mark_vec > most) most = w.mark_vec;
  long long blocks = (most + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(stack_init_kernel, dim3((unsigned)blocks), dim3(256), 0, s, w);
}

hipError_t launch_stack(hipStream_t s, const StackArgs &sa, bool cooperative) {
  const RecArgs &a = sa.c;
  stack_fn fn = pick(a.ks, (a.flags & 7) | ((a.flags & 8) ? 0 : 8), a.T == 1 && sa.row_tiles == 1);
  if (!fn || sa.L < 1 || sa.L > 8) return hipErrorInvalidValue;
  StackArgs args = sa;
  void *params[] = {&args};
  // one workgroup per compute unit, GS per XCD: all of them have to be resident at once (see launch_rec)
  const dim3 grid(8 * a.GS);
  if (cooperative)
    return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(fn), grid, dim3(512), params,
                                      (unsigned)stack_lds_bytes(sa), s);
  return hipLaunchKernel(reinterpret_cast<const void *>(fn), grid, dim3(512), params, (unsigned)stack_lds_bytes(sa), s);
}

}  // namespace lstm_int

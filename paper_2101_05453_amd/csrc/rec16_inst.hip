// The 16-row recurrent kernel: host side (the instantiations are in rec16_inst_4/10/16.hip).
#include "persistent.h"

#include "lstm_int_math.h"

namespace lstm_int {

static const int kKS16[] = {4, 10, 16};

typedef void (*rec_fn)(RecArgs);
rec_fn rec16_pick_4(int fl, int tag);   // rec16_inst_4.hip
rec_fn rec16_pick_10(int fl, int tag);  // rec16_inst_10.hip
rec_fn rec16_pick_16(int fl, int tag);  // rec16_inst_16.hip
static rec_fn pick16(int ks16, int fl, int tag) {
  if (ks16 == 4) return rec16_pick_4(fl, tag);
  if (ks16 == 10) return rec16_pick_10(fl, tag);
  if (ks16 == 16) return rec16_pick_16(fl, tag);
  return nullptr;
}

typedef void (*rec16_pair_fn)(RecArgs2);
rec16_pair_fn rec16_pick_pair_4(int fl, int tag);
rec16_pair_fn rec16_pick_pair_10(int fl, int tag);
rec16_pair_fn rec16_pick_pair_16(int fl, int tag);
static rec16_pair_fn pick16_pair(int ks16, int fl, int tag) {
  if (ks16 == 4) return rec16_pick_pair_4(fl, tag);
  if (ks16 == 10) return rec16_pick_pair_10(fl, tag);
  if (ks16 == 16) return rec16_pick_pair_16(fl, tag);
  return nullptr;
}

// the kernel's FORM
static int rec16_form(int flags) { return !(flags & kTaggedState) ? 0 : !(flags & 8) ? 1 : flags & kMemberStats ? 3 : 2; }

bool rec16_supported(int N, int H, int flags, int B, int *ks16, int *groups) {
  if (N > 2048 || B < 1) return false;
  if (!(flags & 8) && H != N) return false;
  const int GS = (N + 63) / 64;
  const int need = (((H + 127) / 128) * 128 + 63) / 64;
  int k = 0;
  for (int cand : kKS16)
    if (!k && cand >= need) k = cand;
  if (!k) return false;
  const int max_groups = 8 * (32 / GS);
  const int g = (B + 15) / 16;
  if (g > max_groups) return false;  // larger batches take the 32-row kernel
  *ks16 = k;
  *groups = g;
  return true;
}

size_t rec16_lds_bytes(const RecArgs &a) {
  const int items = 64;
  const bool proj = a.flags & 8;
  size_t tile = (((size_t)16 * (a.ks16 * 64 + 16) + 1023) / 1024 + 1) * 1024 + (a.flags & kTaggedState && !(a.flags & (4 | 8)) ? 1024 : 0);
  if (proj && tile < 8 * 2 * 64 * 16) tile = 8 * 2 * 64 * 16;
  size_t n = tile + (size_t)items * 8 + (size_t)items * sizeof(LnRow2) + 2 * 4 * 64 * 8 + 4 * 64 * 4 + 4 * 64 * 2 +
             256 /* PrmLds */ + 16 + 16 * 8 + 3 * 32 /* LutLds */;
  for (int i = 0; i < 3; ++i)
    if (i < 2 || a.lut[2].blob != a.lut[1].blob) n += (size_t)lut_wide_lds_bytes(a.lut[i].dom, a.lut[i].sh, a.lut[i].tail != 0);
  if (proj) {
    const int per_cu = (a.ptiles + a.GS - 1) / a.GS;
    n += ((size_t)per_cu * 32 * (a.npadp + 16) + 1023) / 1024 * 1024;  // loaded in whole 1 KB chunks
  }
  return n;
}

hipError_t rec16_init() {
  for (int ks : kKS16)
    for (int i = 0; i < 32; ++i) {
      const int fl = i & 7, tag = i >> 3;
      if (tag == 3 && !pick16(ks, fl, tag)) continue;
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick16(ks, fl, tag)),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (e != hipSuccess) return e;
      if (tag == 3) continue;
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick16_pair(ks, fl, tag)), hipFuncAttributeMaxDynamicSharedMemorySize,
                              160 * 1024);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

hipError_t launch_rec16(hipStream_t s, const RecArgs &a, bool cooperative) {
  rec_fn fn = pick16(a.ks16, a.flags & 7, rec16_form(a.flags));
  if (!fn || !a.R2h) return hipErrorInvalidValue;
  const int slots = a.GS * ((a.groups + 7) / 8);
  RecArgs args = a;
  void *params[] = {&args};
  if (cooperative)
    return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(fn), dim3(8 * slots), dim3(512), params,
                                      (unsigned)rec16_lds_bytes(a), s);
  return hipLaunchKernel(reinterpret_cast<const void *>(fn), dim3(8 * slots), dim3(512), params,
                         (unsigned)rec16_lds_bytes(a), s);
}

hipError_t launch_rec16_pair(hipStream_t s, const RecArgs2 &a, bool cooperative) {
  const RecArgs &f = a.d[0], &b = a.d[1];
  rec16_pair_fn fn = pick16_pair(f.ks16, f.flags & 7, rec16_form(f.flags));
  if (!fn || !f.R2h || !b.R2h || f.GS != b.GS || f.ks16 != b.ks16 || f.flags != b.flags || f.groups + b.groups > 8 * (32 / f.GS))
    return hipErrorInvalidValue;
  const int slots = f.GS * ((f.groups + b.groups + 7) / 8);
  const size_t lf = rec16_lds_bytes(f), lb = rec16_lds_bytes(b);
  RecArgs2 args = a;
  void *params[] = {&args};
  const auto launch = cooperative ? [](const void *k, dim3 g, dim3 t, void **p, size_t l, hipStream_t st) { return hipLaunchCooperativeKernel(k, g, t, p, (unsigned)l, st); }
                                  : [](const void *k, dim3 g, dim3 t, void **p, size_t l, hipStream_t st) { return hipLaunchKernel(k, g, t, p, l, st); };
  return launch(reinterpret_cast<const void *>(fn), dim3(8 * slots), dim3(512), params, lf > lb ? lf : lb, s);
}

}  // namespace lstm_int

// The four-row recurrent kernel (quad_kernel.inc.h): host side (the instantiations are in quad_inst_8/10/16.hip).
#include "persistent.h"

#include "lstm_int_math.h"

namespace lstm_int {

typedef void (*quad_fn)(RecArgs2);
quad_fn quad_pick_8(int fl);   // quad_inst_8.hip
quad_fn quad_pick_10(int fl);  // quad_inst_10.hip
quad_fn quad_pick_16(int fl);  // quad_inst_16.hip

static int quad_ks(int H) { return H <= 512 ? 8 : H <= 640 ? 10 : H <= 1024 ? 16 : 0; }
static quad_fn pick_quad(int ks16, int fl) {
  if (ks16 == 8) return quad_pick_8(fl);
  if (ks16 == 10) return quad_pick_10(fl);
  if (ks16 == 16) return quad_pick_16(fl);
  return nullptr;
}

// Wherever its groups fit one launch: it is the faster one at every size measured (quad_kernel.inc.h).  A workgroup stores
// 64 columns of the output and projects 64 outputs at most.
bool quad_supported(int N, int H, int flags, int B, int share, int *groups) {
  if (N > 2048 || B < 1 || !quad_ks(H) || (!(flags & 8) && H != N)) return false;
  const int GS = (N + 63) / 64;
  const int g = (B + 3) / 4;
  if (GS < 2 || H > 64 * GS || g * share > 8 * (32 / GS)) return false;
  *groups = g;
  return true;
}

size_t quad_lds_bytes(const RecArgs &a) {
  const bool proj = a.flags & 8;
  const size_t LS = (size_t)quad_ks(a.H) * 64 + 16, MLS = (size_t)((a.N + 63) & ~63) + 16;
  size_t n = 2 * 4 * LS + (proj ? 4 * MLS : 0) + 2 * 2048 + 16 * 8 + 16 * sizeof(LnRow2) + 16;
  n = (n + 1023) & ~(size_t)1023;
  for (int i = 0; i < 3; ++i)
    if (i < 2 || a.lut[2].blob != a.lut[1].blob) n += (size_t)lut_wide_lds_bytes(a.lut[i].dom, a.lut[i].sh, a.lut[i].tail != 0);
  if (proj) n += (size_t)(((a.H + 15) / 16 + a.GS - 1) / a.GS) * 16 * MLS;
  return n;
}

hipError_t quad_init() {
  for (int ks : {8, 10, 16})
    for (int fl = 0; fl < 8; ++fl) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick_quad(ks, fl)),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

hipError_t launch_quad(hipStream_t s, const RecArgs2 &a, bool cooperative) {
  const RecArgs &f = a.d[0], &b = a.d[1];
  quad_fn fn = pick_quad(quad_ks(f.H), f.flags & 7);
  const int groups = f.groups + b.groups;
  if (!fn || !f.R2h || f.rows_pg != 4 || f.groups != (f.B + 3) / 4 || groups > 8 * (32 / f.GS) ||
      (b.groups > 0 && (!b.R2h || b.N != f.N || b.H != f.H || f.flags != b.flags || b.rows_pg != 4 || b.groups != (b.B + 3) / 4)))
    return hipErrorInvalidValue;
  size_t lds = quad_lds_bytes(f);
  if (b.groups > 0) lds = lds > quad_lds_bytes(b) ? lds : quad_lds_bytes(b);
  RecArgs2 args = a;
  void *params[] = {&args};
  const dim3 grid(8 * f.GS * ((groups + 7) / 8));
  // all workgroups have to be resident at once (see launch_rec)
  if (cooperative)
    return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(fn), grid, dim3(256), params, (unsigned)lds, s);
  return hipLaunchKernel(reinterpret_cast<const void *>(fn), grid, dim3(256), params, lds, s);
}

}  // namespace lstm_int

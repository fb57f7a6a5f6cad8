// The one-workgroup recurrent kernel (solo_kernel.inc.h): instantiations and host side.
#include "solo_kernel.inc.h"

namespace lstm_int {

// cells one workgroup takes in each of the three forms
static const int kSoloCells[3] = {64, 128, 256};
static int solo_form(int N, int H) {
  for (int i = 0; i < 3; ++i)
    if (N <= kSoloCells[i] && H <= kSoloCells[i]) return i;
  return -1;
}
static solo_fn pick_solo(int form, int fl) {
  if (form == 0) return solo_pick_size<4, 1>(fl);
  if (form == 1) return solo_pick_size<8, 2>(fl);
  if (form == 2) return solo_pick_size<16, 4>(fl);
  return nullptr;
}

// Where it is the faster one (up to 256 rows row_kernel is faster still, row_inst.hip).  Time per step, us, this kernel (16 or 1024 rows alike; without - with a projection) / groups of
// 16 rows over several workgroups, up to 1024 rows:
//   64 cells 0.7-0.8 / 2.6,      with layer norm 1.5-1.6 / 4.4,      and peephole 2.1-2.3 / 5.9
//  128 cells 0.8-1.0 / 3.0-3.3,                  1.8-2.0 / 4.7-5.1,               2.4-2.7 / 6.1-6.6
//  256 cells 1.4-1.9 / 3.2-3.7,                  3.0-3.5 / 4.8-5.4,               3.6-4.1 / 6.2-6.6
// From 1025 rows on a second round of workgroups doubles it: still less up to 128 cells.
bool solo_supported(int N, int H, int flags, int B) {
  const int form = solo_form(N, H);
  return form >= 0 && ((flags & 8) || H == N) && B <= (form == 2 ? 1024 : 2048);
}

size_t solo_lds_bytes(const RecArgs &a) {
  const int form = solo_form(a.N, a.H);
  if (form < 0) return (size_t)1 << 30;
  const size_t NC = kSoloCells[form], LS = NC + 16;
  size_t n = 3 * 4 * LS + 16 * 8 + 16 * sizeof(LnRow2) + 16 + (form == 2 && (a.flags & 4) ? 2 * 4 * NC * 8 : 0);
  n = (n + 1023) & ~(size_t)1023;
  for (int i = 0; i < 3; ++i)
    if (i < 2 || a.lut[2].blob != a.lut[1].blob) n += (size_t)lut_wide_lds_bytes(a.lut[i].dom, a.lut[i].sh, a.lut[i].tail != 0);
  if (a.flags & 8) n += (size_t)((a.H + 15) & ~15) * LS;
  return n;
}

hipError_t solo_init() {
  for (int form = 0; form < 3; ++form)
    for (int fl = 0; fl < 16; ++fl) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick_solo(form, fl)),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

hipError_t launch_solo(hipStream_t s, const RecArgs2 &a) {
  const RecArgs &f = a.d[0], &b = a.d[1];
  const int form = solo_form(f.N, f.H);
  solo_fn fn = pick_solo(form, f.flags & 15);
  if (!fn || !f.R2h || f.rows_pg != 4 || f.groups != (f.B + 3) / 4 ||
      (b.groups > 0 && (!b.R2h || solo_form(b.N, b.H) != form || f.flags != b.flags || b.rows_pg != 4 || b.groups != (b.B + 3) / 4)))
    return hipErrorInvalidValue;
  size_t lds = solo_lds_bytes(f);
  if (b.groups > 0) lds = lds > solo_lds_bytes(b) ? lds : solo_lds_bytes(b);
  RecArgs2 args = a;
  void *params[] = {&args};
  return hipLaunchKernel(reinterpret_cast<const void *>(fn), dim3(f.groups + b.groups), dim3(form == 0 ? 256 : form == 1 ? 512 : 1024), params, lds, s);
}

}  // namespace lstm_int

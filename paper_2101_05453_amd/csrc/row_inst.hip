// The recurrent kernel with one batch row per workgroup (row_kernel.inc.h): instantiations and host side.
#include "row_kernel.inc.h"

namespace lstm_int {

// cells one workgroup takes in each of the three forms
static const int kRowCells[3] = {64, 128, 256};
static int row_form(int N, int H) {
  for (int i = 0; i < 3; ++i)
    if (N <= kRowCells[i] && H <= kRowCells[i]) return i;
  return -1;
}
static row_fn pick_row(int form, int fl) {
  if (form == 0) return row_pick_size<4, 1>(fl);
  if (form == 1) return row_pick_size<8, 2>(fl);
  if (form == 2) return row_pick_size<16, 4>(fl);
  return nullptr;
}

// Up to 256 rows, a compute unit for each: the launch of four rows per workgroup -> this one, us, 100 steps of 64 rows, input 64
//                 no layer norm    layer norm    and peephole    projection, no layer norm
//   64 cells          79 ->  62     161 -> 109     223 -> 173          92 ->  75
//   128 cells         95 ->  74     197 -> 141     255 -> 229         121 ->  89
//   203 cells        174 -> 125     337 -> 186     389 -> 269         207 -> 153
//   256 cells        173 -> 128     334 -> 195     391 -> 276         214 -> 162
// With 256 rows the gain is 10 to 39 %; with 260, a second round of workgroups, the four-row form is ahead (60 steps: 64 cells
// 56 against 82, 256 cells with layer norm 211 against 260).
bool row_supported(int N, int H, int flags, int rows) {
  const int form = row_form(N, H);
  return form >= 0 && ((flags & 8) || H == N) && rows <= 256;
}

size_t row_lds_bytes(const RecArgs &a) {
  const int form = row_form(a.N, a.H);
  if (form < 0) return (size_t)1 << 30;
  const size_t NC = kRowCells[form];
  size_t n = 3 * NC + 16 * 8 + 4 * sizeof(LnRow2) + 64 + 128;
  n = (n + 1023) & ~(size_t)1023;
  n += row_ahead(NC / 16) * (NC / 16) * 128 + (form == 2 && (a.flags & 4) ? 1024 * 16 : 0);
  for (int i = 0; i < 3; ++i)
    if (i < 2 || a.lut[2].blob != a.lut[1].blob) n += (size_t)lut_wide_lds_bytes(a.lut[i].dom, a.lut[i].sh, a.lut[i].tail != 0);
  if (form == 2 && (a.flags & 8)) n += (size_t)((a.H + 15) & ~15) * (NC + 16);
  return n;
}

hipError_t row_init() {
  for (int form = 0; form < 3; ++form)
    for (int fl = 0; fl < 16; ++fl) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick_row(form, fl)),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

hipError_t launch_row(hipStream_t s, const RecArgs2 &a) {
  const RecArgs &f = a.d[0], &b = a.d[1];
  const int form = row_form(f.N, f.H);
  row_fn fn = pick_row(form, f.flags & 15);
  if (!fn || !f.R2h || f.rows_pg != 1 || f.groups != f.B ||
      (b.groups > 0 && (!b.R2h || row_form(b.N, b.H) != form || f.flags != b.flags || b.rows_pg != 1 || b.groups != b.B)))
    return hipErrorInvalidValue;
  size_t lds = row_lds_bytes(f);
  if (b.groups > 0) lds = lds > row_lds_bytes(b) ? lds : row_lds_bytes(b);
  RecArgs2 args = a;
  void *params[] = {&args};
  return hipLaunchKernel(reinterpret_cast<const void *>(fn), dim3(f.groups + b.groups), dim3(64 * (((f.N > f.H ? f.N : f.H) + 15) / 16)), params, lds, s);
}

}  // namespace lstm_int

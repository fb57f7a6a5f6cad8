// The recurrent kernel with one batch row per workgroup (row_kernel.inc.h): host side (instantiations: row_inst_*.hip).
#include "row_kernel.inc.h"

namespace lstm_int {

// cells one workgroup takes in each of the three forms
static const int kRowCells[3] = {64, 128, 256};
static int row_form(int N, int H) {
  for (int i = 0; i < 3; ++i)
    if (N <= kRowCells[i] && H <= kRowCells[i]) return i;
  return -1;
}
// row_inst_{64,128,192,256}.hip, row_stack_inst_{...}.hip
row_fn row_pick_64(int fl, bool own);
row_fn row_pick_128(int fl, bool own);
row_fn row_pick_192(int fl, bool own);
row_fn row_pick_256(int fl, bool own);
row_fn row_pick_256_128(int fl, bool own);
row_stack_fn row_stack_pick_64(int fl);
row_stack_fn row_stack_pick_128(int fl);
row_stack_fn row_stack_pick_192(int fl);
row_stack_fn row_stack_pick_256(int fl);
row_stack_fn row_stack_pick_256_128(int fl);
// H: outputs, the depth of R h
static row_fn pick_row(int form, int H, int fl, bool own) {
  if (form == 0) return row_pick_64(fl, own);
  if (form == 1) return row_pick_128(fl, own);
  if (form != 2) return nullptr;
  return H <= 128 && (fl & 8) ? row_pick_256_128(fl, own) : H <= 192 ? row_pick_192(fl, own) : row_pick_256(fl, own);
}
static row_stack_fn pick_row_stack(int form, int H, int fl) {
  if (form == 0) return row_stack_pick_64(fl);
  if (form == 1) return row_stack_pick_128(fl);
  if (form != 2) return nullptr;
  return H <= 128 && (fl & 8) ? row_stack_pick_256_128(fl) : H <= 192 ? row_stack_pick_192(fl) : row_stack_pick_256(fl);
}

// Several layers in one launch (row_stack_inst_{64,128,192,256}.hip): T steps of L layers take T + (L - 1) (piece + 1) steps one
// behind the other instead of L T, and a launch instead of one or two per layer; W x of a piece comes to 2 to 5 us.  Layer after layer (or the
// stacked launch, where that is ahead) -> this, us:
//   6 layers of 86 cells, layer norm, 5 rows, 1 step      63 -> 34     3 layers of 128 cells, layer norm, 39 rows, 43 steps   187 -> 117
//   6 layers of 32 cells, layer norm, 16 rows, 100 steps 575 -> 201    4 layers of 219 cells, peephole, 11 rows, 64 steps      366 -> 179
//   2 layers of 203 cells, 131 outputs, 37 rows, 60 steps 217 -> 140    2 layers of 49 cells, 32 rows, 3 steps, two directions   25 -> 22

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

static size_t lds_bytes(const RecArgs &a, int form, size_t term_bytes) {  // term_bytes: of a wave's W x terms
  if (form < 0) return (size_t)1 << 30;
  const size_t NC = kRowCells[form];
  size_t n = 3 * NC + 16 * 8 + 4 * sizeof(LnRow2) + 64 + 128;
  n = (n + 1023) & ~(size_t)1023;
  n += (NC / 16) * term_bytes + (form == 2 && (a.flags & 4) ? 1024 * 16 : 0);
  for (int i = 0; i < 3; ++i)
    if (i < 2 || a.lut[2].blob != a.lut[1].blob) n += (size_t)lut_wide_lds_bytes(a.lut[i].dom, a.lut[i].sh, a.lut[i].tail != 0);
  if (form == 2 && (a.flags & 8)) n += (size_t)((a.H + 15) & ~15) * (NC + 16);
  return n;
}

size_t row_lds_bytes(const RecArgs &a, bool own) {
  const int form = row_form(a.N, a.H);
  return form < 0 ? (size_t)1 << 30 : lds_bytes(a, form, row_terms_bytes(kRowCells[form] / 16, a.T, own));
}
size_t row_stack_lds_bytes(const RecArgs &a, int widest, int term_steps, int x_bytes) {
  return lds_bytes(a, row_form(widest, widest), (size_t)term_steps * 128) + x_bytes;
}

hipError_t row_init() {
  for (int form = 0; form < 3; ++form)
    for (int H = form < 2 ? 256 : 128; H <= 256; H += 64)
      for (int k = 0; k < 32; ++k) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick_row(form, H, k >> 1, k & 1)),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e == hipSuccess && !(k & 1))
          e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick_row_stack(form, H, k >> 1)),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
      }
  return hipSuccess;
}

// The input GEMM's launch takes 5 us and more, its weights and its output on top; W x in the launch itself takes 1.4 us for every
// 16 steps and a microsecond for every 95 KB of weights, which come anew with each.  us per call, GEMM -> in the launch itself:
//     cells, inputs       64, 64          64, 1024        128, 256        128, 1024       256, 64         256, 1024
//     1 row, 4 steps      14.6 -> 11.6    18.0 -> 13.2    16.4 -> 13.6    20.2 -> 16.4    23.9 -> 20.7    27.9 -> 28.5
//     1 row, 16           25.3 -> 21.8    29.4 -> 24.4    30.9 -> 26.4    34.9 -> 31.1    43.9 -> 39.8    48.0 -> 51.8
//     1 row, 32           25.9 -> 24.5    29.6 -> 29.1    30.0 -> 27.9    33.9 -> 37.5
//     256 rows, 32        32.2 -> 25.7    35.5 -> 30.4    37.6 -> 29.1    42.1 -> 39.2
//     1 row, 64           68.1 -> 69.3    72.8 -> 80.6    84.2 -> 84.9    88.5 -> 104.2
bool row_takes_input(int N, int H, int kpad, int T, int B) {
  const int form = row_form(N, H);
  if (form < 0 || T > row_input_steps(kRowCells[form] / 16)) return false;
  const double kb = 4.0 * ((N + 15) / 16 * 16) * kpad / 1024, out_mb = 8e-6 * T * B * N;
  return (T + 15) / 16 * (1.4 + kb / 95) < 5.0 + kpad / 250.0 + out_mb / 3.5;
}

void row_set_input(RowInput &in, const InGemmArgs &g) {
  in.x = g.A;
  in.ldx = g.lda;
  in.cols = g.cols ? g.cols : g.kpad;
  in.W2f = g.W2f;
  in.bx2 = g.bx2;
  in.kx = g.kpad / 64;
  in.pre = g.pre;
  for (int i = 0; i < 4; ++i) {
    in.rs[i] = rescale_hi_prepare(g.M[i], g.r[i]);
    if (in.rs[i].k != 0) in.pre = 2;
  }
}

hipError_t launch_row(hipStream_t s, const RowArgs &a) {
  const RecArgs &f = a.rec.d[0], &b = a.rec.d[1];
  const int form = row_form(f.N, f.H);
  const bool own = a.in[0].x != nullptr;
  row_fn fn = pick_row(form, f.H, f.flags & 15, own);
  if (!fn || !f.R2h || f.rows_pg != 1 || f.groups != f.B ||
      (own && f.T > row_input_steps(kRowCells[form] / 16)) ||
      (b.groups > 0 && (!b.R2h || row_form(b.N, b.H) != form || f.H != b.H || f.flags != b.flags || b.rows_pg != 1 ||
                        b.groups != b.B || own != (a.in[1].x != nullptr))))
    return hipErrorInvalidValue;
  size_t lds = row_lds_bytes(f, own);
  if (b.groups > 0) lds = lds > row_lds_bytes(b, own) ? lds : row_lds_bytes(b, own);
  RowArgs args = a;
  const int blocks = ((f.N > f.H ? f.N : f.H) + 15) / 16;  // a wave each; four at least, which bring the tables in sooner
  void *params[] = {&args};
  return hipLaunchKernel(reinterpret_cast<const void *>(fn), dim3(f.groups + b.groups), dim3(64 * (blocks < 4 ? 4 : blocks)), params, lds, s);
}

void row_stack_layer(RowLayer &to, const RecDirArgs &from) {
  to.T = from.T; to.B = from.B; to.N = from.N; to.H = from.H; to.Hpad = from.Hpad; to.Bp = from.Bp; to.Ncp = from.Ncp;
  to.ks16 = from.ks16; to.npadp = from.npadp; to.ldy = from.ldy; to.rev = from.rev; to.m_c = from.m_c; to.pre_h = from.pre_h;
  to.R2h = from.R2h; to.bh4 = from.bh4; to.Lq4 = from.Lq4; to.qb4 = from.qb4; to.Pq3 = from.Pq3;
  for (int g = 0; g < 4; ++g) {
    to.Mh[g] = from.Mh[g]; to.rh[g] = from.rh[g];
    to.Mln[g] = from.Mln[g]; to.rln[g] = from.rln[g];
  }
  for (int j = 0; j < 3; ++j) {
    to.Mc[j] = from.Mc[j]; to.rc[j] = from.rc[j];
    to.lut[j] = from.lut[j];
  }
  to.Mm = from.Mm; to.rm = from.rm; to.zp_m = from.zp_m;
  to.Mp = from.Mp; to.rp = from.rp; to.zp_h = from.zp_h;
  to.Wp2 = from.Wp2; to.bp2 = from.bp2; to.tx2 = from.tx2; to.h0 = from.h0; to.out = from.out; to.y = from.y;
  to.c_in = from.c_in; to.c_out = from.c_out; to.status = from.status;
}

hipError_t launch_row_stack(hipStream_t s, const RowStackArgs &a, int layers, int flags, int widest, size_t lds) {
  const int form = row_form(widest, widest);
  int H = 0;
  for (int l = 0; l < layers && l < kRowStackLayers; ++l) H = H > a.rec.d[l].H ? H : a.rec.d[l].H;
  row_stack_fn fn = layers < 1 || layers > kRowStackLayers ? nullptr : pick_row_stack(form, H, flags & 15);
  if (!fn || lds > 160 * 1024 || a.dirs < 1 || a.dirs > 2 || layers % a.dirs != 0) return hipErrorInvalidValue;
  for (int i = 0; i < a.dirs; ++i)  // where workgroups that start are counted
    if (a.in[i].done != a.in[0].done + (size_t)i * a.rec.d[0].B * kRowFlagWords || !a.in[0].done) return hipErrorInvalidValue;
  for (int l = 0; l < layers; ++l) {
    const RowInput &in = a.in[l];
    if (a.rec.d[l].B != a.rec.d[0].B || in.piece < 1 || in.piece > 16 || in.term_steps < (in.x ? in.piece : 2 * in.piece) ||
        (in.x && in.x_bytes < 1024 * in.kx) || !a.rec.d[l].R2h || (!in.x && !a.rec.d[l].tx2))
      return hipErrorInvalidValue;
  }
  RowStackArgs args = a;
  const int blocks = (widest + 15) / 16;
  void *params[] = {&args};
  return hipLaunchKernel(reinterpret_cast<const void *>(fn), dim3(layers * a.rec.d[0].B), dim3(64 * (blocks < 4 ? 4 : blocks)), params,
                         lds, s);
}

}  // namespace lstm_int

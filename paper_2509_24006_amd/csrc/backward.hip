// Backward pass, host side: workspace and the order of the launches.
#include "sla_internal.h"

namespace sla {
namespace {

struct BwdWs {
  KvSplit kv;
  float *Ds, *dHZ, *dHZcol, *dQlin, *dWpart;
  int nparts;
  size_t bytes;
};

BwdWs carve_bwd(const Shape& s, char* ws) {
  BwdWs w;
  size_t off = 0;
  auto take = [&](size_t n) {
    float* p = reinterpret_cast<float*>(ws + off);
    off += align_up(n * sizeof(float));
    return p;
  };
  const size_t nd = (size_t)s.BH * s.N * s.d, n = (size_t)s.BH * s.N;
  const size_t st = (size_t)s.BH * s.T * s.state_row();
  w.nparts = s.BH * s.T < 512 ? s.BH * s.T : 512;   // two workgroups per CU
  w.Ds = take(n);
  w.dHZ = take(st);
  w.dHZcol = take(st);
  w.dQlin = take(s.dtype == 0 ? 0 : nd);   // (bf16 with query blocks of several tiles)
  w.dWpart = take((size_t)w.nparts * s.d * s.d);
  w.kv = kv_split(s);
  w.kv.units = reinterpret_cast<int4*>(take((size_t)s.BH * (2 * w.kv.ecap + s.T) * 4));
  w.kv.part = take((size_t)s.BH * 2 * w.kv.ecap * 2 * kBlk * s.d);
  w.bytes = off;
  return w;
}

hipError_t backward_bf16(const Shape& s, const BwdArgs& a, hipStream_t st) {
  const BwdWs w = carve_bwd(s, a.ws);
  const bool lin = s.n_0 > 0;
  SLA_TRY(mfma_backward_query(s, a, w.Ds, w.dHZ, w.dQlin, w.dWpart, w.nparts, w.kv, st));   // dHZ holds bf16 rows
  if (lin) {
    SLA_TRY(mfma_aggregate(w.dHZ, a.indT, s, w.dHZcol,
                           reinterpret_cast<float*>(reinterpret_cast<char*>(w.dHZcol) + state_z_offset(s)), st));
  }
  return mfma_backward_sparse(s, a, w.Ds, lin ? w.dHZcol : nullptr, DwSum{w.dWpart, w.nparts, s.d * s.d, a.dW, a.dW16}, w.kv, st);
}

}  // namespace

// Whether and into what the column lists are cut.  They are very uneven (on video-like inputs the longest holds four
// to thirty times the average), and where a workgroup slot of the chip has few entries the launch lasts as long as
// the longest list.  A cut list costs float sums out and back and a launch that adds them.  So a piece lasts about
// as long as a slot's share of everything (a key block's fixed cost is that of four entries; with floats, where an
// entry takes several times as long, it does not count), and nothing is cut where a third of the longest list there
// can be, T, is shorter than a piece, nor above 256 blocks: there all but a handful of heads are balanced as they
// are (16 x 387 of 19, d = 128, whole -> pieces of a quarter: 644 -> 679; 12 x 512 of 26 776 -> 813), and a head's
// gradients stay the same bits with any number of heads in the call.  Below, the rounding of dK and dV follows the
// pieces and so the number of heads; a rule by T alone would cost many heads more than it gives few (pieces of a
// third, 64 x 254 of 10, d = 64: 585 -> 623; 256 x 42 of 5 241 -> 271).  (Key side with the adding launch, whole ->
// cut, us: 12 x 146 of 7, d = 128, 139 -> 113; 14 x 68 of 2 80 -> 51; 8 x 254 of 10, d = 64, 107 -> 78; 8 x 42 of 7
// 42 -> 30; where the lists happen to be short, 16 x 58 of 2, d = 128, at most 21: 41 -> 48.  Floats: 4 x 122 of 6,
// d = 128, 175 -> 157; 2 x 122 of 12 201 -> 152; 8 x 122 of 6, d = 64, 228 -> 139; 16 x 63 of 5 157 -> 125.)
namespace {
KvSplit split_for(const Shape& s, int parts) {   // parts: workgroups per key block
  const bool f32 = s.dtype == 0;
  const long long slots = s.d == 64 && !f32 ? 768 : 512;
  const long long cols = (long long)s.BH * s.T * parts;
  long long piece = (cols * s.n_h + slots - 1) / slots + (f32 ? 0 : 4 * cols / slots);
  piece = piece < 12 ? 12 : piece;
  if (s.n_h == 0 || s.T > 256 || 3 * piece > s.T) return KvSplit{0x7fffffff, 0, nullptr, nullptr};
  return KvSplit{(int)piece, (int)((long long)s.T * s.n_h / piece), nullptr, nullptr};
}
}  // namespace
KvSplit kv_split(const Shape& s) { return split_for(s, s.dtype != 0 ? 1 : f32_key_quarters(s) ? 4 : 2); }

// Quarters fill the chip where there are few blocks; with more the tiles that they fetch cost more.  Where the long
// lists are cut the line is lower, as the longest list no longer sets the length of the launch.
// (Key side with the adding launch, quarters -> halves, us.  Lists cut: 3 heads x 64 blocks, d = 64, 50 -> 72;
// 2 x 122 of 12, d = 128, 152 -> 160; 4 x 122 of 6 169 -> 157; 12 x 63 of 6 252 -> 236; the number of blocks does
// not separate them all: 1 x 127 of 19, below the line, 141 -> 129.  Whole lists: 1 x 500 of 25, d = 128, 622 -> 986;
// 2 x 300 of 15 519 -> 801; 1 x 625 of 31, d = 64, 477 -> 706; too dense to cut, d = 64, 3 x 160 of 32
// 310 -> 430, 8 x 48 of 14 124 -> 160, too short, 24 x 30 of 3 71 -> 82; 4 x 122 of 24, d = 128, 484 -> 523.)
bool f32_key_quarters(const Shape& s) {
  const int blocks = s.BH * s.T;
  return blocks < 384 || (blocks < 768 && split_for(s, 2).ecap == 0);
}

size_t backward_ws_bytes(const Shape& s) { return carve_bwd(s, nullptr).bytes; }

hipError_t backward(const Shape& s, const BwdArgs& a, hipStream_t st) {
  if (s.dtype != 0) return backward_bf16(s, a, st);
  const BwdWs w = carve_bwd(s, a.ws);
  return f32_backward(s, a, w.Ds, w.dHZ, w.dHZcol, w.dWpart, w.nparts, w.kv, st);
}

}  // namespace sla

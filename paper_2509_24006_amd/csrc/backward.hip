// Backward pass, host side: workspace and the order of the launches.
#include <algorithm>

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
  w.kv.units = reinterpret_cast<int4*>(take(w.kv.ecap ? (size_t)s.BH * (w.kv.ecap + s.T + w.kv.cuts) * 4 : 0));
  w.kv.part = take((size_t)s.BH * (w.kv.ecap + w.kv.cuts) * 2 * kBlk * s.d);
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
// the longest list.  A piece of its own costs float sums out and back and its share of a launch that adds them.
// Nothing is cut above 256 blocks: there all but a handful of heads are balanced as they are (16 x 387 of 19, d = 128,
// whole -> pieces of a quarter: 644 -> 679; 12 x 512 of 26 776 -> 813).
//
// bf16: the pieces follow from a head's own shape, so that the rounding of its dK and dV is the same in any call; the
// number of heads decides only who walks them.  With few heads, while a slot's share of the launch (a key block's
// fixed cost is that of four entries) is below a third of the longest list there can be, T, the pieces are shared
// out; with more one workgroup walks all of them, which costs the sums of its long lists out and back.  Shorter pieces
// balance a few heads better and cost the others more, and lists of average length should stay whole: hence T / 6 and
// one and a half times the average.  Key side with the adding launch and dW's sums, us:
//                                            d    whole   T / 8   T / 6   T / 4
//   1 head x 146 blocks of 7                128      58      39      45      58
//   12 x 146 of 7, the longest 66           128     101     116     109     109
//   the same, b_q = 128, the longest 100    128     137     122     118     111
//   3 x 254 of 10                            64     108      59      61      74
//   40 x 146 of 7, one workgroup a list     128     309     319     318     318
//   64 x 254 of 10, one workgroup a list     64     553     565     566     556
// Where the lists happen to be short nothing is gained: 16 x 58 of 2, d = 128, at most 22, whole 42, shared out 50.
// (2 x 250 of 50, d = 128, pieces of 50, 75, 100: 135, 141, 171; 64 x 128 of 13, one workgroup a list, pieces of 16, 20,
// 26: 637, 624, 615, whole 605.)
//
// Floats, whose sums depend on the number of heads in any case (f32_key_quarters): a piece lasts about as long as a
// slot's share of everything, and nothing is cut where a third of T is shorter than that.  (Key side with the
// adding launch, whole -> cut, us: 4 x 122 of 6, d = 128, 175 -> 157; 2 x 122 of 12 201 -> 152; 8 x 122 of 6, d = 64,
// 228 -> 139; 16 x 63 of 5 157 -> 125.)
namespace {
KvSplit split_f32(const Shape& s, int parts) {   // parts: workgroups per key block
  const long long cols = (long long)s.BH * s.T * parts;
  const long long piece = std::max((cols * s.n_h + 511) / 512, 12ll);
  if (s.n_h == 0 || s.T > 256 || 3 * piece > s.T) return KvSplit{0x7fffffff, 0, 0, nullptr, nullptr};
  return KvSplit{(int)piece, (int)(s.T * s.n_h / piece), (int)(s.T * s.n_h / (piece + 1)), nullptr, nullptr};
}
KvSplit split_bf16(const Shape& s) {
  const int piece = (std::max({12, s.T / 6, 3 * s.n_h / 2}) + 1) & ~1;   // (even: the kernel's loop takes two entries)
  if (s.n_h == 0 || s.T > 256 || 2 * piece > s.T) return KvSplit{0x7fffffff, 0, 0, nullptr, nullptr};
  const long long slots = s.d == 64 ? 768 : 512;
  const bool shared = 3ll * s.BH * (s.n_h + 4) <= slots;
  return KvSplit{piece, shared ? s.T * s.n_h / piece : 0, s.T * s.n_h / (piece + 1), nullptr, nullptr};
}
}  // namespace
KvSplit kv_split(const Shape& s) { return s.dtype != 0 ? split_bf16(s) : split_f32(s, f32_key_quarters(s) ? 4 : 2); }

// Quarters fill the chip where there are few blocks; with more the tiles that they fetch cost more.  Where the long
// lists are cut the line is lower, as the longest list no longer sets the length of the launch.
// (Key side with the adding launch, quarters -> halves, us.  Lists cut: 3 heads x 64 blocks, d = 64, 50 -> 72;
// 2 x 122 of 12, d = 128, 152 -> 160; 4 x 122 of 6 169 -> 157; 12 x 63 of 6 252 -> 236; the number of blocks does
// not separate them all: 1 x 127 of 19, below the line, 141 -> 129.  Whole lists: 1 x 500 of 25, d = 128, 622 -> 986;
// 2 x 300 of 15 519 -> 801; 1 x 625 of 31, d = 64, 477 -> 706; too dense to cut, d = 64, 3 x 160 of 32
// 310 -> 430, 8 x 48 of 14 124 -> 160, too short, 24 x 30 of 3 71 -> 82; 4 x 122 of 24, d = 128, 484 -> 523.)
bool f32_key_quarters(const Shape& s) {
  const int blocks = s.BH * s.T;
  return blocks < 384 || (blocks < 768 && split_f32(s, 2).ecap == 0);
}

size_t backward_ws_bytes(const Shape& s) { return carve_bwd(s, nullptr).bytes; }

hipError_t backward(const Shape& s, const BwdArgs& a, hipStream_t st) {
  if (s.dtype != 0) return backward_bf16(s, a, st);
  const BwdWs w = carve_bwd(s, a.ws);
  return f32_backward(s, a, w.Ds, w.dHZ, w.dHZcol, w.dWpart, w.nparts, w.kv, st);
}

}  // namespace sla

// Backward pass, host side: workspace and the order of the launches.
#include "sla_internal.h"

namespace sla {
namespace {

struct BwdWs {
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
  w.bytes = off;
  return w;
}

hipError_t backward_bf16(const Shape& s, const BwdArgs& a, hipStream_t st) {
  const BwdWs w = carve_bwd(s, a.ws);
  const bool lin = s.n_0 > 0;
  SLA_TRY(mfma_backward_query(s, a, w.Ds, w.dHZ, w.dQlin, w.dWpart, w.nparts, st));   // dHZ holds bf16 rows
  if (lin) {
    SLA_TRY(mfma_aggregate(w.dHZ, a.indT, s, w.dHZcol,
                           reinterpret_cast<float*>(reinterpret_cast<char*>(w.dHZcol) + state_z_offset(s)), st));
  }
  return mfma_backward_sparse(s, a, w.Ds, lin ? w.dHZcol : nullptr, DwSum{w.dWpart, w.nparts, s.d * s.d, a.dW, a.dW16}, st);
}

}  // namespace

size_t backward_ws_bytes(const Shape& s) { return carve_bwd(s, nullptr).bytes; }

hipError_t backward(const Shape& s, const BwdArgs& a, hipStream_t st) {
  if (s.dtype != 0) return backward_bf16(s, a, st);
  const BwdWs w = carve_bwd(s, a.ws);
  return f32_backward(s, a, w.Ds, w.dHZ, w.dHZcol, w.dWpart, w.nparts, st);
}

}  // namespace sla

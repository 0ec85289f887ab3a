// Backward pass, host side: workspace, the order of the launches, and the reduction of dW's
// partial sums that both storage types share.
#include "sla_internal.h"

namespace sla {
namespace {

// dW = sum of the partial d x d sums.  A workgroup owns 64 consecutive elements; its four waves
// take every fourth partial each (one element per lane, 256 contiguous bytes per load) and meet
// in LDS.
__global__ __launch_bounds__(256) void dw_reduce_kernel(const float* __restrict__ part, int nparts, int dd,
                                                        float* __restrict__ dW) {
  __shared__ float red[4][64];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int idx = blockIdx.x * 64 + l;
  float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
  if (idx < dd) {
    int p = w;
    for (; p + 12 < nparts; p += 16) {
      s0 += part[(size_t)p * dd + idx];
      s1 += part[(size_t)(p + 4) * dd + idx];
      s2 += part[(size_t)(p + 8) * dd + idx];
      s3 += part[(size_t)(p + 12) * dd + idx];
    }
    for (; p < nparts; p += 4) s0 += part[(size_t)p * dd + idx];
  }
  red[w][l] = (s0 + s1) + (s2 + s3);
  __syncthreads();
  if (w == 0 && idx < dd) dW[idx] = (red[0][l] + red[1][l]) + (red[2][l] + red[3][l]);
}

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
  SLA_TRY(mfma_backward_query(s, a, w.Ds, w.dHZ, w.dQlin, st));   // dHZ holds bf16 rows
  SLA_TRY(mfma_backward_dw(s, a, w.dWpart, w.nparts, st));
  SLA_TRY(launch_dw_reduce(w.dWpart, w.nparts, s.d * s.d, a.dW, st));
  if (lin) {
    SLA_TRY(mfma_aggregate(w.dHZ, a.indT, s, w.dHZcol,
                           reinterpret_cast<float*>(reinterpret_cast<char*>(w.dHZcol) + state_z_offset(s)), st));
  }
  return mfma_backward_sparse(s, a, w.Ds, lin ? w.dHZcol : nullptr, st);
}

}  // namespace

size_t backward_ws_bytes(const Shape& s) { return carve_bwd(s, nullptr).bytes; }

hipError_t launch_dw_reduce(const float* part, int nparts, int dd, float* dW, hipStream_t st) {
  KernelTimer kt("dw_reduce", st);
  dw_reduce_kernel<<<(dd + 63) / 64, 256, 0, st>>>(part, nparts, dd, dW);
  return hipGetLastError();
}

hipError_t backward(const Shape& s, const BwdArgs& a, hipStream_t st) {
  if (s.dtype != 0) return backward_bf16(s, a, st);
  const BwdWs w = carve_bwd(s, a.ws);
  return f32_backward(s, a, w.Ds, w.dHZ, w.dHZcol, w.dWpart, w.nparts, st);
}

}  // namespace sla

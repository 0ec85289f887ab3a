// Backward pass, host side: workspace, the order of the launches, and the reduction of dW's
// partial sums that both storage types share.
#include "sla_internal.h"

namespace sla {
namespace {

// dW = sum of the partial d x d sums.  Bound by the latency of its loads (64 partials of 16 KB and
// up, 512 of them in a large call), so a workgroup owns only 32 consecutive elements (128 bytes) and
// deals the partials to 64 groups of eight lanes: up to 512 partials, every load of a thread is in
// flight at once.  The groups meet by shuffles and in LDS, in an order fixed by nparts alone.
// (512 partials with the launch gap, d = 64: 10.3 -> 4.9 us, d = 128: 12.1 -> 7.0 us.)
__global__ __launch_bounds__(512) void dw_reduce_kernel(const float* __restrict__ part, int nparts, int dd,
                                                        float* __restrict__ dW) {
  __shared__ __attribute__((aligned(16))) float red[8][32];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63, q = threadIdx.x & 7;
  const float* src = part + blockIdx.x * 32 + 4 * q;   // (dd is a multiple of 32)
  float4 s = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int p0 = threadIdx.x >> 3; p0 < nparts; p0 += 512) {
    float4 x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {   // (past the end: the last partial again, not added)
      x[k] = *reinterpret_cast<const float4*>(src + (size_t)min(p0 + 64 * k, nparts - 1) * dd);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (p0 + 64 * k >= nparts) break;
      s.x += x[k].x;
      s.y += x[k].y;
      s.z += x[k].z;
      s.w += x[k].w;
    }
  }
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) {
    s.x += __shfl_xor(s.x, o);
    s.y += __shfl_xor(s.y, o);
    s.z += __shfl_xor(s.z, o);
    s.w += __shfl_xor(s.w, o);
  }
  if (l < 8) *reinterpret_cast<float4*>(&red[w][4 * q]) = s;
  __syncthreads();
  if (threadIdx.x < 32) {
    float t = red[0][threadIdx.x];
#pragma unroll
    for (int k = 1; k < 8; ++k) t += red[k][threadIdx.x];
    dW[blockIdx.x * 32 + threadIdx.x] = t;
  }
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
  dw_reduce_kernel<<<dd / 32, 512, 0, st>>>(part, nparts, dd, dW);
  return hipGetLastError();
}

hipError_t backward(const Shape& s, const BwdArgs& a, hipStream_t st) {
  if (s.dtype != 0) return backward_bf16(s, a, st);
  const BwdWs w = carve_bwd(s, a.ws);
  return f32_backward(s, a, w.Ds, w.dHZ, w.dHZcol, w.dWpart, w.nparts, st);
}

}  // namespace sla

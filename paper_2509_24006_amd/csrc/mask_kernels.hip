// Mask step of SLA on gfx950: block mean-pooling, pooled scores, three-way classification
// (Eq. 2, Eq. 3, Alg. 1 mask line) and the row / column lookup tables of Appendix A.3.
//
// All arithmetic that decides the mask is float in one fixed order so that the integer
// result is reproducible: sequential add over a block's tokens, one IEEE division, a
// fused multiply-add chain over the features, one multiply by 1/sqrt(d).
#include <type_traits>

#include "mask_parts.h"

namespace sla {
namespace {

// ---------------------------------------------------------------- pool
template <typename T, int D>
__global__ __launch_bounds__(256) void pool_kernel(PoolArgs a) {
  pool_part<T, D>(a, blockIdx.x);
}

// ---------------------------------------------------------------- scores
// 16 R x 16 R output tile per workgroup, R x R outputs per thread, features staged through LDS in
// chunks of 64 and read four at a time; each output keeps one fused multiply-add chain in
// ascending feature order.
// acc[a][b] = sum over features (ascending, one fused multiply-add chain) of
// qb[i0 + ty + 16 a][.] kb[j0 + tx + 16 b][.]; past Tq / T the last row counts again (a select
// between a row and zeros went through scratch memory).  A chunk is on its way while the one before
// it is multiplied.  (Chunks one after the other through that select -> now, us a launch: 12 heads x 73 x 146
// scores 8.3 -> 7.0, 40 x 1182 x 1182 236 -> 203; the same in the mask kernel of short sequences, 2 x 18, 12.6 ->
// 10.7; d = 128.)
template <int R>
__device__ __forceinline__ void score_tile(const float* __restrict__ qb, const float* __restrict__ kb, int Tq, int T,
                                           int d, int i0, int j0, float (*qs)[68], float (*ks)[68],
                                           float (&acc)[R][R]) {
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
#pragma unroll
  for (int a = 0; a < R; ++a)
#pragma unroll
    for (int b = 0; b < R; ++b) acc[a][b] = 0.0f;
  // thread t brings 16 bytes: piece t % 16 of rows t / 16 + 16 q (d is a multiple of 64)
  const int c = 4 * tx;
  typedef float f4 __attribute__((ext_vector_type(4)));
  f4 qn[R], kn[R];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      qn[q] = *reinterpret_cast<const f4*>(qb + (size_t)min(i0 + ty + 16 * q, Tq - 1) * d + k0 + c);
      kn[q] = *reinterpret_cast<const f4*>(kb + (size_t)min(j0 + ty + 16 * q, T - 1) * d + k0 + c);
    }
  };
  fetch(0);
  for (int k0 = 0; k0 < d; k0 += 64) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      *reinterpret_cast<f4*>(&qs[ty + 16 * q][c]) = qn[q];
      *reinterpret_cast<f4*>(&ks[ty + 16 * q][c]) = kn[q];
    }
    __syncthreads();
    if (k0 + 64 < d) fetch(k0 + 64);
#pragma unroll 4
    for (int k = 0; k < 64; k += 4) {
      float4 av[R], bv[R];
#pragma unroll
      for (int a = 0; a < R; ++a) av[a] = *reinterpret_cast<const float4*>(&qs[ty + 16 * a][k]);
#pragma unroll
      for (int b = 0; b < R; ++b) bv[b] = *reinterpret_cast<const float4*>(&ks[tx + 16 * b][k]);
#pragma unroll
      for (int a = 0; a < R; ++a)
#pragma unroll
        for (int b = 0; b < R; ++b) {
          float x = acc[a][b];
          x = __fmaf_rn(av[a].x, bv[b].x, x);
          x = __fmaf_rn(av[a].y, bv[b].y, x);
          x = __fmaf_rn(av[a].z, bv[b].z, x);
          x = __fmaf_rn(av[a].w, bv[b].w, x);
          acc[a][b] = x;
        }
    }
    __syncthreads();
  }
}

template <int R>
__global__ __launch_bounds__(256) void score_kernel(const float* __restrict__ qbar,
                                                    const float* __restrict__ kbar, int Tq, int T, int d,
                                                    float scale, float* __restrict__ s) {
  __shared__ __attribute__((aligned(16))) float qs[16 * R][68];
  __shared__ __attribute__((aligned(16))) float ks[16 * R][68];
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  const int bh = blockIdx.z, i0 = blockIdx.y * 16 * R, j0 = blockIdx.x * 16 * R;
  float acc[R][R];
  score_tile<R>(qbar + (size_t)bh * Tq * d, kbar + (size_t)bh * T * d, Tq, T, d, i0, j0, qs, ks, acc);
#pragma unroll
  for (int a = 0; a < R; ++a) {
    const int i = i0 + ty + 16 * a;
    if (i >= Tq) continue;
#pragma unroll
    for (int b = 0; b < R; ++b) {
      const int j = j0 + tx + 16 * b;
      if (j < T) s[((size_t)bh * Tq + i) * T + j] = __fmul_rn(acc[a][b], scale);
    }
  }
}

// ---------------------------------------------------------------- classify
// Order-preserving map float -> uint32 (larger float <=> larger key); +0 and -0 coincide.
__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t b = __float_as_uint(f);
  if (b == 0x80000000u) b = 0u;
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Marks with `label` the k entries that come first under (key descending, index ascending) among
// the entries with a non-zero key.  The threshold, the largest t with #{key >= t} >= k, is found bit
// by bit, with the row in registers (entry j = 64 i + lane in slot i, key 0 past the end): every
// count is a handful of wave votes tallied on the scalar side, no LDS and no cross-lane shuffles.
// Bound by the issue of these tallies (two scalar instructions per slot and bit), so the search
// ends as soon as exactly k keys reach the candidate: the lower bits of the threshold cannot
// change which keys those are, and the labels are one comparison a slot.  (40 heads x 1182 rows of
// 1182, with 19 slots a lane instead of 32: 515 -> 237 us a launch, with the labels by one
// comparison 221 -> 207; 12 x 512 of 512: 25 -> 20 -> 18.6 us.  Rows of more than 2048 entries in
// LDS, with shuffles: 2 x 2500 360 -> 100 us, 8 x 3000 2550 -> 449.)
template <int KPL>
__device__ __forceinline__ void mark_top_reg(const uint32_t (&key)[KPL], int8_t (&lab)[KPL], int k, int8_t label,
                                             int lane) {
  if (k <= 0) return;
  uint32_t thr = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = thr | (1u << bit);
    int c = 0;
#pragma unroll
    for (int i = 0; i < KPL; ++i) c += __popcll(__ballot(key[i] >= cand));
    if (c >= k) thr = cand;
    if (c == k) {   // no entries equal to the threshold to choose among
#pragma unroll
      for (int i = 0; i < KPL; ++i) lab[i] = key[i] >= cand ? label : lab[i];
      return;
    }
  }
  int need = k;
#pragma unroll
  for (int i = 0; i < KPL; ++i) need -= __popcll(__ballot(key[i] > thr));
  asm volatile("" : "+s"(thr));   // compared anew: the votes above would be kept, two scalar registers a slot
#pragma unroll
  for (int i = 0; i < KPL; ++i) {   // ascending index: slot by slot, lane by lane
    const bool eq = key[i] == thr;
    const unsigned long long m = __ballot(eq);
    const int before = __popcll(m & ((1ull << lane) - 1ull));
    if (key[i] > thr || (eq && before < need)) lab[i] = label;
    need -= __popcll(m);
  }
}

// One wavefront per row of the score matrix, rows of at most 64 KPL entries.
template <int KPL>
__global__ __launch_bounds__(256) void classify_reg_kernel(const float* __restrict__ s, int rows, int Tq, int rq,
                                                           int T, int n_h, int n_l, int8_t* __restrict__ Mc,
                                                           int32_t* __restrict__ row_idx,
                                                           int32_t* __restrict__ col_cnt) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + wave;
  if (row >= rows) return;   // (no barriers in this kernel)
  // the query tiles of this row of the mask: each gets a copy of the row's table entries
  const size_t t0 = (size_t)(row / Tq) * T + (size_t)(row % Tq) * rq;
  const int nrep = min(rq, T - (int)(row % Tq) * rq);
  if (lane < nrep) col_cnt[t0 + lane] = 0;   // one counter per (head, key block), cleared for the column count that follows
  const float* sr = s + (size_t)row * T;
  uint32_t key[KPL];
  int8_t lab[KPL];
#pragma unroll
  for (int i = 0; i < KPL; ++i) {
    const int j = 64 * i + lane;
    key[i] = j < T ? order_key(sr[j]) : 0u;
    lab[i] = 0;
  }
  mark_top_reg<KPL>(key, lab, n_h, (int8_t)1, lane);
  // negligible: lowest scores among the rest = largest inverted keys; critical entries and the
  // slots past the end get key 0 and drop out
#pragma unroll
  for (int i = 0; i < KPL; ++i) key[i] = (lab[i] == 1 || 64 * i + lane >= T) ? 0u : ~key[i];
  mark_top_reg<KPL>(key, lab, n_l, (int8_t)-1, lane);
  int base = 0;
#pragma unroll
  for (int i = 0; i < KPL; ++i) {
    const int j = 64 * i + lane;
    if (j < T) Mc[(size_t)row * T + j] = lab[i];
    const unsigned long long m = __ballot(lab[i] == 1);
    if (lab[i] == 1) {
      const int pos = base + __popcll(m & ((1ull << lane) - 1ull));
      for (int r = 0; r < nrep; ++r) row_idx[(t0 + r) * n_h + pos] = j;
    }
    base += __popcll(m);
  }
}

// ---------------------------------------------------------------- column tables (CSC)

// Marginal indicator as bit masks and the column counts, over query tiles i (of 64 tokens: label
// m(i, j) = Mc[i / rq][j]).  Bit b of ind[i][q] is set iff m(i, 64 q + b) == 0 (and the column
// exists), bit b of indT[j][q] iff m(64 q + b, j) == 0;
// cnt[j] (cleared by the classification kernel) receives the number of critical blocks of column
// j.  A workgroup takes a 64 x 64 tile of Mc, sixteen rows per wave.  (40 heads x 1182 blocks: 102 ->
// 47 us a launch, 12 x 146: 10.2 -> 4.7 us.)
__global__ __launch_bounds__(256) void indicator_kernel(const int8_t* __restrict__ Mc, int Tq, int rq, int T, int Tw,
                                                        unsigned long long* __restrict__ ind,
                                                        unsigned long long* __restrict__ indT,
                                                        int32_t* __restrict__ cnt) {
  __shared__ __attribute__((aligned(8))) unsigned short marg[64][4], crit[64][4];   // [column][wave]
  const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bh = blockIdx.z, i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
  const ColumnVotes<16> v = column_votes<16, true>(Mc + (size_t)bh * Tq * T, T, rq, i0 + 16 * w, j0, l);
  if (l < 16 && i0 + 16 * w + l < T) ind[((size_t)bh * T + i0 + 16 * w + l) * Tw + blockIdx.x] = v.row;
  marg[l][w] = (unsigned short)v.marg[0];
  crit[l][w] = (unsigned short)v.crit[0];
  __syncthreads();
  if (w == 0 && j0 + l < T) {
    indT[((size_t)bh * T + j0 + l) * Tw + blockIdx.y] = *reinterpret_cast<const unsigned long long*>(marg[l]);
    const int ncrit = __popcll(*reinterpret_cast<const unsigned long long*>(crit[l]));
    if (ncrit) atomicAdd(cnt + (size_t)bh * T + j0 + l, ncrit);
  }
}

template <int NW>
__global__ __launch_bounds__(64 * NW) void col_tables_kernel(ColArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  col_tables_part<NW>(smem, a, blockIdx.x, blockIdx.y);
}

// ---------------------------------------------------------------- short sequences
// At most 64 key blocks: scores, classification and all tables of a head in one workgroup.  At
// that size each of the four kernels above is a few microseconds of work behind as many
// microseconds of launch.  Same arithmetic, same tables.  With `given` the scores are read
// instead of computed (classification of given scores).
// Bound by latency: one workgroup per head, a chain of short phases, so the workgroup is as wide as
// it can be (a row of M_c per wave at 16 blocks) and forms only the scores of a T x T corner: TT x TT
// per thread, 32 TT >= T.  (256 heads of 16 blocks, d = 64:
// 14.5 -> 8.5 us a launch with the gap before it; 2 of 18, d = 128: 19 -> 10.3 us.)
constexpr int kSmallWaves = 16;
struct NoPool {};
// PT: the tensors' type where the head's blocks are pooled here too (D features), or NoPool.
template <int TT, typename PT, int D>
__global__ __launch_bounds__(64 * kSmallWaves) void mask_small_kernel(
    PoolArgs pool, const float* qbar, const float* kbar, const float* __restrict__ given, int Tq, int rq,
    int T, int d, float scale, int n_h, int n_l, float* __restrict__ s_out, int8_t* __restrict__ Mc,
    int32_t* __restrict__ row_idx, unsigned long long* __restrict__ ind, unsigned long long* __restrict__ indT,
    int32_t* __restrict__ col_ptr, int32_t* __restrict__ col_order, int32_t* __restrict__ col_rows) {
  __shared__ __attribute__((aligned(16))) float qs[64][68];
  __shared__ __attribute__((aligned(16))) float ks[64][68];
  __shared__ float sc[64][65];
  __shared__ int8_t lab[64][68];   // labels of the rows of M_c; 2 past the end of a row
  __shared__ int cnt[64], cptr[64];
  const int bh = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned long long below = (1ull << lane) - 1ull;
  if constexpr (!std::is_same_v<PT, NoPool>) {
    pool_head<PT, D>(pool, bh, kSmallWaves);
    __syncthreads();
  }
  if (given) {
    const float* g = given + (size_t)bh * Tq * T;
    for (int e = tid; e < Tq * T; e += 64 * kSmallWaves) sc[e / T][e % T] = g[e];
  } else {
    // thread (ty, tx): rows ty + 32 a, columns tx + 32 b; one fused multiply-add chain per score in
    // ascending feature order, as in score_tile
    const float* qb = qbar + (size_t)bh * Tq * d;
    const float* kb = kbar + (size_t)bh * T * d;
    const int ty = tid >> 5, tx = tid & 31, lr = tid >> 4, lc = 4 * (tid & 15);
    float acc[TT][TT];
#pragma unroll
    for (int a = 0; a < TT; ++a)
#pragma unroll
      for (int b = 0; b < TT; ++b) acc[a][b] = 0.0f;
    const float* qr = qb + (size_t)min(lr, Tq - 1) * d + lc;
    const float* kr = kb + (size_t)min(lr, T - 1) * d + lc;
    float4 qn = *reinterpret_cast<const float4*>(qr), kn = *reinterpret_cast<const float4*>(kr);
    for (int k0 = 0; k0 < d; k0 += 64) {
      *reinterpret_cast<float4*>(&qs[lr][lc]) = qn;
      *reinterpret_cast<float4*>(&ks[lr][lc]) = kn;
      __syncthreads();
      if (k0 + 64 < d) {
        qn = *reinterpret_cast<const float4*>(qr + k0 + 64);
        kn = *reinterpret_cast<const float4*>(kr + k0 + 64);
      }
#pragma unroll 4
      for (int k = 0; k < 64; k += 4) {
        float4 av[TT], bv[TT];
#pragma unroll
        for (int a = 0; a < TT; ++a) {
          av[a] = *reinterpret_cast<const float4*>(&qs[ty + 32 * a][k]);
          bv[a] = *reinterpret_cast<const float4*>(&ks[tx + 32 * a][k]);
        }
#pragma unroll
        for (int a = 0; a < TT; ++a)
#pragma unroll
          for (int b = 0; b < TT; ++b) {
            float x = acc[a][b];
            x = __fmaf_rn(av[a].x, bv[b].x, x);
            x = __fmaf_rn(av[a].y, bv[b].y, x);
            x = __fmaf_rn(av[a].z, bv[b].z, x);
            x = __fmaf_rn(av[a].w, bv[b].w, x);
            acc[a][b] = x;
          }
      }
      __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < TT; ++a)
#pragma unroll
      for (int b = 0; b < TT; ++b) {
        const int i = ty + 32 * a, j = tx + 32 * b;
        if (i < Tq && j < T) {
          const float v = __fmul_rn(acc[a][b], scale);
          sc[i][j] = v;
          s_out[((size_t)bh * Tq + i) * T + j] = v;
        }
      }
  }
  __syncthreads();
  // classification: a wave per row of M_c, the row in one register per lane
  for (int i = wave; i < Tq; i += kSmallWaves) {
    uint32_t key[1];
    int8_t lb[1];
    key[0] = lane < T ? order_key(sc[i][lane]) : 0u;
    lb[0] = 0;
    mark_top_reg<1>(key, lb, n_h, (int8_t)1, lane);
    key[0] = (lb[0] == 1 || lane >= T) ? 0u : ~key[0];
    mark_top_reg<1>(key, lb, n_l, (int8_t)-1, lane);
    if (lane < T) Mc[((size_t)bh * Tq + i) * T + lane] = lb[0];
    lab[i][lane] = lane < T ? lb[0] : (int8_t)2;
    const unsigned long long m = __ballot(lb[0] == 1);
    if (lb[0] == 1) {
      const int pos = __popcll(m & below);
      const int nrep = min(rq, T - i * rq);   // the query tiles of this row
      for (int r = 0; r < nrep; ++r) row_idx[((size_t)bh * T + i * rq + r) * n_h + pos] = lane;
    }
  }
  __syncthreads();
  // bit masks and column counts over query tiles: tile r has the labels of row r / rq
  for (int r = wave; r < 64; r += kSmallWaves) {
    const int8_t rv = (r < T) ? lab[r / rq][lane] : (int8_t)2;                 // row r, column = lane
    const int8_t cv = (r < T && lane < T) ? lab[lane / rq][r] : (int8_t)2;     // column r, query tile = lane
    const unsigned long long rowbits = __ballot(rv == 0), colbits = __ballot(cv == 0);
    const int ncrit = __popcll(__ballot(cv == 1));
    if (lane == 0) {
      cnt[r] = ncrit;
      if (r < T) {
        ind[(size_t)bh * T + r] = rowbits;
        indT[(size_t)bh * T + r] = colbits;
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    const int c = cnt[lane];
    int incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o);
      if (lane >= o) incl += v;
    }
    cptr[lane] = incl - c;
    if (lane < T) {
      col_ptr[(size_t)bh * (T + 1) + lane] = incl - c;
      if (lane == T - 1) col_ptr[(size_t)bh * (T + 1) + T] = incl;
      int rank = 0;
      for (int k = 0; k < T; ++k) rank += (cnt[k] > c) || (cnt[k] == c && k < lane);
      col_order[(size_t)bh * T + rank] = lane;
    }
  }
  __syncthreads();
  if (n_h == 0) return;
  for (int j = wave; j < T; j += kSmallWaves) {   // the critical query tiles of column j, ascending
    const bool crit = lane < T && lab[lane / rq][j] == 1;
    const unsigned long long m = __ballot(crit);
    if (crit) col_rows[(size_t)bh * T * n_h + cptr[j] + __popcll(m & below)] = lane;
  }
}

}  // namespace

PoolArgs pool_args(const void* Q, const void* K, const Shape& s, float* qbar, float* kbar) {
  const int bpw = s.dtype == 0 ? 256 / s.d : 512 / s.d;   // blocks per wavefront
  return PoolArgs{Q, K, s.BH, s.N, s.Tq, s.rq * kBlk, s.T, kBlk, (s.BH * s.T + 4 * bpw - 1) / (4 * bpw), s.lay(), qbar, kbar};
}

hipError_t launch_pool(const PoolArgs& a, const Shape& s, hipStream_t st) {
  KernelTimer kt("pool", st);
  auto kern = s.dtype == 0 ? (s.d == 64 ? pool_kernel<float, 64> : pool_kernel<float, 128>)
                           : (s.d == 64 ? pool_kernel<__hip_bfloat16, 64> : pool_kernel<__hip_bfloat16, 128>);
  kern<<<2 * a.wgs, 256, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_scores(const float* qbar, const float* kbar, const Shape& s, float* scores,
                         hipStream_t st) {
  // Tiles of 64 x 64 scores read half as much from LDS per product as those of 32 x 32, but up to two of them
  // per CU leave most of the chip idle.  (Tiles of 64 -> 32, us, before chunks were fetched ahead: 12 heads x 73 x 146 scores, 72 tiles of 64,
  // 13.6 -> 8.4; 4 x 122 x 122, 16 tiles, 13.3 -> 8.3; 24 x 250 x 250, d = 64, 384 tiles, 11.1 -> 10.6;
  // 12 x 512 x 512, 768 tiles, 20.2 -> 22.9; 40 x 1182 x 1182 235 -> 297.)
  const bool wide = (s.T + 63) / 64 * ((s.Tq + 63) / 64) * s.BH > 512;
  const int t = wide ? 64 : 32;
  auto kern = wide ? score_kernel<4> : score_kernel<2>;
  KernelTimer kt("score", st);
  kern<<<dim3((s.T + t - 1) / t, (s.Tq + t - 1) / t, s.BH), 256, 0, st>>>(qbar, kbar, s.Tq, s.T, s.d, s.scale, scores);
  return hipGetLastError();
}

hipError_t launch_classify(const float* scores, const Shape& s, int8_t* Mc, int32_t* row_idx,
                           int32_t* col_cnt, hipStream_t st) {
  const int rows = s.BH * s.Tq;
  {
    KernelTimer kt("classify", st);
    const dim3 grid((rows + 3) / 4);
    // slots per lane as the row needs them (the kernel's time goes with the slots): the fewest
    // instances with which no row pays for more than a fifth more slots than it needs
    const int slots = (s.T + 63) / 64;
    auto kern = slots <= 2 ? classify_reg_kernel<2>
              : slots <= 3 ? classify_reg_kernel<3> : slots <= 4 ? classify_reg_kernel<4>
              : slots <= 6 ? classify_reg_kernel<6> : slots <= 8 ? classify_reg_kernel<8>
              : slots <= 10 ? classify_reg_kernel<10> : slots <= 13 ? classify_reg_kernel<13>
              : slots <= 16 ? classify_reg_kernel<16> : slots <= 19 ? classify_reg_kernel<19>
              : slots <= 22 ? classify_reg_kernel<22> : slots <= 27 ? classify_reg_kernel<27>
              : slots <= 32 ? classify_reg_kernel<32> : slots <= 39 ? classify_reg_kernel<39>
              : classify_reg_kernel<48>;
    static_assert(kMaxT <= 48 * 64);
    kern<<<grid, 256, 0, st>>>(scores, rows, s.Tq, s.rq, s.T, s.n_h, s.n_l, Mc, row_idx, col_cnt);
  }
  return hipGetLastError();
}

hipError_t launch_indicator(const int8_t* Mc, const Shape& s, int32_t* col_cnt, unsigned long long* ind,
                            unsigned long long* indT, hipStream_t st) {
  const int Tw = (s.T + 63) / 64;
  KernelTimer kt("indicator", st);
  indicator_kernel<<<dim3(Tw, Tw, s.BH), 256, 0, st>>>(Mc, s.Tq, s.rq, s.T, Tw, ind, indT, col_cnt);
  return hipGetLastError();
}

hipError_t launch_col_tables(const ColArgs& a, const Shape& s, hipStream_t st) {
  const int Tw = (s.T + 63) / 64;
  KernelTimer kt("col_tables", st);
  // The waves of a workgroup share its row tiles, of which they walk one after the other, so more than four row
  // tiles take eight waves; sixteen pay where there are many and the workgroups leave the chip idle.  (4, 8, 16
  // waves, us: 24 heads x 250 blocks 10.1, 9.7, 9.8; 12 x 512 15.6, 11.4, 11.2, 20 % critical 20.3, 14.0, 13.8; 40 x
  // 512 20.2, 19.0, 22.2; 40 x 1182 48.7, 45.2, 52.4; 2 x 2500 56.6, 36.2, 28.3; 512 x 130 17.5, 22.1, 39.0.)
  const int nw = Tw <= 4 ? 4 : Tw > 16 && Tw * s.BH <= 256 ? 16 : 8;
  auto kern = nw == 4 ? col_tables_kernel<4> : nw == 8 ? col_tables_kernel<8> : col_tables_kernel<16>;
  kern<<<dim3(Tw, s.BH), 64 * nw, col_tables_lds(Tw, nw), st>>>(a);
  return hipGetLastError();
}

hipError_t launch_mask_small(const PoolArgs* pool, const float* qbar, const float* kbar, const float* given,
                             const Shape& s, float* scores, int8_t* Mc, int32_t* row_idx, unsigned long long* ind,
                             unsigned long long* indT, int32_t* col_ptr, int32_t* col_order, int32_t* col_rows,
                             hipStream_t st) {
  KernelTimer kt("mask_small", st);
  typedef __hip_bfloat16 bf;
  auto pick = [&](auto t1, auto t2) { return s.T <= 32 ? t1 : t2; };
  auto kern = !pool ? pick(mask_small_kernel<1, NoPool, 64>, mask_small_kernel<2, NoPool, 64>)
            : s.dtype == 0 ? (s.d == 64 ? pick(mask_small_kernel<1, float, 64>, mask_small_kernel<2, float, 64>)
                                        : pick(mask_small_kernel<1, float, 128>, mask_small_kernel<2, float, 128>))
                           : (s.d == 64 ? pick(mask_small_kernel<1, bf, 64>, mask_small_kernel<2, bf, 64>)
                                        : pick(mask_small_kernel<1, bf, 128>, mask_small_kernel<2, bf, 128>));
  kern<<<s.BH, 64 * kSmallWaves, 0, st>>>(pool ? *pool : PoolArgs{}, qbar, kbar, given, s.Tq, s.rq, s.T, s.d, s.scale,
                                          s.n_h, s.n_l, scores, Mc, row_idx, ind, indT, col_ptr, col_order, col_rows);
  return hipGetLastError();
}

}  // namespace sla

// Pooling and the column tables as device functions: kernels of their own (mask_kernels.hip), and the first
// workgroups of the key-block state kernels in a call that builds the mask and runs the forward pass.
#ifndef SLA_MASK_PARTS_H_
#define SLA_MASK_PARTS_H_

#include "sla_internal.h"

namespace sla {

// ---------------------------------------------------------------- pool
// A lane owns the 16 bytes of a token row that hold V adjacent features and walks the rows of
// its block in order (the sum over a block's tokens is sequential, so that the mask is reproducible); D / V lanes cover
// a block, so a wavefront pools 64 V / D blocks at once and each of its loads fetches whole
// rows.  The first half of the 2 a.wgs workgroups takes Q (blocks of len0 tokens, Tn0 per head), the
// other K (len1, Tn1).
template <typename T, int D>
struct PoolWave {
  static constexpr int V = 16 / sizeof(T), LPB = D / V, BPW = 64 / LPB;   // lanes per block, blocks per wave
};
// block i of head bh (or none, lane by lane) by the LPB lanes that share it
template <typename T, int D>
__device__ __forceinline__ void pool_block(const PoolArgs& a, bool second, int bh, int i) {
  constexpr int V = PoolWave<T, D>::V, LPB = PoolWave<T, D>::LPB;
  const T* X = reinterpret_cast<const T*>(second ? a.X1 : a.X0);
  float* out = second ? a.out1 : a.out0;
  const int Tn = second ? a.Tn1 : a.Tn0, len = second ? a.len1 : a.len0;
  const Lay lay = a.lay;
  const int fl = (threadIdx.x & 63) % LPB;
  const int cnt = min(len, a.N - i * len);
  const T* p = X + lay.head(bh) + (size_t)i * len * lay.ts + fl * V;
  float s[V];
#pragma unroll
  for (int v = 0; v < V; ++v) s[v] = 0.0f;
  // 16 rows are requested before the first is added (the sum itself stays in token order)
  int r = 0;
  for (; r + 16 <= cnt; r += 16) {
    uint4 raw[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) raw[k] = *reinterpret_cast<const uint4*>(p + (size_t)(r + k) * lay.ts);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const T* e = reinterpret_cast<const T*>(&raw[k]);
#pragma unroll
      for (int v = 0; v < V; ++v) s[v] = s[v] + to_f32(e[v]);
    }
  }
  for (; r < cnt; ++r) {
    const uint4 raw = *reinterpret_cast<const uint4*>(p + (size_t)r * lay.ts);
    const T* e = reinterpret_cast<const T*>(&raw);
#pragma unroll
    for (int v = 0; v < V; ++v) s[v] = s[v] + to_f32(e[v]);
  }
  const float c = (float)cnt;
  float* o = out + ((size_t)bh * Tn + i) * D + fl * V;
#pragma unroll
  for (int v = 0; v < V; v += 4)
    *reinterpret_cast<float4*>(o + v) = float4{__fdiv_rn(s[v], c), __fdiv_rn(s[v + 1], c), __fdiv_rn(s[v + 2], c),
                                               __fdiv_rn(s[v + 3], c)};
}

template <typename T, int D>
__device__ __forceinline__ void pool_part(const PoolArgs& a, int wg) {
  using P = PoolWave<T, D>;
  const bool second = wg >= a.wgs;
  const int Tn = second ? a.Tn1 : a.Tn0;
  const long blk = ((long)(second ? wg - a.wgs : wg) * 4 + (threadIdx.x >> 6)) * P::BPW + (threadIdx.x & 63) / P::LPB;
  if (blk < (long)a.BH * Tn) pool_block<T, D>(a, second, (int)(blk / Tn), (int)(blk % Tn));
}

// both tensors of one head by the `waves` waves of a workgroup
template <typename T, int D>
__device__ __forceinline__ void pool_head(const PoolArgs& a, int bh, int waves) {
  using P = PoolWave<T, D>;
  const int u0 = (a.Tn0 + P::BPW - 1) / P::BPW, u1 = (a.Tn1 + P::BPW - 1) / P::BPW;
  for (int u = threadIdx.x >> 6; u < u0 + u1; u += waves) {
    const bool second = u >= u0;
    const int i = (second ? u - u0 : u) * P::BPW + (threadIdx.x & 63) / P::LPB;
    if (i < (second ? a.Tn1 : a.Tn0)) pool_block<T, D>(a, second, bh, i);
  }
}

// ---------------------------------------------------------------- column tables (CSC)

// Labels of query tiles i0 .. i0 + R - 1 (tile i has the labels of row i / rq of the head's M_c) in
// column j = j0 + lane, as bit masks over the tiles: the wave walks the rows, one byte per lane and
// row, all R rows in flight, and every lane collects the bits of its own column, so that nothing
// crosses lanes and nothing goes through LDS.  With ROWS, lane r also receives the marginal bits of
// row i0 + r.  Columns past T have no bits.
template <int R>
struct ColumnVotes {
  unsigned crit[(R + 31) / 32], marg[(R + 31) / 32];
  unsigned long long row;
};
template <int R, bool ROWS>
__device__ __forceinline__ ColumnVotes<R> column_votes(const int8_t* __restrict__ src, int T, int rq, int i0, int j0,
                                                       int lane) {
  ColumnVotes<R> v = {};
  const bool jok = j0 + lane < T;
  const int8_t* col = src + min(j0 + lane, T - 1);
  int q = i0 / rq, rem = i0 - q * rq;   // row of M_c of the next tile, its place in that row's group
  const int qlast = (T - 1) / rq;
  int8_t x[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    x[r] = col[(size_t)min(q, qlast) * T];   // (past the last tile: the last row again, no bits)
    if (++rem == rq) {
      rem = 0;
      ++q;
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool ok = jok && i0 + r < T;
    const bool m = ok && x[r] == 0;
    v.crit[r >> 5] |= (ok && x[r] == 1) ? 1u << (r & 31) : 0u;
    v.marg[r >> 5] |= m ? 1u << (r & 31) : 0u;
    if (ROWS) {
      const unsigned long long b = __ballot(m);
      if (lane == r) v.row = b;
    }
  }
  return v;
}

// From the column counts of a head: col_ptr (exclusive prefix sums, T + 1 entries), col_order
// (col_order[rank] = j, rank = position of column j under count descending, index ascending: the
// column-wise backward kernel takes the longest lists first) and col_rows (the critical rows of
// every column, ascending).  A workgroup owns 64 columns of one head; every workgroup forms the
// prefix sum up to its columns from the head's counts by itself.  Bound by latency (a few hundred
// workgroups, each a chain of short phases): the waves vote different row tiles with no barrier in
// between, counts and column indices are compared as one number, four per LDS read, and the rows of
// a tile are written the cheaper of two ways: short lists by a lane per column (a store touches 64
// lists, so the longest one counts), long ones by the whole wave, column by column (a store is one
// piece of a list, and every column costs the same).  (5 % critical, 40 heads x 1182 blocks: 152 -> 58
// us a launch; 12 x 146, whose rows are not 16-byte aligned: 20 -> 9.6 us.  A lane per column alone,
// both: 40 x 512 with 10 % critical in few columns 35 -> 22.9, with 20 % 51 -> 23.9, with all 92 ->
// 24.8 us; 4096 x 65, all 160 -> 59.)
constexpr int kLongList = 12;   // rows of a column's list in a tile from which the wave writes it
constexpr int kManyLong = 24;   // such columns in a tile from which it writes all 64 without a choice
constexpr int kKeyBits = 12;   // column index in a sort key: kMaxT of the interface is below 2^12
__host__ __device__ constexpr int col_tables_lds(int Tw, int waves) {
  return 64 * Tw * 4 + 64 * Tw * 8 + (waves * 64 + 64 + waves) * 4;
}

// columns [64 jt, +64) of head bh by NW waves; smem: col_tables_lds bytes
template <int NW>
__device__ __forceinline__ void col_tables_part(unsigned char* smem, const ColArgs& a, int jt, int bh) {
  const int8_t* __restrict__ Mc = a.Mc;
  const int32_t* __restrict__ cnt_g = a.cnt;
  int32_t *__restrict__ ptr = a.ptr, *__restrict__ order = a.order, *__restrict__ rows = a.rows;
  const int Tq = a.Tq, rq = a.rq, T = a.T, n_h = a.n_h;
  const int Tw = (T + 63) / 64;
  uint32_t* key = reinterpret_cast<uint32_t*>(smem);   // (count, column descending) of the head; 0 past T
  unsigned long long* crit = reinterpret_cast<unsigned long long*>(smem + 64 * Tw * 4);   // [row tile][column]
  int (*part)[64] = reinterpret_cast<int (*)[64]>(smem + 64 * Tw * 12);   // [wave][column]
  int *cptr = part[NW], *wsum = part[NW + 1];
  const int j0 = jt * 64;
  const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t* cg = cnt_g + (size_t)bh * T;
  int before = 0;   // this thread's share of the counts of the columns before j0
  for (int j = tid; j < 64 * Tw; j += 64 * NW) {
    const int c = j < T ? cg[j] : 0;
    key[j] = j < T ? (uint32_t)c << kKeyBits | (uint32_t)((1 << kKeyBits) - 1 - j) : 0u;
    if (j < j0) before += c;
  }
  if (n_h > 0)
    for (int t = w; t < Tw; t += NW) {
      const ColumnVotes<64> v = column_votes<64, false>(Mc + (size_t)bh * Tq * T, T, rq, 64 * t, j0, l);
      crit[64 * t + l] = (unsigned long long)v.crit[1] << 32 | v.crit[0];
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  if (l == 0) wsum[w] = before;
  __syncthreads();
  // pointers of this workgroup's columns: wave 0 scans its 64 counts
  const uint32_t mine = key[j0 + l];
  if (w == 0) {
    const int j = j0 + l;
    const int c = (int)(mine >> kKeyBits);
    int incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(incl, o);
      if (l >= o) incl += v;
    }
    int p = incl - c;
#pragma unroll
    for (int x = 0; x < NW; ++x) p += wsum[x];
    cptr[l] = p;
    if (j < T) ptr[(size_t)bh * (T + 1) + j] = p;
    if (j == T - 1) ptr[(size_t)bh * (T + 1) + T] = p + c;
  }
  // rank of this workgroup's columns; the waves share the comparisons of a column
  {
    int rank = 0;
    const uint4* k4 = reinterpret_cast<const uint4*>(key) + 16 / NW * Tw * w;
#pragma unroll 4
    for (int k = 0; k < 16 / NW * Tw; ++k) {
      const uint4 x = k4[k];
      rank += (x.x > mine) + (x.y > mine) + (x.z > mine) + (x.w > mine);
    }
    part[w][l] = rank;
  }
  __syncthreads();
  if (w == 0 && j0 + l < T) {
    int rank = 0;
#pragma unroll
    for (int x = 0; x < NW; ++x) rank += part[x][l];
    order[(size_t)bh * T + rank] = j0 + l;
  }
  if (n_h == 0) return;
  // rows of the critical blocks: wave w writes those of the row tiles it voted
  int32_t* out = rows + (size_t)bh * T * n_h;
  int pos = cptr[l];   // where the rows of the next row tile go
  for (int t = 0; t < Tw; ++t) {
    const unsigned long long m = crit[64 * t + l];
    if (t % NW == w) {
      const unsigned mlo = (unsigned)m, mhi = (unsigned)(m >> 32);
      auto column = [&](int c) {   // the wave writes column c's rows
        const unsigned lo = __builtin_amdgcn_readlane(mlo, c), hi = __builtin_amdgcn_readlane(mhi, c);
        const unsigned p = __builtin_amdgcn_readlane(pos, c) + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
        if (__builtin_amdgcn_inverse_ballot_w64((unsigned long long)hi << 32 | lo)) out[p] = 64 * t + l;
      };
      unsigned long long longs = __ballot(__popcll(m) > kLongList);
      if (__popcll(longs) >= kManyLong) {
#pragma unroll 8
        for (int c = 0; c < 64; ++c) column(c);
      } else {
        if (__popcll(m) <= kLongList) {
          unsigned p = pos;
#pragma unroll
          for (int h = 0; h < 2; ++h)
            for (unsigned x = h ? mhi : mlo; x; x &= x - 1) out[p++] = 64 * t + 32 * h + __ffs(x) - 1;
        }
        for (; longs; longs &= longs - 1) column(__ffsll(longs) - 1);
      }
    }
    pos += __popcll(m);
  }
}

}  // namespace sla
#endif

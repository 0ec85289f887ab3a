// Float SLA path for gfx950: every contraction of Algorithm 1 and Algorithm 2 on
// v_mfma_f32_16x16x4_f32 (float products, float accumulation: the same arithmetic as fused
// multiply-adds, at twice the rate of the vector unit and with a sixteenth of its LDS reads).
//
// One instruction multiplies A (16 x 4) by B (4 x 16) into C (16 x 16).  Lane l = 16 g + n:
//   A: row n, k = g        B: column n, k = g        C: column n, rows 4 g + i in registers i
// Any assignment of k-indices to (instruction, g) is right as long as A and B use the same one.
// All kernels take k = 16 t + 4 g + s for instruction s of group t, which gives two things: an
// operand whose k-index runs along a row is read 16 bytes at a time, and a C tile (rows 16 t + 4 g
// + i) is the B operand of the next product as it stands, with no exchange between lanes.  A lane
// therefore owns one token (column n) and the features {16 t + 4 g + s} of it, in every product.
//
// 64 x D tiles lie in LDS row by row, unpadded, filled by direct global -> LDS loads; the 16-byte
// chunk c of row r sits at chunk position c ^ (r % 16).  Both reads are then free of bank
// conflicts: 16 rows at one chunk (operand read by rows) hit 16 different positions, and 4 rows of
// 16 adjacent floats (operand contracted over tile rows) hit four different 64-byte pieces.
#include "mask_parts.h"
#include "mfma_common.h"

namespace sla {
namespace {

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 zero4() { return f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }

template <int D>
struct FTile {
  static constexpr int CPR = D / 4;              // 16-byte chunks per row
  static constexpr int ROWB = 4 * D;
  static constexpr int BYTES = kBlk * ROWB;
  static constexpr int RPI = 1024 / ROWB;        // rows per wave-wide load
  static constexpr int IPW = kBlk / RPI / 4;     // loads per wave and tile (four waves fill a tile)
};

// Direct loads of 64-row tiles whose rows lie tsB bytes apart, behind a descriptor that spans the
// whole head (rows past its end read as zeros: the part of an offset that may pass the end rides on
// the per-lane offset, which the range check covers; the tile's own offset is always inside).
// N tsB is below 2^31, so offsets of rows past the end of a sequence of 62 rows and more stay below
// 2^32.  Shorter ones (a single tile) with rows 64 MB and more apart would come back into range:
// their rows past the end get an offset that is out of range in any case.
template <int D>
struct FLoader {
  using T = FTile<D>;
  static constexpr int kFar = 1 << 26;   // 64 rows of this pitch: 2^32 bytes
  int voff[2];    // this lane's byte offset for even and odd loads (the swizzle has period 16 rows)
  int kend;       // this lane's loads from kend on are of rows past the end (only where rows are far apart)
  int kstep, tile_step;
  unsigned lds0;
  // N: rows of the head (a packed matrix needs none: its rows are near)
  __device__ __forceinline__ void init(unsigned lds_base_addr, int w, int l, int tsB, int N = 0) {
    const int r0 = T::RPI * w + l / T::CPR;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int row = r0 + 4 * T::RPI * k;
      voff[k] = r0 * tsB + (((l % T::CPR) ^ (row & 15)) << 4);
    }
    kend = tsB < kFar ? T::IPW : (N - r0 + 4 * T::RPI - 1) / (4 * T::RPI);
    kstep = 4 * T::RPI * tsB;
    tile_step = kBlk * tsB;
    lds0 = lds_base_addr + wave_uniform(w) * 1024;
  }
  // tile number `tile` of the buffer -> LDS offset `slot`
  __device__ __forceinline__ void load(BufDesc desc, int tile, int slot) const {
#pragma unroll
    for (int k = 0; k < T::IPW; ++k)
      load_to_lds16(desc, k < kend ? voff[k & 1] + k * kstep : 0x7ffffff0, tile * tile_step, lds0 + slot + 4096 * k);
  }
};

template <int D>
__device__ __forceinline__ BufDesc head_rsrc_f32(const float* head_base, int N, int tsB) {
  return tile_rsrc(head_base, (N - 1) * tsB + 4 * D);
}
// a packed matrix of `rows` rows of D floats
template <int D>
__device__ __forceinline__ BufDesc matrix_rsrc_f32(const float* M, int rows) {
  return tile_rsrc(M, rows * 4 * D);
}

// Per-lane addresses of the two operand reads.
template <int D>
struct FAddr {
  int rb, rx;      // by rows: base, swizzle of the chunk index
  int tb[4], tx;   // over rows: base for row 4 g + i, swizzle of the 16-float piece
  __device__ __forceinline__ void init(int l) {
    const int g = l >> 4, n = l & 15;
    rb = n * FTile<D>::ROWB + (((g ^ n) & 3) << 4);
    rx = (n >> 2) << 6;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      tb[i] = (4 * g + i) * FTile<D>::ROWB + ((((n >> 2) ^ i) & 3) << 4) + ((n & 3) << 2);
    tx = g << 6;
  }
  // four k-values (features 16 t + 4 g ..) of tile row r0 + n; r0 a multiple of 16
  __device__ __forceinline__ f32x4 row(const unsigned char* tile, int r0, int t) const {
    return *reinterpret_cast<const f32x4*>(tile + r0 * FTile<D>::ROWB + rb + ((t << 6) ^ rx));
  }
  // feature 16 f + n of tile row r0 + 4 g + i; r0 a multiple of 16
  __device__ __forceinline__ float over(const unsigned char* tile, int r0, int i, int f) const {
    return *reinterpret_cast<const float*>(tile + r0 * FTile<D>::ROWB + tb[i] + ((f << 6) ^ tx));
  }
};

// sum / maximum over the four lanes that hold a token
__device__ __forceinline__ float tok_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}
__device__ __forceinline__ float tok_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}

// features {16 t + 4 g + s} of one token row (zeros if !ok)
template <int NT>
__device__ __forceinline__ void load_frag(const float* __restrict__ row, bool ok, int g, f32x4 (&x)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
    x[t] = ok ? *reinterpret_cast<const f32x4*>(row + 16 * t + 4 * g) : zero4();
}
template <int NT>
__device__ __forceinline__ void store_frag(float* __restrict__ row, int g, const f32x4 (&x)[NT]) {
#pragma unroll
  for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4*>(row + 16 * t + 4 * g) = x[t];
}
template <int NT>
__device__ __forceinline__ float dot_frag(const f32x4 (&a)[NT], const f32x4 (&b)[NT]) {
  f32x4 s = zero4();
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = fmaf(a[t][i], b[t][i], s[i]);
  return tok_sum((s[0] + s[1]) + (s[2] + s[3]));
}

// phi of one token: softmax over its features (phi = 0) or elu + 1
template <int NT>
__device__ __forceinline__ void phi_frag(const f32x4 (&x)[NT], int phi, f32x4 (&y)[NT]) {
  if (phi != 0) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) y[t][i] = x[t][i] > 0.0f ? x[t][i] + 1.0f : expf(x[t][i]);
    return;
  }
  float mx = x[0][0];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) mx = fmaxf(mx, x[t][i]);
  mx = tok_max(mx);
  f32x4 s = zero4();
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      y[t][i] = expf(x[t][i] - mx);
      s[i] += y[t][i];
    }
  const float sum = tok_sum((s[0] + s[1]) + (s[2] + s[3]));
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) y[t][i] = y[t][i] / sum;
}

// acc[r] (rows 16 r .. of the result) += tile rows 16 (r0 + r) .. (k along the rows) times the
// fragment b
template <int D, int NR, int NT>
__device__ __forceinline__ void mm_rows(const FAddr<D>& ad, const unsigned char* tile, const f32x4 (&b)[NT],
                                        f32x4 (&acc)[NR]) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    f32x4 a[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) a[r] = ad.row(tile, 16 * r, t);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int r = 0; r < NR; ++r) acc[r] = mfma16(a[r][s], b[t][s], acc[r]);
  }
}

// acc[f] (features 16 f .. of the tile) += (tile rows 0 .. 16 NK)^T contracted over the rows with
// the C-layout operand b
template <int D, int NK, int NF>
__device__ __forceinline__ void mm_over(const FAddr<D>& ad, const unsigned char* tile, const f32x4 (&b)[NK],
                                        f32x4 (&acc)[NF]) {
#pragma unroll
  for (int k = 0; k < NK; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float a[NF];
#pragma unroll
      for (int f = 0; f < NF; ++f) a[f] = ad.over(tile, 16 * k, i, f);
#pragma unroll
      for (int f = 0; f < NF; ++f) acc[f] = mfma16(a[f], b[k][i], acc[f]);
    }
}

// X^T Y of two 64 x D tiles, both contracted over their rows, into a packed D x D matrix stored
// transposed: out[e][c] = sum_r Y[r][e] X[r][c].  Wave w owns rows e in [D / 4 w, + D / 4).
template <int D>
__device__ __forceinline__ void outer_product(const FAddr<D>& ad, const unsigned char* X, const unsigned char* Y,
                                              int w, f32x4 (&acc)[D / 64][D / 16]) {
  constexpr int NT = D / 16, NE = D / 64;
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float y[NE], x[NT];
#pragma unroll
      for (int e = 0; e < NE; ++e) y[e] = ad.over(Y, 16 * k, i, w * NE + e);
#pragma unroll
      for (int c = 0; c < NT; ++c) x[c] = ad.over(X, 16 * k, i, c);
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int c = 0; c < NT; ++c) acc[e][c] = mfma16(x[c], y[e], acc[e][c]);   // lane = e, registers = c
    }
}
template <int D>
__device__ __forceinline__ void zero_outer(f32x4 (&acc)[D / 64][D / 16]) {
#pragma unroll
  for (int e = 0; e < D / 64; ++e)
#pragma unroll
    for (int c = 0; c < D / 16; ++c) acc[e][c] = zero4();
}
template <int D>
__device__ __forceinline__ void store_outer(float* __restrict__ out, const f32x4 (&acc)[D / 64][D / 16], int w, int l) {
  const int g = l >> 4, n = l & 15;
#pragma unroll
  for (int e = 0; e < D / 64; ++e)
#pragma unroll
    for (int c = 0; c < D / 16; ++c)
      *reinterpret_cast<f32x4*>(out + (size_t)(16 * (w * (D / 64) + e) + n) * D + 16 * c + 4 * g) = acc[e][c];
}

// writes the fragment of this lane's token into row `row` of a swizzled tile
template <int D>
__device__ __forceinline__ void put_frag(unsigned char* tile, int row, int g, const f32x4 (&x)[D / 16]) {
#pragma unroll
  for (int t = 0; t < D / 16; ++t)
    *reinterpret_cast<f32x4*>(tile + row * FTile<D>::ROWB + (((4 * t + g) ^ (row & 15)) << 4)) = x[t];
}
// element c of row r of a swizzled tile
template <int D>
__device__ __forceinline__ float tile_elem(const unsigned char* tile, int r, int c) {
  return *reinterpret_cast<const float*>(tile + r * FTile<D>::ROWB + ((((c >> 2) ^ (r & 15))) << 4) + ((c & 3) << 2));
}

// ------------------------------------------------------------------ key-block states
// Alg. 1 precompute line: h_j = phi(K_j)^T V_j, z_j = rowsum(phi(K_j)^T), one workgroup per key
// block; stored as a state row (h transposed, then z).
// BESIDE: what the first workgroups do, as in the bf16 path: pool Q and K (1), form the column tables (2).
// (4 heads x 122 blocks, d = 128: tables and states 11.1 + 23.1 -> 23.3 us; 2 x 16, d = 64: pooling 6.1 + 7.5 -> 7.5.)
template <int D, int BESIDE>
__global__ __launch_bounds__(256, 2) void f32_states_kernel(const float* __restrict__ K, const float* __restrict__ V,
                                                            int N, int Tn, Lay lay, int phi, float* __restrict__ hz,
                                                            PoolArgs pool, ColArgs col) {
  constexpr int NT = D / 16, TB = FTile<D>::BYTES;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, w = wave_uniform(tid >> 6), l = tid & 63, g = l >> 4, n = l & 15;
  int j = blockIdx.x, bh = blockIdx.y;
  if constexpr (BESIDE != 0) {   // (one row of workgroups, those beside the states first)
    const int Tw = (Tn + 63) / 64, first = BESIDE == 1 ? 2 * pool.wgs : Tw * pool.BH;
    if (j < first) {
      if constexpr (BESIDE == 1) pool_part<float, D>(pool, j);
      else col_tables_part<4>(smem, col, j % Tw, j / Tw);
      return;
    }
    j -= first;
    bh = j / Tn;
    j -= bh * Tn;
  }
  const int n0 = j * kBlk, cnt = min(kBlk, N - n0), row = 16 * w + n;
  const float* Kh = K + lay.head(bh);
  FLoader<D> ld;
  ld.init(lds_base(smem), w, l, 4 * lay.ts, N);
  ld.load(head_rsrc_f32<D>(V + lay.head(bh), N, 4 * lay.ts), j, TB);
  f32x4 x[NT], y[NT];
  load_frag<NT>(Kh + (size_t)(n0 + row) * lay.ts, row < cnt, g, x);
  phi_frag<NT>(x, phi, y);
  if (row >= cnt)   // rows past the end of the sequence contribute nothing, also to z_j
#pragma unroll
    for (int t = 0; t < NT; ++t) y[t] = zero4();
  put_frag<D>(smem, row, g, y);
  wait_vm0();
  __syncthreads();
  FAddr<D> ad;
  ad.init(l);
  f32x4 acc[D / 64][NT];
  zero_outer<D>(acc);
  outer_product<D>(ad, smem, smem + TB, w, acc);
  float* out = hz + ((size_t)bh * Tn + j) * (D * D + D);
  store_outer<D>(out, acc, w, l);
  if (tid < D) {
    float z = 0.0f;
    for (int r = 0; r < kBlk; ++r) z += tile_elem<D>(smem, r, tid);
    out[(size_t)D * D + tid] = z;
  }
}

// ------------------------------------------------------------------ aggregation
// out[i] = sum of the state rows in[k] over the k whose bit is set in ind[i]: the indicator (1 or 0)
// times the states on the matrix cores.  A float is the sum of three bf16 values exactly (24 bits in pieces of
// eight) and their products with 1 and 0 are exact, so three v_mfma_f32_32x32x16_bf16 do in 96 cycles, with the
// same float accumulation, what eight v_mfma_f32_32x32x2_f32 do in 512: that was the bound (122 blocks x 4
// heads, d = 128: 37.6 -> 17.9 us a launch, 12 x 100 77 -> 33, 64 x 8, d = 64, 12.5 -> 9.3).  The sums are closer to
// those in 64 bits than before (relative error 2.4e-7 -> 1.9e-7, 1.9e-7 -> 1.7e-7, 1.65e-7 -> 1.62e-7): the
// accumulators are rounded less often.  A wave owns 32 columns and 32 MT rows i and reads every state
// once, straight into the B operand (lane = column, 128 contiguous bytes per half wave), so no LDS and
// no barriers.  The k-index runs over rows such that the two of a dword lie 16 apart, as their indicator
// bits then do in the dword's place (bits16bf).  The last bits of the last piece of a value below 2^-110 would
// lie below the smallest bf16 there is, 2^-133, so the pieces are those of 2^16 times the value.  A state that is not
// finite would reach every row through its product with 0, and one above 2^99 could overflow the scaled sum of 3072:
// such values are taken out of the product and added only to the rows that hold the bit.
constexpr float kAggScale = 65536.0f, kAggMax = 0x1p99f;

template <int MT>
__global__ __launch_bounds__(256) void f32_aggregate_kernel(const float* __restrict__ in,
                                                            const unsigned long long* __restrict__ ind, int T, int Tw,
                                                            int row_len, float* __restrict__ out) {
  const int w = wave_uniform(threadIdx.x >> 6), l = threadIdx.x & 63, g = l >> 5, n = l & 31;
  const int c0 = (blockIdx.x * 4 + w) * 32, m0 = blockIdx.y * 32 * MT, bh = blockIdx.z;
  if (c0 >= row_len) return;   // (row_len is a multiple of 32)
  const unsigned long long* ib = ind + (size_t)bh * T * Tw;
  const float* src = in + (size_t)bh * T * row_len + c0 + n;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(in + (size_t)bh * T * row_len), 0, T * row_len * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t orsrc =
      __builtin_amdgcn_make_buffer_rsrc(out + (size_t)bh * T * row_len, 0, T * row_len * 4, 0x00020000);
  const int pitch = row_len * 4, voff = 4 * g * pitch + (c0 + n) * 4;
  constexpr int CH = 16;       // values of a chunk of 32 states: slots (u, p, h) = state 8 u + 4 g + p + 16 h
  f32x16 acc[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) acc[m] = zero_f32x16();
  auto fetch = [&](int k0, float (&x)[CH]) {
#pragma unroll
    for (int q = 0; q < CH; ++q)   // (rows past T read as zeros)
      x[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
          rsrc, voff + (k0 + 8 * (q >> 3) + ((q >> 1) & 3) + 16 * (q & 1)) * pitch, 0, 0));
  };
  float x[CH], nx[CH];
  bool bad = false;
  fetch(0, x);
  // indicator words of the lane's rows, a word ahead (rows past T are not stored)
  unsigned long long wb[MT], nwb[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) nwb[m] = ib[(size_t)min(m0 + 32 * m + n, T - 1) * Tw];
  for (int k0 = 0; k0 < T; k0 += 2 * CH) {
    if ((k0 & 63) == 0) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        wb[m] = nwb[m];
        nwb[m] = ib[(size_t)min(m0 + 32 * m + n, T - 1) * Tw + min((k0 >> 6) + 1, Tw - 1)];
      }
    }
    if (k0 + 2 * CH < T) fetch(k0 + 2 * CH, nx);
    unsigned part[3][CH / 2];   // [piece][dword]: the pieces of two states, most significant first
#pragma unroll
    for (int q = 0; q < CH; q += 2) {
      unsigned y[2][3];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bool in_range = fabsf(x[q + h]) <= kAggMax;
        bad |= !in_range;
        float v = in_range ? x[q + h] * kAggScale : 0.0f;
#pragma unroll
        for (int e = 0; e < 3; ++e) {   // the top 16 bits are a bf16, and what is left of v is exact
          y[h][e] = __float_as_uint(v) & 0xffff0000u;
          v -= __uint_as_float(y[h][e]);
        }
      }
#pragma unroll
      for (int e = 0; e < 3; ++e) part[e][q / 2] = y[1][e] | y[0][e] >> 16;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      bf16x8 b[3];
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const u32x4 t = {part[e][4 * u], part[e][4 * u + 1], part[e][4 * u + 2], part[e][4 * u + 3]};
        b[e] = __builtin_bit_cast(bf16x8, t);
      }
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        const unsigned bits = (unsigned)(wb[m] >> (k0 & 32)) >> (8 * u + 4 * g);
        const u32x4 t = {bits16bf<0>(bits), bits16bf<1>(bits), bits16bf<2>(bits), bits16bf<3>(bits)};
        const bf16x8 a = __builtin_bit_cast(bf16x8, t);
#pragma unroll
        for (int e = 2; e >= 0; --e) acc[m] = mfma32(a, b[e], acc[m]);
      }
    }
#pragma unroll
    for (int q = 0; q < CH; ++q) x[q] = nx[q];
  }
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int r = 0; r < 16; ++r)   // row m0 + 32 m + c_row(r, g); rows past T are dropped
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[m][r] * (1.0f / kAggScale)), orsrc,
                                            (m0 + 32 * m + c_row(r, g)) * pitch + (c0 + n) * 4, 0, 0);
  if (!__any(bad)) return;
  // this lane's column again, for the rows it has just written
  for (int i = m0 + 4 * g; i < min(T, m0 + 32 * MT); i += (i & 3) == 3 ? 5 : 1) {
    float* o = out + ((size_t)bh * T + i) * row_len + c0 + n;
    for (int k = 0; k < T; ++k) {
      const float v = src[(size_t)k * row_len];
      if (!(fabsf(v) <= kAggMax) && ((ib[(size_t)i * Tw + (k >> 6)] >> (k & 63)) & 1ull)) *o += v;
    }
  }
}

// The same for the shortest sequences, where the matrix form's 32 states and 32 rows are nearly all
// padding: a thread owns V columns, holds them of every state and writes the sums of every row, so
// that the states are read once and nothing but the traffic is left.  (One block, d = 64: 256 heads
// 31.9 -> 6.6 us a launch, 4096 heads 396 -> 24.6; four blocks, 256 heads, d = 128: 103 -> 23.)
template <int kFew, int V>
__global__ __launch_bounds__(256) void f32_aggregate_few_kernel(const float* __restrict__ in,
                                                                const unsigned long long* __restrict__ ind, int T,
                                                                int row_len, float* __restrict__ out) {
  typedef float vec __attribute__((ext_vector_type(V)));
  const int c = V * (blockIdx.x * 256 + threadIdx.x), bh = blockIdx.y;
  if (c >= row_len) return;   // (row_len is a multiple of 4)
  const size_t o = (size_t)bh * T * row_len + c;
  vec x[kFew];
#pragma unroll
  for (int k = 0; k < kFew; ++k) x[k] = k < T ? *reinterpret_cast<const vec*>(in + o + (size_t)k * row_len) : vec(0.0f);
#pragma unroll
  for (int i = 0; i < kFew; ++i) {
    if (i >= T) break;
    const unsigned bits = (unsigned)ind[(size_t)bh * T + i];   // (one word a row; no bits past T)
    vec s = vec(0.0f);
#pragma unroll
    for (int k = 0; k < kFew; ++k)
      if ((bits >> k) & 1u) s += x[k];
    *reinterpret_cast<vec*>(out + o + (size_t)i * row_len) = s;
  }
}

// ------------------------------------------------------------------ forward
// One workgroup per query block: critical-block loop (Alg. 1 inner loop, M_c = 1 branch), then
// the closing line and Eq. 6.  Wave w owns queries 16 w .. 16 w + 15 (lane n = query) against all
// 64 keys of a step, so that the waves share nothing but the tiles.  Bound by the matrix cores:
// K and V have one slot each; K_{s+1} is requested when the scores of step s are formed and lands
// under the second product, V_{s+1} lands under the scores of step s + 1; two workgroups per CU.
template <int D>
__global__ __launch_bounds__(256, 2) void f32_forward_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, const float* __restrict__ W,
    const int32_t* __restrict__ row_idx, const float* __restrict__ HZ, int N, int Tn, Lay lay, int n_h, int n_0,
    int phi, float scale, float* __restrict__ O, float* __restrict__ Os, float* __restrict__ Ol,
    float* __restrict__ L) {
  constexpr int NT = D / 16, TB = FTile<D>::BYTES;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, w = wave_uniform(tid >> 6), l = tid & 63, g = l >> 4, n = l & 15;
  const int i = blockIdx.x, bh = blockIdx.y;
  const int q0 = i * kBlk, rows = min(kBlk, N - q0), row = 16 * w + n;
  const bool ok = row < rows;
  const size_t qb = ((size_t)bh * N + q0 + row) * D;                       // in the library's packed tensors
  const size_t uq = lay.head(bh) + (size_t)(q0 + row) * lay.ts;            // in the caller's tensors
  FLoader<D> ld, lm;   // the caller's tensors; packed D x D matrices
  ld.init(lds_base(smem), w, l, 4 * lay.ts, N);
  lm.init(lds_base(smem), w, l, 4 * D);
  const BufDesc dK = head_rsrc_f32<D>(K + lay.head(bh), N, 4 * lay.ts);
  const BufDesc dV = head_rsrc_f32<D>(V + lay.head(bh), N, 4 * lay.ts);
  const float* Hrow = HZ + ((size_t)bh * Tn + i) * (D * D + D);
  const BufDesc dH = matrix_rsrc_f32<D>(Hrow, D), dW = matrix_rsrc_f32<D>(W, D);
  const int32_t* lut = row_idx + ((size_t)bh * Tn + i) * n_h;
  // what follows the loop: H_i into the K slot (and, for D = 128, its second half into the V slot)
  auto issue_h0 = [&]() { if (n_0 > 0) lm.load(dH, 0, 0); };
  auto issue_h1 = [&]() { if (n_0 > 0) lm.load(D > kBlk ? dH : dW, D > kBlk ? 1 : 0, TB); };
  int j = 0;
  if (n_h > 0) {
    j = lut[0];
    ld.load(dK, j, 0);
    ld.load(dV, j, TB);
  } else {
    issue_h0();
    issue_h1();
  }
  f32x4 qf[NT], acc[NT];
  load_frag<NT>(Q + uq, ok, g, qf);
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = zero4();
  float m = -INFINITY, lsum = 0.0f;
  FAddr<D> ad;
  ad.init(l);
  wait_vm0();
  __syncthreads();
  for (int s = 0; s < n_h; ++s) {
    const int cols = min(kBlk, N - j * kBlk);
    const bool last = s + 1 == n_h;
    const int jn = last ? 0 : lut[s + 1];
    f32x4 p[4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) p[kt] = zero4();
    mm_rows<D, 4, NT>(ad, smem, qf, p);     // S^T: registers = keys 16 kt + 4 g + i, lane = query
    wait_vm0();
    __syncthreads();                        // V_s is there, the K slot is free
    if (last) issue_h0();
    else ld.load(dK, jn, 0);
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[kt][r] = 16 * kt + 4 * g + r < cols ? p[kt][r] * scale : -INFINITY;
        mx = fmaxf(mx, p[kt][r]);
      }
    const float mnew = fmaxf(m, tok_max(mx));
    f32x4 sum = zero4();
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        p[kt][r] = expf(p[kt][r] - mnew);
        sum[r] += p[kt][r];
      }
    const float alpha = expf(m - mnew);
    lsum = alpha * lsum + tok_sum((sum[0] + sum[1]) + (sum[2] + sum[3]));
    m = mnew;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[t][r] *= alpha;
    mm_over<D, 4, NT>(ad, smem + TB, p, acc);   // O^T += V^T P^T
    wait_vm0();
    __syncthreads();                        // K_{s+1} is there, the V slot is free
    if (last) issue_h1();
    else ld.load(dV, jn, TB);
    j = jn;
  }
  // closing line of Alg. 1, sparse part
  const float inv = n_h > 0 ? 1.0f / lsum : 0.0f;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[t][r] *= inv;
  if (Os && ok) store_frag<NT>(Os + qb, g, acc);
  if (L && ok && g == 0) L[(size_t)bh * N + q0 + row] = n_h > 0 ? m + logf(lsum) : -INFINITY;
  f32x4 ol[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) ol[t] = zero4();
  if (n_0 > 0) {
    // O^l_i = phi(Q_i) H_i / (phi(Q_i) Z_i); the LDS matrix holds H_i^T (rows e, k along the row)
    f32x4 y[NT], z[NT];
    phi_frag<NT>(qf, phi, y);
    load_frag<NT>(Hrow + D * D, true, g, z);
    const float den = dot_frag<NT>(y, z);
    wait_vm0();
    __syncthreads();
    mm_rows<D, NT, NT>(ad, smem, y, ol);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) ol[t][r] = ol[t][r] / den;
    // Eq. 6: O = O^s + O^l W, i.e. O^T += W^T (O^l)^T
    constexpr int WS = D > kBlk ? 0 : TB;   // where W lies
    if (D > kBlk) {
      __syncthreads();
      lm.load(dW, 0, 0);
      lm.load(dW, 1, TB);
      wait_vm0();
      __syncthreads();
    }
    mm_over<D, NT, NT>(ad, smem + WS, ol, acc);
  }
  if (!ok) return;
  store_frag<NT>(O + uq, g, acc);
  if (Ol) store_frag<NT>(Ol + qb, g, ol);
}

// dW = sum over tokens of (O^l)^T dO: part p of `parts` sums the 64-token tiles p, p + parts, .. into its own d x d
// matrix; dw_sum adds the parts.  They are the last workgroups of the query-side launch (it forms nothing they
// need) and run where its last round leaves CUs idle (4 heads
// x 122 blocks, d = 128: 119.5 + 20.0 us in two launches -> 127.2).
template <int D>
__device__ __forceinline__ void f32_dw_part(unsigned char* smem, const float* __restrict__ Ol, const float* __restrict__ dO,
                                            int p, int parts, int BH, int N, int Tn, Lay lay, float* __restrict__ part) {
  constexpr int NT = D / 16, TB = FTile<D>::BYTES;
  const int tid = threadIdx.x, w = wave_uniform(tid >> 6), l = tid & 63;
  FLoader<D> lo, lg;
  lo.init(lds_base(smem), w, l, 4 * D);
  lg.init(lds_base(smem), w, l, 4 * lay.ts, N);
  FAddr<D> ad;
  ad.init(l);
  f32x4 acc[D / 64][NT];
  zero_outer<D>(acc);
  for (int t = p; t < BH * Tn; t += parts) {
    const int bh = t / Tn, i = t - bh * Tn;
    lo.load(matrix_rsrc_f32<D>(Ol + (size_t)bh * N * D, N), i, TB);
    lg.load(head_rsrc_f32<D>(dO + lay.head(bh), N, 4 * lay.ts), i, 0);
    wait_vm0();
    __syncthreads();
    outer_product<D>(ad, smem, smem + TB, w, acc);
    __syncthreads();
  }
  store_outer<D>(part + (size_t)p * D * D, acc, w, l);   // rows c of O^l along the lanes
}

// ------------------------------------------------------------------ backward, query side
// One workgroup per query block, waves as in the forward kernel (lane = query).  D line of Alg. 2
// (dO^l = dO W^T, D^s, D^l), then its first loop: dH_i, dZ_i and dQ^phi_i through phi, then the
// dQ_i accumulation of the second loop over the row table, so that each dQ_i has one owner.  dO^l
// and the linear part of dQ never leave the registers; K and V go through one slot each: V_{s+1}
// lands under the scores and dQ of step s, K_{s+1} under dP of step s + 1.
template <int D>
__global__ __launch_bounds__(256, 2) void f32_bwd_query_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, const float* __restrict__ W,
    const float* __restrict__ dO, const float* __restrict__ Os, const float* __restrict__ Ol,
    const float* __restrict__ L, const float* __restrict__ HZ, const int32_t* __restrict__ row_idx, int N, int Tn,
    Lay lay, int n_h, int n_0, int phi, float scale, float* __restrict__ Ds, float* __restrict__ dHZ,
    float* __restrict__ dQ, int BH, float* __restrict__ dWpart, int nparts, KvPlanArgs plan) {
  constexpr int NT = D / 16, TB = FTile<D>::BYTES;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if ((int)blockIdx.x >= Tn * BH) {   // the last workgroups: units of the key side, then the parts of dW
    const int p = blockIdx.x - Tn * BH, plans = kv_plan_wgs(plan.split, BH);
    if (p >= plans) f32_dw_part<D>(smem, Ol, dO, p - plans, nparts, BH, N, Tn, lay, dWpart);
    else if (4 * p + (int)(threadIdx.x >> 6) < BH) kv_plan(plan, Tn, 4 * p + (threadIdx.x >> 6));
    return;
  }
  float* dls = reinterpret_cast<float*>(smem + 2 * TB);   // D^l / (phi(Q) Z) of the 64 queries
  const int tid = threadIdx.x, w = wave_uniform(tid >> 6), l = tid & 63, g = l >> 4, n = l & 15;
  const int i = blockIdx.x % Tn, bh = blockIdx.x / Tn;
  const int q0 = i * kBlk, rows = min(kBlk, N - q0), row = 16 * w + n;
  const bool ok = row < rows;
  const size_t qi = (size_t)bh * N + q0 + row;
  const size_t uq = lay.head(bh) + (size_t)(q0 + row) * lay.ts;
  FLoader<D> ld, lm;
  ld.init(lds_base(smem), w, l, 4 * lay.ts, N);
  lm.init(lds_base(smem), w, l, 4 * D);
  FAddr<D> ad;
  ad.init(l);
  f32x4 qf[NT], gf[NT], dql[NT];
  load_frag<NT>(Q + uq, ok, g, qf);
  load_frag<NT>(dO + uq, ok, g, gf);
  float Dr;
  {
    f32x4 os[NT];
    load_frag<NT>(Os + qi * D, ok, g, os);
    Dr = dot_frag<NT>(gf, os);
    if (ok && g == 0) Ds[qi] = Dr;
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) dql[t] = zero4();
  if (n_0 > 0) {
    const BufDesc dW = matrix_rsrc_f32<D>(W, D);
    const float* Hrow = HZ + ((size_t)bh * Tn + i) * (D * D + D);
    const BufDesc dH = matrix_rsrc_f32<D>(Hrow, D);
    lm.load(dW, 0, 0);
    lm.load(D > kBlk ? dW : dH, D > kBlk ? 1 : 0, TB);
    f32x4 y[NT], gl[NT], z[NT];
    phi_frag<NT>(qf, phi, y);
    load_frag<NT>(Hrow + D * D, true, g, z);
    const float inv = ok ? 1.0f / dot_frag<NT>(y, z) : 0.0f;
#pragma unroll
    for (int t = 0; t < NT; ++t) gl[t] = zero4();
    wait_vm0();
    __syncthreads();
    mm_rows<D, NT, NT>(ad, smem, gf, gl);   // dO^l: rows c of W, k = e
    {
      f32x4 ol[NT];
      load_frag<NT>(Ol + qi * D, ok, g, ol);
      const float Dl = dot_frag<NT>(gl, ol) * inv;
      if (g == 0) dls[row] = Dl;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          gl[t][r] *= inv;
          dql[t][r] = -Dl * z[t][r];
        }
    }
    constexpr int HS = D > kBlk ? 0 : TB;   // where H_i^T lies
    if (D > kBlk) {
      __syncthreads();
      lm.load(dH, 0, 0);
      lm.load(dH, 1, TB);
      wait_vm0();
      __syncthreads();
    }
    // dQ^phi = (dO^l / den) H^T - (D^l / den) Z, then the Jacobian of phi
    mm_over<D, NT, NT>(ad, smem + HS, gl, dql);
    if (phi == 0) {
      const float dot = dot_frag<NT>(dql, y);
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) dql[t][r] = y[t][r] * (dql[t][r] - dot);
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) dql[t][r] *= qf[t][r] > 0.0f ? 1.0f : expf(qf[t][r]);
    }
    // dH_i^T[e][c] = sum_r (dO^l[r][e] / den_r) phi(Q)[r][c], contracted over the 64 queries
    if (!ok)
#pragma unroll
      for (int t = 0; t < NT; ++t) y[t] = zero4();
    __syncthreads();
    put_frag<D>(smem, row, g, y);
    put_frag<D>(smem + TB, row, g, gl);
    __syncthreads();
    float* out = dHZ + ((size_t)bh * Tn + i) * (D * D + D);
    f32x4 o[D / 64][NT];
    zero_outer<D>(o);
    outer_product<D>(ad, smem, smem + TB, w, o);
    store_outer<D>(out, o, w, l);
    if (tid < D) {
      float s = 0.0f;
      for (int r = 0; r < kBlk; ++r) s = fmaf(tile_elem<D>(smem, r, tid), dls[r], s);
      out[(size_t)D * D + tid] = -s;
    }
    __syncthreads();
  }
  f32x4 dq[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) dq[t] = zero4();
  if (n_h > 0) {
    const BufDesc dK = head_rsrc_f32<D>(K + lay.head(bh), N, 4 * lay.ts);
    const BufDesc dV = head_rsrc_f32<D>(V + lay.head(bh), N, 4 * lay.ts);
    const int32_t* lut = row_idx + ((size_t)bh * Tn + i) * n_h;
    int j = lut[0];
    ld.load(dV, j, TB);
    ld.load(dK, j, 0);
    const float Lr = ok ? L[qi] : 0.0f;
    wait_vm0();
    __syncthreads();
    for (int s = 0; s < n_h; ++s) {
      const int cols = min(kBlk, N - j * kBlk);
      const int jn = s + 1 < n_h ? lut[s + 1] : -1;
      f32x4 p[4], dp[4];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) p[kt] = dp[kt] = zero4();
      mm_rows<D, 4, NT>(ad, smem + TB, gf, dp);    // dP^T = V dO^T
      wait_vm0();
      __syncthreads();                             // K_s is there, the V slot is free
      if (jn >= 0) ld.load(dV, jn, TB);
      mm_rows<D, 4, NT>(ad, smem, qf, p);          // S^T = K Q^T
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float e = ok && 16 * kt + 4 * g + r < cols ? expf(p[kt][r] * scale - Lr) : 0.0f;
          dp[kt][r] = e * (dp[kt][r] - Dr);
        }
      mm_over<D, 4, NT>(ad, smem, dp, dq);         // dQ^T += K^T dS^T
      wait_vm0();
      __syncthreads();                             // V_{s+1} is there, the K slot is free
      if (jn >= 0) ld.load(dK, jn, 0);
      j = jn;
    }
  }
  if (!ok) return;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) dq[t][r] = dq[t][r] * scale + dql[t][r];
  store_frag<NT>(dQ + uq, g, dq);
}

// ------------------------------------------------------------------ backward, key side
// dK_j, dV_j: second loop of Alg. 2 (M_c = 1 branch) over the column table, then its last line.
// Columns hold between none and T critical blocks, and the heaviest list alone would outlast the
// rest of the launch: a workgroup therefore owns only 64 / QW keys of a key block, the waves that
// share 16 of them (lane = key) split the 64 queries of every step in QW parts, and the
// workgroups start with the longest lists of all heads.  The partial sums of the QW waves meet in
// LDS once, after the loop; each then finishes its share of the features.  Q and dO go through
// one slot each; every load lands under a product that reads the other one.  Lists that would still outlast
// the rest are cut: the first workgroups walk pieces of them and leave their sums as rows of a slot, which
// f32_kv_merge_kernel adds to what the first piece of the list gave.
template <int QW, int M>
__device__ __forceinline__ void pick_tiles(const f32x4* x, int wq, f32x4 (&y)[M]) {
  // y[m] = x[wq + QW m] with wq uniform, without indexing registers
#pragma unroll
  for (int m = 0; m < M; ++m) {
    y[m] = x[QW * m];
#pragma unroll
    for (int q = 1; q < QW; ++q)
#pragma unroll
      for (int r = 0; r < 4; ++r) y[m][r] = wq == q ? x[QW * m + q][r] : y[m][r];
  }
}

// a slot: the 64 rows of dK, then those of dV
template <int D>
__device__ __forceinline__ float* f32_kv_slot(const KvSplit& kv, int bh, int slot) {
  return kv.part + ((size_t)bh * (kv.ecap + kv.cuts) + slot) * (2 * kBlk * D);
}
// dK_j, dV_j of the key blocks whose lists were cut += the sums of the extras, in order; a workgroup per
// 16 rows of the two
template <int D>
__global__ __launch_bounds__(256) void f32_kv_merge_kernel(KvSplit kv, int BH, int N, int Tn, Lay lay,
                                                           float* __restrict__ dK, float* __restrict__ dV) {
  const int bh = blockIdx.x % BH, r = blockIdx.x / BH;
  const int4 unit = kv.units[(size_t)bh * (kv.ecap + Tn + kv.cuts) + kv.ecap + Tn + r];
  if (unit.z == 0) return;
  constexpr int C = D / 4;   // 16-byte pieces of a row
  for (int i = blockIdx.y * 16 * C + threadIdx.x; i < (blockIdx.y + 1) * 16 * C; i += 256) {
    const int row = i / C, c = 4 * (i % C), key = unit.x * kBlk + row % kBlk;
    if (key >= N) continue;
    float* o = (row < kBlk ? dK : dV) + lay.head(bh) + (size_t)key * lay.ts + c;
    f32x4 s = *reinterpret_cast<const f32x4*>(o);
#pragma unroll 4
    for (int e = 0; e < unit.z; ++e)
      s += *reinterpret_cast<const f32x4*>(f32_kv_slot<D>(kv, bh, unit.y + e) + (size_t)row * D + c);
    *reinterpret_cast<f32x4*>(o) = s;
  }
}

template <int D>
constexpr int f32_bwd_key_lds() { return 2 * FTile<D>::BYTES + 512 + 256; }   // + L, D^s of 64 queries + dot products

template <int D, int QW>
__global__ __launch_bounds__(256, 2) void f32_bwd_key_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    const float* __restrict__ dO, const float* __restrict__ L, const float* __restrict__ Ds,
    const int32_t* __restrict__ col_ptr, const int32_t* __restrict__ col_rows, const int32_t* __restrict__ col_order,
    const float* __restrict__ dHZcol, int N, int Tn, Lay lay, int n_h, int n_0, int phi, float scale,
    float* __restrict__ dK, float* __restrict__ dV, DwSum dw, KvSplit kv) {
  static_assert(QW == 2 || QW == 4, "waves that share a group of 16 keys");
  constexpr int NT = D / 16, TB = FTile<D>::BYTES, NQ = 4 / QW, NO = NT / QW;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int y = (int)blockIdx.y - kv.ecap * QW;   // below zero: extras
  if (y >= Tn * QW) {   // the last rows of the grid: dW
    const int block = (y - Tn * QW) * gridDim.x + blockIdx.x;
    if (block < dw.dd / kDwPiece) dw_sum(dw, block, smem);
    return;
  }
  const unsigned char* stat = smem + 2 * TB;
  float* dots = reinterpret_cast<float*>(smem + 2 * TB + 512);
  const int tid = threadIdx.x, w = wave_uniform(tid >> 6), l = tid & 63, g = l >> 4, n = l & 15;
  const int wk = w / QW, wq = w % QW;
  const int bh = blockIdx.x, kg = blockIdx.y % QW;
  int j, t0 = 0, t1 = 0, slot = 0;
  if (kv.ecap > 0) {
    const int4 unit = kv.units[(size_t)bh * (kv.ecap + Tn + kv.cuts) + blockIdx.y / QW];
    j = unit.x;
    t0 = unit.y;
    t1 = t0 + unit.z;
    slot = unit.w;
    if (y < 0 && unit.z == 0) return;
  } else {
    j = col_order[(size_t)bh * Tn + blockIdx.y / QW];
    const int32_t* ptr = col_ptr + (size_t)bh * (Tn + 1);
    if (n_h > 0) {
      t0 = ptr[j];
      t1 = ptr[j + 1];
    }
  }
  const int k0 = j * kBlk + kg * (kBlk / QW);      // first key of this workgroup
  if (k0 >= N) return;
  const int key = k0 + 16 * wk + n;
  const bool ok = key < N;
  const size_t uk = lay.head(bh) + (size_t)key * lay.ts;
  f32x4 kf[NT], vf[NT], dk[NT], dv[NT];
  load_frag<NT>(K + uk, ok, g, kf);
  load_frag<NT>(V + uk, ok, g, vf);
#pragma unroll
  for (int t = 0; t < NT; ++t) dk[t] = dv[t] = zero4();
  FLoader<D> ld;
  ld.init(lds_base(smem), w, l, 4 * lay.ts, N);
  FAddr<D> ad;
  ad.init(l);
  const BufDesc dQd = head_rsrc_f32<D>(Q + lay.head(bh), N, 4 * lay.ts);
  const BufDesc dOd = head_rsrc_f32<D>(dO + lay.head(bh), N, 4 * lay.ts);
  const BufDesc dSt = tile_rsrc((w == 0 ? L : Ds) + (size_t)bh * N, N * 4);
  // Q_i into slot 0, with L and D^s of its queries
  auto issue_q = [&](int i) {
    ld.load(dQd, i, 0);
    if (w < 2) load_to_lds4(dSt, (i * kBlk + l) * 4, lds_base(smem) + 2 * TB + 256 * w);
  };
  const int32_t* list = col_rows + (size_t)bh * Tn * n_h;
  if (t0 < t1) {
    int i = list[t0];
    ld.load(dOd, i, TB);
    issue_q(i);
    wait_vm0();
    __syncthreads();
    const unsigned char* Qs = smem + 16 * NQ * wq * FTile<D>::ROWB;         // this wave's queries
    const unsigned char* Gs = Qs + TB;
    const unsigned char* st = stat + 4 * (16 * NQ * wq + 4 * g);
    for (int t = t0; t < t1; ++t) {
      const int in = t + 1 < t1 ? list[t + 1] : -1;
      f32x4 p[NQ], dp[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) p[q] = dp[q] = zero4();
      mm_rows<D, NQ, NT>(ad, Gs, vf, dp);          // dP = dO V^T: registers = queries, lane = key
      wait_vm0();
      __syncthreads();                             // Q_i is there
      mm_rows<D, NQ, NT>(ad, Qs, kf, p);           // S = Q K^T
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const f32x4 Lr = *reinterpret_cast<const f32x4*>(st + 64 * q);
        const f32x4 Dr = *reinterpret_cast<const f32x4*>(st + 64 * q + 256);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool in_row = i * kBlk + 16 * (NQ * wq + q) + 4 * g + r < N;
          p[q][r] = in_row ? expf(p[q][r] * scale - Lr[r]) : 0.0f;
          dp[q][r] = p[q][r] * (dp[q][r] - Dr[r]);
        }
      }
      mm_over<D, NQ, NT>(ad, Gs, p, dv);           // dV^T += dO^T P
      __syncthreads();                             // the dO slot is free
      if (in >= 0) ld.load(dOd, in, TB);
      mm_over<D, NQ, NT>(ad, Qs, dp, dk);          // dK^T += Q^T dS
      wait_vm0();
      __syncthreads();                             // dO_{i'} is there, the Q slot is free
      if (in >= 0) issue_q(in);
      i = in;
    }
  }
  // wave wq of the QW that share a key group gets the feature tiles wq, wq + QW, ...
  f32x4 ok_[NO], ov[NO];
  {
    f32x4* x = reinterpret_cast<f32x4*>(smem);      // [wave][dK, dV][tile][lane]
#pragma unroll
    for (int f = 0; f < NT; ++f) {
      x[(2 * w * NT + f) * 64 + l] = dk[f];
      x[((2 * w + 1) * NT + f) * 64 + l] = dv[f];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NO; ++m) {
      ok_[m] = ov[m] = zero4();
#pragma unroll
      for (int q = 0; q < QW; ++q) {
        const int b = (2 * (wk * QW + q) * NT + wq + QW * m) * 64 + l;
        const f32x4 a = x[b], c = x[b + NT * 64];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          ok_[m][r] += a[r];
          ov[m][r] += c[r];
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < NO; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) ok_[m][r] *= scale;
  if (y < 0) {
    float* o = f32_kv_slot<D>(kv, bh, slot) + (size_t)(key - j * kBlk) * D;
#pragma unroll
    for (int m = 0; m < NO; ++m) {
      *reinterpret_cast<f32x4*>(o + 16 * (wq + QW * m) + 4 * g) = ok_[m];
      *reinterpret_cast<f32x4*>(o + kBlk * D + 16 * (wq + QW * m) + 4 * g) = ov[m];
    }
    return;
  }
  if (n_0 > 0) {
    // last line of Alg. 2: dK^phi = V dH^T + dZ (then through phi), dV += phi(K) dH, with dH, dZ
    // the sums over the marginal query blocks of this key block; LDS holds dH^T (rows e)
    const float* Hrow = dHZcol + ((size_t)bh * Tn + j) * (D * D + D);
    FLoader<D> lm;
    lm.init(lds_base(smem), w, l, 4 * D);
    const BufDesc dH = matrix_rsrc_f32<D>(Hrow, D);
    lm.load(dH, 0, 0);
    if (D > kBlk) lm.load(dH, 1, TB);
    f32x4 y[NT], gk[NO], yo[NO], ko[NO];
    phi_frag<NT>(kf, phi, y);
    pick_tiles<QW, NO>(y, wq, yo);
    pick_tiles<QW, NO>(kf, wq, ko);
#pragma unroll
    for (int m = 0; m < NO; ++m) gk[m] = *reinterpret_cast<const f32x4*>(Hrow + D * D + 16 * (wq + QW * m) + 4 * g);
    wait_vm0();
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      f32x4 a[NO];
#pragma unroll
      for (int m = 0; m < NO; ++m) a[m] = ad.row(smem + 16 * wq * FTile<D>::ROWB, 16 * QW * m, t);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        float b[NO];
#pragma unroll
        for (int m = 0; m < NO; ++m) b[m] = ad.over(smem, 16 * t, s, wq + QW * m);
#pragma unroll
        for (int m = 0; m < NO; ++m) {
          ov[m] = mfma16(a[m][s], y[t][s], ov[m]);
          gk[m] = mfma16(b[m], vf[t][s], gk[m]);
        }
      }
    }
    if (phi == 0) {
      float dot = dot_frag<NO>(gk, yo);
      if (g == 0) dots[16 * w + n] = dot;
      __syncthreads();
      dot = 0.0f;
#pragma unroll
      for (int q = 0; q < QW; ++q) dot += dots[16 * (wk * QW + q) + n];
#pragma unroll
      for (int m = 0; m < NO; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) ok_[m][r] += yo[m][r] * (gk[m][r] - dot);
    } else {
#pragma unroll
      for (int m = 0; m < NO; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) ok_[m][r] += gk[m][r] * (ko[m][r] > 0.0f ? 1.0f : expf(ko[m][r]));
    }
  }
  if (!ok) return;
#pragma unroll
  for (int m = 0; m < NO; ++m) {
    const size_t o = uk + 16 * (wq + QW * m) + 4 * g;
    *reinterpret_cast<f32x4*>(dK + o) = ok_[m];
    *reinterpret_cast<f32x4*>(dV + o) = ov[m];
  }
}

// out[i] = sum over k with bit k of ind[i] set of the state rows in[k]
hipError_t f32_aggregate(const float* in, const unsigned long long* ind, const Shape& s, float* out, hipStream_t st) {
  const int row_len = s.state_row(), Tw = (s.T + 63) / 64;
  const int gx = (row_len / 32 + 3) / 4;
  KernelTimer kt("aggregate", st);
  // Up to eight blocks the short form, whatever the number of heads, which must not change a head's sums.  With many it
  // runs at the memory's rate (matrix -> short form, us: five blocks, 256 heads, d = 128, 63 -> 28; eight, 512 heads,
  // d = 64, 39 -> 23); with few it has one column a thread, as four leave most CUs without a workgroup
  // (16 heads x 8, d = 64, matrix 6.6, four columns 8.0, one 6.6; matrix -> one column: 16 x 5, d = 128, 10.0 -> 7.5,
  // 40 x 8 14.7 -> 11.3).
  if (s.T <= 8) {
    const bool one = s.T > 4 && (long long)s.BH * row_len < 512 * 1024;
    auto few = s.T <= 4 ? f32_aggregate_few_kernel<4, 4> : one ? f32_aggregate_few_kernel<8, 1> : f32_aggregate_few_kernel<8, 4>;
    const int columns = one ? 256 : 1024;
    few<<<dim3((row_len + columns - 1) / columns, s.BH), 256, 0, st>>>(in, ind, s.T, row_len, out);
    return hipGetLastError();
  }
  // up to 128 rows per wave (the states are read ceil(T / 128) times), in tiles of 32 dealt evenly
  const int ny = (s.T + 127) / 128, mt = ((s.T + 31) / 32 + ny - 1) / ny;
  auto kern = mt == 1 ? f32_aggregate_kernel<1> : mt == 2 ? f32_aggregate_kernel<2>
            : mt == 3 ? f32_aggregate_kernel<3> : f32_aggregate_kernel<4>;
  kern<<<dim3(gx, ny, s.BH), 256, 0, st>>>(in, ind, s.T, Tw, row_len, out);
  return hipGetLastError();
}

template <int D>
hipError_t states_impl(const Shape& s, const FwdArgs& a, const Beside& b, hipStream_t st) {
  const int Tw = (s.T + 63) / 64;
  constexpr int tiles = 2 * FTile<D>::BYTES;
  const int lds = b.col ? max(tiles, col_tables_lds(Tw, 4)) : tiles;
  const int first = b.pool ? 2 * b.pool->wgs : b.col ? Tw * s.BH : 0;
  PoolArgs pool = {};
  if (b.pool) pool = *b.pool;
  pool.BH = s.BH;
  auto kern = b.pool ? f32_states_kernel<D, 1> : b.col ? f32_states_kernel<D, 2> : f32_states_kernel<D, 0>;
  SLA_TRY(ensure_dyn_lds(kern, lds));
  KernelTimer kt(b.pool ? "states_pool" : b.col ? "states_cols" : "states", st);
  const dim3 grid = first ? dim3(first + s.T * s.BH) : dim3(s.T, s.BH);
  kern<<<grid, 256, lds, st>>>((const float*)a.K, (const float*)a.V, s.N, s.T, s.lay(), s.phi, a.hz, pool,
                               b.col ? *b.col : ColArgs{});
  return hipGetLastError();
}

template <int D>
hipError_t forward_impl(const Shape& s, const FwdArgs& a, hipStream_t st) {
  const dim3 grid(s.T, s.BH);
  const size_t lds = 2 * FTile<D>::BYTES;
  if (s.n_0 > 0) {
    SLA_TRY(f32_aggregate(a.hz, a.ind, s, a.HZ, st));
  } else {
    SLA_TRY(launch_fill_zero(a.HZ, (size_t)s.BH * s.T * s.state_row(), st));
  }
  SLA_TRY(ensure_dyn_lds(f32_forward_kernel<D>, lds));
  {
    KernelTimer kt("forward", st);
    f32_forward_kernel<D><<<grid, 256, lds, st>>>((const float*)a.Q, (const float*)a.K, (const float*)a.V,
                                                  (const float*)a.W, a.row_idx, a.HZ, s.N, s.T, s.lay(), s.n_h, s.n_0,
                                                  s.phi, s.scale, (float*)a.O, (float*)a.Os, (float*)a.Ol, a.L);
  }
  return hipGetLastError();
}

template <int D, int QW>
hipError_t launch_key(const Shape& s, const BwdArgs& a, const float* Ds, const float* dHZcol, const DwSum& dw,
                      const KvSplit& kv, hipStream_t st) {
  SLA_TRY(ensure_dyn_lds(f32_bwd_key_kernel<D, QW>, f32_bwd_key_lds<D>()));
  {
    KernelTimer kt("bwd_sparse_kv", st);
    f32_bwd_key_kernel<D, QW><<<dim3(s.BH, (kv.ecap + s.T) * QW + (dw.dd / kDwPiece + s.BH - 1) / s.BH), 256, f32_bwd_key_lds<D>(), st>>>(
        (const float*)a.Q, (const float*)a.K, (const float*)a.V, (const float*)a.dO, a.L, Ds, a.col_ptr, a.col_rows,
        a.col_order, dHZcol, s.N, s.T, s.lay(), s.n_h, s.n_0, s.phi, s.scale, (float*)a.dK, (float*)a.dV, dw, kv);
  }
  if (kv.ecap > 0) {
    KernelTimer kt("kv_merge", st);
    f32_kv_merge_kernel<D><<<dim3(s.BH * kv.cuts, 8), 256, 0, st>>>(kv, s.BH, s.N, s.T, s.lay(), (float*)a.dK, (float*)a.dV);
  }
  return hipGetLastError();
}

template <int D>
hipError_t backward_impl(const Shape& s, const BwdArgs& a, float* Ds, float* dHZ, float* dHZcol, float* dWpart,
                         int nparts, const KvSplit& kv, hipStream_t st) {
  const size_t lds_q = 2 * FTile<D>::BYTES + 4 * kBlk;
  SLA_TRY(ensure_dyn_lds(f32_bwd_query_kernel<D>, lds_q));
  {
    KernelTimer kt("bwd_query", st);
    f32_bwd_query_kernel<D><<<s.T * s.BH + kv_plan_wgs(kv, s.BH) + nparts, 256, lds_q, st>>>(
        (const float*)a.Q, (const float*)a.K, (const float*)a.V, (const float*)a.W, (const float*)a.dO,
        (const float*)a.Os, (const float*)a.Ol, a.L, a.HZ, a.row_idx, s.N, s.T, s.lay(), s.n_h, s.n_0, s.phi, s.scale,
        Ds, dHZ, (float*)a.dQ, s.BH, dWpart, nparts, KvPlanArgs{kv, a.col_ptr, a.col_order});
  }
  const DwSum dw{dWpart, nparts, D * D, a.dW, a.dW16};
  if (s.n_0 > 0) SLA_TRY(f32_aggregate(dHZ, a.indT, s, dHZcol, st));
  if (f32_key_quarters(s)) return launch_key<D, 4>(s, a, Ds, dHZcol, dw, kv, st);
  return launch_key<D, 2>(s, a, Ds, dHZcol, dw, kv, st);
}

}  // namespace

hipError_t f32_backward(const Shape& s, const BwdArgs& a, float* Ds, float* dHZ, float* dHZcol, float* dWpart,
                        int nparts, const KvSplit& kv, hipStream_t st) {
  return s.d == 64 ? backward_impl<64>(s, a, Ds, dHZ, dHZcol, dWpart, nparts, kv, st)
                   : backward_impl<128>(s, a, Ds, dHZ, dHZcol, dWpart, nparts, kv, st);
}

hipError_t f32_states(const Shape& s, const FwdArgs& a, const Beside& b, hipStream_t st) {
  return s.d == 64 ? states_impl<64>(s, a, b, st) : states_impl<128>(s, a, b, st);
}

hipError_t f32_forward(const Shape& s, const FwdArgs& a, hipStream_t st) {
  return s.d == 64 ? forward_impl<64>(s, a, st) : forward_impl<128>(s, a, st);
}

}  // namespace sla

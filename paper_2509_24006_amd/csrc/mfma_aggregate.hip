// State aggregation of the linear branch as a dense matrix-core GEMM.
//
// Alg. 1 adds h_j, z_j into H_i, Z_i for every marginal block of row i, and Alg. 2 adds dH_i,
// dZ_i into the sums of key block j for every marginal block of column j.  Over all rows that is
//   out[i][:] = sum_k ind[i][k] in[k][:],   ind = 1 where the block is marginal, else 0,
// a T x T by T x (d*d + d) product per head.  The indicator is exact in bf16, the products are
// bf16 x bf16 with float accumulation.  Compared with adding the marginal blocks one by one
// (or subtracting the others from the total, App. A.3) the state rows are read once per 256
// output rows instead of once per row.
//
// The kernel is bound by HBM traffic (one read of the states, one write of the sums), so the
// design keeps everything else small: the indicator comes as bit masks, 8 bytes per row and
// k-step; the state tiles go global -> LDS directly (row-major, swizzled) through a ring of stages
// and are read with the transposing LDS read; the product is formed with the output rows along the
// lanes, so that the sums leave as whole 128-byte row pieces.  A workgroup of four waves owns 128 or 256
// output rows by 64 columns and four of them share a CU: while one fills its ring or stores its
// sums (a store drains the wave's whole memory queue: loads and stores complete in no fixed order
// relative to each other, so nothing can be waited for selectively behind it), the other computes.
// The workgroups that own the same columns run back to back on one XCD, so that the second read
// of the states comes from its L2.
#include "mfma_common.h"

namespace sla {
namespace {

constexpr int kCols = 64;            // columns of one workgroup
constexpr int kStage = kBlk * 2 * kCols;        // one k-step of states: 64 rows x kCols columns of bf16
constexpr int kStages = 4;           // ring of state tiles
constexpr int kAggLds = kStages * kStage;
constexpr int kColStage = 32 * (2 * kCols + 16);   // store_rows_bf16 area of one wave, laid over the ring
static_assert(4 * kColStage <= kAggLds, "staging of four waves fits in the ring");
constexpr int kOutStage = 32 * (64 * 4 + 16);      // the same for the 128 columns of a short sequence's wave

// two adjacent indicator bits (bits s, s + 1 of x) -> a dword holding two bf16 (1.0 or 0.0)
__device__ __forceinline__ unsigned bits2bf(unsigned x, int s) {
  const unsigned y = (x >> s) & 3u;
  return (((y << 15) | y) & 0x00010001u) * 0x3f80u;
}

// (The main kernel keeps the rows of a stage in the order that makes neighbours of rows 16 apart, stage_row, for
// bits16bf's half the instructions: 40 heads x 1182 blocks, d = 128, 1751 -> 1633 us a launch; 12 x 512 107 us either
// way, there the traffic is the bound.)
// which of a k-step's 64 state rows is row r of the stage
__device__ __forceinline__ int stage_row(int r) { return (r & 32) | ((r >> 1) & 15) | ((r & 1) << 4); }

// Column tile ct covers columns [64 ct, +64) of a state row: below dd the matrix part, written in bf16,
// from there on the vector part (the last d entries), written in float.  A wave owns 32 MT output rows.
// 64 columns and not 128, so that four workgroups share a CU: a workgroup of a few k-steps is mostly
// its first loads and its last stores (128 -> 64 columns: 12 heads x 146 blocks, d = 128, 30.7 -> 24.4 us a
// launch, 12 x 512 112 -> 109, 8 x 1182 even; 64 x 128, d = 64, 30.1 -> 23.8, 8 x 1182 96 -> 92).
// An XCD takes a run of neighbouring column tiles, which share cache lines' neighbours in memory, the runs
// rotated from head to head, as the last is the shortest; the row tiles of a column tile follow
// one another, so that the second read of the states comes from the XCD's L2 (32 x 256, d = 128: 107 -> 102
// us against column tiles dealt one by one).
template <int MT>
__global__ __launch_bounds__(256, 4) void aggregate_mfma_kernel(const bf16* __restrict__ in,
                                                                const unsigned long long* __restrict__ ind,
                                                                int T, int Tw, int row_len, int dd, int mtiles,
                                                                bf16* __restrict__ outH, float* __restrict__ outZ) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, g = l >> 5, ln = l & 31;
  constexpr int NT = kCols / 32, CPR = kCols / 8;   // 32-column tiles, 16-byte chunks of a stage's row
  constexpr int NW = 4;                             // k-steps whose indicator words are held
  const int bh = blockIdx.y, rr = blockIdx.x >> 3, run = gridDim.x / (8 * mtiles);
  const int ct = ((blockIdx.x + bh) & 7) * run + rr / mtiles, mh = rr % mtiles;
  const int nbase = ct * kCols, m0 = mh * 128 * MT;
  if (nbase >= row_len) return;
  const bool zpart = nbase >= dd;
  const unsigned long long* ib = ind + (size_t)bh * T * Tw;
  const bf16* inb = in + (size_t)bh * T * row_len;
  const BufDesc rsrc = tile_rsrc(inb, T * row_len * 2);
  const int pitch = row_len * 2;
  const int wu = wave_uniform(w);
  const unsigned lds0 = lds_base(smem);
  f32x16 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = zero_f32x16();
  const int ksteps = (T + kBlk - 1) / kBlk;
  // one wave-wide load deposits 1 KB, 64 / CPR rows; wave w takes the runs w, w + 4, .. of a stage; rows past T read as zeros (the vector part of a narrow head reads on into
  // the next row: those columns are not written)
  int vo[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    const int row = 64 / CPR * (4 * k + w) + l / CPR, pc = l % CPR;
    vo[k] = stage_row(row) * pitch + nbase * 2 + ((pc ^ swz<kCols>(row)) << 4);
  }
  int iks = 0, istage = 0;   // the next tile to request and its stage
  auto issue_next = [&]() {
    if (iks >= ksteps) return;
#pragma unroll
    for (int k = 0; k < NT; ++k)
      load_to_lds16(rsrc, vo[k], iks * kBlk * pitch, lds0 + istage * kStage + (4 * k + wu) * 1024);
    istage = istage == kStages - 1 ? 0 : istage + 1;
    ++iks;
  };
  // per-lane offsets of the transposing reads inside a stage: [8-row half][column tile]
  TileAddr<kCols> ad;
  ad.init(0, l);
  int tro[2][NT];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) tro[h][nt] = ad.tr(h, nt);
  constexpr int RB = 16 * SwzTile<kCols>::ROW_BYTES;
  const int row0 = m0 + 32 * MT * w + ln;   // this lane's output rows: row0 (and row0 + 32)
#pragma unroll
  for (int k = 0; k < kStages - 1; ++k) issue_next();
  int stage = 0;
  for (int ks0 = 0; ks0 < ksteps; ks0 += NW) {
    // indicator words of the next NW k-steps for the lane's rows
    unsigned long long wb[MT][NW];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        const int i = row0 + 32 * mt;
        wb[mt][q] = (i < T && ks0 + q < Tw) ? ib[(size_t)i * Tw + ks0 + q] : 0ull;
      }
    // (waited for here, once per NW k-steps, rather than at each first use below; the wait
    // also drains the tile loads in flight, which at the start are the ones needed first anyway)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int q = 0; q < NW; ++q) pin_loaded(wb[mt][q]);
#pragma unroll
    for (int q = 0; q < NW; ++q) {
      const int ks = ks0 + q;
      if (ks >= ksteps) break;
      // the lane's bits of this k-step, moved so that those of lane half g sit where those of half 0 do
      unsigned xs[MT][2];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        xs[mt][0] = (unsigned)wb[mt][q] >> (2 * g);
        xs[mt][1] = (unsigned)(wb[mt][q] >> 32) >> (2 * g);
      }
      // the tile has landed; the kStages - 2 tiles requested after it may still be in flight
      if (ks + kStages - 2 < ksteps) wait_vm<NT * (kStages - 2)>();
      else wait_vm0();
      __syncthreads();   // ... for every wave, and the stage of the previous tile is free
      issue_next();
      const int so = stage * kStage;
      stage = stage == kStages - 1 ? 0 : stage + 1;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        // slots 0..3 <- stage rows 16 u + 4 g .. + 3, slots 4..7 <- 16 u + 8 + 4 g .. + 3 (the order in
        // which the transposing read hands over the rows): bits 8 (u & 1) + 2 g + {0, 1, 4, 5}, and the
        // bits 16 above them, of half u >> 1 of the word
        bf16x8 b[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const unsigned x = xs[mt][u >> 1] >> (8 * (u & 1));
          u32x4 packed = {bits16bf<0>(x), bits16bf<1>(x), bits16bf<4>(x), bits16bf<5>(x)};
          b[mt] = *reinterpret_cast<bf16x8*>(&packed);
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf16x8 a = lds_tr<kCols>(smem, tro[0][nt] + so + u * RB, tro[1][nt] + so + u * RB);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = mfma32(a, b[mt], acc[mt][nt]);
        }
      }
    }
  }
  // C tiles: lane = output row, registers = columns 32 nt + c_row(r, g)
  if (zpart) {
    const int dz = row_len - dd;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int row = row0 + 32 * mt;
      if (row >= T) continue;
      float* o = outZ + ((size_t)bh * T + row) * dz;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const int c = nbase - dd + 32 * nt + 8 * r4 + 4 * g;
          if (c < dz)
            *reinterpret_cast<f32x4*>(o + c) = f32x4{acc[mt][nt][4 * r4], acc[mt][nt][4 * r4 + 1],
                                                      acc[mt][nt][4 * r4 + 2], acc[mt][nt][4 * r4 + 3]};
        }
    }
  } else {
    __syncthreads();   // every wave has read the last tile: the ring becomes the staging areas
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int r0 = m0 + 32 * MT * w + 32 * mt;
      if (r0 < T)
        store_rows_bf16<NT>(smem + wu * kColStage, acc[mt], outH + ((size_t)bh * T + r0) * dd + nbase, dd, T - r0, l);
    }
  }
}

// Short sequences (T <= 64: one k-step, one indicator word per row): a workgroup's four waves
// take four column tiles of the same 32 MT output rows, each wave with a stage of its own, so
// that no wave waits for another; the rows of the stage past T are fetched as zeros.  Each wave
// waits for its loads once and stores once, so what hides that is other workgroups: a stage has
// room for 32 MT rows only, which lets four workgroups share a CU up to 32 blocks.  (256 heads of
// 16 blocks, d = 64: 16.2 -> 15.5 us a launch with the gap before it.)
template <int MT>
constexpr int kShortStage = 32 * MT * 256 > kOutStage ? 32 * MT * 256 : kOutStage;
template <int MT>
__global__ __launch_bounds__(256, MT == 1 ? 4 : 2) void aggregate_short_kernel(const bf16* __restrict__ in,
                                                                 const unsigned long long* __restrict__ ind,
                                                                 int T, int row_len, int dd,
                                                                 bf16* __restrict__ outH, float* __restrict__ outZ) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, g = l >> 5, ln = l & 31;
  const int ct = blockIdx.x * 4 + w, bh = blockIdx.y;
  if (ct > dd / 128) return;   // (no barriers in this kernel)
  const bool zpart = ct == dd / 128;
  const int nbase = ct * 128;
  const unsigned long long* ib = ind + (size_t)bh * T;
  const bf16* inb = in + (size_t)bh * T * row_len;
  const BufDesc rsrc = tile_rsrc(inb, T * row_len * 2);
  const int pitch = row_len * 2;
  const int wu = wave_uniform(w);
  unsigned char* stage = smem + wu * kShortStage<MT>;
  const unsigned lds0 = lds_base(smem) + wu * kShortStage<MT>;
  const int nu = (T + 15) / 16;   // 16-row groups that hold valid rows
  for (int k = 0; k < 4 * nu; ++k) {
    const int row = 4 * k + (l >> 4), pc = l & 15;
    load_to_lds16(rsrc, row * pitch + nbase * 2 + ((pc ^ swz<128>(row)) << 4), 0, lds0 + k * 1024);
  }
  unsigned long long wb[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) wb[mt] = (ln + 32 * mt < T) ? ib[ln + 32 * mt] : 0ull;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) pin_loaded(wb[mt]);
  wait_vm0();
  TileAddr<128> ad;
  ad.init(0, l);
  constexpr int RB = 16 * SwzTile<128>::ROW_BYTES;
  f32x16 acc[MT][4];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = zero_f32x16();
  for (int u = 0; u < nu; ++u) {
    bf16x8 b[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const unsigned long long x = wb[mt] >> (4 * g);
      const unsigned half = (unsigned)(x >> (16 * u));   // u < 4: bits 16 u + 4 g ..
      u32x4 packed = {bits2bf(half, 0), bits2bf(half, 2), bits2bf(half, 8), bits2bf(half, 10)};
      b[mt] = *reinterpret_cast<bf16x8*>(&packed);
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      const bf16x8 a = lds_tr<128>(stage, ad.tr(0, nt) + u * RB, ad.tr(1, nt) + u * RB);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = mfma32(a, b[mt], acc[mt][nt]);
    }
  }
  if (zpart) {
    const int dz = row_len - dd;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int row = ln + 32 * mt;
      if (row >= T) continue;
      float* o = outZ + ((size_t)bh * T + row) * dz;
#pragma unroll
      for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const int c = 32 * nt + 8 * r4 + 4 * g;
          if (c < dz)
            *reinterpret_cast<f32x4*>(o + c) = f32x4{acc[mt][nt][4 * r4], acc[mt][nt][4 * r4 + 1],
                                                      acc[mt][nt][4 * r4 + 2], acc[mt][nt][4 * r4 + 3]};
        }
    }
  } else {
    // the wave's own stage becomes its staging area (LDS serves a wave's accesses in order)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (32 * mt < T)
        store_rows_bf16<4>(stage, acc[mt], outH + ((size_t)bh * T + 32 * mt) * dd + nbase, dd, T - 32 * mt, l);
  }
}

}  // namespace

// out[i] = sum over k with bit k of ind[i] set of the bf16 state rows in[k] (d*d + d values each);
// ind is [BH][T][ceil(T/64)] 64-bit masks.  The d x d part goes to outH (bf16 [BH][T][d*d]), the d
// part to outZ (float).
hipError_t mfma_aggregate(const void* in, const unsigned long long* ind, const Shape& s, void* outH,
                          float* outZ, hipStream_t st) {
  const int row_len = s.state_row(), dd = s.d * s.d;
  const int Tw = (s.T + 63) / 64;
  if (dd % 128 != 0 || row_len - dd > 128) return hipErrorInvalidValue;
  const int ntile = dd / 128 + 1;
  if (s.T <= 64) {
    auto kern = s.T <= 32 ? aggregate_short_kernel<1> : aggregate_short_kernel<2>;
    const int lds = 4 * (s.T <= 32 ? kShortStage<1> : kShortStage<2>);
    SLA_TRY(ensure_dyn_lds(kern, lds));
    KernelTimer kt("aggregate", st);
    kern<<<dim3((ntile + 3) / 4, s.BH), 256, lds, st>>>((const bf16*)in, ind, s.T, row_len, dd, (bf16*)outH, outZ);
    return hipGetLastError();
  }
  // Up to 128 rows a wave owns 32 of them and not 64, of which half would be past the end (64 heads x 65
  // blocks, d = 128: 69 -> 58 us a launch, x 100 91 -> 78, x 128 100 -> 97).
  auto kern = s.T <= 128 ? aggregate_mfma_kernel<1> : aggregate_mfma_kernel<2>;
  SLA_TRY(ensure_dyn_lds(kern, kAggLds));
  KernelTimer kt("aggregate", st);
  const int nt = (row_len + kCols - 1) / kCols;
  const int rows = s.T <= 128 ? 128 : 256, mtiles = (s.T + rows - 1) / rows;
  kern<<<dim3(8 * ((nt + 7) / 8) * mtiles, s.BH), 256, kAggLds, st>>>((const bf16*)in, ind, s.T, Tw, row_len, dd, mtiles,
                                                                 (bf16*)outH, outZ);
  return hipGetLastError();
}

}  // namespace sla

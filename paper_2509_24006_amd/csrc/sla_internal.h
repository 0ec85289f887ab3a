// Internal declarations shared by the HIP translation units of the SLA library.
#ifndef SLA_INTERNAL_H_
#define SLA_INTERNAL_H_

#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#define SLA_TRY(x)                      \
  do {                                  \
    hipError_t e_ = (x);                \
    if (e_ != hipSuccess) return e_;    \
  } while (0)

namespace sla {

constexpr int kBlk = 64;  // tile of every kernel: b_kv, and b_q or the unit b_q is a multiple of (Section 6.1)
constexpr int kMaxT = 3072;  // longest sequence in blocks: classification keeps 48 entries of a row per lane

// Where the caller's Q, K, V, O, dO, dQ, dK, dV keep token n of head bh = b H + h: element
// offset head(bh) + n ts.  [B,H,N,d]: ts = d; [B,N,H,d]: ts = H d.  (Everything the library
// itself lays out -- saved tensors, workspaces -- is packed per head with rows d apart.)
struct Lay {
  long long bs, hs;   // elements between batches, between heads of a batch
  int ts, H;          // elements between tokens of a head; heads per batch
  __host__ __device__ size_t head(int bh) const { return (size_t)(bh / H) * bs + (size_t)(bh % H) * hs; }
};

// Shape of one call, derived on the host.
struct Shape {
  int BH, N, d, T, n_h, n_l, n_0;
  int Tq, rq;  // rows of M_c = query blocks of b_q = 64 rq tokens; row r of the 64-token grid has the labels of M_c row r / rq
  int phi;    // 0 softmax over features, 1 elu+1
  int dtype;  // 0 float, 1 bf16
  float scale;  // float 1/sqrt(d)
  Lay layv;     // where the caller's tensors keep their rows
  __host__ __device__ int state_row() const { return d * d + d; }
  Lay lay() const { return layv; }
};

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(__hip_bfloat16 x) { return __bfloat162float(x); }

// ---- mask step (mask_kernels.hip)
// block means of X0 = Q (blocks of 64 rq tokens) and X1 = K (64) -> out0 (float [BH][Tq][d]), out1 (float [BH][T][d])
struct PoolArgs {
  const void *X0, *X1;
  int BH, N, Tn0, len0, Tn1, len1;
  int wgs;   // workgroups per tensor
  Lay lay;
  float *out0, *out1;
};
PoolArgs pool_args(const void* Q, const void* K, const Shape& s, float* qbar, float* kbar);
hipError_t launch_pool(const PoolArgs& a, const Shape& s, hipStream_t st);
hipError_t launch_scores(const float* qbar, const float* kbar, const Shape& s, float* scores,
                         hipStream_t st);
// col_cnt: [BH][T] ints of scratch: cleared by the classification, filled by the table build
hipError_t launch_classify(const float* scores, const Shape& s, int8_t* Mc, int32_t* row_idx,
                           int32_t* col_cnt, hipStream_t st);
hipError_t launch_indicator(const int8_t* Mc, const Shape& s, int32_t* col_cnt, unsigned long long* ind,
                            unsigned long long* indT, hipStream_t st);
struct ColArgs {
  const int8_t* Mc;
  int Tq, rq, T, n_h;
  const int32_t* cnt;            // critical blocks per column
  int32_t *ptr, *order, *rows;
};
hipError_t launch_col_tables(const ColArgs& a, const Shape& s, hipStream_t st);
// What the state kernel's launch does besides the states: nothing, the pooling, or the column tables.
struct Beside {
  const PoolArgs* pool = nullptr;
  const ColArgs* col = nullptr;
};

// T <= 64: with `pool` the block means first (into qbar and kbar); scores (computed from qbar, kbar and written to
// `scores`, or read from `given`), classification and all tables in one launch
hipError_t launch_mask_small(const PoolArgs* pool, const float* qbar, const float* kbar, const float* given,
                             const Shape& s, float* scores, int8_t* Mc, int32_t* row_idx, unsigned long long* ind,
                             unsigned long long* indT, int32_t* col_ptr, int32_t* col_order, int32_t* col_rows,
                             hipStream_t st);

// n floats from p on become 0 (mfma_fwd.hip)
hipError_t launch_fill_zero(float* p, size_t n, hipStream_t st);

// ---- float path (mfma_f32.hip)
struct FwdArgs {
  const void *Q, *K, *V, *W;
  const unsigned long long* ind;   // marginal indicator bit masks
  const int32_t* row_idx;
  void* O;
  void *Os, *Ol;   // may be null (inference)
  float* L;        // may be null
  float* HZ;       // [BH,T] state rows (saved or workspace)
  float* hz;       // [BH,T] state rows of the key blocks (workspace)
};
hipError_t f32_states(const Shape& s, const FwdArgs& a, const Beside& b, hipStream_t st);   // (only with marginal blocks)
hipError_t f32_forward(const Shape& s, const FwdArgs& a, hipStream_t st);                  // what follows the states

struct BwdArgs {
  const void *Q, *K, *V, *W, *dO;
  const unsigned long long* indT;  // marginal indicator bit masks, transposed
  const int32_t *row_idx, *col_ptr, *col_rows, *col_order;
  const void *Os, *Ol;
  const float *L, *HZ;
  void *dQ, *dK, *dV;
  void* dW;    // float, or bf16 with dW16
  bool dW16;
  char* ws;  // workspace, ws_backward_bytes
};
size_t backward_ws_bytes(const Shape& s);   // (backward.hip)
// How the key-side kernel walks the column lists.  A list longer than `piece` entries is summed in pieces of that
// many (the last is shorter), each from zero, and the sums are added in order.
// With ecap > 0 a piece is a unit of work: those behind the first, at most ecap per head, go to workgroups of their
// own, which leave float sums in a slot of `part`, and a second launch adds them up.  Every unit is four ints, written
// by a wave per head of the query-side launch (kv_plan):
//   extra e < ecap             key block, first entry, entries (0: none), slot e
//   ecap + r, r < T            the first piece of the list of rank r: key block, first entry, entries, slot ecap + r
//                              where the list was cut (these are the first ranks), else -1
//   ecap + T + r, r < cuts     a key block that was cut, or zeros: key block, slot of the first extra, extras, 0
// With ecap = 0 (bf16) one workgroup walks all pieces, and the sum so far of the list of rank r waits in slot r.
struct KvSplit {
  int piece, ecap, cuts;   // cuts: at most this many lists of a head are longer than a piece
  int4* units;   // [BH][ecap + T + cuts]
  float* part;   // [BH][ecap + cuts] slots of 2 x 64 x d floats
};
KvSplit kv_split(const Shape& s);   // piece, ecap and cuts (backward.hip)
struct KvPlanArgs {
  KvSplit split;
  const int32_t *col_ptr, *col_order;
};
// The sum of dW's partial d x d sums, done by extra workgroups of the key-side kernel's launch.
struct DwSum {
  const float* part;
  int nparts, dd;
  void* dW;
  bool bf16;
};
// critical-block gradients on the matrix cores (mfma_bwd.hip).  dQlin: linear-branch part of dQ.
// dHZcol: dH and dZ summed over the marginal blocks of each key block (bf16 matrices, then float
// vectors at state_z_offset); the dK/dV kernel turns them into the linear-branch parts of dK and
// dV itself.  Both may be null (no marginal block).
hipError_t mfma_backward_sparse(const Shape& s, const BwdArgs& a, const float* Ds, const void* dHZcol, const DwSum& dw,
                                const KvSplit& kv, hipStream_t st);
// the float path's backward pass; the workspace pieces are carved by backward()
hipError_t f32_backward(const Shape& s, const BwdArgs& a, float* Ds, float* dHZ, float* dHZcol, float* dWpart,
                        int nparts, const KvSplit& kv, hipStream_t st);
bool f32_key_quarters(const Shape& s);   // whether a workgroup of its key side owns a quarter of a key block, or half of one (backward.hip)
hipError_t backward(const Shape& s, const BwdArgs& a, hipStream_t st);

// ---- bf16 matrix-core path (mfma_fwd.hip)
size_t mfma_forward_ws_bytes(const Shape& s);
hipError_t mfma_states(const Shape& s, const FwdArgs& a, char* ws, const Beside& b, hipStream_t st);
hipError_t mfma_forward(const Shape& s, const FwdArgs& a, char* ws, hipStream_t st);
// out[i] = sum over k with bit k of ind[i] set of the bf16 state rows in[k] (mfma_aggregate.hip)
hipError_t mfma_aggregate(const void* in, const unsigned long long* ind, const Shape& s, void* outH, float* outZ,
                          hipStream_t st);
// bf16 tensors keep the aggregated states as a bf16 block [BH][T][d*d] (matrices, transposed)
// followed by a float block [BH][T][d] (vectors); this is the byte offset of the second block.
inline size_t state_z_offset(const Shape& s) { return ((size_t)s.BH * s.T * s.d * s.d * 2 + 255) / 256 * 256; }

// the same sums by additions (method 1), pre-aggregation (2) or Four Russians tables (3), for
// comparison (aggregate_alt.hip)
size_t aggregate_alt_ws_bytes(const Shape& s, int method);
hipError_t aggregate_alt(int method, const void* in, const unsigned long long* ind, const Shape& s, void* outH,
                         float* outZ, void* ws, hipStream_t st);

// query side on the matrix cores (mfma_bwd_query.hip): D^s, dH_i / dZ_i rows (dHZ16), dQ.  dQlin:
// scratch for the linear part of dQ (only used with query blocks of two or four tiles).
// dWpart: nparts partial sums of dW = sum O^l^T dO.
hipError_t mfma_backward_query(const Shape& s, const BwdArgs& a, float* Ds, void* dHZ16, float* dQlin, float* dWpart,
                               int nparts, const KvSplit& kv, hipStream_t st);

// Brackets one kernel launch with events when profiling is on (profile.hip).
class KernelTimer {
 public:
  KernelTimer(const char* name, hipStream_t st);
  ~KernelTimer();
 private:
  hipStream_t st_;
  long idx_;
};

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// Raises the dynamic-LDS limit of a kernel to `bytes`, once per kernel and device (profile.hip);
// every later call is a table lookup on the host.
hipError_t ensure_dyn_lds(const void* kernel, int bytes);
template <typename K>
hipError_t ensure_dyn_lds(K kernel, size_t bytes) {
  return ensure_dyn_lds(reinterpret_cast<const void*>(kernel), (int)bytes);
}

// Whether query blocks of an even number of tiles run the eight-wave kernels (sla_wide_query_tiles;
// profile.hip holds the flag).
bool wide_query_tiles();

}  // namespace sla
#endif

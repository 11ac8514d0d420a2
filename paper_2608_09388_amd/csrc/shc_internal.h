// Internal declarations shared by the HIP translation units of libshc.so.
// Nothing here is part of the public ABI (include/shc.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace shc {

// ---------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) {
  return __uint_as_float(h << 16);
}

// fp32 -> bf16 bits, round to nearest, ties to even; NaN -> quiet NaN.
// Adding 0x7FFF plus the lowest kept bit to the fp32 pattern carries into the
// kept part exactly when the dropped half is above one half ulp, or equal to
// it with an odd kept part.
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u | ((u >> 16) & 0x8000u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}

template <typename T>
__device__ __forceinline__ T ceil_div(T a, T b) {
  return (a + b - 1) / b;
}

// Tile of workgroup b of n.  Workgroups are dealt to the eight XCDs in turn
// (b runs on XCD b % 8); each XCD takes a contiguous range of tiles, so that
// rows that neighbouring tiles both read stay in its L2.
__device__ __forceinline__ int xcd_tile(int b, int n) {
  const int x = b & 7, q = n >> 3, r = n & 7;
  return x * q + (x < r ? x : r) + (b >> 3);
}

// Rows of a workgroup sorted by their first sparse slot (a slot present in fewer
// than half of the rows), so that rows sharing it share 16-row blocks and a
// block's slot is more often present in none of its rows: a counting sort over
// buckets 0 (dense slots only), 1 + j (first sparse slot j), K + 1 (past the
// last row).  LDS: srcs_in [K][R] by row and cnt [K] (rows present per slot) are
// read behind a barrier, hist [K + 2] is zero; srcs [K][R] by position and perm
// [R] (position -> row) are written, placed(position, the row's slots) called
// for every row.  The order inside a bucket is whatever the atomics give, which
// no result may depend on.
template <int R, int NT, typename Placed>
__device__ __forceinline__ void sort_by_first_slot(int K, int nrows, const int32_t* srcs_in,
                                                   const int32_t* cnt, int32_t* hist,
                                                   int32_t* srcs, int32_t* perm, Placed&& placed) {
  constexpr int RPT = (R + NT - 1) / NT;  // rows per thread
  const int tid = threadIdx.x, lane = tid & 63;
  int bkt[RPT];
  uint32_t rm[RPT];
  uint32_t dense = 0;
  for (int j = 0; j < K; ++j) dense |= (2 * cnt[j] >= nrows ? 1u : 0u) << j;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int t = tid + i * NT;
    rm[i] = 0;
    bkt[i] = -1;
    if (t < R) {
      for (int j = 0; j < K; ++j) rm[i] |= (srcs_in[j * R + t] >= 0 ? 1u : 0u) << j;
      const uint32_t key = rm[i] & ~dense;
      bkt[i] = t >= nrows ? K + 1 : (key ? 1 + __builtin_ctz(key) : 0);
      atomicAdd(&hist[bkt[i]], 1);
    }
  }
  __syncthreads();
  if (tid < 64) {  // exclusive scan of the K + 2 <= 34 counts, one per lane
    const int c = lane < K + 2 ? hist[lane] : 0;
    int inc = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(inc, d, 64);
      if (lane >= d) inc += y;
    }
    if (lane < K + 2) hist[lane] = inc - c;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int t = tid + i * NT;
    if (t < R) {
      const int pos = atomicAdd(&hist[bkt[i]], 1);
      perm[pos] = t;
      for (int j = 0; j < K; ++j) srcs[j * R + pos] = srcs_in[j * R + t];
      placed(pos, rm[i]);
    }
  }
}

// ---------------------------------------------------------------------------
// launchers (host side, enqueue only; arguments already validated)
// ---------------------------------------------------------------------------

// the calling thread's last-error message (shc_last_error), for entry points
// defined outside the file that owns it; set_error returns `code`
int set_error(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

// compaction: number of blocks and per-block element span for a mask of `total` entries
void compact_plan(int64_t total, int32_t* nblocks, int64_t* per_block);

hipError_t launch_compact(const uint8_t* mask, int32_t B, int32_t V, int32_t* coords, int32_t* inv,
                          int32_t* row_ptr, int32_t* n_active, int64_t* n_host, int64_t cap,
                          int32_t* block_counts, hipStream_t stream);

// the same over a table [K][n] of rows, entry active when >= 0: pairs (slot,
// row) in order, pair_ptr [K + 1]
hipError_t launch_compact_present(const int32_t* table, int32_t K, int32_t n, int32_t* pairs,
                                  int32_t* pair_ptr, int32_t* count, int32_t* block_counts,
                                  hipStream_t stream);

// compaction that also writes the neighbour-row table of the active set
// (table[j * N' + i], as launch_neighbor_table), one block per body: the body's
// row numbering lives in LDS, 8 bytes per vertex
constexpr int32_t kCompactTableMaxV = 19456;
bool compact_table_supported(int32_t V, int32_t K);
hipError_t launch_compact_table(const uint8_t* mask, int32_t B, int32_t V, int32_t* coords,
                                int32_t* inv, int32_t* row_ptr, int32_t* n_active,
                                int64_t* n_host, int64_t cap, const int32_t* nbr, int32_t K,
                                int32_t* table, int32_t* block_counts, hipStream_t stream);

hipError_t launch_gather(const void* x, const int32_t* coords, int64_t n_rows, int32_t B,
                         int32_t V, int32_t row_bytes, void* S, hipStream_t stream);

int group_norm_split(int32_t B, int32_t C, int32_t G, int is_bf16, int num_cus);
hipError_t launch_group_norm(const void* S, const int32_t* row_ptr, int64_t n_rows, int32_t B,
                             int32_t C, int32_t G, float eps, int is_bf16, void* out,
                             int num_cus, hipStream_t stream);
// mask scores (scores.hip)
constexpr int kMaxScoreMasks = 64;
void mask_scores_plan(int32_t K, int64_t N, int32_t C, int* tile, int* tiles, int* splits,
                      int64_t* rows_per_split, int* chunks);
size_t mask_scores_workspace_bytes(int32_t K, int64_t N, int32_t C);
hipError_t launch_mask_scores(const void* O, int32_t K, int64_t N, int32_t C,
                              const double* alpha_in, double* alpha_out, double* sim,
                              int32_t kappa, int32_t* top, void* ws, hipStream_t stream);
// backward of the linear and conv layers (backward.hip)
constexpr int kMaxVirtualSlots = 64;
struct BwdPlan {
  int T, tiles, L, splits;
  int64_t max_chunks, rps;
  size_t off_dz, off_colpart, off_pairs, off_rowptr, off_mask, off_part, total;
};
void backward_plan(int64_t n, int32_t K, int32_t Cin, int32_t Cout, int is_bf16, int conv,
                   BwdPlan* p);
int backward_dgrad_supported(int32_t Kw, int32_t Cin, int32_t Cout, int is_bf16);
size_t transpose_neighbors_ws_bytes(int32_t V, int32_t K);
hipError_t launch_transpose_neighbors(const int32_t* nbr, int32_t V, int32_t K, int32_t* nbr_t,
                                      int32_t* slot_of, int32_t* off_dev, void* ws,
                                      hipStream_t stream);
hipError_t launch_transposed_table(const int32_t* coords, const int32_t* inv, int64_t n, int32_t B,
                                   int32_t V, const int32_t* nbr_t, int32_t Kt, int32_t* table_t,
                                   uint64_t* row_slots, hipStream_t stream);
hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t stream);
size_t slot_pairs_ws_bytes(int64_t n, int32_t K);
hipError_t launch_slot_pairs(const int32_t* table, int64_t n, int32_t K, int32_t* pairs,
                             int32_t* pair_ptr, void* ws, hipStream_t stream);
hipError_t launch_layer_backward(int conv, const void* S, const int32_t* table,
                                 const int32_t* pairs, const int32_t* pair_ptr,
                                 const int32_t* table_t, const uint64_t* row_slots,
                                 const int32_t* slot_of, const void* W, const void* Y,
                                 const void* dY, int64_t n, int32_t K, int32_t Cin, int32_t Cout,
                                 int is_bf16, int act, void* dS, float* dW, float* db, void* ws,
                                 hipStream_t stream);
hipError_t launch_clear_inactive(const int32_t* inv, int32_t B, int32_t V, int32_t row_bytes,
                                 void* D, hipStream_t stream);
hipError_t launch_scatter_update(const void* S, const int32_t* inv, const int32_t* coords,
                                 int64_t n_rows, const int32_t* prev_coords, int64_t prev_rows,
                                 int32_t B, int32_t V, int32_t row_bytes, void* D,
                                 hipStream_t stream);
hipError_t launch_gather_ext(const void* x, const uint8_t* me, int mask_mode,
                             const int32_t* coords, int64_t n_rows, int32_t B, int32_t Bx,
                             int32_t V, int32_t row_bytes, void* S, hipStream_t stream);
hipError_t launch_combine(const void* Y, int32_t kappa, int64_t rows, int32_t row_bytes, int op,
                          int is_bf16, void* out, hipStream_t stream);
hipError_t launch_row_activity(const uint8_t* me, int32_t B, int32_t V, int32_t C, uint8_t* m,
                               hipStream_t stream);
hipError_t launch_scatter(const void* S, const int32_t* inv, const int32_t* coords,
                          int64_t n_rows, int32_t B, int32_t V, int32_t row_bytes, int zero_fill,
                          void* D, hipStream_t stream);

hipError_t launch_segment_max(const void* S, const int32_t* row_ptr, int64_t n_rows, int32_t B,
                              int32_t C, int is_bf16, float empty_value, void* P,
                              hipStream_t stream);

// neighbour-row table of the active set: table[j * n_rows + i] = row of slot j's
// neighbour of active row i, or -1
hipError_t launch_neighbor_table(const int32_t* coords, const int32_t* inv, int64_t n_rows,
                                 int32_t B, int32_t V, const int32_t* nbr, int32_t K,
                                 int32_t* table, hipStream_t stream);

struct GemmArgs {
  const void* S;        // [n_rows][Cin]
  const int32_t* coords;  // conv only
  const int32_t* inv;     // conv only
  const int32_t* nbr;     // conv only, [V][K]
  const int32_t* table;   // conv from a neighbour-row table, [K][n_rows]; else null
  const void* W;        // [K][Cin][Cout] (linear: K = 1)
  const float* bias;    // [Cout] or null
  void* out;            // [n_rows][Cout]
  int64_t n_rows;
  int32_t B, V, K, Cin, Cout;
  int32_t relu;
  int32_t gather;       // linear only: input row i is S[coords b_i * V + v_i] (S = dense x)
  uint32_t cin_magic;   // ceil(2^32 / Cin), filled in by the launcher
  // conv from a table, weight-stationary kernel only: write the active set's
  // plan (index lists, sort, job lists per row group) to plan_out instead of
  // computing, or read it from plan; images plan_stride bytes apart
  void* plan_out;
  const void* plan;
  int64_t plan_stride;
};

hipError_t launch_gather_gemm(const GemmArgs& a, bool conv, bool bf16, hipStream_t stream);

// weight-stationary variant (conv_ws.hip): LDS plan, all sizes in bytes
struct WsPlan {
  int ws;         // output-column slice width held in LDS
  int wrow;       // padded LDS row of the weight slice
  int wbytes;     // weight slice
  int rows;       // active rows per workgroup (multiple of 16)
  int idx_bytes;  // index lists
  int scratch;    // epilogue staging (all waves)
  int total;
};
bool ws_plan(const GemmArgs& a, bool conv, bool bf16, int num_cus, WsPlan* plan);
// Bytes of the plan of a conv from a table with this shape (0: the shape
// takes no plan), and the distance between two row groups' images.
int64_t conv_plan_bytes(const GemmArgs& a, bool bf16, int num_cus, int64_t* stride);
// The largest row count whose conv takes a plan (0: none), and the largest
// plan of any row count up to a.n_rows.
int64_t conv_plan_max_rows(const GemmArgs& a, bool bf16, int num_cus);
int64_t conv_plan_bytes_upto(const GemmArgs& a, bool bf16, int num_cus);
hipError_t launch_ws_gemm(const GemmArgs& a, bool conv, bool bf16, const WsPlan& plan,
                          hipStream_t stream);
// the kernel of a conv or linear layer (gemm.hip)
enum class GemmKernel { kSlotMajor, kWalk, kWalkSplit, kWeightStationary, kTiled };
GemmKernel gemm_kernel_of(const GemmArgs& a, bool conv, bool bf16, int cus, WsPlan* plan);
// slot-walking conv for any shape whose buffers stay below 2 GiB
// (conv_walk.hip), and whether its smallest workgroups (16 rows x 64 columns)
// all run at once, or its middle ones (128 x 32) at per_cu to a CU
bool conv_walk_supported(const GemmArgs& a, bool bf16);
bool conv_walk_small(const GemmArgs& a, int num_cus);
bool conv_walk_medium(const GemmArgs& a, int num_cus, int per_cu);
// split: fp32 products of large shapes from six bf16 ones (not the other
// kernels' bits; the error against 64 bits is below theirs)
hipError_t launch_conv_walk(const GemmArgs& a, bool bf16, bool split, int num_cus,
                            hipStream_t stream);
// slot-major conv from a neighbour-row table (conv_sm.hip): bf16, C_in and
// C_out in {64, 128}, K <= 32, no plan
bool conv_sm_supported(const GemmArgs& a, bool bf16);
bool conv_sm_two(const GemmArgs& a);  // its workgroups fit two to a CU
hipError_t launch_conv_sm(const GemmArgs& a, int num_cus, hipStream_t stream);
// conv from a neighbour-row table with slot 0 and the other slots apart
// (conv_split.hip): bf16, C_in and C_out in {64, 128, 256}, K <= 32; the
// other slots' partial rows go through an fp32 workspace of
// conv_split_workspace_bytes bytes
int64_t conv_split_workspace_bytes(int64_t n_rows, int32_t K, int32_t Cout);
bool conv_split_supported(int64_t n_rows, int32_t K, int32_t Cin, int32_t Cout);
hipError_t launch_conv_split(const void* S, const int32_t* table, int64_t n_rows, int32_t K,
                             const void* W, const float* bias, int32_t Cin, int32_t Cout,
                             int32_t relu, void* out, float* workspace, int num_cus,
                             hipStream_t stream);

// conv from a neighbour-row table with every slot's weights in registers
// (conv_packed.hip): bf16, C_in and C_out in {64, 128}, K <= 9, weights
// pre-arranged by launch_pack_conv_weights into conv_packed_weights_bytes
bool conv_packed_supported(int64_t n_rows, int32_t K, int32_t Cin, int32_t Cout);
int64_t conv_packed_weights_bytes(int32_t K, int32_t Cin, int32_t Cout);
hipError_t launch_pack_conv_weights(const void* W, int32_t K, int32_t Cin, int32_t Cout,
                                    void* Wp, hipStream_t stream);
hipError_t launch_conv_packed(const void* S, const int32_t* table, int64_t n_rows, int32_t K,
                              const void* Wp, const float* bias, int32_t Cin, int32_t Cout,
                              int32_t relu, void* out, int num_cus, hipStream_t stream);
// its plan: the rows' grouping and slot entries of every chunk, built once per
// active set (launch_build_packed_plan) and read by every packed layer of the
// shape (launch_conv_packed_planned)
int64_t conv_packed_plan_bytes(int64_t n_rows, int32_t Cin, int32_t Cout, int num_cus);
int64_t conv_packed_plan_bytes_upto(int64_t n_rows, int32_t Cin, int32_t Cout, int num_cus);
hipError_t launch_build_packed_plan(const int32_t* table, int64_t n_rows, int32_t K, int32_t Cin,
                                    int32_t Cout, void* plan, int num_cus, hipStream_t stream);
hipError_t launch_conv_packed_planned(const void* S, const void* plan, int64_t n_rows, int32_t K,
                                      const void* Wp, const float* bias, int32_t Cin,
                                      int32_t Cout, int32_t relu, void* out, int num_cus,
                                      hipStream_t stream);

}  // namespace shc

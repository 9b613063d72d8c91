// Internal declarations shared by the HIP translation units of libdci (gfx950 only).
#ifndef DCI_INTERNAL_H_
#define DCI_INTERNAL_H_

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "dci.h"

constexpr int kPresampleRun = 16;  // batches that dci_presample_count times between two waits for the GPU

struct dci_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  char* static_scratch = nullptr;  // this GPU's copy of the library's static scratch array (DCI_STATIC_SCRATCH_BYTES)
  int num_cus = 256;
  hipEvent_t ev[2 * kPresampleRun + 1] = {nullptr};  // dci_presample_count's stage times; it makes those beyond the first three
  char err[512] = {0};
  // optional per-kernel-class timing
  uint32_t timing_mask = 0;
  hipEvent_t* t_events = nullptr;  // 2 * DCI_TIMING_MAX_LAUNCHES, created on first enable
  int8_t* t_class = nullptr;
  int t_used = 0;
  unsigned* host_flag = nullptr;  // pinned host word (64 bytes): a kernel raises it when a batch had to be voided
  unsigned long long* host_scal = nullptr;  // eight pinned words behind it: what dci_fill_caches reads back
  unsigned relabel_spin_limit = 1u << 24;  // DCI_OPT_RELABEL_SPIN_LIMIT
  unsigned test_first_ticket = 0;          // DCI_OPT_TEST_RELABEL_FIRST_TICKET
  // what the last call that returned DCI_ERR_CAPACITY needed (dci_last_required)
  int64_t req_nodes[DCI_MAX_HOPS + 1] = {0};
  int64_t req_edges[DCI_MAX_HOPS] = {0};
  size_t req_workspace = 0;
  int relabel_tile_iters = 0;  // DCI_OPT_RELABEL_TILE_ITERS: 0 = by frontier size (1, 2, 4 or 8), else 2, 4 or 8 rows per lane group
  int input_layer = 0;    // DCI_OPT_INPUT_LAYER: 0 by shape, 1 aggregation and dense layer as two kernels, 2 / 3 one kernel where the shape allows (weights in registers / 64-row tiles)
  int fused_input = 0;    // DCI_OPT_FUSED_INPUT: dci_infer_batches lets the first layer read cached rows in place
  int linear_split = 0;   // DCI_OPT_LINEAR_SPLIT: 0 = by shape, n = at most n workgroups per tile
  int linear_kernel = 0;  // DCI_OPT_LINEAR_KERNEL: 0 by shape, 1 tile kernel, 2 wide kernel where the shape allows
};

namespace dci {

constexpr int kWave = 64;
constexpr size_t kAlign = 256;

// The frontier scan numbers the tiles of a hop by tickets, so that a tile waits only for workgroups that are running already.  A hop of few
// tiles numbers them by workgroup instead, which spares it the ticket (1 us); every tile that another one waits for must then get to run
// whatever the others do.  Only workgroups that wait could keep it from that (all others end by themselves), so they must leave it a
// place.  A compute unit has kRelabelPerCu places; kScansAtOnce scans may be on the card, or on the part of it that the process sees, at a
// time, those of other processes among them (16 processes with four hardware queues each).  That makes 16 tiles with 256 compute units, 2 with
// 32 of them.
constexpr int kRelabelPerCu = 4, kScansAtOnce = 64;
constexpr unsigned unticketed_tiles(int num_cus) { return (unsigned)(num_cus * kRelabelPerCu / kScansAtOnce); }

inline int32_t fail(dci_ctx* ctx, int32_t code, const char* fmt, ...) {
  if (ctx) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(ctx->err, sizeof(ctx->err), fmt, ap);
    va_end(ap);
  }
  return code;
}

#define DCI_HIP(ctx, call)                                                                          \
  do {                                                                                              \
    hipError_t e_ = (call);                                                                         \
    if (e_ != hipSuccess)                                                                           \
      return dci::fail((ctx), DCI_ERR_HIP, "%s failed: %s (%s:%d)", #call, hipGetErrorString(e_),   \
                       __FILE__, __LINE__);                                                         \
  } while (0)

#define DCI_LAUNCH_CHECK(ctx)                                                                       \
  do {                                                                                              \
    hipError_t e_ = hipGetLastError();                                                              \
    if (e_ != hipSuccess)                                                                           \
      return dci::fail((ctx), DCI_ERR_HIP, "kernel launch failed: %s (%s:%d)", hipGetErrorString(e_), \
                       __FILE__, __LINE__);                                                         \
  } while (0)

// Brackets the launches issued during its lifetime with a pair of events when the class is timed.
struct Timed {
  dci_ctx* ctx;
  int idx = -1;
  Timed(dci_ctx* c, int cls) : ctx(c) {
    if ((c->timing_mask >> cls) & 1u) {
      if (c->t_used < DCI_TIMING_MAX_LAUNCHES) {
        idx = c->t_used++;
        c->t_class[idx] = (int8_t)cls;
        (void)hipEventRecord(c->t_events[2 * idx], c->stream);
      }
    }
  }
  ~Timed() {
    if (idx >= 0) (void)hipEventRecord(ctx->t_events[2 * idx + 1], ctx->stream);
  }
};

inline size_t align_up(size_t x, size_t a = kAlign) { return (x + a - 1) / a * a; }

// Bump allocator over the context's workspace.  Every call carves its temporaries from the
// start: calls on one context are ordered on one stream, so they never hold it at the same time.
struct Arena {
  char* base;
  size_t cap;
  size_t off = 0;
  Arena(char* b, size_t c) : base(b), cap(c) {}
  template <class T>
  T* take(size_t n) {
    size_t bytes = align_up(n * sizeof(T));
    T* p = reinterpret_cast<T*>(base + off);
    off += bytes;
    return p;
  }
  bool ok() const { return off <= cap && (base != nullptr || off == 0); }
};

inline uint64_t next_pow2(uint64_t x) {
  uint64_t p = 1;
  while (p < x) p <<= 1;
  return p;
}

// -- device helpers -----------------------------------------------------------------------

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

__device__ __forceinline__ long long wave_incl_scan64(long long x) {
  const int lane = lane_id();
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    long long y = __shfl_up(x, d, kWave);
    if (lane >= d) x += y;
  }
  return x;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long x) {
#pragma unroll
  for (int d = kWave / 2; d >= 1; d >>= 1) x += __shfl_down(x, d, kWave);
  return x;  // valid in lane 0
}

// Fills `bytes` (a multiple of 16) at a 16-byte aligned address with the 32-bit pattern.
__global__ void k_fill_u32x4(uint4* __restrict__ p, size_t n16, uint32_t pattern);

int32_t fill_bytes(dci_ctx* ctx, void* p, size_t bytes, uint32_t pattern);
// After a wait on the context's stream: reports (and clears) a failure that a kernel flagged.
int32_t check_device_flag(dci_ctx* ctx);
// What the closing workgroups of a batch do (close_batch)
struct CloseArgs {
  long long* counts;
  int hop, fanout;  // of the last hop
  const int* tmp_slot;
  const long long* blk_indptr;
  const void* table;
  unsigned shift;
  int* blk_src;
  long long* counts_host;
  const unsigned* batch_flag;
  unsigned* host_flag;
  bool direct;
  int wgs = 0;
};
constexpr int kCloseBesidePerCu = 2;  // closing workgroups of another launch, at most, per compute unit
// dci_sample_khop with its temporaries at ws_base; close (nullable): what is left to do for the batch, instead of the closing kernel
int32_t sample_khop_in(dci_ctx* ctx, const dci_graph* graph, const dci_cache* cache, const int64_t* seeds, int64_t n_seeds,
                       uint64_t batch_index, const int32_t* fanouts, int32_t n_hops, uint64_t rng_seed, dci_blocks* out, uint64_t* stats,
                       char* ws_base, size_t ws_bytes, const char* ws_name, CloseArgs* close);
// A whole batch of dci_infer_batches without statistics, closed beside the gather.  *done = false and nothing done where the workspace
// does not hold the sampler's temporaries beside those of the other stages, where an argument is wrong (the calls in
// sequence then say what is), or where it would not be quicker.
int32_t infer_joint(dci_ctx* ctx, const dci_graph* graph, const dci_cache* cache, const int64_t* seeds, int64_t n_seeds,
                    uint64_t batch_index, const int32_t* fanouts, int32_t n_hops, uint64_t rng_seed, dci_blocks* blocks, float* x,
                    const int32_t* dims, int32_t model, const float* const* w_self, const float* const* w_neigh,
                    const float* const* bias, float* logits, bool in_place, bool* done);
// partials_buf: gather_partials_bytes(ctx) bytes of device scratch, needed when stats != NULL
// rowref / n_dense_dev: nullptr for the plain gather; otherwise the selective form (see k_gather_select),
// n_dense_max bounding *n_dense_dev
// add_partials / fold_partials (plain gather only): several launches of one n_max that are folded into stats once - the
// first starts the partial sums, later ones add to them, the last folds them
// split (nullable): weights to be laid out as parts by workgroups of their own in the same launch
// close (nullable): a batch to be closed by workgroups of the same launch
struct SplitArgs;
int32_t gather_launch(dci_ctx* ctx, const dci_graph* g, const dci_cache* cache, const int64_t* ids,
                      int64_t n_max, const int64_t* n_dev, float* out, uint64_t* stats, void* partials_buf,
                      int32_t* rowref, const int64_t* n_dense_dev, int64_t n_dense_max, bool add_partials = false,
                      bool fold_partials = true, const SplitArgs* split = nullptr, const CloseArgs* close = nullptr);
size_t gather_partials_bytes(const dci_ctx* ctx);
// dci_gather_features' checks
int32_t check_gather(dci_ctx* ctx, const dci_graph* graph, const dci_cache* cache, const int64_t* node_ids, int64_t n_max, const float* out);
// dci_gather_features of a whole batch and dci_gnn_forward on its rows, in one call
int32_t gather_all_forward(dci_ctx* ctx, const dci_graph* graph, const dci_cache* cache, const dci_blocks* blocks, float* x,
                           int32_t n_layers, const int32_t* dims, int32_t model, const float* const* w_self,
                           const float* const* w_neigh, const float* const* bias, float* logits);

// One layer of the forward pass in one kernel (dci_layer.hip)
struct LayerArgs {
  const long long* counts;  // rows = counts[hop]
  int hop;
  const long long* blk_indptr;
  const int* blk_src;
  const float* x;      // [*, D] rows of the layer's input
  const int* rowref;   // not nullptr: the row of source s is cache[rowref[s]] where that is not negative, else x[s]
  const float* cache;
  const float* w_self;   // [D, N] row-major (not read for GCN)
  const float* w_neigh;  // [D, N]
  const float* bias;     // [N]
  float* y;              // [rows, N]
  int D, N, relu;
  int mode;  // DCI_MODEL_*
  int n_col_groups;
  long long cap_rows;     // bound on the rows
  const void* w_split;    // the weights as parts (k_sage_layer)
};
struct LayerPlan {
  int D, N, C;  // C: -1 not one of these kernels, 0 k_sage_layer_small, else k_sage_layer with 16 C columns per wavefront
  int64_t cap_rows;
  void* w_split;
  int cols, rs;  // k_sage_layer: multiplying wavefronts side by side, and how many of them share columns (each takes a part of the rows)
};
// Plans every layer of a forward pass; scratch is where the weights' parts may
// go.  false: none of the layers is for these kernels, because an input is too narrow or the scratch too small.
bool layers_plan(const dci_ctx* ctx, const dci_blocks* blocks, int32_t model, const int32_t* dims, void* scratch,
                 size_t scratch_bytes, LayerPlan* plans);
// The parts to lay out for the layers from `first` on
SplitArgs layers_split_args(int32_t model, int32_t first, int32_t n_layers, const LayerPlan* plans, const float* const* w_self,
                            const float* const* w_neigh);
int32_t layers_split_weights(dci_ctx* ctx, const SplitArgs& args);
int32_t layer_launch(dci_ctx* ctx, const LayerPlan& plan, const LayerArgs& args);

}  // namespace dci

#endif  // DCI_INTERNAL_H_

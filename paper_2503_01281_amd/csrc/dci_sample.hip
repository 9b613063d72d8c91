// Cache-aware multi-hop neighbour sampling, mini-batch block construction and pre-sampling
// access counting (Section II-C; Section IV; Section IV-B, first and third paragraphs).
//
// One batch is one clear of the batch's node table, two kernels per hop and one closing kernel (the clear and the first hops of small batches
// are one kernel, k_first_hops):
//   k_sample_hop  - one lane group per frontier node (a whole wavefront for fan-outs above 32, a
//                   half / quarter / eighth for smaller ones): read the node's list bounds from the
//                   adjacency cache or the host CSR (a position is served by the cache iff it lies
//                   below the node's cached length, which is the whole list for every node but the
//                   one an element-granular fill may have cached in part), draw the positions (Floyd's subset algorithm
//                   on Philox4x32-10, one lane per slot), read the neighbour ids, store them at the
//                   padded position row*fanout + slot and register every id in the node table with
//                   an atomic minimum over that padded position.  A row's list bounds are noted for the
//                   batch's later hops, which sample the same row again and then need neither the slot
//                   look-up nor - for a miss - a second trip over the host link.  At hop 0 the same kernel turns
//                   the seeds into F_0; at later hops its first workgroups write the previous
//                   hop's edge ids, whose inputs are final by then.
//   k_relabel_hop - a lane is the "first appearance" of its node iff the table still holds its own
//                   padded position.  Counts them per row, prefix-sums edge counts and first
//                   appearances over all rows (chained scan with decoupled look-back), appends the
//                   first appearances to the frontier in (row, slot) order, publishes their
//                   local ids in the table and writes them as those edges' ids.
//   k_write_src   - the last hop's remaining edge ids, the batch sizes for the host, in pre-sampling the visits of the
//                   input nodes, and the totals of the batch's statistics.
// Should a tile of the scan ever give up waiting for its predecessors, the batch is voided: a status
// word makes the batch's remaining kernels return at once, k_write_src zeroes the batch's sizes and
// raises the context's host flag, and the next dci_sync reports it.
// A node's value in the table is either a final local id (below 2^31) or 2^31 + the smallest padded
// position seen so far, so one atomic minimum serves both "already in the frontier" and "who came first".
// The table is hashed (a 64-bit word per entry, node id in the high half, value in the low half) or direct
// (a 32-bit value per node of the graph): see table_is_direct.
#include "dci_close.h"

namespace dci {

constexpr unsigned int kTentative = 0x80000000u;
constexpr HashEntry kEmptyEntry = ~0ull;
constexpr int kBlock = 256;
// row_cnt[i]: bits 0..7 sampled edges of row i; bits 8..15 how many of them were read from the host although
// the node has a cache slot (only the node cached in part has any); bits 16..22 the distinct 128-byte lines
// of graph->indices the row read, bits 23..24 those of graph->indptr (both only counted when statistics are
// on); bit 30 set if the node has a slot
constexpr int kRowHitBit = 1 << 30;
constexpr int kRowCntMask = 0xFF;
constexpr int kRowHostShift = 8;
constexpr int kRowLinesShift = 16;
constexpr int kRowLinesMask = 0x7F;
constexpr int kRowBoundLinesShift = 23;
constexpr int kRowBoundLinesMask = 0x3;
constexpr int kHostLineLog2 = 7;  // the host link moves 128-byte lines: smaller reads cost a whole request each
template <bool DIRECT>
__device__ __forceinline__ void entry_set_val(HashEntry* table, unsigned shift, unsigned slot, unsigned v) {
  reinterpret_cast<unsigned*>(table)[(size_t)slot << (DIRECT ? shift : 1u)] = v;
}

// ---- Philox4x32-10 (Salmon et al., SC'11), counter-based ---------------------------------
__device__ __forceinline__ unsigned long long philox_u64(unsigned c0, unsigned c1, unsigned c2, unsigned c3,
                                                         unsigned k0, unsigned k1) {
  constexpr unsigned M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const unsigned h0 = __umulhi(M0, c0), l0 = M0 * c0;
    const unsigned h1 = __umulhi(M1, c2), l1 = M1 * c2;
    c0 = h1 ^ c1 ^ k0;
    c1 = l1;
    c2 = h0 ^ c3 ^ k1;
    c3 = l0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return (unsigned long long)c0 | ((unsigned long long)c1 << 32);
}

__device__ __forceinline__ unsigned long long uniform_below(unsigned k0, unsigned k1, long long node, unsigned batch,
                                                            int hop, int slot, unsigned long long m) {
  const unsigned long long u = philox_u64((unsigned)(unsigned long long)node,
                                          (unsigned)((unsigned long long)node >> 32), batch,
                                          ((unsigned)hop << 24) | (unsigned)slot, k0, k1);
  return __umul64hi(u, m);
}

// ---- node table -----------------------------------------------------------------------------
// Direct: the node's word is looked at and, if v is smaller, lowered by an atomic minimum whose
// result nobody waits for; one dependent access per edge where the hashed table has two or more (look, claim,
// probe on).  An id outside the graph stays inside the table (its last word).
// Hashed: finds or creates the entry of node u (open addressing, linear probing) and lowers its value to
// v if v is smaller; returns the slot and, in *candidate, whether v may have become the entry's
// value (the slot was empty, or held a larger value when it was looked at).  A call for which that
// is false can never be the node's first appearance; the reverse need not hold.
// For an entry that already holds u, key and value move as one word, so a single 64-bit atomic
// minimum does it; an empty slot is claimed by compare-and-swap.  Values only decrease and keys
// never change, so a stale read costs a redundant atomic at most, and any cache may serve it.
template <bool DIRECT>
__device__ __forceinline__ unsigned table_insert_min(HashEntry* table, unsigned entries, unsigned shift, unsigned last_node,
                                                     long long u, unsigned v, bool* candidate) {
  if (DIRECT) {
    const unsigned own = (unsigned long long)u < last_node ? (unsigned)u : last_node;
    unsigned* const word = reinterpret_cast<unsigned*>(table) + ((size_t)own << shift);
    *candidate = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > v;
    if (*candidate) atomicMin(word, v);
    return own;
  }
  // multiplicative hash, its high 32 bits scaled to [0, entries): the table need not be a power of two
  unsigned slot = __umulhi((unsigned)(((unsigned long long)u * 0x9E3779B97F4A7C15ull) >> 32), entries);
  const HashEntry mine = ((HashEntry)u << 32) | v;
  *candidate = false;
  for (;;) {
    HashEntry w = __hip_atomic_load(&table[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (w == kEmptyEntry) {
      w = atomicCAS(&table[slot], kEmptyEntry, mine);
      if (w == kEmptyEntry) {
        *candidate = true;
        return slot;
      }
    }
    if ((long long)(w >> 32) == u) {
      if ((unsigned)w > v) {
        atomicMin(&table[slot], mine);
        *candidate = true;
      }
      return slot;
    }
    slot = slot + 1 == entries ? 0u : slot + 1;
  }
}

template <int G>
__device__ __forceinline__ unsigned long long group_bits(unsigned long long ballot, int grp_in_wave) {
  if (G == 64) return ballot;
  return (ballot >> (grp_in_wave * G)) & ((1ull << (G & 63)) - 1ull);
}

// Lane S of every group of G lanes, for all of the group.  Every lane of the wavefront must be active.
template <int G, int S>
__device__ __forceinline__ int group_bcast(int x) {
  if constexpr (G == 64) return __builtin_amdgcn_readlane(x, S);
  else if constexpr (G == 16) return __builtin_amdgcn_update_dpp(0, x, 0x150 + S, 0xF, 0xF, false);  // row_newbcast
  else return __builtin_amdgcn_ds_swizzle(x, (S << 5) | (G == 8 ? 0x18 : 0));                         // (lane & 24 or 0) | S
}

// Whether an earlier lane of the group has the same 64-bit number.  The comparisons do not depend on one another and the broadcasts need no
// address.  All lanes take part in every broadcast: nothing here may become a branch.
template <int G, int S = 0>
__device__ __forceinline__ void least_difference(unsigned lo, unsigned hi, int gl, unsigned& least) {
  if constexpr (S + 1 < G) {
    const unsigned differ = ((unsigned)group_bcast<G, S>((int)lo) ^ lo) | ((unsigned)group_bcast<G, S>((int)hi) ^ hi);
    const unsigned seen = gl > S ? differ : ~0u;
    least = seen < least ? seen : least;
    if constexpr (S % 4 == 3) asm volatile("" : "+v"(least));  // four at a time: all at once would cost wavefronts their registers
    least_difference<G, S + 1>(lo, hi, gl, least);
  }
}
template <int G>
__device__ __forceinline__ bool earlier_equal(unsigned long long x, int gl) {
  unsigned least = ~0u;
  least_difference<G>((unsigned)x, (unsigned)(x >> 32), gl, least);
  return least == 0u;
}

// Inclusive sums over the wavefront on the vector ALU (no trips through LDS).  Every lane must be active.
__device__ __forceinline__ int wave_scan_dpp(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);   // row_shr:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast:15 to rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast:31 to rows 2 and 3
  return x;
}

// ---- kernels ----------------------------------------------------------------------------------

struct HopArgs {
  const long long* seeds;  // hop 0 only: the seeds become F_0 inside this kernel
  long long n_seeds;
  long long* nodes;
  long long* counts;
  int hop;
  int fanout;
  const long long* indptr;
  const long long* indices;
  const int* adj_remap;
  const long long* c_indptr;
  const long long* c_indices;
  long long partial_node;  // the node whose list is cached in part (-1: none) and its full length
  long long partial_deg;
  unsigned k0, k1, batch;
  long long* tmp_u;
  int* tmp_slot;
  int* row_cnt;
  HashEntry* table;
  unsigned entries;    // of a hashed table
  unsigned shift;      // of a direct table's slot, to its 32-bit word
  unsigned last_node;  // the graph's last node id (direct table)
  unsigned* adj_count;
  unsigned* edge_count;
  // previous hop, whose edges get their local ids at the start of this kernel (hop >= 1)
  int prev_fanout;
  const int* prev_tmp_slot;
  const long long* prev_blk_indptr;
  int* prev_blk_src;
  int n_write_blocks;  // leading workgroups that only do the previous hop's edge ids
  const unsigned* batch_flag;  // != kBatchOk: an earlier kernel of this batch failed, do nothing
  int count_lines;             // statistics are on: count the host lines every row touches
  // List bounds of the frontier's rows, kept for the batch's later hops (F_h is a prefix of F_{h+1}, and every
  // hop samples all of its frontier): row i -> (start in the array that serves it, length | served-by-cache << 62),
  // or a negative second word for the one node cached in part, whose bounds are looked up again.
  longlong2* row_memo;
  int last_hop;                // no later hop will read what this one would note
  long long cap_rows;          // bound on the rows: what the arrays have room for
};

// Closing kernel of a batch: the last hop's edge ids, and the batch sizes for the host.
// Hit statistics of a batch: every relabel tile leaves (rows with a cache slot, edges read from the cache) in
// its hop's array of partial sums; the closing kernel adds them up and updates the caller's counters with
// one atomic each.  (Per-tile atomics on the same few words cost 12 us per batch on a 56 k-row frontier.)
constexpr int kStatPartWords = 4;  // per relabel tile: rows with a slot, edges from the cache, lines of ids, lines of bounds
struct StatFold {
  unsigned long long* stats;                    // nullptr: no statistics
  const unsigned long long* part[DCI_MAX_HOPS]; // [kStatPartWords * tiles] per hop
  int tile_rows[DCI_MAX_HOPS];
  int n_hops;
};

template <bool DIRECT>
__global__ __launch_bounds__(kBlock) void k_write_src(CloseArgs close, StatFold sf, const long long* nodes, int n_hops,
                                                      unsigned* feat_count) {
  if (!close_batch<DIRECT>(close, (int)blockIdx.x, (int)gridDim.x)) return;
  const long long* const counts = close.counts;
  if (feat_count) {  // pre-sampling: one visit for every input node
    const long long n = counts[n_hops];
    for (long long i = blockIdx.x * (long long)kBlock + threadIdx.x; i < n; i += (long long)gridDim.x * kBlock)
      atomicAdd(&feat_count[nodes[i]], 1u);
  }
  if (sf.stats && blockIdx.x == gridDim.x - 1) {
    __shared__ unsigned long long s_r[kBlock / kWave], s_e[kBlock / kWave];
    __shared__ unsigned long long s_l[kBlock / kWave], s_b[kBlock / kWave];
    unsigned long long hr = 0, he = 0, hl = 0, hb = 0, rows = 0, edges = 0;
    for (int h = 0; h < sf.n_hops; ++h) {
      const long long n_rows = counts[h];
      const long long n_tiles = (n_rows + sf.tile_rows[h] - 1) / sf.tile_rows[h];
      for (long long t = threadIdx.x; t < n_tiles; t += kBlock) {
        hr += sf.part[h][kStatPartWords * t];
        he += sf.part[h][kStatPartWords * t + 1];
        hl += sf.part[h][kStatPartWords * t + 2];
        hb += sf.part[h][kStatPartWords * t + 3];
      }
      rows += (unsigned long long)n_rows;
      edges += (unsigned long long)counts[DCI_MAX_HOPS + 1 + h];
    }
    hr = wave_sum_u64(hr);
    he = wave_sum_u64(he);
    hl = wave_sum_u64(hl);
    hb = wave_sum_u64(hb);
    if (lane_id() == 0) {
      s_r[threadIdx.x / kWave] = hr;
      s_e[threadIdx.x / kWave] = he;
      s_l[threadIdx.x / kWave] = hl;
      s_b[threadIdx.x / kWave] = hb;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      hr = 0;
      he = 0;
      hl = 0;
      hb = 0;
      for (int w = 0; w < kBlock / kWave; ++w) {
        hr += s_r[w];
        he += s_e[w];
        hl += s_l[w];
        hb += s_b[w];
      }
      if (edges) atomicAdd(&sf.stats[DCI_STAT_EDGES_SAMPLED], edges);
      if (hr) atomicAdd(&sf.stats[DCI_STAT_ADJ_NODE_HITS], hr);
      if (rows - hr) atomicAdd(&sf.stats[DCI_STAT_ADJ_NODE_MISSES], rows - hr);
      if (he) atomicAdd(&sf.stats[DCI_STAT_ADJ_EDGE_HITS], he);
      if (edges - he) atomicAdd(&sf.stats[DCI_STAT_ADJ_EDGE_MISSES], edges - he);
      atomicAdd(&sf.stats[DCI_STAT_INPUT_NODES], (unsigned long long)counts[sf.n_hops]);
      // a frontier node costs its pair of list bounds (16 bytes), a sampled edge its neighbour id (8 bytes),
      // charged to the tier that served them
      if (hr | he) atomicAdd(&sf.stats[DCI_STAT_BYTES_HBM], 16ull * hr + 8ull * he);
      if ((rows - hr) | (edges - he)) atomicAdd(&sf.stats[DCI_STAT_BYTES_HOST], 16ull * (rows - hr) + 8ull * (edges - he));
      if (hl) atomicAdd(&sf.stats[DCI_STAT_LINES_IDS], hl);
      if (hb) atomicAdd(&sf.stats[DCI_STAT_LINES_BOUNDS], hb);
    }
  }
}

// A hop's frontier: in the table already, the seeds, or nodes that are not in the table yet
enum { kRegistered, kSeeds, kUnregistered };

// What a frontier row reads: its list bounds and, for lane `gl` of its group, where the id at that lane's drawn position stands.
struct RowDraw {
  const long long* src;  // of this lane's neighbour id
  long long start, pos;
  bool hit, active;      // the node has a cache slot; this lane has an edge
  int c, n_host, n_lines, n_bound_lines;  // edges; those read from the host although it has a slot; as in row_cnt
};

// A row's list: where it starts in the array that serves it, its length, how much of it the cache holds.
struct RowBounds {
  long long start, d, cached_len;
  bool hit;
};
// b0, b1: the row's pair of bounds, in the cache's list or the graph's
__device__ __forceinline__ RowBounds row_bounds(const HopArgs& a, long long v, bool hit, long long b0, long long b1) {
  return RowBounds{b0, hit && v == a.partial_node ? a.partial_deg : b1 - b0, hit ? b1 - b0 : 0, hit};
}
__device__ __forceinline__ RowBounds noted_bounds(longlong2 memo) {
  const long long d = memo.y & ((1ll << 62) - 1);
  return RowBounds{memo.x, d, d, (memo.y >> 62) != 0};
}
__device__ __forceinline__ RowBounds look_up_bounds(const HopArgs& a, long long v) {
  const int r = a.adj_remap ? a.adj_remap[v] : -1;
  const long long* const p = r >= 0 ? a.c_indptr + r : a.indptr + v;
  return row_bounds(a, v, r >= 0, p[0], p[1]);
}
__device__ __forceinline__ void note_bounds(const HopArgs& a, long long i, long long v, const RowBounds& b) {
  a.row_memo[i] = longlong2{b.start, v == a.partial_node ? -1ll : (b.d | (b.hit ? (1ll << 62) : 0ll))};
}

// noted: the bounds come from a note.  Every lane of the wavefront must be active.
template <int G>
__device__ __forceinline__ RowDraw draw_row(const HopArgs& a, int hop, int f, bool row_ok, long long v, bool noted, const RowBounds& b, int gl,
                                            int grp_in_wave) {
  const long long start = b.start, d = b.d, cached_len = b.cached_len;
  const bool hit = b.hit;
  const long long* list = hit ? a.c_indices : a.indices;
  const int c = d < (long long)f ? (int)d : f;
  long long pos = gl;
  const bool floyd = row_ok && d > (long long)f;
  if (__ballot(floyd) != 0ull) {
    // Slot s draws t_s below j_s + 1, j_s = d - f + s; it keeps t_s unless an earlier slot already holds that value, in which
    // case it takes j_s.  What earlier slots hold is every earlier t, and j_k of every earlier slot k that took its own: so
    // slot s takes j_s if an earlier t is the same, or if t_s = j_k and slot k took j_k.
    const long long j = d - f + gl;
    long long t = 0;
    if (floyd && gl < f) t = (long long)uniform_below(a.k0, a.k1, v, a.batch, hop, gl, (unsigned long long)(j + 1));
    const bool own = floyd && gl < f;
    bool taken = earlier_equal<G>((unsigned long long)t, gl) && own;
    const long long k = t - (d - f);
    const bool depends = own && k >= 0 && k < gl;
    if (__ballot(depends) != 0ull) {
      for (;;) {
        const unsigned long long bits = group_bits<G>(__ballot(taken), grp_in_wave);
        const bool more = depends && !taken && ((bits >> (k & 63)) & 1ull) != 0ull;
        if (__ballot(more) == 0ull) break;
        taken = taken || more;
      }
    }
    if (floyd) pos = taken ? j : t;
  }
  const bool active = row_ok && gl < c;
  // position p of a node with a slot is served by the cache iff p < cached length (Section IV-B, third
  // paragraph); beyond it - possible only for the one node cached in part - the host list is read
  const bool from_host = active && hit && pos >= cached_len;
  const int n_host = __popcll(group_bits<G>(__ballot(from_host), grp_in_wave));
  const long long* src = from_host ? a.indices + (a.indptr[v] + pos) : list + (start + pos);
  int n_lines = 0, n_bound_lines = 0;
  if (a.count_lines) {
    // Miss-path traffic of the row in the unit a host link moves (128-byte lines): the distinct lines of
    // the neighbour ids it reads from graph->indices, and the lines its list bounds in graph->indptr lie in.
    const bool host_read = active && (from_host || !hit);
    if (__ballot(host_read) != 0ull) {
      // (lanes that read nothing there have numbers of their own)
      const unsigned long long line = host_read ? (unsigned long long)reinterpret_cast<uintptr_t>(src) >> kHostLineLog2 : ~(unsigned long long)gl;
      const bool leader = host_read & !earlier_equal<G>(line, gl);
      n_lines = __popcll(group_bits<G>(__ballot(leader), grp_in_wave));
    }
    if (row_ok && hit && n_host > 0) n_bound_lines = 1;  // the partly cached node: where its host list starts
    if (row_ok && !hit && !noted) {  // (a noted row's bounds came from the batch's own note in HBM)
      const uintptr_t b0 = reinterpret_cast<uintptr_t>(a.indptr + v), b1 = reinterpret_cast<uintptr_t>(a.indptr + v + 1);
      n_bound_lines = (b0 >> kHostLineLog2) == (b1 >> kHostLineLog2) ? 1 : 2;
    }
  }
  return RowDraw{src, start, pos, hit, active, c, n_host, n_lines, n_bound_lines};
}

// Phase 1 of a hop.  INIT (hop 0): row i first turns seed i into frontier entry i (final local id
// i in the table; an atomic minimum, so it also wins against a neighbour lane that registered
// the same node a moment earlier), and REGISTER (after k_first_hops) does the same with the frontier's nodes.  Otherwise the kernel starts by finishing the previous hop
// (write_block_sources), which only needs values that are already final.
//   Bound by the length of its chain of dependent reads, and in large frontiers by the number of random reads: the arguments are fetched
// together; the frontier's sizes, the batch's status, the group's first node and that node's note are asked for together, before it is
// known whether the row exists (the arrays have room for the bound), and the next row's while this one is sampled.  Microseconds before /
// after, third hops: 18 k rows 14.7 / 13.7, 53 k rows 32.4 / 29.5.
struct HopRow {
  long long v;
  longlong2 memo;
};

template <int G, bool COUNT, int FRONTIER, bool DIRECT>
__global__ __launch_bounds__(kBlock, 8) void k_sample_hop(HopArgs a) {
  constexpr bool INIT = FRONTIER == kSeeds, REGISTER = FRONTIER == kUnregistered;
  const int lane = lane_id();
  const int gl = lane & (G - 1);
  const int grp_in_wave = lane / G;
  constexpr int kGroups = kBlock / G;
  const int grp_in_block = (int)threadIdx.x / G;
  const int f = a.fanout;
  const int block = (int)blockIdx.x - (INIT ? 0 : a.n_write_blocks);
  const int n_blocks = (int)gridDim.x - (INIT ? 0 : a.n_write_blocks);
  auto read_row = [&](long long i) {
    HopRow r;
    if (INIT) {
      r.v = a.seeds[i];
    } else {
      r.v = a.nodes[i];
      r.memo = a.row_memo[i];
    }
    return r;
  };
  long long n_rows, n_noted = 0;  // rows below n_noted were rows of the previous hop as well
  HopRow next = {0, {0, 0}};
  if (INIT) {
    n_rows = a.n_seeds;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.counts[0] = n_rows;
    const long long i = (long long)block * kGroups + grp_in_block;
    if (i < n_rows) next = read_row(i);
  } else {
    asm volatile("" ::"s"(a.tmp_slot), "s"(a.row_cnt), "s"(a.table), "s"(a.indices), "s"(a.c_indices), "s"(a.indptr), "s"(a.k0), "s"(a.k1),
                 "s"(a.batch), "s"(a.row_memo), "s"(a.nodes), "s"(a.counts), "s"(a.batch_flag), "s"(a.last_node), "s"(a.shift));
    const unsigned flag = *a.batch_flag;
    n_rows = a.counts[a.hop];
    n_noted = a.counts[a.hop - 1];
    const long long i = (long long)block * kGroups + grp_in_block;
    if (block >= 0 && i < a.cap_rows) next = read_row(i);
    asm volatile("" ::"s"(flag), "s"(n_rows), "s"(n_noted), "v"(next.v));  // all of them on their way before the first is waited for
    if (flag != kBatchOk) return;  // an earlier relabel tile gave up: the closing kernel voids the batch
    if (block < 0) {
      // the first few workgroups finish the previous hop while the others sample this one
      write_block_sources<DIRECT>(n_noted, a.prev_fanout, a.prev_tmp_slot, a.prev_blk_indptr,
                                  a.table, a.shift, a.prev_blk_src, (int)blockIdx.x, a.n_write_blocks);
      return;
    }
  }

  const long long step = (long long)n_blocks * kGroups;
  for (long long base = (long long)block * kGroups; base < n_rows; base += step) {
    const long long i = base + grp_in_block;
    const bool row_ok = i < n_rows;
    const long long v = next.v;
    const longlong2 memo = next.memo;
    if (i + step < n_rows) next = read_row(i + step);
    const bool noted = !INIT && row_ok && i < n_noted && memo.y >= 0;
    if ((INIT || REGISTER) && row_ok && gl == 0) {
      if (INIT) a.nodes[i] = v;
      bool ignored;
      (void)table_insert_min<DIRECT>(a.table, a.entries, a.shift, a.last_node, v, (unsigned)i, &ignored);
    }
    RowBounds b = {0, 0, 0, false};
    if (row_ok) {
      if (noted) {
        b = noted_bounds(memo);
      } else {
        b = look_up_bounds(a, v);
        if (!a.last_hop && gl == 0) note_bounds(a, i, v, b);
      }
    }
    const RowDraw r = draw_row<G>(a, a.hop, f, row_ok, v, noted, b, gl, grp_in_wave);
    if (r.active) {
      const long long u = *(__attribute__((address_space(1))) const long long*)r.src;
      const int p = (int)(i * f + gl);
      bool candidate;
      const unsigned slot =
          table_insert_min<DIRECT>(a.table, a.entries, a.shift, a.last_node, u, kTentative | (unsigned)p, &candidate);
      if (!DIRECT) a.tmp_u[p] = u;  // (a direct table's slot is the id)
      a.tmp_slot[p] = candidate ? (int)slot : -2 - (int)slot;  // the relabel kernel looks at the candidates only
      if (COUNT && a.edge_count) {
        const long long host_start = r.hit ? a.indptr[v] : r.start;
        atomicAdd(&a.edge_count[host_start + r.pos], 1u);
      }
    } else if (row_ok && gl < f) {
      a.tmp_slot[(int)(i * f + gl)] = -1;  // no edge here: lets the later kernels read the slots without the row count
    }
    if (row_ok && gl == 0) {
      // the hit flag rides in bit 30 so that the relabel kernel can total the hit statistics
      a.row_cnt[i] = r.c | (r.n_host << kRowHostShift) | (r.n_lines << kRowLinesShift) |
                     (r.n_bound_lines << kRowBoundLinesShift) | (r.hit ? kRowHitBit : 0);
      if (COUNT && r.c > 0) atomicAdd(&a.adj_count[v], (unsigned)r.c);
    }
  }
}

// Phase 2 of a hop, one pass: count the first appearances of every row, prefix-sum edge counts and
// first-appearance counts over all rows, and give the first appearances their local ids.
// The prefix sums run as a chained scan over tiles of rows with decoupled look-back: a workgroup
// takes the next tile number from a ticket counter (so every earlier tile is already running),
// publishes its own totals, and adds up its predecessors' published values until it meets one
// that already carries an inclusive prefix.  Status word: flag (2 bits) | firsts (31) | edges (31);
// the all-ones fill pattern reads as "not yet published".  A status word carries its whole
// message, so the atomic accesses are relaxed: release / acquire at device scope would add an
// L2 write-back / invalidate to every publish and every poll.
// Rows per tile = (lane groups per workgroup) x (rows per group, kTileItersMax at most).  Many rows per
// group keep several independent loads in flight per lane; few rows per group give more tiles, i.e. more
// workgroups to hide the tile's chain of dependent phases behind.  Which wins depends on how many tiles a
// frontier makes, so the count is picked per hop from the frontier's capacity (tile_iters_for).
constexpr int kTileItersMax = 8;
// 512 threads to a tile: the tickets of the chained scan are atomics on one word and serialise (12 - 19 ns each), so larger tiles wait
// less; but a compute unit takes about three clocks for each of a tile's scattered accesses, so they are longer at them.  Rows of 16 slots
// per tile / microseconds, direct table: 4 k rows (10 sources) 32 / 6.6, 64 / 6.5, 128 / 7.2, 256 / 8.7; 18 k (15) 32 / 16.2, 64 / 10.7, 128 / 8.5, 256 /
// 9.1; 53 k (15) 64 / 25, 128 / 17.4, 256 / 13.9, and with 1,024 threads 512 / 15.8.
constexpr int kRelabelBlock = 512;
static_assert(kRelabelBlock == 4 * kWave * 2, "a workgroup is two wavefronts to each of a compute unit's four SIMDs");
constexpr unsigned long long kStInvalid = 3ull, kStAggregate = 1ull, kStInclusive = 2ull;
// The look-back polls at most dci_ctx::relabel_spin_limit times (default 2^24: far beyond any real wait, ends a wedged launch).

__device__ __forceinline__ unsigned long long st_pack(unsigned long long flag, unsigned long long firsts,
                                                      unsigned long long edges) {
  return (flag << 62) | (firsts << 31) | edges;
}

struct RelabelArgs {
  long long* counts;
  int hop;
  int fanout;
  const int* row_cnt;
  const long long* tmp_u;
  int* tmp_slot;  // read; the first appearances are marked kSlotDone
  HashEntry* table;
  unsigned shift;  // of a direct table's slot, to its 32-bit word
  long long* nodes;
  long long* blk_indptr;
  int* blk_src;   // the first appearances' local ids are written here, the other edges' by the next kernel
  unsigned long long* status;  // one word per tile, filled with ones beforehand
  unsigned* ticket;            // filled with ones beforehand: the first ticket is 0xFFFFFFFF + 1 = 0
  unsigned long long* stat_part;  // [kStatPartWords * tiles] per tile, or nullptr
  unsigned* batch_flag;   // set to 0 by a tile that gives up; != kBatchOk on entry: do nothing
  unsigned spin_limit;    // polls of the look-back before a tile gives up
  unsigned first_ticket;  // tiles are numbered from here (0 except under the failure-handling test hook)
  unsigned unticketed;    // up to this many tiles are numbered by their workgroup (unticketed_tiles)
};

template <int G, int kTileIters, bool DIRECT>
__global__ __launch_bounds__(kRelabelBlock, kTileIters < kTileItersMax ? 2 * kRelabelPerCu : 4) void k_relabel_hop(RelabelArgs a) {
  constexpr int kGroups = kRelabelBlock / G;
  constexpr int TR = kGroups * kTileIters;  // rows per tile, at most kRelabelBlock
  constexpr int kWaves = kRelabelBlock / kWave;
  static_assert(TR <= kRelabelBlock, "one thread per tile row in the block scan");
  static_assert(TR * G < 65536, "edge and first-appearance counts of a tile share a word");
  __shared__ unsigned s_cf[TR];  // edges | first appearances << 16
  __shared__ unsigned s_w[kWaves];
  __shared__ unsigned long long s_hr[kWaves], s_he[kWaves], s_hl[kWaves], s_hb[kWaves];
  __shared__ unsigned s_tile;
  __shared__ long long s_ec;
  __shared__ int s_ef;
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int gl = lane & (G - 1), grp_in_wave = lane / G, grp = tid / G;
  const unsigned flag = *a.batch_flag;
  const long long n_rows = a.counts[a.hop];
  asm volatile("" ::"s"(flag), "s"(n_rows));  // (one trip for both)
  if (flag != kBatchOk) return;  // an earlier hop failed (uniform over the launch: set before it began)
  // The grid is sized for the frontier's bound; only as many workgroups as the frontier has tiles take a
  // ticket (left to the whole grid the tickets were most of this kernel's time).  Which workgroups those are does not matter for
  // progress: a tile waits only for smaller tickets, and those are held by workgroups that are already running.
  const long long n_tiles = (n_rows + TR - 1) / TR;
  long long takers = n_tiles - (long long)a.first_ticket;
  if (takers < 1) takers = 1;  // an empty frontier (or a test hook beyond it) still needs one workgroup
  if ((long long)blockIdx.x >= takers) return;
  unsigned tile = blockIdx.x + a.first_ticket;
  if (takers > (long long)a.unticketed) {
    if (tid == 0) s_tile = atomicAdd(a.ticket, 1u) + 1u + a.first_ticket;
    __syncthreads();
    tile = s_tile;
  }
  const long long row0 = (long long)tile * TR;
  if (row0 >= n_rows) {
    // (test hook: when even the first numbered tile lies beyond the frontier nobody would notice the
    // missing tiles, so that tile voids the batch itself)
    if (a.first_ticket != 0 && tile == a.first_ticket && tid == 0)
      __hip_atomic_store(a.batch_flag, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tile == 0 && tid == 0) {  // empty frontier: the hop adds nothing
      a.blk_indptr[0] = 0;
      a.counts[a.hop + 1] = n_rows;
      a.counts[DCI_MAX_HOPS + 1 + a.hop] = 0;
    }
    return;
  }
  const int f = a.fanout;

  // per row: sampled edges, first appearances (the table still holds the lane's own position).
  // Row counts and table slots are independent loads, the table values depend on the slots; each
  // group is issued for all of the lane's rows at once, so that the tile pays the memory latency
  // twice, not 24 times.
  int raw[kTileIters], slot[kTileIters];
  unsigned val[kTileIters];
#pragma unroll
  for (int it = 0; it < kTileIters; ++it) {
    const long long i = row0 + it * kGroups + grp;
    raw[it] = i < n_rows ? a.row_cnt[i] : 0;
  }
#pragma unroll
  for (int it = 0; it < kTileIters; ++it) {
    const long long i = row0 + it * kGroups + grp;
    slot[it] = (i < n_rows && gl < f) ? a.tmp_slot[i * f + gl] : -1;  // -1 where the row has no edge
  }
#pragma unroll
  for (int it = 0; it < kTileIters; ++it) val[it] = slot[it] >= 0 ? entry_val<DIRECT>(a.table, a.shift, (unsigned)slot[it]) : 0u;
  unsigned first_bits = 0;
  long long new_u[kTileIters];
#pragma unroll
  for (int it = 0; it < kTileIters; ++it) {
    const int r = it * kGroups + grp;
    const int c = raw[it] & kRowCntMask;
    const unsigned p = (unsigned)((row0 + r) * f + gl);
    const bool first = slot[it] >= 0 && val[it] == (kTentative | p);
    const unsigned long long bits = group_bits<G>(__ballot(first), grp_in_wave);
    if (first) first_bits |= 1u << it;
    // the ids of the first appearances are only needed once the tile knows its offsets; asked for here, they
    // arrive while the tile scans and looks back
    new_u[it] = !first ? 0 : DIRECT ? (long long)slot[it] : a.tmp_u[(row0 + r) * f + gl];
    if (gl == 0) s_cf[r] = (unsigned)c | (unsigned)__popcll(bits) << 16;
  }
  if (a.stat_part) {
    unsigned long long hit_rows = 0, hit_edges = 0, host_lines = 0, bound_lines = 0;
    if (gl == 0) {
#pragma unroll
      for (int it = 0; it < kTileIters; ++it) {
        if (raw[it] & kRowHitBit) {
          hit_rows += 1;
          hit_edges += (unsigned)((raw[it] & kRowCntMask) - ((raw[it] >> kRowHostShift) & 0xFF));
        }
        host_lines += (unsigned)((raw[it] >> kRowLinesShift) & kRowLinesMask);
        bound_lines += (unsigned)((raw[it] >> kRowBoundLinesShift) & kRowBoundLinesMask);
      }
    }
    hit_rows = wave_sum_u64(hit_rows);
    hit_edges = wave_sum_u64(hit_edges);
    host_lines = wave_sum_u64(host_lines);
    bound_lines = wave_sum_u64(bound_lines);
    if (lane == 0) {
      s_hr[wave] = hit_rows;
      s_he[wave] = hit_edges;
      s_hl[wave] = host_lines;
      s_hb[wave] = bound_lines;
    }
  }
  __syncthreads();

  // scan of the tile's rows, one thread per row
  const unsigned cf = tid < TR ? s_cf[tid] : 0u;
  const unsigned incl = (unsigned)wave_scan_dpp((int)cf);
  if (lane == kWave - 1) s_w[wave] = incl;
  __syncthreads();
  unsigned off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) off += s_w[w];
    tot += s_w[w];
  }
  const unsigned tot_c = tot & 0xFFFFu, tot_f = tot >> 16;
  const unsigned row_cf = off + incl;  // of row tid, inclusive
  if (tid < TR) s_cf[tid] = row_cf - (cf & 0xFFFF0000u);  // edges inclusive, first appearances exclusive
  // publish this tile, then look back over the earlier ones (first wavefront)
  if (tid == 0)
    __hip_atomic_store(&a.status[tile], st_pack(tile == 0 ? kStInclusive : kStAggregate, tot_f, tot_c), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  if (wave == 0) {
    long long ec = 0;
    int ef = 0;
    if (tile != 0) {
      // Look back over the earlier tiles, kLookWindows x 64 status words per round trip (lane l of window k
      // reads tile j - 64 k - l), nearest first.  A window is resolved once every word nearer than its
      // nearest inclusive one (or, if it has none, every word) is published; the sum stops at the first
      // inclusive word.  A lane adds its words up as they are (edges and first appearances of all tiles stay below 2^31
      // each); the lanes' sums meet at the end.
      constexpr int kLookWindows = 4;
      long long j = (long long)tile - 1;
      unsigned polls = 0;
      bool found = false, timed_out = false;
      unsigned sum_c = 0, sum_f = 0;
      while (!found && !timed_out) {
        unsigned long long st[kLookWindows];
#pragma unroll
        for (int k = 0; k < kLookWindows; ++k) {
          const long long idx = j - (long long)k * kWave - lane;
          st[k] = idx >= 0 ? __hip_atomic_load(&a.status[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                           : st_pack(kStInclusive, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < kLookWindows; ++k) {
          if (!found && !timed_out) {
            const long long idx = j - (long long)k * kWave - lane;
            int first_inc;
            for (;;) {
              const unsigned long long inv = __ballot((st[k] >> 62) == kStInvalid);
              const unsigned long long inc = __ballot((st[k] >> 62) == kStInclusive);
              first_inc = inc ? (int)__ffsll((long long)inc) - 1 : kWave;  // nearest tile with a prefix
              const unsigned long long nearer = first_inc >= kWave ? ~0ull : ((1ull << first_inc) - 1ull);
              if ((inv & nearer) == 0ull) break;
              if (polls >= a.spin_limit) {
                timed_out = true;
                break;
              }
              __builtin_amdgcn_s_sleep(1);
              ++polls;
              if ((st[k] >> 62) == kStInvalid)
                st[k] = __hip_atomic_load(&a.status[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (lane <= first_inc && (st[k] >> 62) != kStInvalid) {
              sum_c += (unsigned)(st[k] & 0x7FFFFFFFull);
              sum_f += (unsigned)((st[k] >> 31) & 0x7FFFFFFFull);
            }
            if (!timed_out && first_inc < kWave) found = true;
          }
        }
        j -= (long long)kLookWindows * kWave;
      }
      if (timed_out && lane == 0) {
        // Gave up: a predecessor never published.  The tile goes on with what it has - every index it
        // forms stays at or below the true one, hence inside the batch's buffers - and voids the batch,
        // so that no later kernel reads what this hop leaves behind.
        __hip_atomic_store(a.batch_flag, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      ec = (long long)__builtin_amdgcn_readlane(wave_scan_dpp((int)sum_c), kWave - 1);
      ef = __builtin_amdgcn_readlane(wave_scan_dpp((int)sum_f), kWave - 1);
      if (lane == 0)
        __hip_atomic_store(&a.status[tile], st_pack(kStInclusive, (unsigned)ef + tot_f, (unsigned long long)ec + tot_c),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) {
      s_ec = ec;
      s_ef = ef;
    }
  }
  __syncthreads();
  const long long ec = s_ec;
  const int ef = s_ef;
  if (tid < TR && row0 + tid < n_rows) a.blk_indptr[row0 + tid + 1] = ec + (row_cf & 0xFFFFu);

  // first appearances take the next local ids, in (row, slot) order
#pragma unroll
  for (int it = 0; it < kTileIters; ++it) {
    const int r = it * kGroups + grp;
    const bool first = (first_bits >> it) & 1u;
    const unsigned long long bits = group_bits<G>(__ballot(first), grp_in_wave);
    if (first) {
      const unsigned row = s_cf[r];
      const long long new_id = n_rows + ef + (int)(row >> 16) + __popcll(bits & ((1ull << gl) - 1ull));
      a.nodes[new_id] = new_u[it];
      entry_set_val<DIRECT>(a.table, a.shift, (unsigned)slot[it], (unsigned)new_id);
      // this edge's local id is known right here: write it (the row's edges sit at its sampled slots
      // 0 .. c-1, and s_cf holds the row's inclusive edge count within the tile), and spare the edge-id pass
      // the table look-up
      a.blk_src[ec + (row & 0xFFFFu) - (raw[it] & kRowCntMask) + gl] = (int)new_id;
      a.tmp_slot[(row0 + r) * f + gl] = kSlotDone;
    }
  }

  if (tid == 0) {
    if (tile == 0) a.blk_indptr[0] = 0;
    const bool last_tile = row0 + TR >= n_rows;
    if (last_tile) {
      a.counts[a.hop + 1] = n_rows + ef + tot_f;
      a.counts[DCI_MAX_HOPS + 1 + a.hop] = ec + tot_c;
    }
    if (a.stat_part) {
      unsigned long long hr = 0, he = 0, hl = 0, hb = 0;
      for (int w = 0; w < kWaves; ++w) {
        hr += s_hr[w];
        he += s_he[w];
        hl += s_hl[w];
        hb += s_hb[w];
      }
      a.stat_part[kStatPartWords * (size_t)tile] = hr;      // added up by the batch's closing kernel
      a.stat_part[kStatPartWords * (size_t)tile + 1] = he;
      a.stat_part[kStatPartWords * (size_t)tile + 2] = hl;
      a.stat_part[kStatPartWords * (size_t)tile + 3] = hb;
    }
  }
}

// The first hops of a batch with few seeds, in one launch: the first workgroup samples and relabels them with a node table of its own in LDS
// while the others clear the batch's table for the hops behind, the next of which puts this frontier into it (kUnregistered).
//   Bound by the same chain of reads as a hop's two kernels (seed, slot, bounds, ids), but without their launches, the clear's and the trips
// to the table in memory: two hops of 16 seeds take 12 us, where the clear and four kernels took 24 and the gaps between them.  A pass,
// fan-outs 5, 10, 15, before / after: 4 seeds 63.6 / 56.1 us, 16 72.3 / 65.8, 64 (one hop) 89.4 / 86.4, 128 89.5 / 86.5; 2, 4, 8: 64 seeds 66.7 / 59.3.
//   At most kFirstSlots slots (lanes of all rows' groups) to a hop: with 2,048, two rows to every group, one compute unit's reads take as long as
// the launches do (256 seeds 100.5 / 100.0 us, over the host link 133.4 / 133.7, two hops 55.3 / 55.5).
// (Every workgroup has the 83 KB of LDS that only the first needs, so the others clear one to a compute unit at a time.)
constexpr int kFirstThreads = 1024, kFirstIters = 2, kFirstSlots = 1536, kFirstEntries = 8192, kFirstNodes = kFirstEntries / 2;

struct FirstArgs {
  HopArgs a;   // what the hops have in common
  int n_hops;  // made here, all but the batch's last at most
  int fanout[DCI_MAX_HOPS];
  long long* blk_indptr[DCI_MAX_HOPS];
  int* blk_src[DCI_MAX_HOPS];
  unsigned long long* stat_part[DCI_MAX_HOPS];  // nullptr: no statistics
  uint4* clear;  // the region to fill with ones
  size_t clear_n16;
};

// As table_insert_min, in LDS: at most kFirstNodes different ids come, so half of the entries stay empty.
__device__ __forceinline__ unsigned first_insert_min(HashEntry* table, unsigned u, unsigned v) {
  const HashEntry mine = ((HashEntry)u << 32) | v;
  unsigned slot = (u * 0x9E3779B9u) >> 19;
  static_assert(kFirstEntries == 1 << 13, "the hash's bits");
  for (;;) {
    HashEntry w = table[slot];
    if (w == kEmptyEntry) {
      w = atomicCAS(&table[slot], kEmptyEntry, mine);
      if (w == kEmptyEntry) return slot;
    }
    if ((unsigned)(w >> 32) == u) {
      if ((unsigned)w > v) atomicMin(&table[slot], mine);
      return slot;
    }
    slot = (slot + 1) & (kFirstEntries - 1);
  }
}

template <int G, bool COUNT>
__global__ __launch_bounds__(kFirstThreads) void k_first_hops(FirstArgs fa) {
  if (blockIdx.x != 0) {
    const size_t n = (size_t)(gridDim.x - 1) * kFirstThreads;
    for (size_t q = (size_t)(blockIdx.x - 1) * kFirstThreads + threadIdx.x; q < fa.clear_n16; q += n) fa.clear[q] = make_uint4(~0u, ~0u, ~0u, ~0u);
    return;
  }
  constexpr int kGroups = kFirstThreads / G, kRows = kGroups * kFirstIters, kWaves = kFirstThreads / kWave;
  static_assert(kRows <= kFirstThreads && kFirstSlots <= kFirstThreads * kFirstIters, "one thread per row in the scan, a lane for every slot");
  __shared__ HashEntry s_table[kFirstEntries];
  __shared__ unsigned s_node[kFirstNodes];
  __shared__ unsigned s_cf[kRows];  // edges | first appearances << 16
  __shared__ unsigned s_w[kWaves];
  __shared__ unsigned s_stat[kStatPartWords];
  const HopArgs& a = fa.a;
  const int tid = (int)threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int gl = lane & (G - 1), grp_in_wave = lane / G, grp = tid / G;
  int n_rows = (int)a.n_seeds, n_noted = 0;
  const long long seed = tid < n_rows ? a.seeds[tid] : 0;
  for (int q = tid; q < kFirstEntries; q += kFirstThreads) s_table[q] = kEmptyEntry;
  __syncthreads();
  if (tid < n_rows) {
    a.nodes[tid] = seed;
    s_node[tid] = (unsigned)seed;
    (void)first_insert_min(s_table, (unsigned)seed, (unsigned)tid);
  }
  if (tid == 0) a.counts[0] = n_rows;
  for (int h = 0; h < fa.n_hops; ++h) {
    const int f = fa.fanout[h];
    if (tid < kStatPartWords) s_stat[tid] = 0;
    __syncthreads();
    // each step for all of a group's rows before the next: the reads of a step are on their way together
    int raw[kFirstIters], look[kFirstIters];
    unsigned slot[kFirstIters], u[kFirstIters];
    long long v[kFirstIters], b0[kFirstIters], b1[kFirstIters];
    RowDraw r[kFirstIters];
#pragma unroll
    for (int it = 0; it < kFirstIters; ++it) {
      const int i = it * kGroups + grp;
      v[it] = s_node[i < n_rows ? i : n_rows - 1];
      look[it] = a.adj_remap && i >= n_noted ? a.adj_remap[v[it]] : -1;
    }
#pragma unroll
    for (int it = 0; it < kFirstIters; ++it) {
      const int i = it * kGroups + grp;
      const long long* const p = i < n_noted ? &a.row_memo[i].x : look[it] >= 0 ? a.c_indptr + look[it] : a.indptr + v[it];
      if (i < n_rows) {
        b0[it] = p[0];
        b1[it] = p[1];
      }
    }
#pragma unroll
    for (int it = 0; it < kFirstIters; ++it) {
      const int i = it * kGroups + grp;
      RowBounds b = {0, 0, 0, false};
      const bool noted = i < n_noted && b1[it] >= 0;
      if (noted) b = noted_bounds(longlong2{b0[it], b1[it]});
      else if (i < n_noted) b = look_up_bounds(a, v[it]);
      else if (i < n_rows) b = row_bounds(a, v[it], look[it] >= 0, b0[it], b1[it]);
      if (i >= n_noted && i < n_rows && gl == 0) note_bounds(a, i, v[it], b);
      r[it] = draw_row<G>(a, h, f, i < n_rows, v[it], noted, b, gl, grp_in_wave);
      raw[it] = r[it].c | (r[it].n_host << kRowHostShift) | (r[it].n_lines << kRowLinesShift) | (r[it].n_bound_lines << kRowBoundLinesShift) |
                (r[it].hit ? kRowHitBit : 0);
    }
#pragma unroll
    for (int it = 0; it < kFirstIters; ++it)
      if (r[it].active) u[it] = (unsigned)*(__attribute__((address_space(1))) const long long*)r[it].src;
#pragma unroll
    for (int it = 0; it < kFirstIters; ++it) {
      const int i = it * kGroups + grp;
      if (r[it].active) {
        slot[it] = first_insert_min(s_table, u[it], kTentative | (unsigned)(i * f + gl));
        if (COUNT && a.edge_count) atomicAdd(&a.edge_count[(r[it].hit ? a.indptr[v[it]] : r[it].start) + r[it].pos], 1u);
      }
      if (COUNT && i < n_rows && gl == 0 && r[it].c > 0) atomicAdd(&a.adj_count[v[it]], (unsigned)r[it].c);
    }
    __syncthreads();
    unsigned first_bits = 0;
#pragma unroll
    for (int it = 0; it < kFirstIters; ++it) {
      const int i = it * kGroups + grp, c = raw[it] & kRowCntMask;
      const bool first = gl < c && (unsigned)s_table[slot[it]] == (kTentative | (unsigned)(i * f + gl));
      const unsigned long long bits = group_bits<G>(__ballot(first), grp_in_wave);
      if (first) first_bits |= 1u << it;
      if (gl == 0) {
        s_cf[i] = (unsigned)c | (unsigned)__popcll(bits) << 16;
        if (fa.stat_part[h] && raw[it] != 0) {
          if (raw[it] & kRowHitBit) {
            atomicAdd(&s_stat[0], 1u);
            atomicAdd(&s_stat[1], (unsigned)(c - ((raw[it] >> kRowHostShift) & 0xFF)));
          }
          atomicAdd(&s_stat[2], (unsigned)((raw[it] >> kRowLinesShift) & kRowLinesMask));
          atomicAdd(&s_stat[3], (unsigned)((raw[it] >> kRowBoundLinesShift) & kRowBoundLinesMask));
        }
      }
    }
    __syncthreads();
    const unsigned cf = tid < kRows ? s_cf[tid] : 0u;
    const unsigned incl = (unsigned)wave_scan_dpp((int)cf);
    if (lane == kWave - 1) s_w[wave] = incl;
    __syncthreads();
    unsigned off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) off += s_w[w];
      tot += s_w[w];
    }
    const unsigned row_cf = off + incl;
    if (tid < kRows) s_cf[tid] = row_cf - cf;
    if (tid < n_rows) fa.blk_indptr[h][tid + 1] = row_cf & 0xFFFFu;
    if (tid == 0) {
      fa.blk_indptr[h][0] = 0;
      a.counts[h + 1] = n_rows + (int)(tot >> 16);
      a.counts[DCI_MAX_HOPS + 1 + h] = tot & 0xFFFFu;
    }
    if (fa.stat_part[h] && tid < kStatPartWords) fa.stat_part[h][tid] = s_stat[tid];
    __syncthreads();
    // first appearances take the next local ids, in (row, slot) order
#pragma unroll
    for (int it = 0; it < kFirstIters; ++it) {
      const bool first = (first_bits >> it) & 1u;
      const unsigned long long bits = group_bits<G>(__ballot(first), grp_in_wave);
      if (first) {
        const unsigned new_id = (unsigned)n_rows + (s_cf[it * kGroups + grp] >> 16) + (unsigned)__popcll(bits & ((1ull << gl) - 1ull));
        a.nodes[new_id] = (long long)u[it];
        s_node[new_id] = u[it];
        reinterpret_cast<unsigned*>(s_table)[2 * slot[it]] = new_id;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kFirstIters; ++it)
      if (gl < (raw[it] & kRowCntMask)) fa.blk_src[h][(s_cf[it * kGroups + grp] & 0xFFFFu) + gl] = (int)(unsigned)s_table[slot[it]];
    n_noted = n_rows;
    n_rows = __builtin_amdgcn_readfirstlane(n_rows + (int)(tot >> 16));
  }
}

__global__ void k_add_u64(unsigned long long* p, unsigned long long v) { atomicAdd(p, v); }

// ---- host side ----------------------------------------------------------------------------------

struct SampleWs {
  HashEntry* table;        // the table, the tile status words and the tickets are one region,
  uint64_t table_entries;  // cleared with a single all-ones fill per batch
  bool direct;             // which kind of table
  unsigned table_shift;    // of a direct table's slot, to its 32-bit word
  unsigned long long* status[DCI_MAX_HOPS];
  unsigned* ticket;        // [DCI_MAX_HOPS]
  unsigned* batch_flag;    // one word after the tickets, also in the cleared region
  size_t clear_bytes;
  long long* tmp_u;
  int* tmp_slot[2];  // by hop parity: a hop's slots are still read while the next hop samples
  int* row_cnt[2];
  longlong2* row_memo;     // list bounds of the frontier's rows, noted for the batch's later hops
  unsigned long long* stat_part[DCI_MAX_HOPS];  // per hop: two words per relabel tile
};

// Twice the bound on the batch's distinct nodes (load factor at most one half), even so that the
// region is a whole number of 16-byte words for the clear.
static uint64_t table_entries_for(int64_t cap_nodes_last) {
  uint64_t want = (uint64_t)(cap_nodes_last > 0 ? cap_nodes_last : 1) * 2;
  return want < 1024 ? 1024 : want;
}

// Direct table: 4 bytes per node of the graph, where that is no more to clear than the hashed table's 8 bytes for
// each of twice the bound on the batch's nodes.  At equal bytes the direct one is the quicker of the two (no
// claim to wait for, no probing, no second copy of the ids); a graph many times the batch's bound would pay
// for its clear with more than that (24 M nodes, bound 4.3 M: direct 3,185 us a pass, hashed 3,168).  Slots double as
// negative codes in tmp_slot, hence the limit of 2^30.
// Both measured, hashed / direct: eight 4,096-seed batches of a 2.4 M-node graph on four lanes 2,002 / 1,917 us (clear 39 /
// 10 MB a batch); an 8,192-seed batch of two hops on 4.0 M nodes 353 / 346 us; 4,096 seeds on 1.6 M nodes 366 / 357 us.
static bool table_is_direct(int64_t num_nodes, uint64_t hashed_bytes) {
  return num_nodes < ((int64_t)1 << 30) && 4 * (uint64_t)num_nodes <= hashed_bytes;
}

// A small direct table is spread out, up to four words per node, as long as it stays within 4 MB (cleared in 2 us) and
// the hashed table's bytes: packed 32 to a 128-byte line, the nodes of a dense graph queue for their line.  1,024 seeds on
// 233 k nodes of 490 neighbours: packed 334 us, spread 331 (hashed 331; runs of one kind differ by 0.3 %).  Other graphs gain
// nothing from it and lose nothing: of 28 cases no other changed by more than its own runs differ, nor did any with 16 MB in
// the place of 4.
constexpr size_t kSpreadBytes = (size_t)4 << 20;
static unsigned direct_shift(int64_t num_nodes, size_t hashed_bytes) {
  const size_t limit = hashed_bytes < kSpreadBytes ? hashed_bytes : kSpreadBytes;
  unsigned shift = 0;
  while (shift < 2 && ((size_t)4 * (size_t)num_nodes << (shift + 1)) <= limit) ++shift;
  return shift;
}

static int group_for(int fanout) { return fanout <= 8 ? 8 : fanout <= 16 ? 16 : fanout <= 32 ? 32 : 64; }

static int64_t tiles_for(int64_t rows, int fanout, int iters) {
  const int64_t tr = (int64_t)(kRelabelBlock / group_for(fanout)) * iters;
  const int64_t t = (rows + tr - 1) / tr;
  return t < 1 ? 1 : t;
}
constexpr int kTileItersMin = 1;  // the workspace is sized for the smallest tiles

// Rows per lane group of a relabel tile (DCI_OPT_RELABEL_TILE_ITERS overrides): the fewest that make no more than 200 tiles of the rows
// that a frontier has about (cap_rows bounds them: seeds fill the bound, batches half or so of the next one and a fifth to a third of
// those behind).  See kRelabelBlock for both sides.
static int tile_iters_for(const dci_ctx* ctx, int hop, int64_t cap_rows, int fanout) {
  if (ctx->relabel_tile_iters) return ctx->relabel_tile_iters;
  const int64_t rows = cap_rows / (hop < 2 ? hop + 1 : 3);
  int iters = kTileItersMin;
  while (iters < kTileItersMax && tiles_for(rows, fanout, iters) > 200) iters *= 2;
  return iters;
}

static void carve_sample_ws(Arena& ar, int64_t num_nodes, const int64_t* cap_nodes, const int64_t* cap_edges,
                            const int32_t* fanouts, int32_t n_hops, SampleWs* ws) {
  int64_t max_edges = 1, max_rows = 1;
  size_t status_words = 0;
  for (int32_t h = 0; h < n_hops; ++h) {
    if (cap_edges[h] > max_edges) max_edges = cap_edges[h];
    if (cap_nodes[h] > max_rows) max_rows = cap_nodes[h];
    status_words += (size_t)tiles_for(cap_nodes[h], fanouts[h], kTileItersMin);
  }
  ws->table_entries = table_entries_for(cap_nodes[n_hops]);
  size_t table_bytes = ws->table_entries * sizeof(HashEntry);
  const size_t sync_bytes = align_up(status_words * 8 + (DCI_MAX_HOPS + 1) * 4, 16);
  char* region = ar.take<char>(table_bytes + sync_bytes);  // the hashed table's size either way
  ws->direct = table_is_direct(num_nodes, table_bytes);
  ws->table_shift = 0;
  if (ws->direct) {
    ws->table_shift = direct_shift(num_nodes, table_bytes);
    // both are multiples of 16: at most the hashed table's bytes
    table_bytes = align_up((size_t)4 * (size_t)num_nodes << ws->table_shift, 16);
  }
  ws->table = reinterpret_cast<HashEntry*>(region);
  unsigned long long* st = reinterpret_cast<unsigned long long*>(region + table_bytes);
  for (int32_t h = 0; h < n_hops; ++h) {
    ws->status[h] = st;
    st += tiles_for(cap_nodes[h], fanouts[h], kTileItersMin);
  }
  ws->ticket = reinterpret_cast<unsigned*>(st);
  ws->batch_flag = ws->ticket + DCI_MAX_HOPS;
  ws->clear_bytes = table_bytes + sync_bytes;
  ws->tmp_u = ar.take<long long>((size_t)max_edges);
  for (int k = 0; k < 2; ++k) {
    ws->tmp_slot[k] = ar.take<int>((size_t)max_edges);
    ws->row_cnt[k] = ar.take<int>((size_t)max_rows);
  }
  ws->row_memo = ar.take<longlong2>((size_t)max_rows);
  for (int32_t h = 0; h < n_hops; ++h)
    ws->stat_part[h] = ar.take<unsigned long long>(kStatPartWords * (size_t)tiles_for(cap_nodes[h], fanouts[h], kTileItersMin));
}

static void carve_blocks(Arena& ar, const int64_t* cap_nodes, const int64_t* cap_edges, int32_t n_hops,
                         dci_blocks* b) {
  std::memset(b, 0, sizeof(*b));
  b->n_hops = n_hops;
  b->cap_nodes = cap_nodes[n_hops];
  b->nodes = reinterpret_cast<int64_t*>(ar.take<long long>((size_t)(cap_nodes[n_hops] > 0 ? cap_nodes[n_hops] : 1)));
  for (int32_t h = 0; h < n_hops; ++h) {
    b->cap_rows[h] = cap_nodes[h];
    b->cap_edges[h] = cap_edges[h];
    b->blk_indptr[h] = reinterpret_cast<int64_t*>(ar.take<long long>((size_t)cap_nodes[h] + 1));
    b->blk_src[h] = ar.take<int>((size_t)(cap_edges[h] > 0 ? cap_edges[h] : 1));
  }
  b->counts = reinterpret_cast<int64_t*>(ar.take<long long>(2 * DCI_MAX_HOPS + 1));
}

static int grid_for_rows(const dci_ctx* ctx, int64_t rows, int groups_per_block) {
  int64_t blocks = (rows + groups_per_block - 1) / groups_per_block;
  int64_t cap = (int64_t)ctx->num_cus * 8;
  if (blocks > cap) blocks = cap;
  if (blocks < 1) blocks = 1;
  return (int)blocks;
}

// frontier: as for k_sample_hop
template <int G, bool DIRECT>
static int32_t launch_hop(dci_ctx* ctx, const HopArgs& ha, RelabelArgs& ra, bool count, int frontier, int64_t cap_rows) {
  const int grid = grid_for_rows(ctx, cap_rows, kBlock / G) + ha.n_write_blocks;
  {
    Timed t(ctx, DCI_K_SAMPLE);
    auto* const kernel = frontier == kSeeds          ? (count ? k_sample_hop<G, true, kSeeds, DIRECT> : k_sample_hop<G, false, kSeeds, DIRECT>)
                         : frontier == kUnregistered ? (count ? k_sample_hop<G, true, kUnregistered, DIRECT> : k_sample_hop<G, false, kUnregistered, DIRECT>)
                                                     : (count ? k_sample_hop<G, true, kRegistered, DIRECT> : k_sample_hop<G, false, kRegistered, DIRECT>);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kBlock), 0, ctx->stream, ha);
  }
  DCI_LAUNCH_CHECK(ctx);
  {
    Timed t(ctx, DCI_K_RELABEL);
    const int iters = tile_iters_for(ctx, ha.hop, cap_rows, ha.fanout);
    // (tiles of the most rows need more registers than that many places leave, and are many: tickets, but for a single one)
    ra.unticketed = iters < kTileItersMax ? unticketed_tiles(ctx->num_cus) : 1;
    const dim3 grid_r((unsigned)tiles_for(cap_rows, ha.fanout, iters));
    if (iters == 1)
      hipLaunchKernelGGL((k_relabel_hop<G, 1, DIRECT>), grid_r, dim3(kRelabelBlock), 0, ctx->stream, ra);
    else if (iters == 2)
      hipLaunchKernelGGL((k_relabel_hop<G, 2, DIRECT>), grid_r, dim3(kRelabelBlock), 0, ctx->stream, ra);
    else if (iters == 4)
      hipLaunchKernelGGL((k_relabel_hop<G, 4, DIRECT>), grid_r, dim3(kRelabelBlock), 0, ctx->stream, ra);
    else
      hipLaunchKernelGGL((k_relabel_hop<G, 8, DIRECT>), grid_r, dim3(kRelabelBlock), 0, ctx->stream, ra);
  }
  DCI_LAUNCH_CHECK(ctx);
  return DCI_OK;
}

template <int G>
static void launch_first(dci_ctx* ctx, const FirstArgs& fa, bool count) {
  const int64_t want = (int64_t)((fa.clear_n16 + kFirstThreads - 1) / kFirstThreads), most = (int64_t)ctx->num_cus * 2;
  hipLaunchKernelGGL((count ? k_first_hops<G, true> : k_first_hops<G, false>), dim3((unsigned)(1 + (want < most ? want : most))),
                     dim3(kFirstThreads), 0, ctx->stream, fa);
}

// How many of the batch's hops k_first_hops makes.
static int first_hops(int64_t n_seeds, const int32_t* fanouts, int32_t n_hops, const dci_blocks* out, int* group) {
  int n = 0, g = 8;
  if (n_seeds < 1) return 0;
  for (int32_t h = 0; h + 1 < n_hops; ++h) {
    if (group_for(fanouts[h]) > g) g = group_for(fanouts[h]);
    if (out->cap_rows[h] * g > kFirstSlots || out->cap_rows[h + 1] > kFirstNodes) break;
    n = h + 1;
    *group = g;
  }
  return n;
}

// Enqueues the sampling of one batch: one clear, two kernels per hop (or one kernel for the clear and the first hops), one closing kernel.
// `adj_count` non-null turns on the pre-sampling counters.  left (nullable; neither counters nor statistics then): the closing is left
// to the caller.
static int32_t sample_batch(dci_ctx* ctx, const dci_graph* g, const dci_cache* cache, const int64_t* seeds,
                            int64_t n_seeds, uint64_t batch_index, const int32_t* fanouts, int32_t n_hops,
                            uint64_t rng_seed, const dci_blocks* out, const SampleWs& ws, uint64_t* stats,
                            uint32_t* feat_count, uint32_t* adj_count, uint32_t* edge_count, CloseArgs* left = nullptr) {
  int rc = DCI_OK, first_group = 8;
  const int n_first = first_hops(n_seeds, fanouts, n_hops, out, &first_group);
  if (n_first == 0) {
    Timed t(ctx, DCI_K_TABLE_CLEAR);
    rc = fill_bytes(ctx, ws.table, ws.clear_bytes, 0xFFFFFFFFu);
  }
  if (rc != DCI_OK) return rc;
  long long* counts = reinterpret_cast<long long*>(out->counts);
  long long* nodes = reinterpret_cast<long long*>(out->nodes);
  const bool count = adj_count != nullptr;
  for (int32_t h = n_first > 0 ? n_first - 1 : 0; h < n_hops; ++h) {
    HopArgs ha;
    ha.seeds = reinterpret_cast<const long long*>(seeds);
    ha.n_seeds = n_seeds;
    ha.nodes = nodes;
    ha.counts = counts;
    ha.hop = h;
    ha.fanout = fanouts[h];
    ha.indptr = reinterpret_cast<const long long*>(g->indptr);
    ha.indices = reinterpret_cast<const long long*>(g->indices);
    ha.adj_remap = cache ? cache->adj_remap : nullptr;
    ha.c_indptr = cache ? reinterpret_cast<const long long*>(cache->c_indptr) : nullptr;
    ha.c_indices = cache ? reinterpret_cast<const long long*>(cache->c_indices) : nullptr;
    ha.partial_node = cache ? cache->adj_partial_node : -1;
    ha.partial_deg = cache ? cache->adj_partial_deg : 0;
    ha.k0 = (unsigned)rng_seed;
    ha.k1 = (unsigned)(rng_seed >> 32);
    ha.batch = (unsigned)batch_index;
    ha.tmp_u = ws.tmp_u;
    ha.tmp_slot = ws.tmp_slot[h & 1];
    ha.row_cnt = ws.row_cnt[h & 1];
    ha.table = ws.table;
    ha.entries = (unsigned)ws.table_entries;
    ha.shift = ws.table_shift;
    ha.last_node = (unsigned)(g->num_nodes - 1);
    ha.adj_count = adj_count;
    ha.edge_count = edge_count;
    const bool first = h < n_first, finished = h <= n_first;  // the hop is k_first_hops'; the hop before has its edge ids
    ha.prev_fanout = h > 0 ? fanouts[h - 1] : 1;
    ha.prev_tmp_slot = ws.tmp_slot[(h + 1) & 1];
    ha.prev_blk_indptr = h > 0 ? reinterpret_cast<const long long*>(out->blk_indptr[h - 1]) : nullptr;
    ha.prev_blk_src = h > 0 ? out->blk_src[h - 1] : nullptr;
    ha.n_write_blocks = !finished ? grid_for_rows(ctx, out->cap_rows[h - 1] * fanouts[h - 1], kBlock * 4) : 0;
    ha.batch_flag = ws.batch_flag;
    ha.count_lines = stats ? 1 : 0;
    ha.row_memo = ws.row_memo;
    ha.last_hop = h == n_hops - 1 ? 1 : 0;
    ha.cap_rows = out->cap_rows[h];
    if (first) {
      FirstArgs fa;
      fa.a = ha;
      fa.n_hops = n_first;
      for (int32_t k = 0; k < n_first; ++k) {
        fa.fanout[k] = fanouts[k];
        fa.blk_indptr[k] = reinterpret_cast<long long*>(out->blk_indptr[k]);
        fa.blk_src[k] = out->blk_src[k];
        fa.stat_part[k] = stats ? ws.stat_part[k] : nullptr;
      }
      fa.clear = reinterpret_cast<uint4*>(ws.table);
      fa.clear_n16 = ws.clear_bytes / 16;  // (16-byte words: carve_sample_ws)
      Timed t(ctx, DCI_K_SAMPLE);
      switch (first_group) {
        case 8: launch_first<8>(ctx, fa, count); break;
        case 16: launch_first<16>(ctx, fa, count); break;
        case 32: launch_first<32>(ctx, fa, count); break;
        default: launch_first<64>(ctx, fa, count); break;
      }
      DCI_LAUNCH_CHECK(ctx);
      continue;
    }
    const int frontier = h == 0 ? kSeeds : h == n_first ? kUnregistered : kRegistered;
    RelabelArgs ra;
    ra.counts = counts;
    ra.hop = h;
    ra.fanout = fanouts[h];
    ra.row_cnt = ws.row_cnt[h & 1];
    ra.tmp_u = ws.tmp_u;
    ra.tmp_slot = ws.tmp_slot[h & 1];
    ra.table = ws.table;
    ra.shift = ws.table_shift;
    ra.nodes = nodes;
    ra.blk_indptr = reinterpret_cast<long long*>(out->blk_indptr[h]);
    ra.blk_src = out->blk_src[h];
    ra.status = ws.status[h];
    ra.ticket = ws.ticket + h;
    ra.stat_part = stats ? ws.stat_part[h] : nullptr;
    ra.batch_flag = ws.batch_flag;
    ra.spin_limit = ctx->relabel_spin_limit;
    ra.first_ticket = ctx->test_first_ticket;
    // launch shapes follow the frontier bound of this call; with zero seeds one workgroup still
    // runs so that the (empty) sizes get written
    const int64_t rows = out->cap_rows[h];
    switch (group_for(fanouts[h])) {
      case 8: rc = (ws.direct ? launch_hop<8, true> : launch_hop<8, false>)(ctx, ha, ra, count, frontier, rows); break;
      case 16: rc = (ws.direct ? launch_hop<16, true> : launch_hop<16, false>)(ctx, ha, ra, count, frontier, rows); break;
      case 32: rc = (ws.direct ? launch_hop<32, true> : launch_hop<32, false>)(ctx, ha, ra, count, frontier, rows); break;
      default: rc = (ws.direct ? launch_hop<64, true> : launch_hop<64, false>)(ctx, ha, ra, count, frontier, rows); break;
    }
    if (rc != DCI_OK) return rc;
  }
  {
    const int32_t h = n_hops - 1;
    const int64_t positions = out->cap_rows[h] * fanouts[h];
    CloseArgs close;
    close.counts = counts;
    close.hop = h;
    close.fanout = fanouts[h];
    close.tmp_slot = ws.tmp_slot[h & 1];
    close.blk_indptr = reinterpret_cast<const long long*>(out->blk_indptr[h]);
    close.table = ws.table;
    close.shift = ws.table_shift;
    close.blk_src = out->blk_src[h];
    close.counts_host = reinterpret_cast<long long*>(out->counts_host);
    close.batch_flag = ws.batch_flag;
    close.host_flag = ctx->host_flag;
    close.direct = ws.direct;
    close.wgs = grid_for_rows(ctx, positions, kBlock);
    if (left) {
      // beside other work no more workgroups than two to a compute unit: as many as for a launch of its own (eight) keep the copy from
      // starting (a pass over 798 k edges, all rows gathered, 314 us, with two 308)
      if (close.wgs > kCloseBesidePerCu * ctx->num_cus) close.wgs = kCloseBesidePerCu * ctx->num_cus;
      *left = close;
      return DCI_OK;
    }
    StatFold sf;
    sf.stats = reinterpret_cast<unsigned long long*>(stats);
    sf.n_hops = n_hops;
    for (int32_t k = 0; k < DCI_MAX_HOPS; ++k) {
      sf.part[k] = k < n_hops ? ws.stat_part[k] : nullptr;
      sf.tile_rows[k] = k < n_first ? kFirstThreads : k < n_hops ? (kRelabelBlock / group_for(fanouts[k])) * tile_iters_for(ctx, k, out->cap_rows[k], fanouts[k]) : 1;
    }
    Timed t(ctx, feat_count ? DCI_K_COUNT_NODES : DCI_K_WRITE_SRC);
    hipLaunchKernelGGL(ws.direct ? k_write_src<true> : k_write_src<false>, dim3(close.wgs), dim3(kBlock), 0, ctx->stream, close, sf,
                       (const long long*)nodes, n_hops, feat_count);
  }
  DCI_LAUNCH_CHECK(ctx);
  return DCI_OK;
}

static int32_t check_common(dci_ctx* ctx, const dci_graph* g, const int64_t* seeds, int64_t n_seeds,
                            const int32_t* fanouts, int32_t n_hops, uint64_t last_batch_index) {
  if (!g || !g->indptr || !g->indices || g->num_nodes < 1 || g->num_edges < 0)
    return fail(ctx, DCI_ERR_INVALID_ARG, "graph: null arrays or bad sizes");
  if (g->num_nodes >= ((int64_t)1 << 31)) return fail(ctx, DCI_ERR_UNSUPPORTED, "more than 2^31-1 nodes");
  if (n_seeds < 0 || (!seeds && n_seeds > 0)) return fail(ctx, DCI_ERR_INVALID_ARG, "seeds: null or negative count");
  if (!fanouts || n_hops < 1 || n_hops > DCI_MAX_HOPS)
    return fail(ctx, DCI_ERR_INVALID_ARG, "n_hops must be 1..%d", DCI_MAX_HOPS);
  for (int32_t h = 0; h < n_hops; ++h)
    if (fanouts[h] < 1 || fanouts[h] > DCI_MAX_FANOUT)
      return fail(ctx, DCI_ERR_INVALID_ARG, "fanouts[%d] = %d outside 1..%d", h, fanouts[h], DCI_MAX_FANOUT);
  if (last_batch_index >> 32) return fail(ctx, DCI_ERR_INVALID_ARG, "batch index must be below 2^32");
  return DCI_OK;
}

static int32_t check_cache(dci_ctx* ctx, const dci_cache* cache) {
  if (cache && (!cache->adj_remap || !cache->feat_remap || (cache->adj_nodes > 0 && (!cache->c_indptr || (cache->adj_edges > 0 && !cache->c_indices)))))
    return fail(ctx, DCI_ERR_INVALID_ARG, "cache: null arrays");
  return DCI_OK;
}

}  // namespace dci

using namespace dci;

extern "C" {

size_t dci_sample_workspace_bytes(int64_t num_nodes, int64_t n_seeds, const int32_t* fanouts, int32_t n_hops) {
  int64_t cap_nodes[DCI_MAX_HOPS + 1], cap_edges[DCI_MAX_HOPS];
  if (dci_blocks_bounds(num_nodes, n_seeds, fanouts, n_hops, cap_nodes, cap_edges) != DCI_OK) return 0;
  Arena ar(nullptr, 0);
  SampleWs ws;
  dci_blocks b;
  carve_sample_ws(ar, num_nodes, cap_nodes, cap_edges, fanouts, n_hops, &ws);
  carve_blocks(ar, cap_nodes, cap_edges, n_hops, &b);
  (void)ar.take<char>(256 * 1024);  // room for the gather statistics of the pre-sampling pass
  return ar.off;
}

}  // extern "C"

namespace dci {

// Shared body of dci_sample_khop, dci_sample_khop_static and infer_joint: they differ in where the
// temporaries live (`ws_base`, `ws_bytes`; `ws_name` names that memory in the error message) and in who closes the batch.
int32_t sample_khop_in(dci_ctx* ctx, const dci_graph* graph, const dci_cache* cache, const int64_t* seeds,
                       int64_t n_seeds, uint64_t batch_index, const int32_t* fanouts, int32_t n_hops,
                       uint64_t rng_seed, dci_blocks* out, uint64_t* stats, char* ws_base, size_t ws_bytes,
                       const char* ws_name, CloseArgs* close) {
  int32_t rc = check_common(ctx, graph, seeds, n_seeds, fanouts, n_hops, batch_index);
  if (rc != DCI_OK) return rc;
  if ((rc = check_cache(ctx, cache)) != DCI_OK) return rc;
  if (!out || !out->nodes || !out->counts || out->n_hops != n_hops)
    return fail(ctx, DCI_ERR_INVALID_ARG, "blocks: null arrays or n_hops mismatch");
  int64_t cap_nodes[DCI_MAX_HOPS + 1], cap_edges[DCI_MAX_HOPS];
  rc = dci_blocks_bounds(graph->num_nodes, n_seeds, fanouts, n_hops, cap_nodes, cap_edges);
  if (rc != DCI_OK) return fail(ctx, rc, "batch bounds reach 2^31");
  {  // remembered for dci_last_required, should one of the capacity checks below fail
    Arena probe(nullptr, 0);
    SampleWs unused;
    carve_sample_ws(probe, graph->num_nodes, cap_nodes, cap_edges, fanouts, n_hops, &unused);
    std::memset(ctx->req_nodes, 0, sizeof(ctx->req_nodes));
    std::memset(ctx->req_edges, 0, sizeof(ctx->req_edges));
    for (int32_t h = 0; h <= n_hops; ++h) ctx->req_nodes[h] = cap_nodes[h];
    for (int32_t h = 0; h < n_hops; ++h) ctx->req_edges[h] = cap_edges[h];
    ctx->req_workspace = probe.off;
  }
  if (out->cap_nodes < cap_nodes[n_hops])
    return fail(ctx, DCI_ERR_CAPACITY, "blocks.nodes holds %lld entries, %lld needed", (long long)out->cap_nodes,
                (long long)cap_nodes[n_hops]);
  for (int32_t h = 0; h < n_hops; ++h) {
    if (!out->blk_indptr[h] || !out->blk_src[h]) return fail(ctx, DCI_ERR_INVALID_ARG, "blocks: null array at hop %d", h);
    if (out->cap_rows[h] < cap_nodes[h] || out->cap_edges[h] < cap_edges[h])
      return fail(ctx, DCI_ERR_CAPACITY, "block %d holds %lld rows / %lld edges, %lld / %lld needed", h,
                  (long long)out->cap_rows[h], (long long)out->cap_edges[h], (long long)cap_nodes[h],
                  (long long)cap_edges[h]);
  }
  Arena ar(ws_base, ws_bytes);
  SampleWs ws;
  carve_sample_ws(ar, graph->num_nodes, cap_nodes, cap_edges, fanouts, n_hops, &ws);
  if (!ar.ok())
    return fail(ctx, DCI_ERR_CAPACITY, "%s holds %zu bytes, sampling a batch of these bounds needs %zu", ws_name,
                ws_bytes, ar.off);
  // launch shapes follow the bounds of this call, not the (possibly larger) capacities
  dci_blocks view = *out;
  for (int32_t h = 0; h < n_hops; ++h) view.cap_rows[h] = cap_nodes[h];
  view.cap_nodes = cap_nodes[n_hops];
  return sample_batch(ctx, graph, cache, seeds, n_seeds, batch_index, fanouts, n_hops, rng_seed, &view, ws, stats,
                      nullptr, nullptr, nullptr, close);
}

}  // namespace dci

extern "C" {

int32_t dci_sample_khop(dci_ctx* ctx, const dci_graph* graph, const dci_cache* cache, const int64_t* seeds,
                        int64_t n_seeds, uint64_t batch_index, const int32_t* fanouts, int32_t n_hops,
                        uint64_t rng_seed, dci_blocks* out, uint64_t* stats) {
  if (!ctx) return DCI_ERR_INVALID_ARG;
  return sample_khop_in(ctx, graph, cache, seeds, n_seeds, batch_index, fanouts, n_hops, rng_seed, out, stats,
                        ctx->ws, ctx->ws_bytes, "workspace", nullptr);
}

int32_t dci_sample_khop_static(dci_ctx* ctx, const dci_graph* graph, const dci_cache* cache, const int64_t* seeds,
                               int64_t n_seeds, uint64_t batch_index, const int32_t* fanouts, int32_t n_hops,
                               uint64_t rng_seed, dci_blocks* out, uint64_t* stats) {
  if (!ctx) return DCI_ERR_INVALID_ARG;
  if (!ctx->static_scratch) return fail(ctx, DCI_ERR_HIP, "the static scratch array has no address on this device");
  return sample_khop_in(ctx, graph, cache, seeds, n_seeds, batch_index, fanouts, n_hops, rng_seed, out, stats,
                        ctx->static_scratch, (size_t)DCI_STATIC_SCRATCH_BYTES, "the static scratch array", nullptr);
}

size_t dci_sample_khop_scratch_bytes(int64_t num_nodes, int64_t n_seeds, const int32_t* fanouts, int32_t n_hops) {
  int64_t cap_nodes[DCI_MAX_HOPS + 1], cap_edges[DCI_MAX_HOPS];
  if (dci_blocks_bounds(num_nodes, n_seeds, fanouts, n_hops, cap_nodes, cap_edges) != DCI_OK) return 0;
  Arena ar(nullptr, 0);
  SampleWs ws;
  carve_sample_ws(ar, num_nodes, cap_nodes, cap_edges, fanouts, n_hops, &ws);
  return ar.off;
}

int32_t dci_presample_count(dci_ctx* ctx, const dci_graph* graph, const dci_cache* cache, const int64_t* seeds,
                            int64_t n_seeds, int32_t batch_size, int64_t first_batch, int64_t n_batches,
                            uint64_t rng_batch0, const int32_t* fanouts, int32_t n_hops, uint64_t rng_seed,
                            uint32_t* feat_count, uint32_t* adj_count, uint32_t* edge_count, float* feat_scratch,
                            uint64_t* stats) {
  if (!ctx) return DCI_ERR_INVALID_ARG;
  if (batch_size < 1 || first_batch < 0 || n_batches < 0)
    return fail(ctx, DCI_ERR_INVALID_ARG, "batch_size / first_batch / n_batches out of range");
  int32_t rc = check_common(ctx, graph, seeds, n_seeds, fanouts, n_hops,
                            rng_batch0 + (uint64_t)(n_batches > 0 ? n_batches - 1 : 0));
  if (rc != DCI_OK) return rc;
  if ((rc = check_cache(ctx, cache)) != DCI_OK) return rc;
  if (!feat_count || !adj_count) return fail(ctx, DCI_ERR_INVALID_ARG, "feat_count / adj_count are required");
  if (feat_scratch && !graph->feat) return fail(ctx, DCI_ERR_INVALID_ARG, "feat_scratch given but graph.feat is NULL");
  int64_t cap_nodes[DCI_MAX_HOPS + 1], cap_edges[DCI_MAX_HOPS];
  rc = dci_blocks_bounds(graph->num_nodes, batch_size, fanouts, n_hops, cap_nodes, cap_edges);
  if (rc != DCI_OK) return fail(ctx, rc, "batch bounds reach 2^31");
  Arena ar(ctx->ws, ctx->ws_bytes);
  SampleWs ws;
  dci_blocks blk;
  carve_sample_ws(ar, graph->num_nodes, cap_nodes, cap_edges, fanouts, n_hops, &ws);
  carve_blocks(ar, cap_nodes, cap_edges, n_hops, &blk);
  void* gather_partials = ar.take<char>(gather_partials_bytes(ctx));
  if (!ar.ok())
    return fail(ctx, DCI_ERR_CAPACITY, "workspace holds %zu bytes, pre-sampling needs %zu", ctx->ws_bytes, ar.off);
  // The batches run back to back: the stage times come from events between them, read once per kPresampleRun batches
  // (a wait after every batch left the GPU idle for the length of the host's round trip), and the gather's
  // statistics are folded once per run.
  double ms_sample = 0.0, ms_feature = 0.0;
  int64_t batches = (n_seeds + batch_size - 1) / batch_size - first_batch;  // those that have seeds
  if (batches > n_batches) batches = n_batches;
  for (int64_t i = 0; feat_scratch && i <= 2 * (batches < kPresampleRun ? batches : kPresampleRun); ++i)
    if (!ctx->ev[i]) DCI_HIP(ctx, hipEventCreate(&ctx->ev[i]));
  int in_run = 0;
  for (int64_t k = 0; k < batches; ++k) {
    const int64_t lo = (first_batch + k) * batch_size;
    const int64_t hi = lo + batch_size < n_seeds ? lo + batch_size : n_seeds;
    if (feat_scratch && in_run == 0) DCI_HIP(ctx, hipEventRecord(ctx->ev[0], ctx->stream));
    rc = sample_batch(ctx, graph, cache, seeds + lo, hi - lo, rng_batch0 + (uint64_t)k, fanouts, n_hops, rng_seed,
                      &blk, ws, stats, feat_count, adj_count, edge_count);
    if (rc != DCI_OK) return rc;
    if (!feat_scratch) continue;
    const bool last = in_run + 1 == kPresampleRun || k + 1 == batches;
    DCI_HIP(ctx, hipEventRecord(ctx->ev[2 * in_run + 1], ctx->stream));
    rc = gather_launch(ctx, graph, cache, blk.nodes, cap_nodes[n_hops], blk.counts + n_hops, feat_scratch, stats,
                       gather_partials, nullptr, nullptr, 0, in_run > 0, last);
    if (rc != DCI_OK) return rc;
    DCI_HIP(ctx, hipEventRecord(ctx->ev[2 * in_run + 2], ctx->stream));
    ++in_run;
    if (!last) continue;
    DCI_HIP(ctx, hipEventSynchronize(ctx->ev[2 * in_run]));
    if ((rc = check_device_flag(ctx)) != DCI_OK) return rc;
    for (int j = 0; j < in_run; ++j) {
      float a = 0.f, b = 0.f;
      DCI_HIP(ctx, hipEventElapsedTime(&a, ctx->ev[2 * j], ctx->ev[2 * j + 1]));
      DCI_HIP(ctx, hipEventElapsedTime(&b, ctx->ev[2 * j + 1], ctx->ev[2 * j + 2]));
      ms_sample += a;
      ms_feature += b;
    }
    in_run = 0;
  }
  if (feat_scratch && stats) {
    unsigned long long* st = reinterpret_cast<unsigned long long*>(stats);
    hipLaunchKernelGGL(k_add_u64, dim3(1), dim3(1), 0, ctx->stream, st + DCI_STAT_T_SAMPLE_NS,
                       (unsigned long long)(ms_sample * 1.0e6));
    DCI_LAUNCH_CHECK(ctx);
    hipLaunchKernelGGL(k_add_u64, dim3(1), dim3(1), 0, ctx->stream, st + DCI_STAT_T_FEATURE_NS,
                       (unsigned long long)(ms_feature * 1.0e6));
    DCI_LAUNCH_CHECK(ctx);
  }
  return DCI_OK;
}

}  // extern "C"

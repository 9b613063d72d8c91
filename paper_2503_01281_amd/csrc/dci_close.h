// Closing a batch: what the sampler's last kernel does, or workgroups of the gather's launch.
#ifndef DCI_CLOSE_H_
#define DCI_CLOSE_H_

#include "dci_internal.h"

namespace dci {

// One 64-bit word per entry of a hashed node table: node id in the high half, value in the low half, all ones =
// empty.  Node ids are below 2^31, so a real entry is always smaller than the empty word.
typedef unsigned long long HashEntry;

// The value of a slot: the low half (little endian) of a hashed table's word, or the first of the 2^shift 32-bit words
// that a direct table has per node (its slot is the node's id).  The kind is a template parameter throughout: the kernels of
// small batches are bound by latency, code fetch included, and with the kind as a branch at run time the hashed ones were a
// third longer (six batches of 27 seeds 486 us, as a template 479; 485 seeds 117.2 and 115.3).
template <bool DIRECT>
__device__ __forceinline__ unsigned entry_val(const HashEntry* table, unsigned shift, unsigned slot) {
  return reinterpret_cast<const unsigned*>(table)[(size_t)slot << (DIRECT ? shift : 1u)];
}

// tmp_slot encoding: s >= 0 a table slot whose value this edge may still own; -1 no edge at this
// position; kSlotDone an edge whose local id the relabel kernel has already written (it was its node's first
// appearance); any other s <= -2 the slot -2 - s of an edge that cannot be its node's first appearance.
constexpr int kSlotDone = (int)0x80000000;
__device__ __forceinline__ unsigned slot_of(int s) { return (unsigned)(s >= 0 ? s : -2 - s); }

// Batch status word (in the region that the per-batch clear fills with ones): all ones = fine; anything
// else = a relabel tile gave up waiting for its predecessors, the batch's outputs are void.
constexpr unsigned kBatchOk = 0xFFFFFFFFu;

// blk_src of a finished hop: every edge reads the (by now final) local id of its source.
// One thread per padded position row * fanout + slot (fewer than 2^31 of them).
template <bool DIRECT>
__device__ __forceinline__ void write_block_sources(long long n_rows, int fanout, const int* __restrict__ tmp_slot,
                                                    const long long* __restrict__ blk_indptr,
                                                    const HashEntry* table, unsigned shift,
                                                    int* __restrict__ blk_src,
                                                    int block, int n_blocks) {
  const unsigned total = (unsigned)(n_rows * fanout), step = (unsigned)n_blocks * blockDim.x;
  for (unsigned q = (unsigned)block * blockDim.x + threadIdx.x; q < total; q += step) {
    const unsigned i = q / (unsigned)fanout;
    const int ts = tmp_slot[q];
    const long long first = blk_indptr[i];
    if (ts != -1 && ts != kSlotDone) blk_src[first + (q - i * fanout)] = (int)entry_val<DIRECT>(table, shift, slot_of(ts));
  }
}

// Workgroup `block` of `n_blocks` that close a batch: the last hop's edge ids, and the batch's sizes for the host.  false: a relabel
// tile timed out and the batch is void.  Its sizes are zeroed so that whatever consumes the batch next (gather, forward) finds
// nothing to do, and the context's host flag is raised for dci_sync.
template <bool DIRECT>
__device__ __forceinline__ bool close_batch(const CloseArgs& a, int block, int n_blocks) {
  if (*a.batch_flag != kBatchOk) {
    if (block == 0 && threadIdx.x < 2 * DCI_MAX_HOPS + 1) {
      a.counts[threadIdx.x] = 0;
      if (a.counts_host) a.counts_host[threadIdx.x] = 0;
      if (threadIdx.x == 0) *a.host_flag = 1u;
    }
    return false;
  }
  write_block_sources<DIRECT>(a.counts[a.hop], a.fanout, a.tmp_slot, a.blk_indptr, reinterpret_cast<const HashEntry*>(a.table), a.shift,
                              a.blk_src, block, n_blocks);
  if (a.counts_host && block == 0 && threadIdx.x < 2 * DCI_MAX_HOPS + 1)
    a.counts_host[threadIdx.x] = a.counts[threadIdx.x];  // pinned host memory, visible once the stream is idle
  return true;
}

}  // namespace dci

#endif  // DCI_CLOSE_H_

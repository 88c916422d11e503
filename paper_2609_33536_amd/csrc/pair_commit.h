// Table updates of a transition made in its data launch (internal header;
// also compiled for the host).  One tile's workgroup of each pair, the
// committing one, updates the pair's second table entry; the pair's other
// tiles may read the entry before or after that.
//  - A refinement only checks the entry that changes, and both its values pass
//    or fail together.
//  - A demotion needs member 1's block, which the update overwrites.  The
//    committing workgroup reads the entry, writes the block to freed[i], and
//    only once that write is in memory overwrites the entry with member 0's
//    block.  So a tile that finds the entry equal to member 0's block, as no
//    TARGET pair's is, finds member 1's in freed[i].
// Pair: load_entry, store_entry, load_freed, store_freed (on the device,
// accesses past the caches).
#pragma once

#include <hip/hip_runtime.h>

namespace ekv {

__host__ __device__ inline bool in_pool(int block, int num_blocks) { return (unsigned)block < (unsigned)num_blocks; }

// Demotion: member 1's block, or false (a skipped entry: nothing is freed).
// b0: member 0's block.
template <class Pair>
__host__ __device__ inline bool demotion_block(Pair& pair, bool commits, int b0, int num_blocks, int& b1) {
  b1 = pair.load_entry();
  const bool ok = in_pool(b0, num_blocks) && in_pool(b1, num_blocks);
  if (commits) {
    pair.store_freed(ok ? b1 : -1);
  } else if (ok && b1 == b0) {   // already updated
    b1 = pair.load_freed();
    return in_pool(b1, num_blocks);
  }
  return ok;
}

// Refinement: whether the pair is rebuilt.
template <class Pair>
__host__ __device__ inline bool refinement_ok(Pair& pair, int b0, int new_block, int num_blocks) {
  return in_pool(b0, num_blocks) && in_pool(pair.load_entry(), num_blocks) && in_pool(new_block, num_blocks);
}

}  // namespace ekv

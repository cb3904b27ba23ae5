// Which tree row the chunk-score kernels (retrieval.hip) score.  Callable on the host too, so that its reads can be run there
// against buffers of exact size.
#pragma once

#include <hip/hip_runtime.h>

namespace specext {

// path null: first_row.  Else the acceptance walk's last accepted node, path[*count - 1]; row 0 when nothing was accepted or the
// entry is no node.  A path may be as short as its accepted entries, so no other entry is read, and this one only when the count
// is there: two trips to memory.  (One trip for all n_tree entries and the count: equal where the path is in the L2, 2.72 us per
// launch of 512 chunks, and at most 0.2 us faster in an iteration: 33.65 against 33.85 us with 257 chunks of 16 keys, 22.83 either
// way with 64.)
__host__ __device__ __forceinline__ int scored_row(const int* path, const int* count, int n_tree, int first_row) {
  if (!path) return first_row;
  const int accepted = *count < n_tree ? *count : n_tree;        // never past the tree, whatever the count says
  const int node = accepted > 0 ? path[accepted - 1] : 0;
  return node >= 0 && node < n_tree ? node : 0;
}

}  // namespace specext

// Which tree row the chunk-score kernels (retrieval.hip) score.  Callable on the host too, so that its reads can be run there
// against buffers of exact size.
#pragma once

#include <hip/hip_runtime.h>

namespace specext {

// path null: first_row.  Else the acceptance walk's last accepted node, path[*count - 1]; row 0 when nothing was accepted or the
// entry is no node.  A path may be as short as its accepted entries, so no other entry is read, and this one only when the count
// is there: two trips to memory, which cost nothing against one for all n_tree entries and the count (2.72 us per launch of 512
// chunks either way, 3.22 of two score blocks).
__host__ __device__ __forceinline__ int scored_row(const int* path, const int* count, int n_tree, int first_row) {
  if (!path) return first_row;
  const int accepted = *count < n_tree ? *count : n_tree;        // never past the tree, whatever the count says
  const int node = accepted > 0 ? path[accepted - 1] : 0;
  return node >= 0 && node < n_tree ? node : 0;
}

}  // namespace specext

// What one thread of the commit kernel (accept.hip) copies.  A function of its thread and workgroup numbers, callable
// on the host too, so that its indexing can be run there against buffers of exact size.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

namespace specext {

constexpr int kCommitThreads = 256;

// V: a 16-byte vector.  The accepted rows of K and V of head `lh` (layer * n_kv_heads + head) are items
// (row, K or V, 16-byte piece), K and V of a row next to each other; the `shares` workgroups of the head take them in turns.
// path has min(max_accept, n_tree) entries at least; entries behind the accepted ones may be read, never used.
template <class V>
__host__ __device__ __forceinline__ void commit_rows(const V* __restrict__ k_tree, const V* __restrict__ v_tree,
                                                     V* __restrict__ k_cache, V* __restrict__ v_cache,
                                                     const int* __restrict__ path, const int* __restrict__ n_accept,
                                                     int max_accept, int n_tree, int n_kv_heads, int prefix_len, int row_vecs,
                                                     int64_t tree_sl, int64_t tree_sh, int64_t tree_st, int64_t cache_sy,
                                                     int64_t cache_sh, int64_t cache_sl, int thread, int lh, int share,
                                                     int shares) {
  int item = share * kCommitThreads + thread;
  int row = item / (2 * row_vecs);
  // requested with the count and before it is known; the launch bound may exceed the tree, whose size the path has
  const int known = max_accept < n_tree ? max_accept : n_tree;
  int node = path[row < known ? row : known - 1];
  int n = *n_accept;
  n = n < 0 ? 0 : n < max_accept ? n : max_accept;
  if (row >= known && row < n) node = path[row];
  const int layer = lh / n_kv_heads;
  const int g = lh - layer * n_kv_heads;
  const int64_t src0 = layer * tree_sl + g * tree_sh;
  const int64_t dst0 = layer * cache_sy + g * cache_sh + static_cast<int64_t>(prefix_len) * cache_sl;
  while (row < n) {
    if (node >= 0 && node < n_tree) {
      int piece = item - row * (2 * row_vecs);
      const bool is_v = piece >= row_vecs;
      if (is_v) piece -= row_vecs;
      const V* src = (is_v ? v_tree : k_tree) + src0 + node * tree_st;
      V* dst = (is_v ? v_cache : k_cache) + dst0 + row * cache_sl;
      dst[piece] = src[piece];
    }
    item += shares * kCommitThreads;
    row = item / (2 * row_vecs);
    if (row < n) node = path[row];
  }
}

}  // namespace specext

// What follows the attention in one verification step (SpecExtend Alg. 1): the
// Verify / Correct loop at temperature 0 walked down the draft tree, and the commit of
// the accepted tree tokens' K/V rows into the target cache.
#include "commit_rows.h"
#include "common.h"

namespace specext {
namespace {

// One wavefront; lane i holds nodes i and i + 64 (n_tree <= 128).  At each step the
// children of the current node that carry the wanted token are found with two ballots,
// the lowest index wins, and the next wanted token is read across lanes.  At most
// n_tree steps, so the walk also ends on a malformed parent array.
__global__ __launch_bounds__(64) void accept_greedy_kernel(uint64_t parent_at, uint64_t draft_at, uint64_t target_at,
                                                          uint64_t first_at, int n_tree, uint64_t path_at, uint64_t n_accept_at,
                                                          uint64_t next_at) {
  const int* __restrict__ parent = in_global<const int>(parent_at);
  const int* __restrict__ draft_token = in_global<const int>(draft_at);
  const int* __restrict__ target_token = in_global<const int>(target_at);
  const int* __restrict__ first_target = in_global<const int>(first_at);
  int* __restrict__ path_out = in_global<int>(path_at);
  int* __restrict__ n_accept_out = in_global<int>(n_accept_at);
  int* __restrict__ next_token_out = in_global<int>(next_at);
  const int lane = threadIdx.x;
  const bool has0 = lane < n_tree, has1 = lane + 64 < n_tree;
  const int par0 = has0 ? parent[lane] : -2, par1 = has1 ? parent[lane + 64] : -2;
  const int tok0 = has0 ? draft_token[lane] : 0, tok1 = has1 ? draft_token[lane + 64] : 0;
  const int tgt0 = has0 ? target_token[lane] : 0, tgt1 = has1 ? target_token[lane + 64] : 0;
  int cur = -1;
  int want = *first_target;
  int n = 0;
  for (int step = 0; step < n_tree; ++step) {
    const uint64_t m0 = __ballot(has0 && par0 == cur && tok0 == want);
    const uint64_t m1 = __ballot(has1 && par1 == cur && tok1 == want);
    int c;
    if (m0) c = __builtin_ctzll(m0);
    else if (m1) c = 64 + __builtin_ctzll(m1);
    else break;
    if (lane == 0) path_out[n] = c;
    ++n;
    cur = c;
    want = c < 64 ? __builtin_amdgcn_readlane(tgt0, c) : __builtin_amdgcn_readlane(tgt1, c - 64);
  }
  for (int i = n + lane; i < n_tree; i += 64) path_out[i] = -1;
  if (lane == 0) {
    *n_accept_out = n;
    *next_token_out = want;
  }
}

// grid (layers * KV heads, shares): the workgroups of one (layer, head) copy its accepted rows of K and of V, 16 bytes per
// thread and pass, a row of 256 bytes by 16 threads.  What bounds it is the launch and two trips to memory (the
// accepted count and path, then the rows): so the count and the thread's first path entry are requested together, and
// there is no workgroup per row that may be accepted - 60-node tree, 32 layers of 8 heads: 30720 workgroups, nearly all of
// which found nothing to do, took 8.1 us, these 512 take 2.1 us.  Few rows are accepted as a rule and one share would do; of
// a long accepted chain it takes a pass after the other, hence several shares where the heads leave compute units
// idle: 128 of 128 rows, one layer of 8 heads 7.4 us with one share, 2.1 us with sixteen; 60 of 60 rows, 32 layers
// 5.5 us with one, 4.3 us with two.
constexpr int kCommitBlocks = 512;               // two per compute unit; beyond, the empty ones cost time
// (One struct: twenty arguments of their own, the first ones in registers, took 0.1 us more.)
struct CommitArgs {
  const int *path, *n_accept;
  const uint4 *k_tree, *v_tree;
  uint4 *k_cache, *v_cache;
  int64_t tree_sl, tree_sh, tree_st, cache_sy, cache_sh, cache_sl;      // in 16-byte vectors
  int32_t max_accept, n_tree, row_vecs, n_kv_heads, prefix_len, shares;
};
__global__ __launch_bounds__(kCommitThreads) void commit_tree_kv_kernel(CommitArgs c) {
  commit_rows(c.k_tree, c.v_tree, c.k_cache, c.v_cache, c.path, c.n_accept, c.max_accept, c.n_tree, c.n_kv_heads, c.prefix_len,
              c.row_vecs, c.tree_sl, c.tree_sh, c.tree_st, c.cache_sy, c.cache_sh, c.cache_sl, threadIdx.x, blockIdx.x, blockIdx.y,
              c.shares);
}

}  // namespace

hipError_t launch_accept_greedy(const int32_t* parent, const int32_t* draft_token, const int32_t* target_token,
                                const int32_t* first_target, int32_t n_tree, int32_t* path_out,
                                int32_t* n_accept_out, int32_t* next_token_out, hipStream_t stream) {
  return launch_kernel(accept_greedy_kernel, dim3(1), dim3(64), 0, stream, address_of(parent), address_of(draft_token),
                       address_of(target_token), address_of(first_target), n_tree, address_of(path_out),
                       address_of(n_accept_out), address_of(next_token_out));
}

hipError_t launch_commit_tree_kv(const void* k_tree, const void* v_tree, void* k_cache, void* v_cache,
                                 const int32_t* path, const int32_t* n_accept, int32_t max_accept, int32_t n_tree,
                                 int32_t n_layers, int32_t n_kv_heads, int32_t prefix_len, int32_t row_bytes,
                                 int64_t tree_sl_bytes, int64_t tree_sh_bytes, int64_t tree_st_bytes,
                                 int64_t cache_sy_bytes, int64_t cache_sh_bytes, int64_t cache_sl_bytes,
                                 hipStream_t stream) {
  if (max_accept <= 0) return hipSuccess;
  // several workgroups per (layer, head) while they are no more than kCommitBlocks in all and have a pass each
  const int64_t heads = static_cast<int64_t>(n_layers) * n_kv_heads;
  const int64_t passes = (static_cast<int64_t>(max_accept) * 2 * (row_bytes / 16) + kCommitThreads - 1) / kCommitThreads;
  int64_t share = heads < kCommitBlocks ? kCommitBlocks / heads : 1;
  if (share > passes) share = passes;
  if (share < 1) share = 1;
  const CommitArgs c = {path, n_accept, static_cast<const uint4*>(k_tree), static_cast<const uint4*>(v_tree),
                        static_cast<uint4*>(k_cache), static_cast<uint4*>(v_cache), tree_sl_bytes / 16, tree_sh_bytes / 16,
                        tree_st_bytes / 16, cache_sy_bytes / 16, cache_sh_bytes / 16, cache_sl_bytes / 16, max_accept, n_tree,
                        row_bytes / 16, n_kv_heads, prefix_len, static_cast<int32_t>(share)};
  return launch_kernel(commit_tree_kv_kernel, dim3(static_cast<unsigned>(heads), static_cast<unsigned>(share)), dim3(kCommitThreads), 0,
                       stream, c);
}

}  // namespace specext

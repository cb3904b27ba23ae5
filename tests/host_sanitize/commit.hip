// The commit of accepted rows, thread by thread on the host under AddressSanitizer: every buffer has exactly the size that
// the header asks for, so a read or write outside one ends the program.  Exit code 0 = copied rows are right everywhere.
#include <cstdio>
#include <vector>

#include "commit_rows.h"

struct Vec {
  int x[4];
  bool operator==(const Vec& o) const { return x[0] == o.x[0] && x[1] == o.x[1] && x[2] == o.x[2] && x[3] == o.x[3]; }
};

// layers x heads, rows of row_vecs vectors; `path` in a buffer of exactly its entries
static bool run(int layers, int heads, int n_tree, int max_accept, int row_vecs, int shares, int count, const std::vector<int>& path) {
  const int prefix = 3, cap = prefix + max_accept;
  const int64_t st = row_vecs, sh = n_tree * st, sl = heads * sh, csl = row_vecs + 1, csh = cap * csl, csy = heads * csh;
  std::vector<Vec> kt(layers * sl), vt(layers * sl), kc(layers * csy), vc(layers * csy);
  for (size_t i = 0; i < kt.size(); ++i) kt[i] = Vec{{int(i), 1, 2, 3}}, vt[i] = Vec{{int(i), 4, 5, 6}};
  for (size_t i = 0; i < kc.size(); ++i) kc[i] = Vec{{-int(i) - 1, 0, 0, 0}}, vc[i] = Vec{{-int(i) - 1, 1, 0, 0}};
  std::vector<Vec> want_k = kc, want_v = vc;
  const int n = count < 0 ? 0 : count < max_accept ? count : max_accept;
  for (int lh = 0; lh < layers * heads; ++lh)
    for (int r = 0; r < n; ++r)
      for (int v = 0; v < row_vecs; ++v) {
        if (path[r] < 0 || path[r] >= n_tree) continue;
        const int64_t from = (lh / heads) * sl + (lh % heads) * sh + path[r] * st + v;
        const int64_t to = (lh / heads) * csy + (lh % heads) * csh + (prefix + r) * csl + v;
        want_k[to] = kt[from], want_v[to] = vt[from];
      }
  int* exact_path = new int[path.size()];
  for (size_t i = 0; i < path.size(); ++i) exact_path[i] = path[i];
  int* exact_count = new int(count);
  for (int lh = 0; lh < layers * heads; ++lh)
    for (int s = 0; s < shares; ++s)
      for (int th = 0; th < specext::kCommitThreads; ++th)
        specext::commit_rows(kt.data(), vt.data(), kc.data(), vc.data(), exact_path, exact_count, max_accept, n_tree, heads,
                             prefix, row_vecs, sl, sh, st, csy, csh, csl, th, lh, s, shares);
  delete[] exact_path;
  delete exact_count;
  return kc == want_k && vc == want_v;
}

int main() {
  int failures = 0;
  for (int row_vecs : {1, 3, 8, 16, 32})
    for (int n_tree : {1, 4, 8, 60})
      for (int max_accept : {1, 4, 8, 60, 128})
        for (int shares : {1, 2, 16}) {
          // the path as the acceptance walk leaves it (n_tree entries, -1 behind the accepted ones), some of the nodes invalid
          for (int accepted : {0, 1, n_tree / 2, n_tree}) {
            std::vector<int> path(n_tree, -1);
            for (int i = 0; i < accepted; ++i) path[i] = i % 5 == 3 ? n_tree + i : n_tree - 1 - i;
            if (!run(2, 3, n_tree, max_accept, row_vecs, shares, accepted, path)) {
              std::printf("FAILED row_vecs %d n_tree %d max_accept %d shares %d accepted %d\n", row_vecs, n_tree, max_accept, shares, accepted);
              ++failures;
            }
          }
          // a path of max_accept entries, all of them accepted, nodes repeated where the tree is smaller; a count beyond the bound
          std::vector<int> path(max_accept < n_tree ? n_tree : max_accept);
          for (size_t i = 0; i < path.size(); ++i) path[i] = int(i) % n_tree;
          if (!run(1, 2, n_tree, max_accept, row_vecs, shares, max_accept + 7, path)) {
            std::printf("FAILED row_vecs %d n_tree %d max_accept %d shares %d, full path\n", row_vecs, n_tree, max_accept, shares);
            ++failures;
          }
        }
  if (!failures) std::printf("all rows right\n");
  return failures != 0;
}

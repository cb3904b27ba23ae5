// The choice of the scored tree row on the host under AddressSanitizer: the path has exactly the entries that the header asks
// for, so a read outside it ends the program.  Exit code 0 = the row is right everywhere.
#include <cstdio>

#include "score_row.h"

int main() {
  int failures = 0;
  for (int n_tree : {1, 8, 60, 64, 65, 128})
    for (int count : {-3, 0, 1, 2, 7, 63, 64, 65, 127, 128, 129, 1 << 30}) {
      const int accepted = count < 0 ? 0 : count < n_tree ? count : n_tree;
      for (int last : {0, n_tree - 1, n_tree, -1}) {
        int* path = new int[accepted];
        for (int i = 0; i < accepted; ++i) path[i] = i == accepted - 1 ? last : n_tree;
        int* exact_count = new int(count);
        const int want = accepted > 0 && last >= 0 && last < n_tree ? last : 0;
        if (specext::scored_row(path, exact_count, n_tree, 5) != want) {
          std::printf("FAILED n_tree %d count %d last %d\n", n_tree, count, last);
          ++failures;
        }
        delete[] path;
        delete exact_count;
      }
    }
  if (specext::scored_row(nullptr, nullptr, 8, 5) != 5) ++failures;
  if (!failures) std::printf("all rows right\n");
  return failures != 0;
}

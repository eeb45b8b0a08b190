// Which launches go over pairs of neighbouring blocks (radial_internal.h): for each input line
//   n_blocks sliced ordered mean max_slice codes longest longest_pair alike
// a line with 1 where a forward takes pairs, else 0 (codes 2: where dK/dV does).
#include <stdio.h>

#include "radial_internal.h"

using namespace radial;

int main() {
  WorkMap w = {};
  int codes, alike;
  while (scanf("%d %d %d %d %d %d %d %d %d", &w.n_blocks, &w.sliced, &w.ordered, &w.mean, &w.max_slice, &codes, &w.longest, &w.longest_pair, &alike) == 9) {
    w.alike = alike != 0;
    printf("%d\n", (codes == 2 ? takes_key_pairs(w) : takes_pairs(w, codes != 0)) ? 1 : 0);
  }
  return 0;
}

// The rule for halves at the end of a common backward launch (radial_internal.h) on the host: for each input line
//   items sliced mean
// one line "halved end_whole end_64 end_128 halved_64 halved_128": head dimension 128, the ends its rule goes by, and head dimension 64 in blocks of
// 64 and 128.
#include <stdio.h>

#include "radial_internal.h"

using namespace radial;

int main() {
  long long items;
  WorkMap w = {};
  while (scanf("%lld %d %d", &items, &w.sliced, &w.mean) == 3) {
    const bool laid_out = items <= 6 * kOneRound;
    printf("%d %d %d %d %d %d\n", halved_query_items(w, items), laid_out ? common_launch_end(items, 0) : 0,
           laid_out && items >= 64 ? common_launch_end(items, 64) : 0, laid_out && items >= 128 ? common_launch_end(items, 128) : 0, halved_query_items_64(64, w, items), halved_query_items_64(128, w, items));
  }
  return 0;
}

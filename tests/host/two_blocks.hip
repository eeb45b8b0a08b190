// Which workgroup of a forward over pairs of query blocks takes what (radial_tile.h, radial_internal.h) on the host: for each input line
//   n_blocks sliced ordered mean walk slice[0] .. slice[8]   (walk 0: forward, 1: with 8-bit scores, 2: dK/dV)
// (the order of the pairs is their index, reversed) "takes_pairs grid records", then a line "bh block half form record" for every workgroup that
// has work (and its number; form 0: block and block + 1, 1: a block, 2: half of one) and a line "end".
#include <stdio.h>

#include <vector>

#include "radial_internal.h"
#include "radial_tile.h"

using namespace radial;

int main() {
  int32_t slice[9];
  WorkMap w = {};
  int codes;
  w.slice = slice;
  while (scanf("%d %d %d %d %d", &w.n_blocks, &w.sliced, &w.ordered, &w.mean, &codes) == 5) {
    w.max_slice = 0;
    for (int i = 0; i < 9; ++i) {
      if (scanf("%d", slice + i) != 1) return 1;
      if (i && slice[i] - slice[i - 1] > w.max_slice) w.max_slice = slice[i] - slice[i - 1];
    }
    std::vector<int32_t> order((w.n_blocks + 1) / 2);
    for (size_t i = 0; i < order.size(); ++i) order[i] = (int32_t)(order.size() - 1 - i);
    const TwoMap m = make_two_map(w, order.data(), 1.f, codes == 0 ? TwoWalk::kForward : codes == 1 ? TwoWalk::kCodes : TwoWalk::kKeyGrad);
    const uint32_t grid = m.n_two + 2 * m.n_one + 4 * m.n_half;
    printf("%d %u %lld\n", takes_pairs(w) ? 1 : 0, grid, (long long)trace_records(w.sliced + w.ordered, w.max_slice));
    for (uint32_t id = 0; id < grid; ++id) {
      TwoItem item;
      if (two_item(w, m, id, item)) printf("%d %d %d %d %lld %u\n", item.bh, 2 * item.pair + item.block, item.half, (int)item.form, (long long)item.record, id);
    }
    printf("end\n");
  }
  return 0;
}

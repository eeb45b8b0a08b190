// The launch rules (radial_internal.h) on the host: for each input line
//   head_dim block heads n_blocks nnz longest longest_t
// one line "forward dq dkdv fp8 ordered ordered_q ordered_k": groups of waves per list in each kernel, and the heads that
// go by list length in the forward, dQ and dK/dV kernels.  Run with the word "backward": one line "kind key query kind key query", the
// form of a backward call whose dq has memory of its own, and of one whose dq is the memory of q or dout.  With "forward": one line
// "single halved parts", whether a forward goes in groups of one wave, how many of its last blocks go in halves, and the workgroups
// per block of the 8-bit forward.  With "halves": one line "halved", how many of a backward call's last query blocks (or parts) go in halves.
#include <stdio.h>

#include "radial_internal.h"

using namespace radial;

int main(int argc, char** argv) {
  int D, block, heads, nb, longest, longest_t;
  long long nnz;
  int32_t order = 0;  // only looked at for being there
  while (scanf("%d %d %d %d %lld %d %d", &D, &block, &heads, &nb, &nnz, &longest, &longest_t) == 7) {
    radial_mask m;
    m.block = block;
    m.n_blocks = nb;
    m.n_tokens = nb * block;
    m.nnz = nnz;
    m.longest = longest;
    m.longest_t = longest_t;
    m.max_slice = m.max_slice_t = (nb + 7) / 8;
    if (nb <= kMaxOrdered) m.d_order = m.d_order_t = &order;
    const WorkMap w = make_work_map(&m, Walk::kForward, heads, D), wq = make_work_map(&m, Walk::kQueryGrad, heads, D),
                  wt = make_work_map(&m, Walk::kKeyGrad, heads, D);
    const int64_t items = work_items(w, nb);
    if (argc > 1 && argv[1][0] == 'f') {
      printf("%d %d %d\n", single_waves(block, w, items), halved_items(w, items), fp8_parts(w, items));
      continue;
    }
    if (argc > 1 && argv[1][0] == 'h') {
      const BackwardForm form = backward_form(D, block, wq, wt, items, true);
      printf("%d\n", form.kind == BackwardForm::kTogether && form.key != 4 ? halved_query_items_64(block, wq, items)
                     : form.kind == BackwardForm::kTogetherInPairs ? halved_query_items(wq, items) : 0);
      continue;
    }
    if (argc > 1) {
      const BackwardForm apart = backward_form(D, block, wq, wt, items, true), after = backward_form(D, block, wq, wt, items, false);
      printf("%d %d %d %d %d %d\n", apart.kind, apart.key, apart.query, after.kind, after.key, after.query);
      continue;
    }
    printf("%d %d %d %d %d %d %d\n", query_groups(D, block, w, items, true), query_groups(D, block, wq, items, false),
           key_groups(D, block, wt, items), fp8_groups(w, items), w.ordered, wq.ordered, wt.ordered);
  }
  return 0;
}

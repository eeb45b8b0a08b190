// may_overlap (radial_internal.h) on the host: for each input line
//   B H N D offset, and sb sh sn of the first and of the second tensor (elements; offset: of the second from the first)
// one line: 1 if the tensors may share memory, else 0.
#include <stdio.h>

#include "radial_internal.h"

using namespace radial;

int main() {
  int B, H, N, D;
  long long offset, s[6];
  while (scanf("%d %d %d %d %lld %lld %lld %lld %lld %lld %lld", &B, &H, &N, &D, &offset, s, s + 1, s + 2, s + 3, s + 4, s + 5) == 11) {
    const uintptr_t base = (uintptr_t)1 << 40;  // never read through
    const TensorArg x{(const void*)base, s[0], s[1], s[2]}, y{(const void*)(base + 2 * offset), s[3], s[4], s[5]};
    printf("%d\n", may_overlap(B, H, N, D, x, y));
  }
  return 0;
}

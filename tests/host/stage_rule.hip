// The kernels' token-rule arithmetic (radial_tile.h) on the host: for each input line
//   frames tokens_per_frame extra sink width_num width_den block stage own_is_query
// the N x N visibility that the stages of every block give every token, one byte a pair, to stdout:
// row = the lane's own token, column = the stage's token.
#include <stdio.h>

#include <vector>

#include "radial_internal.h"
#include "radial_tile.h"

using namespace radial;

template <int kBlock, int kStage>
static bool run(const TokenRule& rule, int32_t n, bool own_is_query) {
  std::vector<unsigned char> vis((size_t)n * n, 0);
  for (int32_t token = 0; token < n; ++token) {
    const StagePos own = block_pos(token, rule.s);
    for (int32_t block = 0; block < n; block += kBlock)
      for (int32_t offset = 0; offset < kBlock; offset += kStage) {
        const StagePos at = advance<kBlock - kStage>(block_pos(block, rule.s), offset, rule.s);
        const int32_t hw0 = pair_half_width(rule, own.frame, at.frame, own_is_query), hw1 = pair_half_width(rule, own.frame, at.frame + 1, own_is_query);
        for (int g = 0; g < 2; ++g) {
          const uint32_t hidden = hidden_elements<kStage>(own.pos, at.pos, hw0, hw1, rule.s, g);
          for (int e = 0; e < kStage / 2; ++e) {
            const int32_t other = block + offset + 32 * (e >> 4) + 8 * ((e & 15) >> 2) + 4 * g + (e & 3);
            if (other < n) vis[(size_t)token * n + other] = !(hidden >> e & 1u);
          }
        }
      }
  }
  return fwrite(vis.data(), 1, vis.size(), stdout) == vis.size();
}

int main() {
  int frames, s, extra, sink, num, den, block, stage, own_is_query;
  while (scanf("%d %d %d %d %d %d %d %d %d", &frames, &s, &extra, &sink, &num, &den, &block, &stage, &own_is_query) == 9) {
    radial_mask m;
    m.flags = RADIAL_MASK_TOKEN_EXACT;
    m.frames = frames;
    m.tokens_per_frame = s;
    m.sink_frames = sink;
    m.width_num = num;
    m.width_den = den;
    const TokenRule rule = make_token_rule(&m);
    const int32_t n = frames * s + extra;
    const bool ok = block == 128 ? (stage == 64 ? run<128, 64>(rule, n, own_is_query) : run<128, 32>(rule, n, own_is_query))
                                 : (stage == 64 ? run<64, 64>(rule, n, own_is_query) : run<64, 32>(rule, n, own_is_query));
    if (!ok) return 1;
  }
  return 0;
}

// What the kernels make of the token rule for a wave of 32 tokens that walks a list (span_rule, hidden_elements in radial_tile.h), on
// the host: for each input line
//   frames tokens_per_frame extra sink width_num width_den block stage own_is_query table..., a count and as many half widths (0: the radial rule)
// the N x N visibility that the element masks give, one byte a pair, to stdout (row = the wave's token, column = the stage's).  Exit
// status 2: a stage is said to be seen wholly, or not at all, and its masks say otherwise.
#include <stdio.h>

#include <vector>

#include "radial_internal.h"
#include "radial_tile.h"

using namespace radial;

template <int kBlock, int kStage>
static int run(const TokenRule& rule, int32_t n, bool own_is_query) {
  std::vector<unsigned char> vis((size_t)n * n, 0);
  for (int32_t first = 0; first < n; first += 32) {
    const WaveSpan span = wave_span(first, n, rule.s);
    for (int32_t block = 0; block < n; block += kBlock)
      for (int32_t offset = 0; offset < kBlock; offset += kStage) {
        const StagePos at = advance<kBlock - kStage>(block_pos(block, rule.s), offset, rule.s);
        const SpanRule r = span_rule<kStage>(rule, span, at, own_is_query);
        bool all = true, none = true;
        for (int lane = 0; lane < 64; ++lane) {
          const int g = lane >> 5, token = first + (lane & 31);
          const StagePos own = block_pos(token < n ? token : n - 1, rule.s);
          const int second = own.frame != span.frame;
          const uint32_t hidden = hidden_elements<kStage>(own.pos, at.pos, r.hw[second][0], r.hw[second][1], rule.s, g);
          const uint32_t past = elements_from(n - block - offset - 4 * g);
          for (int e = 0; e < kStage / 2; ++e) {
            const int x = 32 * (e >> 4) + 8 * ((e & 15) >> 2) + 4 * g + (e & 3), other = block + offset + x;
            const bool seen = !(hidden >> e & 1u);
            if (seen) none = false;
            else all = false;
            if ((past >> e & 1u) != (other >= n)) return 1;
            if (token < n && other < n) vis[(size_t)token * n + other] = seen;
          }
        }
        if (all != r.all || none != r.none) return 2;
      }
  }
  return fwrite(vis.data(), 1, vis.size(), stdout) == vis.size() ? 0 : 1;
}

int main() {
  int frames, s, extra, sink, num, den, block, stage, own_is_query, count;
  while (scanf("%d %d %d %d %d %d %d %d %d %d", &frames, &s, &extra, &sink, &num, &den, &block, &stage, &own_is_query, &count) == 10) {
    std::vector<int32_t> table(count);
    for (int32_t& width : table)
      if (scanf("%d", &width) != 1) return 1;
    radial_mask m;
    m.flags = RADIAL_MASK_TOKEN_EXACT;
    m.frames = frames;
    m.tokens_per_frame = s;
    m.sink_frames = sink;
    m.width_num = num;
    m.width_den = den;
    m.d_half_width = count ? table.data() : nullptr;  // (host memory: so are these functions here)
    const TokenRule rule = make_token_rule(&m);
    const int32_t n = frames * s + extra;
    const int rc = block == 128 ? (stage == 64 ? run<128, 64>(rule, n, own_is_query) : run<128, 32>(rule, n, own_is_query))
                                : (stage == 64 ? run<64, 64>(rule, n, own_is_query) : run<64, 32>(rule, n, own_is_query));
    if (rc) return rc;
  }
  return 0;
}

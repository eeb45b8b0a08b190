// Internal declarations shared by the libradial translation units (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "radial.h"

// Device-side description of a block list; owned by radial_mask.
struct radial_mask {
  int32_t n_tokens = 0;
  int32_t block = 0;
  int32_t n_blocks = 0;  // ceil(n_tokens / block): number of query blocks == number of key blocks
  int64_t nnz = 0;
  uint32_t flags = 0;
  int device = 0;
  // owners of the device storage; the pointers below are views into them
  int32_t* d_meta = nullptr;     // totals and launch partitions
  int32_t* d_ptrs = nullptr;     // row_ptr, order (+ col_ptr, order), counts, order of pairs
  int32_t* d_idx = nullptr;      // col_idx (+ row_idx)
  int32_t* d_counts = nullptr;   // [n_blocks] scratch of the build; null above kMaxOrdered blocks
  int32_t* d_row_ptr = nullptr;  // [n_blocks + 1]
  int32_t* d_col_idx = nullptr;  // [nnz]
  int32_t* d_col_ptr = nullptr;  // [n_blocks + 1]  (transpose; only with RADIAL_MASK_TRANSPOSE)
  int32_t* d_row_idx = nullptr;  // [nnz]
  // Launch partition: XCD x of the 8 works on query blocks [slice[x], slice[x+1]) of every
  // (batch, head), so that all XCDs are on the same head at the same time (its K/V then sit
  // in the shared last-level cache) and carry equal weight.  Same for key blocks (backward).
  int32_t* d_slice = nullptr;    // [9]
  int32_t* d_slice_t = nullptr;  // [9]
  // Blocks by falling list length (null above kMaxOrdered blocks): the work order of short launches.
  int32_t* d_order = nullptr;    // [n_blocks]
  int32_t* d_order_t = nullptr;  // [n_blocks]
  int32_t* d_pair_order = nullptr;  // [(n_blocks + 1) / 2]  pairs of query blocks 2p, 2p + 1 by falling length of both lists, an odd last block's counted twice (blocks of 128, without the token rule)
  int32_t* d_pair_order_t = nullptr;  // the same of key blocks
  int32_t max_slice = 0;         // longest slice, in blocks (host copy, sizes the grid)
  int32_t max_slice_t = 0;
  int32_t longest = 0, longest_t = 0;  // entries of the longest list (n_blocks, a bound, where there is no order)
  int32_t longest_pair = 0;            // entries of the longest pair of lists 2p, 2p + 1, both together (0 where there is no order)
  bool alike = true;             // the lists of query blocks 2p and 2p + 1 name some of the same blocks (caller-supplied lists may not)
  int32_t tokens_per_frame = 0;  // geometry of a radial mask (0 for dense / caller-supplied lists)
  int32_t sink_frames = 0;
  int32_t width_num = 1, width_den = 1;  // sparsity knob of a radial mask
  int32_t frames = 0;                    // video frames (tokens from frames*tokens_per_frame on are text tokens)
  int32_t* d_half_width = nullptr;       // [frames + 1] banded patterns only: half width per frame distance
};

namespace radial {

constexpr int kMaxDevices = 64;  // per-device tables of the library are this long

// Records a message for radial_last_error() and returns `code`.
int fail(int code, const char* fmt, ...);

#define RADIAL_HIP_TRY(expr)                                                              \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess)                                                                 \
      return ::radial::fail(RADIAL_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_));  \
  } while (0)

// Lets `kernel` use `bytes` of dynamic LDS (the default limit is 64 KiB).  The attribute belongs to the
// (device, kernel) pair; `done` belongs to the kernel and remembers the devices where it is set.  Setting
// it twice is harmless, so two host threads racing through here only repeat the call.
struct DeviceOnce {
  std::atomic<bool> done[kMaxDevices];
};
inline int allow_dynamic_lds(DeviceOnce& once, const void* kernel, int bytes) {
  int dev = 0;
  RADIAL_HIP_TRY(hipGetDevice(&dev));
  const bool tracked = dev >= 0 && dev < kMaxDevices;
  if (tracked && once.done[dev].load(std::memory_order_acquire)) return RADIAL_OK;
  RADIAL_HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
  if (tracked) once.done[dev].store(true, std::memory_order_release);
  return RADIAL_OK;
}

// Token-level rule of the radial mask, for kernels that apply it inside listed blocks.
struct TokenRule {
  int32_t exact;  // 0: listed blocks are dense
  int32_t s;      // tokens per frame
  int32_t sink;   // key frames below this are visible to everyone
  int32_t frames; // video frames; tokens of later "frames" are text tokens: they see and are seen by everyone
  // sparsity knob c = num/den for frame distances >= 2: the diagonal of band r is
  // floor(c*s / 2^r) = w0 >> r wide, with w0 = floor(s*num/den)
  int32_t w0;
  int32_t den;
  int64_t s_num;  // s * num
  const int32_t* half_width;  // banded patterns: device table by frame distance (null: radial rule)
};

inline TokenRule make_token_rule(const radial_mask* m) {
  TokenRule r;
  r.exact = (m->flags & RADIAL_MASK_TOKEN_EXACT) ? 1 : 0;
  r.s = m->tokens_per_frame;
  r.sink = m->sink_frames;
  r.frames = m->frames;
  r.s_num = (int64_t)m->tokens_per_frame * m->width_num;
  r.den = m->width_den;
  r.w0 = (int32_t)(r.s_num / m->width_den);
  r.half_width = m->d_half_width;
  return r;
}

// Which (batch*head, block) a workgroup works on: the first `sliced` heads by slices, the others by
// falling list length.
struct WorkMap {
  const int32_t* slice;  // [9]
  const int32_t* order;  // [n_blocks]; null only if ordered == 0
  int32_t max_slice;
  int32_t sliced, ordered;  // heads; sum B * H
  int32_t n_blocks;
  int32_t longest, mean;    // entries of the longest and of an average list
  int32_t longest_pair = 0; // of query blocks' lists: entries of the longest two neighbours 2p, 2p + 1
  bool alike = true;        // of query blocks' lists: see radial_mask
  int32_t halved = 0;       // the last items of the launch, taken in two halves each (kernels that have such a form)
};

constexpr int32_t kMaxOrdered = 16384;  // blocks up to which a mask carries the order

// Slices keep the whole chip on one head, but the launch ends on whatever lists come last in the last
// heads: with few heads, or rows that list everything (text tokens), compute units idle there.  Longest
// lists first, each XCD on its own head of the last 8, ends on short lists; it walks the K and V of those
// heads at once, so they have to fit the 256 MB last-level cache (and leave room for Q and O).  Whole
// launches of up to 8 heads within it (forward, 3 heads x 119 026 tokens with text: 9.28 -> 8.35 ms; 5 x 14 040:
// 0.639 -> 0.563 ms; forward+backward under the token rule, 5 x 32 760: 8.91 -> 8.36 ms), and the last heads of
// larger ones, at most 8 and 160 MB (forward, 10 x 14 040: 0.910 -> 0.858 ms, 40 x 32 760: 13.44 -> 13.24 ms,
// 24 x 118 800, 2 heads: 74.1 -> 73.4 ms; with 8 = 490 MB it takes 77.0 ms, with all 24 88.2 ms).  More than 8
// heads by length put several heads on each XCD: 30 x 27 000 tokens in 64-token blocks 6.97 -> 9.35 ms.
// A launch of at most kOneRound items, a workgroup for each compute unit, runs all at once: there is no tail and no
// locality to keep, but slices of unequal length start workgroups without work, which hold up to 128 KiB of LDS as long as they
// wait for their turn.  Such a launch goes by length whatever its number of heads (20 heads x 12 blocks: 288
// workgroups for 240 items; forward, D 128, block 128, two groups: lists of 4 29.4 -> 17.4 us, of 12 55.8 -> 33.0).
// In blocks of 64, where two groups take half a compute unit, that holds up to twice as many (40 heads x 12 blocks: 608
// workgroups for 480 items; D 128, lists of 12, forward 37.3 -> 23.4 us, forward and backward 140 -> 91).
// Blocks of 128 go by length with all their heads, however many, while K and V of all of them are well within the last-level
// cache (160 MB): the grid of slices starts 8 times the longest slice per head, the more of them without work the fewer
// blocks a head has, and ends on whole heads.  By slices but for the last 8 heads / all by length, radial lists, heads x blocks, forward, us: 74 x 9
// 87.9 / 64.1, 42 x 26 273 / 244, 33 x 38 403 / 382, 36 x 47 636 / 609, 15 x 49 303 / 283, 12 x 69 444 / 410, 10 x 110 838 / 812, 10 x 147 1303 / 1304, 20 x 20 79.9 / 79.7;
// D 64 28 x 18 64.6 / 51.4, 26 x 17 60.0 / 46.5, 27 x 140 1892 / 1833; backward 74 x 9 290 / 212, 42 x 26 868 / 783, 12 x 69 1348 / 1354, 10 x 110 2602 / 2618, 10 x 147
// 4430 / 4452 (the runs of one side differ by 1.5 %), D 64 36 x 20 245 / 226, 12 x 64 612 / 579.
constexpr int64_t kOrderedWholeBytes = 256 << 20, kOrderedTailBytes = 160 << 20;
constexpr int64_t kOneRound = 256;
// Blocks of 64 tokens move twice the K and V per product, and by length the blocks that an XCD works on at one time
// are no neighbours: beyond some multiple of its 4 MB L2 the walk over the K and V of its heads is slower than the
// tail is worth, unless single lists are far longer than the others (text tokens) and half as long as the whole
// launch.  An XCD sees one head where their number divides 8 (else some XCDs are on two): (heads + 8 - gcd(heads, 8)) / 8
// on average.
// By slices / by length, ms, D 128 unless said, MB of K and V per XCD in brackets.  Forward, whole launches: 1 / 4 / 8 heads [16]
// 0.497 / 0.388, 1.71 / 1.39, 3.13 / 2.89; 7 heads [29] 2.91 / 2.66; 2 / 8 heads [20] 0.966 / 0.897, 3.74 / 3.41; 1 / 4 / 8 heads
// [27] 0.686 / 0.703, 2.76 / 2.67, 5.37 / 5.30; 5 / 7 heads [31, 36] 2.40 / 2.48, 3.31 / 3.43; 1 / 4 / 8 heads [59]
// 3.18 / 3.73, 12.6 / 14.0, 26.7 / 28.3; D 64, 8 heads [30] 12.8 / 13.1, 2 heads [66] 10.2 / 12.0.  The last 8 of more heads: 12 and 20
// heads [16] 4.86 / 4.69, 8.00 / 8.02, 16 heads [20] 7.34 / 7.77.  The dQ kernel: 4 heads [27] -0.25 of 8.5, 4 heads [61] +0.36
// of 45, 1 head [132] +0.96 of 30.  With text rows (longest / mean): 3 heads of 854 blocks (854 / 301) forward and backward 11.4 / 10.1,
// 6 heads of 1631 blocks 20.9 / 24.1.  dK/dV, and everything in blocks of 128, gain or tie throughout.
constexpr int64_t kForwardXcdBytes64 = 28 << 20, kForwardTailBytes64 = 16 << 20, kQueryGradXcdBytes64 = 64 << 20;
inline int64_t xcd_bytes(int64_t per_head, int32_t heads) {
  const int32_t gcd = heads & 1 ? 1 : heads & 2 ? 2 : heads & 4 ? 4 : 8;
  return heads > 8 ? per_head : per_head * (heads + 8 - gcd) / 8;  // above 8 heads the last 8 go by length
}

enum class Walk { kForward, kQueryGrad, kKeyGrad };

inline WorkMap make_work_map(const radial_mask* m, Walk walk, int32_t heads, int32_t D) {
  WorkMap w;
  const bool transposed = walk == Walk::kKeyGrad;
  w.slice = transposed ? m->d_slice_t : m->d_slice;
  w.order = transposed ? m->d_order_t : m->d_order;
  w.max_slice = transposed ? m->max_slice_t : m->max_slice;
  w.longest = transposed ? m->longest_t : m->longest;
  w.longest_pair = transposed ? 0 : m->longest_pair;
  w.alike = m->alike;
  w.mean = (int32_t)(m->nnz / m->n_blocks);
  const int64_t per_head = 4LL * D * m->n_tokens;  // K and V of one head
  const int64_t fit = (heads <= 8 && per_head * heads <= kOrderedWholeBytes ? kOrderedWholeBytes : kOrderedTailBytes) / per_head;
  const int32_t most = heads < 8 ? heads : 8;
  const int64_t most_bytes = walk == Walk::kQueryGrad ? kQueryGradXcdBytes64 : heads > 8 ? kForwardTailBytes64 : kForwardXcdBytes64;
  const bool long_tail = w.longest >= 2LL * w.mean && 2048LL * w.longest >= (int64_t)w.mean * heads * m->n_blocks;
  const bool scattered = m->block == 64 && !transposed && xcd_bytes(per_head, heads) > most_bytes && !long_tail;
  w.ordered = !w.order ? 0 : (int64_t)heads * m->n_blocks <= (m->block == 64 ? 2 * kOneRound : kOneRound) ? heads : scattered ? 0 : (fit < most ? (int32_t)fit : most);
  if (w.order && m->block == 128 && m->n_blocks >= 8 && heads * per_head <= kOrderedTailBytes) w.ordered = heads;
  w.sliced = heads - w.ordered;
  w.n_blocks = m->n_blocks;
  return w;
}
// Records of a trace: one for every block of every head, by workgroup; pairs of blocks take an even number of every slice.
inline int64_t trace_records(int64_t heads, int32_t max_slice) { return 8 * heads * (max_slice + (max_slice & 1)); }
// (head, block) pairs of a launch, its workgroups, and the most workgroups that any division of the heads could start.
inline int64_t work_grid_bound(const WorkMap& w) { return 8LL * (w.sliced + w.ordered) * w.max_slice; }
inline int64_t work_items(const WorkMap& w, int32_t n_blocks) { return (int64_t)(w.sliced + w.ordered) * n_blocks; }
inline int64_t work_grid(const WorkMap& w, int32_t n_blocks) {
  return 8LL * w.sliced * w.max_slice + (int64_t)w.ordered * n_blocks;
}

// ---- Two query blocks per workgroup (forward, head dimension 128, blocks of 128) ------------------
// Pairs are numbered: those of the sliced heads (n_sliced workgroups), then those of the ordered heads by falling length.  A workgroup each takes
// the first n_two, two workgroups the next n_one, a block each, and four the last n_half, half a block each.
struct TwoMap {
  WorkMap pairs;  // the ordered heads alone, with pairs for blocks
  uint32_t n_sliced, n_two, n_one, n_half;
  float c;  // exp(scale * x) = exp2(c * x); worked out here it is a scalar in the kernel
};
constexpr uint32_t kTwoRound = 512;  // workgroups that the chip holds

// A pair takes 1.75 times as long as a block, so a launch ends as evenly only if its last, shortest lists are taken singly, and the very
// last in halves: whole rounds of pairs, what is left over singly (with slices before them, at least half a round), 64 pairs of that in halves.
// Forward, us, single blocks / 512 pairs, 76 blocks / 512, the last 38 in halves / 448, 38 / 256, 38: 10 heads x 14 040 tokens 829 / 794 / 769 / 776 / 820.
// 3 heads x 119 026 (1395 pairs) 8080 / 1024 pairs 7750, the last 80 in halves 7570, 192 7830, 256 8000; 1136 pairs, 64 in halves 7570, 1280 8060.  With
// slices 40 heads x 32 760 (1024 ordered pairs), none / 512 / 768 of them as pairs 13010 / 12980 / 12960, 24 x 118 800 70.2 / 69.9 / 69.8 ms.
// Over 15 more launches without slices (540 to 1395 pairs) and 8 with them it is faster than single blocks and 0 to 4.5 % behind the best of none, 128 and 256 pairs singly and of 0, 32 and 128
// of them in halves (836 pairs 2927 us, 128 singly 2794; 1000 pairs 6458, none singly 6249; 1140 pairs 11153, no halves 10813; single blocks 2979, 6625, 11790).
// 8-bit scores, which have no halves here: what is left over above rounds of 512 goes singly up to 192 pairs, none up to 256, a pair for each compute unit, what is above those up to
// 384 but at least 64, none beyond; with slices 128 pairs.  At either side of each step (1, 2 and 4 heads, 150 to 460 left over, 78 launches, and 34 others) that is within 2 % of the best of 0,
// 64, 128, 192, all and all above 256, but for 240 to 250 at one head (3 %): 192 / 195 left over 5662 / 6143 us (none singly 5688 / 6084, all 5705 / 6025), 256 / 258 6306 / 6931 (6328 / 6970, 64 6595 /
// 6910), 384 / 387 8292 / 9495 (8984 / 9556, 128 8328 / 9442); single blocks 6227 / 6464, 6900 / 7793, 9593 / 10095: it is the next round that makes the steps.  Single blocks / the best of 0, 64 .. 256 pairs taken singly / this rule, us (pairs in order of length, left over above rounds): 550 (38)
// 763 / 706 / 703, 600 (88) 769 / 727 / 721, 660 (148) 930 / 891 / 891, 700 (188) 990 / 932 / 932, 740 (228) 1146 / 1073 / 1076, 800 (288) 1638 / 1387 / 1390, 832 (320) 1762 / 1530 /
// 1535, 900 (388) 1645 / 1487 / 1471, 1024 (0) 2265 / 2115 / 2098, 1395 (371) 8190 / 7353 / 7297; none singly: 550 800, 800 1525, 1395 8010.
//
// dK/dV, a workgroup to a compute unit: what is left over above rounds of 256 goes singly up to 128 pairs, 64 up to 208, none above.  Single blocks / 0, 64, 128 pairs
// singly, us, training steps: 800 pairs (32 left over) of lists of 20 1229 / 1238, 1188, 1186, radial 6127 / 6210, 5998, 6002, 4370 / 4356, 4212, 4221; 1212 (188) 10750 / 10640,
// 10656, 10636, with text 15370 / 15820, 15490, 15500; 1000 (232) 13240 / 12625, 12780, 12788; 1290 (10) 18353 / 18016, 18096, 17510 (this rule 18140).  128 with slices is hardly better than
// any other number: 40 heads x 126 360 tokens 480 / 466, 467, 467 ms, backward of 20 x 32 760 22.5 / 21.8, 21.6, 21.5, 40 x 14 040 11.3 / 10.8, 10.8, 10.75, 24 x 21 600 14.3 / 13.4, 13.5, 13.5.
enum class TwoWalk { kForward, kCodes, kKeyGrad };
inline TwoMap make_two_map(const WorkMap& w, const int32_t* pair_order, float scale, TwoWalk walk) {
  TwoMap m;
  m.c = scale * 1.4426950408889634f;
  m.pairs = w;
  m.pairs.order = pair_order;
  m.pairs.sliced = 0;
  m.pairs.n_blocks = (w.n_blocks + 1) / 2;
  const uint32_t per_head = (uint32_t)m.pairs.n_blocks, most = ((uint32_t)w.max_slice + 1) / 2;  // pairs of a head; of it to an XCD
  const uint32_t last = (uint32_t)w.sliced % 8u * most;                                       // of the heads that are no full eight to an XCD
  m.n_sliced = 8u * ((uint32_t)w.sliced / 8u * per_head + (last < per_head ? last : per_head));
  const uint32_t ordered = (uint32_t)w.ordered * per_head;
  uint32_t rest;  // pairs at the end that are not taken by one workgroup
  if (walk == TwoWalk::kForward) {
    rest = ordered % kTwoRound;
    if (w.sliced > 0 && rest < kTwoRound / 2 && ordered >= kTwoRound) rest += kTwoRound;
  } else if (w.sliced > 0) {
    rest = ordered < 128u ? ordered : 128u;
  } else if (walk == TwoWalk::kCodes) {
    rest = ordered % kTwoRound;
    if (rest > 192u) rest = rest <= 256u || rest > 384u ? 0u : rest < 320u ? 64u : rest - 256u;
  } else {
    rest = ordered % (kTwoRound / 2);
    if (rest > 128u) rest = rest <= 208u ? 64u : 0u;
  }
  m.n_half = walk != TwoWalk::kForward ? 0u : rest < 64u ? rest : 64u;
  m.n_one = rest - m.n_half;
  m.n_two = m.n_sliced + ordered - rest;  // in the forward a multiple of 8
  return m;
}
// A head of n blocks by slices starts at least 8 workgroups, 8 * max_slice, of which those beyond n have no work; pairs have no such gaps.  Whether there are
// at least eighths / 8 workgroups to a block:
inline bool slices_leave_gaps(const WorkMap& w, int eighths) { return w.sliced > 0 && 64LL * w.max_slice >= (int64_t)eighths * (w.n_blocks + w.n_blocks % 2); }
// A pair begins later than a block (which entries both lists name, and up to three first stages to wait for) and lasts 1.75 times as long, so it takes lists of
// some length, the workgroups without work that slices start, or 8-bit scores, whose kernel for single blocks is slower to begin as well.
// Forward, single blocks / pairs, us, lists of L neighbouring entries unless said.
//   by length, from a whole round of pairs on: 10 heads x 104 blocks 777 / 712, 10 x 120 898 / 869, 8 x 200 1788 / 1716, 10 x 180 1790 / 1778, 14 x 88 759 / 755, 8 x 256
//     2610 / 2535, 5 x 500 4925 / 4710, 4 x 929 13415 / 12250; L 20: 60 x 20 207 / 211, L 40: 32 x 40 422 / 429; below a round: 5 x 110 480 / 487.
//   by slices, hardly a gap: 40 x 128 L 2 168 / 182, 10 477 / 486, 20 865 / 875, 28 1173 / 1169, 40 1632 / 1609; 24 x 256 L 2 201 / 216, 20 1021 / 1049, 40 1935 / 1927;
//     16 x 929 L 2 472 / 504, 10 1382 / 1401, 28 3409 / 3380; 113 x 24 L 3 114 / 119, 12 308 / 314, 24 566 / 563.  With gaps: 290 x 9 L 2 124 / 94, 9 321 / 244, 240 x 11 L 3 129 /
//     117, 190 x 14 L 2 97.5 / 97.1, 149 x 18 L 2 104 / 97, 134 x 20 L 2 99.6 / 97.3, 105 x 25 L 25 617 / 558.  8-bit scores: 40 x 128 L 2 160 / 160, 10 429 / 422, 24 x 256 L 3 232 / 220,
//     20 922 / 883, 16 x 929 L 2 444 / 441.
//   fewer than 8 blocks, where pairs are half of the workgroups with work but a launch of a round or two lasts as long as one of them, and an odd last block is a pair of its
//     own: 1 block 280 heads 25.6 / 15.1, 1200 87 / 39; 2 blocks 140 heads 32.6 / 21.7, 1000 L 1 137 / 55; 3 blocks 96 heads 19.2 / 26.3, 400 60 / 67, 800 L 1 80 / 88, L 3 114 / 115;
//     4 blocks 65 heads 21.9 / 30.4, 100 L 1 18.4 / 20.3, 128 L 1 23.1 / 19.7, L 4 40.0 / 32.8, 600 177 / 120; 5 blocks 53 heads 25.6 / 34.9, 120 47 / 51, 200 L 2 45.1 / 41.0, 400 141 / 121;
//     6 blocks 64 heads 32.6 / 40.0, 120 L 2 32.1 / 34.2, 180 85 / 88, 200 95.6 / 89.8, 400 183 / 151; 7 blocks 40 heads 32.5 / 43.3, 160 93 / 102, 350 L 2 89 / 96, L 7 200 / 203.
//
// Two neighbouring lists far longer than the others (text tokens) are one workgroup's in pairs, and the launch ends no sooner than it does: 1.13 of the time that either
// takes alone.  They start where the heads by length do, so the shorter of them counts against what a
// workgroup of a whole round has of those heads, or of the launch where all heads go by slices.  Single blocks / pairs, us, radial lists and 512 tokens of text unless said, that share in
// brackets: by length 1 head x 1129 blocks [1.10] 4881 / 5537, 1 x 1690 (226 tokens) [0.91] 8090 / 8559, 1 x 1971 (226) [0.84] 9970 / 10177, 1 x 2252 (226) [0.79] 12418 / 12027, 2 x 565 (226) [0.78]
// 3003 / 2982, 2 x 933 [0.60] 6538 / 6142, 3 x 359 (226) [0.81] 1827 / 1909, 3 x 363 [0.85] 1772 / 1880, 2 x 531 [0.95] 2380 / 2506, 4 x 269 [0.75] 1481 / 1497, 4 x 268 [0.72] 1534 / 1491, one long list of a pair 1 x 1127 (226) 4617 / 4052; the last heads by length: lists of 32 and two full ones 40 x 128 [1.9] 1503 / 1588, one 1480 /
// 1444, lists of 40 and two 20 x 256 [1.5] 1854 / 2164; 4 x 1804 [0.88] 36.3 / 32.2 ms, 24 x 114 [0.66] 2218 / 2138; (beside slices they have to be twice the mean: few heads by length are less than a round of their own) all by slices 2 x 3633 [0.31] 52.1 / 55.6 ms, 2 x 2817 [0.35] 37.9 / 40.4, 3 x 2817
// [0.24] 55.9 / 56.1, 4 x 3633 [0.16] 101 / 98, without text 2 x 3629 [0.08] 49.8 / 46.2.  8-bit scores: 1 x 1129 4176 / 4616, 1 x 1409 (226) [0.99] 5521 / 5785, 1 x 1690 7175 / 6988, 40 x 128 1386 /
// 1429, 20 x 256 1732 / 1832, 2 x 3633 48.2 / 46.8 ms.
// One long list that the whole launch waits for is slower beside a usual one in bf16: lists of 64 and a full one by length 4 x 929 [1.9]
// 2425 / 2719; the last heads by length 8 x 929 [3.9] 5013 / 5253, lists of 32 10 x 929 [7.5] 4035 / 4243, 40 x 128 [1.9] 1404 / 1376; 8-bit scores 4 x 929 2953 / 2730.
inline bool long_lists_end_the_launch(const WorkMap& w, bool codes) {
  const int64_t shorter = w.longest_pair - w.longest, entries = (int64_t)w.n_blocks * w.mean;  // of a head
  if (!codes && w.ordered > 0 && w.longest >= 2LL * w.mean && 2LL * kTwoRound * w.longest > (w.sliced ? 6 : 3) * w.ordered * entries) return true;
  if (w.sliced > 0 && shorter < 2LL * w.mean) return false;
  if (w.ordered == 0) return !codes && 5 * kTwoRound * shorter > w.sliced * entries;
  return 20 * kTwoRound * shorter > (codes ? 19 : w.sliced ? 20 : 16) * w.ordered * entries;
}
// Lists that hardly share an entry gain nothing from being walked together and are slower at any length, above all with 8-bit scores, whose kernel for single blocks keeps three waves to a
// SIMD: forward, single blocks / pairs, us, 40 x 128 L 40, nothing shared 1636 / 1668, 8 bits 1437 / 1497; 16 x 929 random lists of a tenth of the blocks 11805 / 11797, 8 bits 9949 / 10301; of a
// quarter 29035 / 28175, 24384 / 24062; 40 x 128 of a quarter 1414 / 1424, 1231 / 1247, of a half 2694 / 2674, 2355 / 2297.  Gaps have to be wider then: 40 x 128 random lists of 2.5
// entries, 9 workgroups to 8 blocks, 194 / 199, 8 bits 179 / 181.
inline bool takes_pairs(const WorkMap& w, bool codes = false) {
  if (w.n_blocks > kMaxOrdered || (w.n_blocks >= 8 && long_lists_end_the_launch(w, codes))) return false;
  const int64_t pairs = (int64_t)(w.sliced + w.ordered) * ((w.n_blocks + 1) / 2);
  if (w.sliced == 0) return w.alike && w.mean >= 64 && pairs >= kTwoRound;
  if (w.n_blocks >= 8) return slices_leave_gaps(w, w.alike ? 9 : 12) || (w.alike && (codes || w.mean >= 28));
  return w.n_blocks <= 2 || (w.n_blocks == 4 && pairs >= 256) || ((w.n_blocks == 5 || w.n_blocks == 6) && pairs >= 600);
}

// dK/dV, above the sizes of a common launch, whatever neighbouring lists share (the kernel sees that itself): lists of 7 entries, fewer than 8 blocks but for 3 and 7, whose last
// pair is a block, or gaps among the slices.  Backward, one block / two, us, lists of L neighbouring entries: 40 heads x 128 blocks L 2 612 / 619, 3 717 / 731, 6 1091 / 1093, 8 1353 / 1336, 10 1596 /
// 1581, 40 5462 / 5192; 16 x 929 L 2 1687 / 1728, 5 2774 / 2781, 10 4618 / 4542; 100 x 40 L 2 477 / 494, 5 770 / 771, 10 1314 / 1264; 200 x 16 L 2 401 / 408, 8 900 / 869; gaps: 400 x 9 L 2 599 / 494, 300 x 11 L 2 472 / 441,
// 5 777 / 684, 220 x 15 (none) L 2 420 / 426; 1600 x 1 433 / 283, 800 x 2 532 / 332, 520 x 3 L 1 184 / 192, L 3 274 / 269, 400 x 4 L 1 240 / 212, 320 x 5 L 2 252 / 211, 260 x 6 L 2 226 / 201, 224 x 7 L 2 209 / 223, L 7 413 / 411.
inline bool takes_key_pairs(const WorkMap& w) {
  if (w.n_blocks > kMaxOrdered || work_items(w, w.n_blocks) <= 6 * kOneRound) return false;
  return w.mean >= 7 || (w.n_blocks < 8 ? w.n_blocks != 3 && w.n_blocks != 7 : slices_leave_gaps(w, 9));
}

// ---- How many groups of waves share a list ------------------------------------------------------
// A workgroup walks its list stage by stage, so a launch that runs in one round lasts as long as its longest
// walk, and S groups cut that by S.  They cost a merge (1 to 4 us) and, once the chip is full, wait for each
// other at the same barriers.  All figures are kernel times in microseconds, one group / the form named,
// on lists of equal length L unless said otherwise.
// `groups` = 4 at block 128 and 2 in the dK/dV kernel at block 128 mean half blocks: two workgroups per block, of 64 rows each.
// The forward asks single_waves first (query_groups' forward figures at 64 items are from before it), the backward
// backward_form: it comes to query_groups and key_groups above the sizes of a common launch and where dq is the memory of q or dout.

// Two groups for 64-token blocks above kOneRound items: four workgroups of one group fit a compute unit, or two of two, so that
// two groups take ceil(items / 512) / 2 walks where one takes ceil(items / 1024).
//   up to 512 items:  a round either way.  Forward, D 128, 300 items: L 8 22.2 / 17.0, L 48 91.9 / 58.9; dQ -5, -48.
//   up to 1024:  one round or two of half the length, which pays for what long lists of unequal length leave over, more so
//     at D 64.  Forward, (items; mean, longest), D 128 / D 64: (568; 103, 115) 194 / 194, 129 / 106; (568; 62, 65) 119 / 125,
//     76.1 / 69.5; (882; 84, 98) 192 / 200, 120 / 115; (879; 236, 293) 513 / 508, 323 / 299; (891; 418, 505) 1113 / 988,
//     576 / 529; with text rows (897; 188, 299) 492 / 413, 271 / 244.  Equal lists: D 128 (835; 167, 167) 356 / 377,
//     (640; 16, 16) 40.6 / 42.5; D 64 (830; 166, 166) 211 / 218.  dQ 0 to -5 % from 90 entries on.
//   up to 1536:  two rounds or three of half the length.  Forward, D 128, 1200 items: L 8 46.1 / 44.6, L 12 62.0 / 56.7,
//     L 48 195 / 172; dQ, L 8 0, L 12 -4, L 48 -36.  L 4, forward: 30.3 / 32.2.
//   above:  D 128 loses (1800 items, L 48 224 / 233; 1880 items on radial lists 359 / 373).
inline bool two_groups_pay_64(int D, const WorkMap& w, int64_t items) {
  if (items <= 512) return w.longest >= 4;
  if (items <= 1024) {
    if (2LL * w.longest >= 3LL * w.mean) return w.mean >= 16;
    return D == 64 ? w.mean >= 24 && 32LL * w.longest > 33LL * w.mean : w.mean >= 96 && 8LL * w.longest > 9LL * w.mean;
  }
  return items <= 1536 && w.mean >= 12;
}

// Forward: groups of a single wave, 32 rows per workgroup, 4 groups at D 128 and 8 at D 64, while all parts of all blocks still get a compute
// unit of their own (the backward at D 64 has the like in both_groups; dK/dV at D 128 has LDS for two such waves only).  The launch
// spreads over 2 (block 64) or 4 (block 128) times the compute units of a workgroup per block, and a wave that shares its
// stage buffers with nobody needs no barrier: in the forms below it waited there for 29 % of its loop (64 items of D 64, block 64).
// Best of the forms below / single waves, us: block 64, D 64, 64 items L 28 15.3 / 11.1; 99 items L 99 36.6 / 23.0; D 128, 22 items
// L 11 15.2 / 11.0; 128 items L 3 8.9 / 7.4, L 1 7.5 / 7.7; block 128, D 128, 64 items L 1 7.8 / 8.3, L 2 10.0 / 8.6, L 8 16.6 /
// 13.5; D 64 L 8 10.2 / 8.2.  (A forward call takes the host 7.7 us.)
inline bool single_waves(int block, const WorkMap& w, int64_t items) { return items * (block / 32) <= kOneRound && w.longest >= 2; }

// Block 128, up to 256 items.  Forward, D 128: half blocks at 64 items L 2 10.5 / 11.0, L 3 12.6 / 12.2, L 16 41.3 / 25.8, at
// 256 items L 16 48.0 / 54.0; two groups at 256 items L 3 15.0 / 15.9, L 4 17.4 / 17.4, L 16 48.0 / 41.6, at 288 items
// (longer lists) 101 / 111.  dQ at 64 items: L 2 -0.6, L 3 -2.3, L 16 -28; 564 items, D 64: +20.
// Block 64, up to 256 items.  Forward, D 128, one / two / four groups: L 3 9.6 / 9.5 / 10.6, L 4 11.1 / 9.4 / 10.7,
// L 8 17.2 / 12.5 / 13.0, L 12 23.1 / 15.8 / 15.6, L 32 52.1 / 31.0 / 27.9; dQ alike (L 32 0 / -26 / -29).
// D 64, block 64, above 1536 items: two workgroups of 4 waves per compute unit walk fewer lists at once than five of 2 waves,
// which pays on long lists: 19 200 items L 16 499 / 526, L 32 912 / 918, L 64 1722 / 1690, L 100 2637 / 2557; 4000 items L 12
// 87.8 / 87.2, L 48 290 / 279; on radial lists (15 800 items) 16.3 / 13.1 ms.
inline int query_groups(int D, int block, const WorkMap& w, int64_t items, bool forward) {
  if (block == 128) {
    if (items <= 128) return w.longest >= (forward ? 3 : 2) ? 4 : 1;
    return items <= kOneRound && w.longest >= 4 ? 2 : 1;
  }
  if (items <= kOneRound && w.longest >= 12) return 4;
  if (two_groups_pay_64(D, w, items)) return 2;
  return forward && D == 64 && items > 1536 && w.mean >= 32 ? 2 : 1;
}

// dK/dV at D 128 by hand holds one wave per SIMD: a compute unit takes one workgroup of 128 keys, one of two groups of 64, or two of
// one group of 64, so that at block 64 two groups take ceil(items / 256) / 2 walks where one takes ceil(items / 512).
//   block 128, half blocks, 64 items: L 1 0, L 2 -3, L 16 -27; 256 items, L 32: +13.
//   block 64, D 64, where two workgroups of either form fit a compute unit: 288 items L 3 +1, L 4 -1, L 8 -5.5, L 16 -10, 512 items L 3 0, L 8 -5.4.
//   block 64, D 128: 256 items L 2 +1, L 3 0, L 8 -7, L 32 -22; 300 items L 8 +2, L 16 -6, L 48 -40; 500 items L 48 +7;
//   572 items L 26 -26 (with dQ); 600 items L 8 +2, L 16 -1, L 48 -34; 700 items L 16 +9, L 48 -33; 1000 items L 48 +18; 1200 items L 16 +23, L 48 -25,
//   radial lists (mean 51, 1140 items) -9; 1300 items, L 48: +5.  One list far longer than the others (text, the sink's
//   columns) makes up for a round: 891 items (mean 418, longest 891) -153 of 3219.
inline int key_groups(int D, int block, const WorkMap& w, int64_t items) {
  if (block == 128) return items <= 128 && w.longest >= 2 ? 2 : 1;
  if (items <= (D == 64 ? 2 * kOneRound : kOneRound)) return w.longest >= 3 ? 2 : 1;
  if (items <= 384) return w.longest >= 16 ? 2 : 1;
  return items <= 1200 && w.mean >= (items <= 768 ? 24 : 32) && ((items - 1) / 256 % 2 == 0 || w.longest >= 2LL * w.mean) ? 2 : 1;
}

// D 64, dK/dV and dQ in one launch: groups of waves per workgroup; 0: two launches, one after the other.
// Each alone leaves compute units idle, a small one because it has too few workgroups or waves, a larger one where it ends.
// Neither needs the other's results, both fit two waves per SIMD, and a workgroup of two groups is half a compute unit's LDS.  Up to 128 parts
// of 32 rows, where each of the 256 workgroups has a compute unit: groups of one wave; up to kOneRound blocks two groups of 64 rows, so that
// two workgroups share a compute unit; above, two groups of a block of 64, or one of a block of 128.
// Backward pass, us, the best forms of two launches / one, (items, list length):
//   one wave, block 64: (64; 32) 30.6 / 20.0, (4; 1) 15.6 / 13.2 (the host takes 13); block 128: (32; 8) 22.2 / 13.6, (32; 32) 48.4 / 29.5, (16; 16)
//     30.1 / 18.2.  At 128 to 256 parts: block 64 (128; 32) 33.0 / 31.5, two groups 28.6; block 128 (64; 16) 33.0 / 31.4, two groups 27.9.
//   two groups, block 64: (192; 4) 17.4 / 13.1, (256; 32) 46.1 / 39.7, (288; 8) 28.4 / 23.1, (384; 32) 71.9 / 59.5, (512; 32) 80.3 / 75.1, (768; 16)
//     74.7 / 65.7, (1024; 32) 152 / 149, (1536; 16) 132 / 124, radial lists (1100; mean 57) 847 / 769.
//   half blocks of two groups, block 128: (128; 2) 18.4 / 13.5, (128; 16) 46.1 / 39.7, (256; 16) 76.9 / 73.6, radial lists (250; 29) 228 / 206.
//   one group, block 128: (288; 4) 43.7 / 36.4, (288; 24) 168 / 144, (512; 16) 143 / 137, (768; 16) 213 / 197, radial lists (550; 57) 939 / 836,
//     (1330; 112) 2085 / 2038.
//   above: radial lists, block 64 (2560) 2996 / 3015, block 128 (2580) 6284 / 6420.
//   lists of one entry in blocks of 64, where two groups share nothing: 512 items 17.1 / 16.5, above 768 22.1 / 23.8, 1024 27.8 / 30.8, 1536 42.2 / 44.1.
inline int both_groups(int block, const WorkMap& w, int64_t items) {
  if (items * (block / 32) <= kOneRound / 2) return 4;
  if (items > 6 * kOneRound || (block == 64 && items > 640 && w.mean < 2)) return 0;
  return block == 128 && items > kOneRound ? 1 : 2;
}

// The same at D 128.  By hand, 4 waves with a compute unit each for either half of the work: while all workgroups of both, of 64 rows,
// have one.  In pairs of waves, blocks of 128 (8 waves for either): up to 6 rounds.  In blocks of 64 the hand-made schedule, one wave per
// SIMD, would hold dQ to one as well.  Backward pass, us, two launches / one, (items, list length):
//   by hand, block 128: (8; 2) 22.1 / 13.5, (40; 8) 37.4 / 25.8, (60; 4) 27.4 / 18.6, (64; 32) 104 / 79.5, above (100; 16) 71.5 / 79.5; block 64: (16; 4) 20.9
//     / 13.3, (64; 16) 37.3 / 25.5, (128; 8) 27.2 / 18.4, (128; 32) 59.4 / 43.9, above (192; 8) 31.5 / 31.3, (256; 32) 77.3 / 76.6.
//   in pairs: (64; 32) 104 / 109, (100; 16) 71.5 / 65.3, (128; 1) 24.7 / 16.3, (128; 32) 135 / 129, (256; 32) 248 / 237, (288; 16) 209 / 164, (384; 32)
//     405 / 355, (512; 16) 252 / 250, (640; 16) 347 / 310, radial lists (550; 57) 1697 / 1452, (1280) 5802 / 5760;
//     above (2070) 8078 / 7960, (2560) 11510 / 11690, (2787) 33460 / 33330, (3000; 16) 1510 / 1553.
//   Either kind of workgroup fills a compute unit, so one launch of equal lists saves a round where the last one would be at most half full;
//   elsewhere it saves only what unequal lists leave over, and lists of a few entries do not pay for dQ in two groups: (384; 1) 48.7 / 46.1, above
//     (512; 1) 56.0 / 60.1, (768; 1) 80.4 / 86.8, (1280; 1) 127.5 / 138.7, (1024; 3) 151 / 162, (1280; 3) 185 / 198, (1536; 3) 225 / 242, (1024; 8) 270 / 275;
//     by hand before the pairs / one (two launches in between): (448; 1) 51.1 / 55.8, (576; 1) 71.0 / 69.8, (640; 2) 89.6 / 84.1, (896; 1) 95.8 / 98.0, (896; 2) 118 / 114,
//     (1408; 1) 144 / 152, (1408; 3) 213 / 209, (448; 4) 84.6 / 84.9.
inline bool both_by_hand(int block, int64_t items) { return items * (block / 64) <= kOneRound / 2; }
inline bool both_in_pairs(const WorkMap& w, int64_t items) {
  if (items > 6 * kOneRound) return false;
  return items <= kOneRound * 3 / 2 || w.mean >= 4 || (w.mean >= 2 && (items - 1) % kOneRound < kOneRound / 2);
}

// What a backward call launches, the groups of waves per list in dK/dV and dQ.  apart: dq shares no memory with q and dout, so that dQ may run
// beside dK/dV.  Where it may not, the kernels alone are best in the forms that either has by itself, not in those of a common launch, which
// leave it half of each compute unit.  Backward pass into the memory of dout, us, equal lists of L, the forms of a common launch one after the
// other / every list whole in one group / these: D 128, block 128, 64 items L 32 142 / 210 / 112, 128 items L 8 64.0 / 68.5 / 45.7, L 32 188 / 213 /
// 116, 1536 items L 3 229 / 199 / 199; D 64, block 128, 64 items L 32 85.4 / 157 / 77.9, block 64, 128 items L 32 49.0 / 64.4 / 46.0, 1024 items
// L 3 41.4 / 33.3 / 33.1; D 128, block 64, 128 items L 32 79.5 / - / 66.4.
struct BackwardForm {
  enum Kind { kOneAfterTheOther, kTogether, kTogetherByHand, kTogetherInPairs } kind;
  int key, query;
};
inline BackwardForm backward_form(int D, int block, const WorkMap& w, const WorkMap& wt, int64_t items, bool apart) {
  if (apart && D == 64) {
    if (const int groups = both_groups(block, w, items)) return {BackwardForm::kTogether, groups, groups};
  } else if (apart) {
    if (both_by_hand(block, items)) return {BackwardForm::kTogetherByHand, 2, 2};
    if (block == 128 && both_in_pairs(w, items)) return {BackwardForm::kTogetherInPairs, 1, 2};
  }
  // D 64 has two waves per SIMD in dK/dV; in blocks of 64 two groups take fewer walks at once, which pays on long lists (3200 items L 16
  // 251 / 261, L 32 454 / 453; radial lists: 2136 items, mean 172, 1620 / 1563)
  const int key = D == 64 && block == 64 && wt.mean >= 32 ? 2 : key_groups(D, block, wt, items);
  return {BackwardForm::kOneAfterTheOther, key, query_groups(D, block, w, items, false)};
}

// Blocks of 128 above one round, whole blocks by one group: the launch takes ceil(items / 256) rounds of a workgroup per compute
// unit (two share one), so the items % 256 last ones keep most of the chip waiting for a whole list.  Up to half a
// round of them are taken in two halves each, of 64 rows and two groups that walk half the list: the
// same threads and stage buffers as a whole block, so that both kinds run in one launch.  They have to be the shortest
// lists of it, so all heads go by length (among slices, 12 to 54 heads: 0.97-1.02).  Whole blocks / with halves, forward, us, equal
// lists: 264 items L 4 23.4 / 20.1, L 64 208 / 161; 320 items L 4 22.9 / 19.5, L 32 114 / 94.5; 368 items L 32 119 / 104; 520 items L 4
// 35.1 / 33.2, L 64 367 / 328; 624 items L 32 196 / 179; 1120 items L 4 61.2 / 59.9, L 32 321 / 303; 1600 items L 64 865 / 825; D 64 264 items L 64 147 / 108,
// 368 items L 32 78.3 / 63.3, 1120 items L 64 373 / 345.  Radial lists: 550 items (64 to 108 entries) 514 / 469, 776 (101 to 153) 990 / 906,
// 2254 (203 to 448; 206 left, not halved) 7327 / 7340 with 206 halved 7428; 910 (65; 142 left) 516 with 142 halved 568.
inline int32_t halved_items(const WorkMap& w, int64_t items) {
  const int64_t rest = items % kOneRound;
  return items > kOneRound && rest <= kOneRound / 2 && w.sliced == 0 && w.longest >= 4 ? (int32_t)rest : 0;
}

// The common backward launch in pairs (D 128, blocks of 128): a compute unit holds one workgroup, dK/dV's go first and dQ's last, so the end of the
// launch waits for a whole dQ list on however few units.  In two halves, of 64 rows and four groups that walk a quarter of the list each, the last
// lists end sooner, at more copies per product (1.16 of the time, as much as 8 % of a launch that ends evenly as it is).  Which it is
// depends on where the rounds fall: the launch is laid out as if lists were equal, a unit at a time to the workgroup that is next, at the
// measured 40 : 31 : 18 of a dK/dV, a dQ and half a dQ list, and halves are taken where that ends 4 % earlier.
// Backward, us, whole lists / (64 or 128 halved), predicted in brackets, radial lists unless said: 129 items 204 / (64) 180 [0.79], 170 194 / (128) 178
// [0.94], 306 305 / (128) 292 [0.92], 294 375 / (128) 366 [0.87], 400 557 / (64) 520 [0.90], 513 equal lists 324 / (128) 306 [0.93], 812 1277 / (128)
// 1245 [0.95]; not taken: 216 218 / (128) 237 [1.07], 238 219 / (128) 237 [1.07], 330 470 / (128) 490 [1.05], 372 795 / (128) 827 [1.05], 450 2812 / (128) 2872
// [0.97], 506 335 / (128) 343 [1.04], 1280 5649 / (128) 5703 [1.01], 1455 3025 / (128) 2964 [0.97].
inline int32_t common_launch_end(int64_t items, int64_t halved) {
  constexpr int32_t kKey = 40, kQuery = 31, kHalf = 18;
  int16_t free_at[640] = {(int16_t)kOneRound};  // units by the time they are free; items <= 6 * kOneRound end before 6 * (kKey + 2 * kHalf) + kKey
  int32_t now = 0, end = 0;
  const auto run = [&](int64_t workgroups, int32_t time) {
    while (workgroups > 0) {
      while (free_at[now] == 0) ++now;
      const int64_t n = workgroups < free_at[now] ? workgroups : free_at[now];
      free_at[now] -= (int16_t)n;
      free_at[now + time] += (int16_t)n;
      end = now + time > end ? now + time : end;
      workgroups -= n;
    }
  };
  run(items, kKey);
  run(items - halved, kQuery);
  run(2 * halved, kHalf);
  return end;
}
inline int32_t halved_query_items(const WorkMap& w, int64_t items) {
  if (w.sliced != 0 || items <= kOneRound / 2 || items > 6 * kOneRound || w.mean < 4) return 0;
  const int32_t whole = common_launch_end(items, 0), some = common_launch_end(items, 64), more = common_launch_end(items, 128);
  const int32_t best = more < some ? more : some;
  return 25 * best > 24 * whole ? 0 : more < some ? 128 : 64;
}

// The same at D 64, where two workgroups share a compute unit.  dQ's parts are laid over what dK/dV, as many workgroups, leave of the units: halves pay
// where that is a little more than half of them (129 to 176 parts), and where the last round of 256 has few parts (1 to 72).
// Backward, us, whole parts / with halves.  Block 64, items: 132 33.9 / 31.3, 168 40.5 / 39.0, 175 36.9 / 35.5 (184 with 96 halved 0.98, 200 1.00, 210 1.05), 260 84.9 / 75.1,
// 304 64.8 / 59.6, 328 71.7 / 68.2 (360 with 192 1.02, 378 1.02), 528 167 / 156, 792 348 / 328, 1032 569 / 549; equal lists 136 L 8 14.9 / 14.5, 272 L 4 17.9 / 16.9, 272 L 8 22.5 / 20.8;
// token rule 294 80.8 / 71.0.  Block 128 (two parts a block up to 256): 66 60.2 / 54.1, 80 71.6 / 66.1 (96 with 96 1.03, 114 1.05, 126 1.05), 132 106 / 94, 148 118 / 110, 164 130 /
// 127 (175 with 192 0.98, 225 1.07), 264 252 / 221, 320 232 / 216 (360 with 192 1.01, 410 1.00, 450 1.04), 528 441 / 406, 816 634 / 603, 784 2541 / 2333 (600 0.99, 1000 1.00, 1104
// 1.00); equal lists 136 L 4 23.8 / 21.8, 280 L 4 46.8 / 46.9; token rule 320 236 / 218.
inline int32_t halved_query_items_64(int block, const WorkMap& w, int64_t items) {
  const int64_t parts = block == 128 && items <= kOneRound ? 2 * items : items, rest = parts % kOneRound;
  if (w.sliced != 0 || w.mean < 4 || parts <= kOneRound / 2) return 0;
  if (parts <= kOneRound) return parts <= 176 ? 96 : 0;
  return rest >= 1 && rest <= 72 ? 192 : 0;
}

// 8-bit scores: three groups of 4 waves (12 waves are what a compute unit holds of this kernel) while every item can
// have a compute unit of its own.  64 items: L 4 16.9 / 17.7, L 6 22.3 / 19.8; 105 items L 5 (with the quantisation) 40.4 / 37.5; 256 items: L 6 24.0 / 22.7, L 32 93.5 / 69.0;
// 288 items (with the quantisation) 127 / 133.
inline int fp8_groups(const WorkMap& w, int64_t items) { return items <= kOneRound && w.longest >= 5 ? 3 : 1; }

// Workgroups per query block, of four groups each that walk stages of 32 keys: 4 (groups of one wave) or 2 (of two waves) while
// every part has a compute unit of its own.  Best of the forms above / 4 parts / 2 parts, us, without the quantisation: 64 items L 1
// 8.5 / 9.4 / 9.5, L 2 10.8 / 9.3 / 9.3, L 4 16.2 / 9.6 / 10.6, L 8 21.8 / 14.2 / 15.4, L 16 34.8 / 23.4 / 24.7; 128 items L 2 11.3 / 17.2 /
// 9.8, L 4 16.7 / 17.5 / 11.4, L 16 35.8 / 45.6 / 26.0 (six groups in 2 parts: 25.1, L 8 17.6 against 16.6); 192 items L 4 16.9 / 25.0 / 20.2.
inline int fp8_parts(const WorkMap& w, int64_t items) { return w.longest < 2 || items > 128 ? 1 : items <= 64 ? 4 : 2; }

struct TensorArg {
  const void* ptr;
  int64_t sb, sh, sn;  // element strides
};

// Whether two bf16 tensors of a call, [B, H, N, D] each, may share memory.  They do not if their extents are apart, or if both stay
// in parts of one period of memory that are apart, as slices of a packed [B, N, 4, H, D] or [B, H, N, 2, D] do.
inline bool may_overlap(int32_t B, int32_t H, int32_t N, int D, const TensorArg& x, const TensorArg& y) {
  const int32_t sizes[] = {B, H, N};
  const auto extent = [&](const TensorArg& t) { return (B - 1) * t.sb + (H - 1) * t.sh + (N - 1) * t.sn + D; };
  const int64_t apart = ((int64_t)(uintptr_t)y.ptr - (int64_t)(uintptr_t)x.ptr) / 2;  // elements; tensors are 16-byte aligned
  if (apart >= extent(x) || -apart >= extent(y)) return false;
  // Elements of one period that the tensor touches, from its first one on; 0: it does not repeat with this period.
  const auto touched = [&](const TensorArg& t, int64_t period) -> int64_t {
    const int64_t strides[] = {t.sb, t.sh, t.sn};
    int64_t n = D;
    for (int i = 0; i < 3; ++i) {
      if (sizes[i] == 1 || strides[i] % period == 0) continue;
      if (strides[i] > period) return 0;
      n += (sizes[i] - 1) * strides[i];
    }
    return n <= period ? n : 0;
  };
  const int64_t periods[] = {x.sb, x.sh, x.sn};
  for (int i = 0; i < 3; ++i) {
    if (sizes[i] == 1 || periods[i] == 0) continue;
    const int64_t of_x = touched(x, periods[i]), of_y = touched(y, periods[i]);
    const int64_t at = (apart % periods[i] + periods[i]) % periods[i];
    if (of_x && of_y && at >= of_x && at + of_y <= periods[i]) return false;
  }
  return true;
}

struct FwdArgs {
  TensorArg q, k, v, o;
  float* lse;  // may be null
  const int32_t* row_ptr;
  const int32_t* col_idx;
  WorkMap work;
  int32_t B, H, N, n_blocks;
  float scale;
  TokenRule rule;
  uint64_t* wg_trace;  // null, or [trace_records][3]: begin, end (100 MHz clock), where the workgroup ran
  const int32_t* pair_order;  // pairs of query blocks by falling length; null where no kernel takes pairs (blocks of 64, token rule, above kMaxOrdered blocks)
};

int launch_fwd(int D, int block, const FwdArgs& a, hipStream_t stream);
// Argument checks of a forward call (as radial_attn_fwd documents them); fills *a, wg_trace = null.
int make_fwd_args(int32_t B, int32_t H, int32_t N, int32_t D, radial_tensor q, radial_tensor k, radial_tensor v,
                  radial_tensor out, float* lse, const radial_mask* mask, float scale, FwdArgs* a);
// Launches a kernel that only issues dependent bf16 MFMAs from registers; *flops_out (host)
// receives the floating-point operations it performs.
int launch_mfma_probe(int64_t iters, hipStream_t stream, double* flops_out);

// 8-bit scores: Q and K as E4M3 codes ([B, H, N, D] bytes, contiguous) with one scale per
// (batch, head, block of tokens).
struct Fp8FwdArgs {
  const uint8_t* q8;
  const uint8_t* k8;
  const float* q_scale;  // [B, H, n_blocks]
  const float* k_scale;
  TensorArg v, o;
  float* lse;  // may be null
  const int32_t* row_ptr;
  const int32_t* col_idx;
  WorkMap work;
  int32_t B, H, N, n_blocks;
  float scale;
  const int32_t* pair_order;  // as in FwdArgs
};
int launch_fwd_fp8(const Fp8FwdArgs& a, hipStream_t stream);
int launch_quantize_fp8(int32_t B, int32_t H, int32_t N, int32_t D, const TensorArg& x, int32_t block, uint8_t* codes,
                        float* scales, hipStream_t stream);

struct BwdArgs {
  TensorArg q, k, v, o, dout, dq, dk, dv;
  const float* lse;
  float* delta;   // workspace: [B, H, N] rowsum(dO * O)
  const int32_t* row_ptr;
  const int32_t* col_idx;
  const int32_t* col_ptr;
  const int32_t* row_idx;
  WorkMap work;    // query blocks
  WorkMap work_t;  // key blocks
  int32_t B, H, N, n_blocks;
  float scale;
  TokenRule rule;
  const int32_t* pair_order_t;  // pairs of key blocks by falling length; null as in FwdArgs
};

int launch_bwd(int D, int block, const BwdArgs& a, hipStream_t stream);

}  // namespace radial

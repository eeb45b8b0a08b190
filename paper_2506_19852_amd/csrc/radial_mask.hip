// Radial block-mask construction on the GPU (integer kernels) and the radial_mask object.
//
// The token-level rule is the formal definition of Sec. 4.2 of the paper plus the attention
// sink of App. A.1.  For one query frame i and one key frame j it keeps, for the query
// positions k in [klo, khi], the key positions
//     sink (j < sink_frames):              the whole frame,
//     b = 2^floor(log2 max(|i-j|,1)) <= s:  l in [klo-(w-1), khi+(w-1)] clipped to the frame, w = floor(s/b),
//     b > s and |i-j| mod ceil(b/s) == 0:   l in [klo, khi]  (single diagonal k == l),
// so the key blocks touched by a query block are a union of contiguous block ranges, one per
// (query frame in the block, key frame).  Each workgroup ORs those ranges into a bitmap in
// LDS; a count pass and a pass in which every row finds its place among the counts turn the bitmaps into
// compressed lists (above kMaxOrdered blocks: count, exclusive scan, fill).
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include "radial_internal.h"

namespace radial {

static thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
  return code;
}

namespace {

constexpr int kThreads = 256;
// Blocks up to which a radial mask's lists get room for every pair, so that nothing has to be known before
// they are written (up to 2 MiB per list; hipMalloc becomes slow from there on, and counting first is then cheaper).
// radial_mask_build and free, four kernels and two waits / two kernels and one wait (then with a copy, see Meta): 110 blocks 61 / 34 us, 720 blocks
// 62 / 35; 929 blocks 65 / 73.  With the transposed lists both come from one hipMalloc, of 2 MiB and more from 512 blocks
// on, which takes most of the gain: 244 blocks 77 / 45, 512 blocks 94 / 90, 720 blocks 149 / 107.
constexpr int32_t kMaxUncounted = 720;
static_assert(kMaxUncounted <= kMaxOrdered, "place_list writes the order");
constexpr int kMaxWords = 15 * 1024;  // 60 KiB of LDS bitmap: up to 491 520 key blocks

struct MaskGeom {
  int32_t f, s, block, sink, n, nb;
  int32_t w0, den;  // sparsity knob c = num/den (frame distances >= 2): w0 = floor(s*num/den)
  int64_t s_num;    // s * num
  // banded patterns: device table [f + 1] of spatial half widths per frame distance (-1: none);
  // null for the radial mask
  const int32_t* half_width;
  int32_t nv;  // video tokens f*s; tokens nv .. n-1 are text tokens (dense rows and columns)
};

__device__ inline int32_t pow2_floor(int32_t d) {
  d = d < 1 ? 1 : d;
  return 1 << (31 - __clz(d));
}

// Bitmap of the key blocks listed for query block qb; words[] is LDS, nwords = ceil(nb/32).
__device__ void row_bitmap(const MaskGeom g, int32_t qb, uint32_t* words, int32_t nwords) {
  for (int32_t w = threadIdx.x; w < nwords; w += blockDim.x) words[w] = 0u;
  __syncthreads();
  const int64_t q0 = (int64_t)qb * g.block;
  int64_t q1 = q0 + g.block - 1;
  if (q1 > (int64_t)g.n - 1) q1 = (int64_t)g.n - 1;
  if (q1 >= g.nv) {  // the block holds a text token: it lists every key block
    for (int32_t w = threadIdx.x; w < nwords; w += blockDim.x) {
      const int32_t left = g.nb - w * 32;
      words[w] = left >= 32 ? 0xffffffffu : ((1u << left) - 1u);
    }
    __syncthreads();
    return;
  }
  if (g.nv < g.n) {  // every video row lists the text tokens' key blocks
    for (int32_t kb = g.nv / g.block + threadIdx.x; kb < g.nb; kb += blockDim.x) atomicOr(&words[kb >> 5], 1u << (kb & 31));
  }
  const int32_t i0 = (int32_t)(q0 / g.s), i1 = (int32_t)(q1 / g.s);
  const int64_t npairs = (int64_t)(i1 - i0 + 1) * g.f;
  for (int64_t p = threadIdx.x; p < npairs; p += blockDim.x) {
    const int32_t i = i0 + (int32_t)(p / g.f);
    const int32_t j = (int32_t)(p % g.f);
    const int64_t fi = (int64_t)i * g.s;
    const int32_t klo = (int32_t)((q0 > fi ? q0 : fi) - fi);
    const int64_t fe = fi + g.s - 1;
    const int32_t khi = (int32_t)((q1 < fe ? q1 : fe) - fi);
    const int32_t d = i > j ? i - j : j - i;
    const int32_t b = pow2_floor(d);
    int64_t llo, lhi;
    if (j < g.sink) {
      llo = 0;
      lhi = g.s - 1;
    } else if (g.half_width) {
      const int64_t hw = g.half_width[d];
      if (hw < 0) continue;
      llo = klo - hw;
      if (llo < 0) llo = 0;
      lhi = khi + hw;
      if (lhi > g.s - 1) lhi = g.s - 1;
    } else if (d < 2 || g.w0 / b >= 1) {
      // diagonal of width floor(s/b), or floor(c*s/b) for the scaled distances d >= 2
      const int64_t w = d < 2 ? g.s : (g.w0 / b < g.s ? g.w0 / b : g.s);
      llo = klo - (w - 1);
      if (llo < 0) llo = 0;
      lhi = khi + (w - 1);
      if (lhi > g.s - 1) lhi = g.s - 1;
    } else {
      const int32_t stride = (int32_t)(((int64_t)b * g.den + g.s_num - 1) / g.s_num);
      if (d % stride != 0) continue;
      llo = klo;
      lhi = khi;
    }
    const int64_t t0 = (int64_t)j * g.s + llo, t1 = (int64_t)j * g.s + lhi;
    const int32_t b0 = (int32_t)(t0 / g.block), b1 = (int32_t)(t1 / g.block);
    for (int32_t w = b0 >> 5; w <= (b1 >> 5); ++w) {
      const int32_t lo = w == (b0 >> 5) ? (b0 & 31) : 0;
      const int32_t hi = w == (b1 >> 5) ? (b1 & 31) : 31;
      const uint32_t m = (hi == 31 ? 0xffffffffu : ((1u << (hi + 1)) - 1u)) & ~((1u << lo) - 1u);
      atomicOr(&words[w], m);
    }
  }
  __syncthreads();
}

// Exclusive scan of one value per thread across the workgroup (blockDim.x == kThreads).
__device__ int32_t block_exclusive_scan(int32_t v, int32_t* total) {
  __shared__ int32_t part[kThreads];
  part[threadIdx.x] = v;
  __syncthreads();
  for (int off = 1; off < kThreads; off <<= 1) {
    int32_t add = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
    __syncthreads();
    part[threadIdx.x] += add;
    __syncthreads();
  }
  const int32_t incl = part[threadIdx.x];
  if (total) *total = part[kThreads - 1];
  __syncthreads();
  return incl - v;
}

__global__ void __launch_bounds__(kThreads) mask_count_kernel(MaskGeom g, int32_t nwords, int32_t* counts) {
  extern __shared__ uint32_t words[];
  row_bitmap(g, blockIdx.x, words, nwords);
  int32_t c = 0;
  for (int32_t w = threadIdx.x; w < nwords; w += blockDim.x) c += __popc(words[w]);
  int32_t total;
  block_exclusive_scan(c, &total);
  if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

// Writes the entries of words[] (a row's bitmap in LDS) to out, ascending.
__device__ void write_row(const uint32_t* words, int32_t nwords, int32_t* out) {
  const int32_t per = (nwords + kThreads - 1) / kThreads;
  const int32_t w0 = threadIdx.x * per;
  const int32_t w1 = w0 + per < nwords ? w0 + per : nwords;
  int32_t c = 0;
  for (int32_t w = w0; w < w1; ++w) c += __popc(words[w]);
  int32_t pos = block_exclusive_scan(c, nullptr);
  for (int32_t w = w0; w < w1; ++w) {
    uint32_t m = words[w];
    while (m) {
      const int32_t bit = __ffs(m) - 1;
      m &= m - 1;
      out[pos++] = w * 32 + bit;
    }
  }
}

__global__ void __launch_bounds__(kThreads) mask_fill_kernel(MaskGeom g, int32_t nwords, const int32_t* row_ptr,
                                                            int32_t* col_idx) {
  extern __shared__ uint32_t words[];
  row_bitmap(g, blockIdx.x, words, nwords);
  write_row(words, nwords, col_idx + row_ptr[blockIdx.x]);
}

// In place: counts[0..n) -> exclusive prefix, counts[n] = total (as int32), *total64 = exact total.
__global__ void __launch_bounds__(kThreads) scan_kernel(int32_t* counts, int32_t n, long long* total64) {
  const int32_t per = (n + kThreads - 1) / kThreads;
  const int32_t a = threadIdx.x * per;
  const int32_t b = a + per < n ? a + per : n;
  long long sum = 0;
  for (int32_t i = a; i < b; ++i) sum += counts[i];
  __shared__ long long part[kThreads];
  part[threadIdx.x] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long run = 0;
    for (int t = 0; t < kThreads; ++t) {
      const long long v = part[t];
      part[t] = run;
      run += v;
    }
    *total64 = run;
    counts[n] = run > 0x7fffffffLL ? 0x7fffffff : (int32_t)run;
  }
  __syncthreads();
  long long run = part[threadIdx.x];
  for (int32_t i = a; i < b; ++i) {
    const int32_t v = counts[i];
    counts[i] = (int32_t)(run > 0x7fffffffLL ? 0x7fffffffLL : run);
    run += v;
  }
}

__global__ void dense_fill_kernel(int32_t nb, int32_t* row_ptr, int32_t* col_idx) {
  const int64_t total = (int64_t)nb * nb;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x)
    col_idx[i] = (int32_t)(i % nb);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= nb; i += (int64_t)gridDim.x * blockDim.x)
    row_ptr[i] = (int32_t)(i * nb);
}

__device__ inline bool row_contains(const int32_t* col_idx, int32_t lo, int32_t hi, int32_t key) {
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    const int32_t v = col_idx[mid];
    if (v == key) return true;
    if (v < key) lo = mid + 1; else hi = mid;
  }
  return false;
}

// Sum of (a, b, c) over the workgroup, to every thread.
__device__ void block_sum3(long long& a, long long& b, int32_t& c) {
  __shared__ long long part_a[kThreads / 64], part_b[kThreads / 64];
  __shared__ int32_t part_c[kThreads / 64];
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_xor(a, off);
    b += __shfl_xor(b, off);
    c += __shfl_xor(c, off);
  }
  if ((threadIdx.x & 63) == 0) {
    part_a[threadIdx.x >> 6] = a;
    part_b[threadIdx.x >> 6] = b;
    part_c[threadIdx.x >> 6] = c;
  }
  __syncthreads();
  a = b = 0;
  c = 0;
  for (int w = 0; w < kThreads / 64; ++w) {
    a += part_a[w];
    b += part_b[w];
    c += part_c[w];
  }
  __syncthreads();
}

// Launch partition: slice[k] = first block r whose weight prefix W(r) = ptr[r] + kItemCost*r
// reaches k/8 of the total (slice[0] = 0, slice[8] = nb): 8 runs of consecutive blocks with
// equal work, one per XCD.  kItemCost stands for the fixed cost of a work item (loading Q,
// storing O) in units of one listed block.
constexpr int kItemCost = 4;
__device__ inline long long slice_target(long long total, int32_t nb, int k) {
  return ((total + (long long)kItemCost * nb) * k + 7) / 8;
}

// What a build finds out about its lists, for the launches (device) and for the host: the kernels write both, so that the host
// has it when it has waited for the stream.  A copy of these 128 bytes to pageable memory behind the kernels costs 10 us of that wait (kernel, copy and wait
// 22.5 us, kernel writing mapped memory and wait 12.0); radial_mask_build and free, 110 blocks, 32.4 / 23.2 us.
// [0..1] total of rows, [2..3] total of columns, [4] longest row, [5] longest column, [6] both rows of the longest pair, [8..16] slice, [20..28] slice_t
constexpr int kMetaInts = 32, kTotal = 0, kTotalT = 2, kLongest = 4, kLongestT = 5, kLongestPair = 6, kSlice = 8, kSliceT = 20;
struct Meta {
  int32_t* device;
  int32_t* host;  // mapped host memory, or null
  __device__ void put(int at, int32_t value) const {
    device[at] = value;
    if (host) host[at] = value;
  }
  __device__ void put_total(int at, long long value) const {
    put(at, (int32_t)(uint32_t)(unsigned long long)value);
    put(at + 1, (int32_t)(value >> 32));
  }
};

// What pairs are ordered by: the entries of the lists of blocks r and r + 1.  The list of an odd last block counts twice: it is walked for as long as one of two, and by its entries alone a
// full one (text tokens) came last and began when the first workgroups ended (of the time of one block per workgroup, by its entries / so: 8-bit forward, 4 heads x 269 blocks 1.09 / 0.94, 5 x 215
// 1.06 / 0.90, bf16 8 x 143 1.05 / 0.97).
__device__ inline int32_t pair_length(const int32_t* counts, int32_t nb, int32_t r) { return counts[r] + counts[r + 1 < nb ? r + 1 : r]; }

// What workgroup r needs to know of all lists to write its own: where it starts.  On the way it writes
// ptr[r], the launch partitions, the longest list and the totals, so that neither a scan nor a partition pass is needed: every
// workgroup reads all counts (nb / 256 rounds), which up to kMaxOrdered blocks costs less than the launches.
// columns: of the transposed lists.  pair_order: of the pairs of neighbouring blocks, or null.
__device__ int32_t place_list(const int32_t* counts, int32_t nb, int32_t r, int32_t* ptr, int32_t* order, int32_t* pair_order, const Meta& meta,
                              bool columns) {
  const int slice = columns ? kSliceT : kSlice;
  const int32_t len = counts[r];
  const bool places_pair = pair_order && r % 2 == 0;
  const int32_t pair_len = places_pair ? pair_length(counts, nb, r) : 0;
  long long before = 0, total = 0;
  int32_t ahead = 0;  // blocks with longer lists, and pairs above bit 16: at most 2^14 and 2^13
  for (int32_t j = threadIdx.x; j < nb; j += kThreads) {
    const int32_t other = counts[j];
    total += other;
    before += j < r ? other : 0;
    ahead += (other > len || (other == len && j < r)) ? 1 : 0;
    if (places_pair && j % 2 == 0) {
      const int32_t other_pair = pair_length(counts, nb, j);
      ahead += (other_pair > pair_len || (other_pair == pair_len && j < r)) ? 1 << 16 : 0;
    }
  }
  block_sum3(before, total, ahead);
  const int32_t pairs_ahead = ahead >> 16;
  ahead &= 0xffff;
  if (threadIdx.x == 0) {
    ptr[r] = (int32_t)before;
    order[ahead] = r;
    if (places_pair) pair_order[pairs_ahead] = r / 2;
    if (places_pair && !columns && pairs_ahead == 0) meta.put(kLongestPair, r + 1 < nb ? pair_len : len);
    if (ahead == 0) meta.put(columns ? kLongestT : kLongest, len);
    if (r == nb - 1) {
      ptr[nb] = (int32_t)total;
      meta.put_total(columns ? kTotalT : kTotal, total);
    }
  }
  if (threadIdx.x <= 8) {
    const int k = threadIdx.x;
    const long long w = before + (long long)kItemCost * r, target = slice_target(total, nb, k);
    if (k == 0 || k == 8) {
      if (r == 0) meta.put(slice + k, k == 0 ? 0 : nb);
    } else if (w >= target && (r == 0 || w - counts[r - 1] - kItemCost < target)) {
      meta.put(slice + k, r);
    } else if (r == nb - 1 && w < target) {
      meta.put(slice + k, nb);
    }
  }
  return (int32_t)before;
}

__global__ void __launch_bounds__(kThreads) mask_lists_kernel(MaskGeom g, int32_t nwords, const int32_t* counts, int32_t* row_ptr,
                                                             int32_t* order, Meta meta, int32_t* col_idx, int32_t* pair_order) {
  extern __shared__ uint32_t words[];
  row_bitmap(g, blockIdx.x, words, nwords);
  const int32_t start = place_list(counts, g.nb, blockIdx.x, row_ptr, order, pair_order, meta, false);
  write_row(words, nwords, col_idx + start);
}

// Transposed lists: workgroup kb looks kb up in every (ascending) row.
__global__ void __launch_bounds__(kThreads) transpose_count_kernel(const int32_t* row_ptr, const int32_t* col_idx,
                                                                  int32_t nb, int32_t* tcounts) {
  const int32_t kb = blockIdx.x;
  int32_t c = 0;
  for (int32_t qb = threadIdx.x; qb < nb; qb += blockDim.x)
    c += row_contains(col_idx, row_ptr[qb], row_ptr[qb + 1], kb) ? 1 : 0;
  int32_t total;
  block_exclusive_scan(c, &total);
  if (threadIdx.x == 0) tcounts[kb] = total;
}

__device__ void write_column(const int32_t* row_ptr, const int32_t* col_idx, int32_t nb, int32_t kb, int32_t pos, int32_t* row_idx) {
  for (int32_t base = 0; base < nb; base += kThreads) {
    const int32_t qb = base + threadIdx.x;
    const int32_t hit = (qb < nb && row_contains(col_idx, row_ptr[qb], row_ptr[qb + 1], kb)) ? 1 : 0;
    int32_t total;
    const int32_t off = block_exclusive_scan(hit, &total);
    if (hit) row_idx[pos + off] = qb;
    pos += total;
  }
}

__global__ void __launch_bounds__(kThreads) transpose_fill_kernel(const int32_t* row_ptr, const int32_t* col_idx,
                                                                 int32_t nb, const int32_t* col_ptr, int32_t* row_idx) {
  write_column(row_ptr, col_idx, nb, blockIdx.x, col_ptr[blockIdx.x], row_idx);
}

__global__ void __launch_bounds__(kThreads) transpose_lists_kernel(const int32_t* row_ptr, const int32_t* col_idx, int32_t nb,
                                                                  const int32_t* counts, int32_t* col_ptr, int32_t* order, Meta meta,
                                                                  int32_t* row_idx, int32_t* pair_order) {
  const int32_t start = place_list(counts, nb, blockIdx.x, col_ptr, order, pair_order, meta, true);
  write_column(row_ptr, col_idx, nb, blockIdx.x, start, row_idx);
}

// Workgroup 0 cuts the slices; the others, a wave per block, place the block (and its pair) at its rank by falling
// list length (equal lengths: by index) if there is an order to fill, and the first writes its length.
__global__ void __launch_bounds__(kThreads) partition_kernel(const int32_t* ptr, int32_t nb, int32_t* order, int32_t* pair_order, Meta meta, bool columns) {
  if (blockIdx.x > 0) {
    const int32_t b = (blockIdx.x - 1) * (kThreads / 64) + (threadIdx.x >> 6);
    if (b >= nb) return;
    const int32_t len = ptr[b + 1] - ptr[b];
    int32_t ahead = 0;
    for (int32_t j = threadIdx.x & 63; j < nb; j += 64) {
      const int32_t other = ptr[j + 1] - ptr[j];
      ahead += (other > len || (other == len && j < b)) ? 1 : 0;
    }
    const bool places_pair = pair_order && b % 2 == 0;
    int32_t pair_len = 0;
    if (places_pair) {
      const auto length = [&](int32_t r) { return r + 1 < nb ? ptr[r + 2] - ptr[r] : 2 * (ptr[r + 1] - ptr[r]); };  // as pair_length
      pair_len = length(b);
      for (int32_t j = 2 * (threadIdx.x & 63); j < nb; j += 128) {
        const int32_t other = length(j);
        ahead += (other > pair_len || (other == pair_len && j < b)) ? 1 << 16 : 0;
      }
    }
    for (int off = 32; off > 0; off >>= 1) ahead += __shfl_xor(ahead, off);  // at most 2^14 blocks, 2^13 pairs
    const int32_t pairs_ahead = ahead >> 16;
    ahead &= 0xffff;
    if ((threadIdx.x & 63) == 0) {
      order[ahead] = b;
      if (places_pair) pair_order[pairs_ahead] = b / 2;
      if (places_pair && !columns && pairs_ahead == 0) meta.put(kLongestPair, b + 1 < nb ? pair_len : len);
      if (ahead == 0) meta.put(columns ? kLongestT : kLongest, len);
    }
    return;
  }
  const int k = threadIdx.x;
  if (k > 8) return;
  const long long target = slice_target(ptr[nb], nb, k);
  int32_t lo = 0, hi = nb;  // smallest r in [0, nb] with W(r) >= target
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if ((long long)ptr[mid] + (long long)kItemCost * mid >= target) hi = mid; else lo = mid + 1;
  }
  meta.put((columns ? kSliceT : kSlice) + k, k == 8 ? nb : (k == 0 ? 0 : lo));
}

int check_common(int64_t n_tokens, int32_t block, uint32_t flags) {
  if (block != 64 && block != 128) return fail(RADIAL_EUNSUPPORTED, "block must be 64 or 128 (got %d)", block);
  if (flags & ~(RADIAL_MASK_TRANSPOSE | RADIAL_MASK_TOKEN_EXACT)) return fail(RADIAL_EINVAL, "unknown mask flag bits 0x%x", flags);
  if (n_tokens < 1 || n_tokens >= (int64_t)0x7fffffff - block)
    return fail(RADIAL_EINVAL, "token count %lld outside [1, 2^31 - block)", (long long)n_tokens);
  const int64_t nb = (n_tokens + block - 1) / block;
  if ((nb + 31) / 32 > kMaxWords) return fail(RADIAL_EUNSUPPORTED, "more than %d key blocks", kMaxWords * 32);
  return RADIAL_OK;
}

// Device storage of a mask is three allocations: `meta` (two 64-bit totals and the two launch
// partitions), `ptrs` (row_ptr, its order and that of its pairs and, with the transposed lists, the same of col_ptr) and `idx` (col_idx and
// row_idx).  The views d_row_ptr, d_col_ptr, ... point into them at 256-byte aligned offsets.
int launch_partition(const int32_t* ptr, int32_t nb, int32_t* order, int32_t* pair_order, const Meta& meta, bool columns, hipStream_t st) {
  const int32_t per = kThreads / 64;
  partition_kernel<<<1 + (order ? (nb + per - 1) / per : 0), kThreads, 0, st>>>(ptr, nb, order, pair_order, meta, columns);
  RADIAL_HIP_TRY(hipGetLastError());
  return RADIAL_OK;
}

// A Meta's host side for the time of one build: a slot of one page of mapped host memory that the process keeps (mapping it anew would
// cost more than it saves).  A build that finds no slot free, or no page, copies instead.  One that ends early waits for what it has
// queued on its stream before the slot goes to another; where the stream cannot be waited for, the slot is not used again.
class HostMeta {
 public:
  explicit HostMeta(hipStream_t stream) : stream_(stream) {
    const std::lock_guard<std::mutex> lock(mutex());
    static int32_t* const page = [] {
      void* p = nullptr;
      if (hipHostMalloc(&p, kSlots * kMetaInts * sizeof(int32_t), hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
        (void)hipGetLastError();  // the build goes on without
        p = nullptr;
      }
      return (int32_t*)p;
    }();
    for (int i = 0; page && i < kSlots && slot_ < 0; ++i)
      if (!(used() >> i & 1u)) slot_ = i;
    if (slot_ < 0) return;
    void* device = nullptr;
    if (hipHostGetDevicePointer(&device, page + slot_ * kMetaInts, 0) != hipSuccess) {
      (void)hipGetLastError();
      slot_ = -1;
      return;
    }
    used() |= 1u << slot_;
    host_ = page + slot_ * kMetaInts;
    device_ = (int32_t*)device;
  }
  HostMeta(const HostMeta&) = delete;
  ~HostMeta() {
    if (slot_ >= 0 && hipStreamSynchronize(stream_) == hipSuccess) release();
  }
  // Once the kernels of the build have ended.
  void release() {
    if (slot_ < 0) return;
    const std::lock_guard<std::mutex> lock(mutex());
    used() &= ~(1u << slot_);
    slot_ = -1;
  }
  const int32_t* host() const { return host_; }  // null: none
  int32_t* device() const { return device_; }

 private:
  static constexpr int kSlots = 32;
  static std::mutex& mutex() {
    static std::mutex m;
    return m;
  }
  static uint32_t& used() {
    static uint32_t bits = 0;
    return bits;
  }
  hipStream_t stream_;
  int slot_ = -1;
  int32_t* host_ = nullptr;
  int32_t* device_ = nullptr;
};

inline int64_t aligned_ints(int64_t n) { return (n + 63) & ~(int64_t)63; }

int alloc_meta_and_ptrs(radial_mask* m) {
  const int64_t np = aligned_ints((int64_t)m->n_blocks + 1);
  RADIAL_HIP_TRY(hipMalloc(&m->d_meta, sizeof(int32_t) * kMetaInts));
  const int64_t no = m->n_blocks <= kMaxOrdered ? aligned_ints(m->n_blocks) : 0;
  const int64_t lists = (m->flags & RADIAL_MASK_TRANSPOSE) ? 2 : 1;
  // Only kernels on blocks of 128 that are dense inside take pairs (a build of 44 to 87 lists of 64 tokens and the forward behind it 78.5 us without their order, 79.1 with).
  const bool paired = no && m->block == 128 && !(m->flags & RADIAL_MASK_TOKEN_EXACT);
  const int64_t pairs = paired ? aligned_ints((m->n_blocks + 1) / 2) : 0;
  RADIAL_HIP_TRY(hipMalloc(&m->d_ptrs, sizeof(int32_t) * ((np + no + pairs) * lists + no)));
  if (no) m->d_counts = m->d_ptrs + (np + no) * lists;
  if (paired) m->d_pair_order = m->d_counts + no;
  if (paired && lists == 2) m->d_pair_order_t = m->d_pair_order + pairs;
  m->d_row_ptr = m->d_ptrs;
  if (no) m->d_order = m->d_ptrs + np;
  m->d_slice = m->d_meta + kSlice;
  if (m->flags & RADIAL_MASK_TRANSPOSE) {
    m->d_col_ptr = m->d_ptrs + np + no;
    if (no) m->d_order_t = m->d_col_ptr + np;
    m->d_slice_t = m->d_meta + kSliceT;
  }
  return RADIAL_OK;
}

// Needs m->nnz (or a bound of it).
int alloc_idx(radial_mask* m) {
  const int64_t ni = aligned_ints(m->nnz > 0 ? m->nnz : 1);
  RADIAL_HIP_TRY(hipMalloc(&m->d_idx, sizeof(int32_t) * ni * ((m->flags & RADIAL_MASK_TRANSPOSE) ? 2 : 1)));
  m->d_col_idx = m->d_idx;
  if (m->flags & RADIAL_MASK_TRANSPOSE) m->d_row_idx = m->d_idx + ni;
  return RADIAL_OK;
}

// Shared tail of the constructors: transposed lists (optional) and launch partitions, then the one
// wait of the call for everything queued on the stream (the partitions come back to the host).
// rows_placed: the rows' launch partitions and their total are written already.  Here and above, every launch is checked before the
// next: a kernel that finds what an earlier one should have written uninitialised reads and writes anywhere.
int finish_mask(radial_mask* m, HostMeta& shared, bool rows_placed, hipStream_t st) {
  const int32_t nb = m->n_blocks;
  const Meta meta = {m->d_meta, shared.device()};
  alignas(8) int32_t h_meta[kMetaInts];
  if (!rows_placed)
    if (int rc = launch_partition(m->d_row_ptr, nb, m->d_order, m->d_pair_order, meta, false, st)) return rc;
  if ((m->flags & RADIAL_MASK_TRANSPOSE) && m->d_counts) {
    transpose_count_kernel<<<nb, kThreads, 0, st>>>(m->d_row_ptr, m->d_col_idx, nb, m->d_counts);
    RADIAL_HIP_TRY(hipGetLastError());
    transpose_lists_kernel<<<nb, kThreads, 0, st>>>(m->d_row_ptr, m->d_col_idx, nb, m->d_counts, m->d_col_ptr, m->d_order_t, meta, m->d_row_idx, m->d_pair_order_t);
    RADIAL_HIP_TRY(hipGetLastError());
  } else if (m->flags & RADIAL_MASK_TRANSPOSE) {
    transpose_count_kernel<<<nb, kThreads, 0, st>>>(m->d_row_ptr, m->d_col_idx, nb, m->d_col_ptr);
    RADIAL_HIP_TRY(hipGetLastError());
    scan_kernel<<<1, kThreads, 0, st>>>(m->d_col_ptr, nb, (long long*)(m->d_meta + kTotalT));
    RADIAL_HIP_TRY(hipGetLastError());
    transpose_fill_kernel<<<nb, kThreads, 0, st>>>(m->d_row_ptr, m->d_col_idx, nb, m->d_col_ptr, m->d_row_idx);
    RADIAL_HIP_TRY(hipGetLastError());
    if (int rc = launch_partition(m->d_col_ptr, nb, m->d_order_t, m->d_pair_order_t, meta, true, st)) return rc;
  }
  hipError_t e = hipSuccess;
  if (!shared.host()) e = hipMemcpyAsync(h_meta, m->d_meta, sizeof h_meta, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return fail(RADIAL_EHIP, "mask kernels failed: %s", hipGetErrorString(e));
  if (shared.host()) memcpy(h_meta, shared.host(), sizeof h_meta);
  shared.release();
  if (rows_placed) memcpy(&m->nnz, h_meta + kTotal, sizeof m->nnz);
  m->longest = m->d_order ? h_meta[kLongest] : nb;
  m->longest_pair = m->d_pair_order ? h_meta[kLongestPair] : 0;
  if (m->flags & RADIAL_MASK_TRANSPOSE) m->longest_t = m->d_order_t ? h_meta[kLongestT] : nb;
  for (int k = 0; k < 8; ++k) {
    const int32_t len = h_meta[kSlice + k + 1] - h_meta[kSlice + k];
    m->max_slice = len > m->max_slice ? len : m->max_slice;
    if (m->flags & RADIAL_MASK_TRANSPOSE) {
      const int32_t len_t = h_meta[kSliceT + k + 1] - h_meta[kSliceT + k];
      m->max_slice_t = len_t > m->max_slice_t ? len_t : m->max_slice_t;
    }
  }
  return RADIAL_OK;
}

}  // namespace
}  // namespace radial

using namespace radial;

extern "C" const char* radial_last_error(void) { return radial::g_err; }

extern "C" void radial_mask_free(radial_mask* m) {
  if (!m) return;
  (void)hipFree(m->d_meta);
  (void)hipFree(m->d_ptrs);
  (void)hipFree(m->d_idx);
  (void)hipFree(m->d_half_width);
  delete m;
}

static int new_mask(int64_t n_tokens, int32_t block, uint32_t flags, radial_mask** out, radial_mask** m) {
  if (!out) return fail(RADIAL_EINVAL, "out is NULL");
  *out = nullptr;
  if (int rc = check_common(n_tokens, block, flags)) return rc;
  radial_mask* mm = new (std::nothrow) radial_mask();
  if (!mm) return fail(RADIAL_ENOMEM, "host allocation failed");
  mm->n_tokens = (int32_t)n_tokens;
  mm->block = block;
  mm->n_blocks = (int32_t)((n_tokens + block - 1) / block);
  mm->flags = flags;
  if (hipGetDevice(&mm->device) != hipSuccess) {
    delete mm;
    return fail(RADIAL_EHIP, "hipGetDevice failed");
  }
  *m = mm;
  return RADIAL_OK;
}

// Lists of a radial mask (m->d_half_width null) or of a banded pattern (table already on the device).
static int build_radial(radial_mask* m, const radial_mask_params* p, hipStream_t st) {
  const int32_t nb = m->n_blocks;
  const int32_t nwords = (nb + 31) / 32;
  const int64_t s_num = (int64_t)p->tokens_per_frame * p->width_num;
  const MaskGeom g{p->frames, p->tokens_per_frame, p->block, p->sink_frames, m->n_tokens, nb,
                   (int32_t)(s_num / p->width_den), p->width_den, s_num, m->d_half_width,
                   (int32_t)((int64_t)p->frames * p->tokens_per_frame)};
  long long total = 0;
  if (int rc = alloc_meta_and_ptrs(m)) return rc;
  if (m->d_counts) {
    mask_count_kernel<<<nb, kThreads, nwords * sizeof(uint32_t), st>>>(g, nwords, m->d_counts);
    RADIAL_HIP_TRY(hipGetLastError());
    if (nb <= kMaxUncounted) {
      m->nnz = (int64_t)nb * nb;
    } else {
      const std::unique_ptr<int32_t[]> counts(new (std::nothrow) int32_t[nb]);
      if (!counts) return fail(RADIAL_ENOMEM, "host allocation failed");
      hipError_t e = hipMemcpyAsync(counts.get(), m->d_counts, sizeof(int32_t) * nb, hipMemcpyDeviceToHost, st);
      if (e == hipSuccess) e = hipStreamSynchronize(st);   // the list storage is sized by the count
      if (e != hipSuccess) return fail(RADIAL_EHIP, "mask count failed: %s", hipGetErrorString(e));
      for (int32_t r = 0; r < nb; ++r) m->nnz += counts[r];  // at most kMaxOrdered^2 = 2^28
    }
    if (int rc = alloc_idx(m)) return rc;
    HostMeta shared(st);
    mask_lists_kernel<<<nb, kThreads, nwords * sizeof(uint32_t), st>>>(g, nwords, m->d_counts, m->d_row_ptr, m->d_order,
                                                                       Meta{m->d_meta, shared.device()}, m->d_col_idx, m->d_pair_order);
    RADIAL_HIP_TRY(hipGetLastError());
    return finish_mask(m, shared, true, st);
  }
  mask_count_kernel<<<nb, kThreads, nwords * sizeof(uint32_t), st>>>(g, nwords, m->d_row_ptr);
  RADIAL_HIP_TRY(hipGetLastError());
  scan_kernel<<<1, kThreads, 0, st>>>(m->d_row_ptr, nb, (long long*)m->d_meta);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpyAsync(&total, m->d_meta, sizeof total, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);   // the list storage is sized by the count
  if (e != hipSuccess) return fail(RADIAL_EHIP, "mask count failed: %s", hipGetErrorString(e));
  if (total > 0x7fffffffLL) return fail(RADIAL_EUNSUPPORTED, "%lld listed block pairs do not fit int32", total);
  m->nnz = total;
  if (int rc = alloc_idx(m)) return rc;
  mask_fill_kernel<<<nb, kThreads, nwords * sizeof(uint32_t), st>>>(g, nwords, m->d_row_ptr, m->d_col_idx);
  RADIAL_HIP_TRY(hipGetLastError());
  HostMeta shared(st);
  return finish_mask(m, shared, false, st);
}

extern "C" int radial_mask_build(const radial_mask_params* p, void* hip_stream, radial_mask** out) {
  if (!p) return fail(RADIAL_EINVAL, "params is NULL");
  if (p->frames < 1 || p->tokens_per_frame < 1 || p->sink_frames < 0 || p->extra_tokens < 0)
    return fail(RADIAL_EINVAL, "need frames >= 1, tokens_per_frame >= 1, sink_frames >= 0, extra_tokens >= 0");
  if ((p->flags & RADIAL_MASK_TOKEN_EXACT) && p->tokens_per_frame < 64)
    return fail(RADIAL_EUNSUPPORTED, "RADIAL_MASK_TOKEN_EXACT needs tokens_per_frame >= 64");
  if (p->width_num < 1 || p->width_num > 32767 || p->width_den < 1 || p->width_den > 32767)
    return fail(RADIAL_EINVAL, "width_num and width_den must be in [1, 32767] (1, 1 for the paper's mask)");
  if ((int64_t)p->tokens_per_frame * p->width_num > 0x7fffffffLL)
    return fail(RADIAL_EINVAL, "tokens_per_frame * width_num must be below 2^31");
  radial_mask* m = nullptr;
  if (int rc = new_mask((int64_t)p->frames * p->tokens_per_frame + p->extra_tokens, p->block, p->flags, out, &m)) return rc;
  m->tokens_per_frame = p->tokens_per_frame;
  m->frames = p->frames;
  m->sink_frames = p->sink_frames;
  m->width_num = p->width_num;
  m->width_den = p->width_den;
  const int rc = build_radial(m, p, (hipStream_t)hip_stream);
  if (rc) {
    radial_mask_free(m);
    return rc;
  }
  *out = m;
  return RADIAL_OK;
}

extern "C" int radial_mask_build_banded(int32_t frames, int32_t tokens_per_frame, int32_t block, int32_t sink_frames,
                                        const int32_t* half_width, uint32_t flags, void* hip_stream,
                                        radial_mask** out) {
  if (frames < 1 || tokens_per_frame < 1 || sink_frames < 0)
    return fail(RADIAL_EINVAL, "need frames >= 1, tokens_per_frame >= 1, sink_frames >= 0");
  if (!half_width) return fail(RADIAL_EINVAL, "half_width is NULL");
  if ((flags & RADIAL_MASK_TOKEN_EXACT) && tokens_per_frame < 64)
    return fail(RADIAL_EUNSUPPORTED, "RADIAL_MASK_TOKEN_EXACT needs tokens_per_frame >= 64");
  radial_mask* m = nullptr;
  if (int rc = new_mask((int64_t)frames * tokens_per_frame, block, flags, out, &m)) return rc;
  m->tokens_per_frame = tokens_per_frame;
  m->frames = frames;
  m->sink_frames = sink_frames;
  // device table with one extra entry: the kernels also look up the distance to the frame after
  // the last one (a stage of keys may run past the end of the sequence)
  std::vector<int32_t> table((size_t)frames + 1, -1);
  // (half widths beyond a frame mean the whole frame; as tokens_per_frame the kernels' sums of positions stay within 32 bits)
  for (int32_t d = 0; d < frames; ++d) table[d] = half_width[d] < -1 ? -1 : half_width[d] < tokens_per_frame ? half_width[d] : tokens_per_frame;
  const hipStream_t st = (hipStream_t)hip_stream;
  int rc = RADIAL_OK;
  if (hipMalloc(&m->d_half_width, sizeof(int32_t) * table.size()) != hipSuccess ||
      hipMemcpyAsync(m->d_half_width, table.data(), sizeof(int32_t) * table.size(), hipMemcpyHostToDevice, st) != hipSuccess)
    rc = fail(RADIAL_EHIP, "copying the half-width table failed");
  if (!rc) {  // `table` stays alive until build_radial has waited for the stream
    const radial_mask_params p{frames, tokens_per_frame, block, sink_frames, flags, 1, 1, 0};
    rc = build_radial(m, &p, st);
  }
  if (rc) {
    radial_mask_free(m);
    return rc;
  }
  *out = m;
  return RADIAL_OK;
}

static int build_dense(radial_mask* m, hipStream_t st) {
  const int64_t nb = m->n_blocks;
  if (nb * nb > 0x7fffffffLL) return fail(RADIAL_EUNSUPPORTED, "%lld block pairs do not fit int32", (long long)(nb * nb));
  m->nnz = nb * nb;
  if (int rc = alloc_meta_and_ptrs(m)) return rc;
  if (int rc = alloc_idx(m)) return rc;
  dense_fill_kernel<<<1024, kThreads, 0, st>>>((int32_t)nb, m->d_row_ptr, m->d_col_idx);
  RADIAL_HIP_TRY(hipGetLastError());
  HostMeta shared(st);
  return finish_mask(m, shared, false, st);
}

extern "C" int radial_mask_build_dense(int32_t n_tokens, int32_t block, uint32_t flags, void* hip_stream,
                                       radial_mask** out) {
  if (flags & RADIAL_MASK_TOKEN_EXACT) return fail(RADIAL_EINVAL, "RADIAL_MASK_TOKEN_EXACT applies to radial_mask_build only");
  radial_mask* m = nullptr;
  if (int rc = new_mask(n_tokens, block, flags, out, &m)) return rc;
  const int rc = build_dense(m, (hipStream_t)hip_stream);
  if (rc) {
    radial_mask_free(m);
    return rc;
  }
  *out = m;
  return RADIAL_OK;
}

// Whether lists 2p and 2p + 1 have at least a fifth of their entries in common, from 64 to 127 pairs spread over all (all of fewer).
static bool neighbours_alike(const int32_t* row_ptr, const int32_t* col_idx, int32_t nb) {
  const int32_t pairs = nb / 2, step = pairs < 64 ? 1 : pairs / 64;
  int64_t entries = 0, common = 0;
  for (int32_t p = 0; p < pairs; p += step) {
    int32_t i = row_ptr[2 * p], j = row_ptr[2 * p + 1];
    const int32_t i_end = j, j_end = row_ptr[2 * p + 2];
    entries += j_end - i;
    while (i < i_end && j < j_end) {
      const int32_t a = col_idx[i], b = col_idx[j];
      common += a == b;
      i += a <= b;
      j += b <= a;
    }
  }
  return 10 * common >= entries;
}

static int build_from_csr(radial_mask* m, const int32_t* row_ptr, const int32_t* col_idx, hipStream_t st) {
  const int32_t nb = m->n_blocks;
  if (row_ptr[0] != 0) return fail(RADIAL_EINVAL, "row_ptr[0] must be 0");
  for (int32_t r = 0; r < nb; ++r) {
    if (row_ptr[r + 1] < row_ptr[r]) return fail(RADIAL_EINVAL, "row_ptr decreases at row %d", r);
    for (int32_t e = row_ptr[r]; e < row_ptr[r + 1]; ++e) {
      if (col_idx[e] < 0 || col_idx[e] >= nb) return fail(RADIAL_EINVAL, "row %d: key block %d out of range", r, col_idx[e]);
      if (e > row_ptr[r] && col_idx[e] <= col_idx[e - 1]) return fail(RADIAL_EINVAL, "row %d is not strictly ascending", r);
    }
  }
  m->nnz = row_ptr[nb];
  m->alike = neighbours_alike(row_ptr, col_idx, nb);
  if (int rc = alloc_meta_and_ptrs(m)) return rc;
  if (int rc = alloc_idx(m)) return rc;
  // the caller's arrays are read until finish_mask has waited for the stream
  RADIAL_HIP_TRY(hipMemcpyAsync(m->d_row_ptr, row_ptr, sizeof(int32_t) * (nb + 1), hipMemcpyHostToDevice, st));
  if (m->nnz > 0)
    RADIAL_HIP_TRY(hipMemcpyAsync(m->d_col_idx, col_idx, sizeof(int32_t) * m->nnz, hipMemcpyHostToDevice, st));
  HostMeta shared(st);
  return finish_mask(m, shared, false, st);
}

extern "C" int radial_mask_from_csr(int32_t n_tokens, int32_t block, uint32_t flags, const int32_t* row_ptr,
                                    const int32_t* col_idx, void* hip_stream, radial_mask** out) {
  if (!row_ptr) return fail(RADIAL_EINVAL, "row_ptr is NULL");
  if (flags & RADIAL_MASK_TOKEN_EXACT) return fail(RADIAL_EINVAL, "RADIAL_MASK_TOKEN_EXACT applies to radial_mask_build only");
  radial_mask* m = nullptr;
  if (int rc = new_mask(n_tokens, block, flags, out, &m)) return rc;
  int rc = RADIAL_OK;
  if (!col_idx && row_ptr[m->n_blocks] != 0) rc = fail(RADIAL_EINVAL, "col_idx is NULL");
  if (!rc) rc = build_from_csr(m, row_ptr, col_idx, (hipStream_t)hip_stream);
  if (rc) {
    radial_mask_free(m);
    return rc;
  }
  *out = m;
  return RADIAL_OK;
}

extern "C" int radial_mask_info(const radial_mask* m, int32_t* n_tokens, int32_t* block, int32_t* n_blocks,
                                int64_t* nnz, uint32_t* flags) {
  if (!m) return fail(RADIAL_EINVAL, "mask is NULL");
  if (n_tokens) *n_tokens = m->n_tokens;
  if (block) *block = m->block;
  if (n_blocks) *n_blocks = m->n_blocks;
  if (nnz) *nnz = m->nnz;
  if (flags) *flags = m->flags;
  return RADIAL_OK;
}

extern "C" int radial_mask_copy_to_host(const radial_mask* m, int32_t* row_ptr, int32_t* col_idx) {
  if (!m) return fail(RADIAL_EINVAL, "mask is NULL");
  if (row_ptr) RADIAL_HIP_TRY(hipMemcpy(row_ptr, m->d_row_ptr, sizeof(int32_t) * (m->n_blocks + 1), hipMemcpyDeviceToHost));
  if (col_idx && m->nnz > 0) RADIAL_HIP_TRY(hipMemcpy(col_idx, m->d_col_idx, sizeof(int32_t) * m->nnz, hipMemcpyDeviceToHost));
  return RADIAL_OK;
}

extern "C" int radial_mask_copy_transpose_to_host(const radial_mask* m, int32_t* col_ptr, int32_t* row_idx) {
  if (!m) return fail(RADIAL_EINVAL, "mask is NULL");
  if (!(m->flags & RADIAL_MASK_TRANSPOSE)) return fail(RADIAL_ESHAPE, "mask was built without RADIAL_MASK_TRANSPOSE");
  if (col_ptr) RADIAL_HIP_TRY(hipMemcpy(col_ptr, m->d_col_ptr, sizeof(int32_t) * (m->n_blocks + 1), hipMemcpyDeviceToHost));
  if (row_idx && m->nnz > 0) RADIAL_HIP_TRY(hipMemcpy(row_idx, m->d_row_idx, sizeof(int32_t) * m->nnz, hipMemcpyDeviceToHost));
  return RADIAL_OK;
}

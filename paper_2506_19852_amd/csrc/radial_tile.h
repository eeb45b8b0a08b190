// Device helpers shared by the attention kernels: MFMA operand types, LDS tile addressing,
// HBM -> LDS copies.  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "radial_internal.h"

namespace radial {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(8))) int i32x8;

// Generic pointer into a __shared__ array -> LDS (address space 3) pointer.
template <class T>
__device__ __forceinline__ __attribute__((address_space(3))) T* lds_cast(const void* p) {
  return (__attribute__((address_space(3))) T*)(p);
}

// LDS address -> LDS pointer.
template <class T>
__device__ __forceinline__ __attribute__((address_space(3))) T* lds_pointer(uint32_t address) {
  return (__attribute__((address_space(3))) T*)(uintptr_t)address;
}

__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)lds_cast<char>(p); }

// v_mfma_f32_32x32x16_bf16: D[32x32] += A[32x16] * B[16x32].
//   A: lane l holds row l%32, k = 8*(l/32) .. +7;   B: lane l holds column l%32, same k;
//   D: lane l holds column l%32, element e is row 8*(e/4) + 4*(l/32) + e%4.
// A and B have the same register layout, so swapping them transposes the product.
__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  f32x2 f = {a, b};
  bf16x2 h = __builtin_convertvector(f, bf16x2);
  return __builtin_bit_cast(uint32_t, h);
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const u32x4 raw = {a, b, c, d};
  return __builtin_bit_cast(bf16x8, raw);
}

// The lane's number again, so that nothing derived from it is held in a register meanwhile.
__device__ __forceinline__ int lane_again() {
  int lane;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
  return lane;
}

// The kernel's first parameter, asked for here and not before.
template <class Args>
__device__ __forceinline__ const Args& own_args() {
  using Own = const Args __attribute__((address_space(4)));
  Own* args = (Own*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(args));  // not known to be the same memory
  return *(const Args*)args;
}

// One 1 KiB HBM -> LDS copy: lane i's 16 bytes land at LDS address lds_addr + 16*i.  Issued
// from assembly so that the compiler does not order later LDS reads after it; the caller
// waits with wait_all_copies() and a barrier before anyone reads the destination.
__device__ __forceinline__ void copy16_to_lds(const void* gptr, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(gptr) : "memory", "m0");
}
// copy16_to_lds with the address split into a wave-uniform 64-bit base (SGPRs) and a per-lane
// 32-bit byte offset, so that walking to the next tile costs scalar arithmetic only.
__device__ __forceinline__ void copy16_to_lds_sv(const void* base, uint32_t byte_offset, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(byte_offset), "s"(base) : "memory", "m0");
}
// copy16_to_lds_sv for the lanes set in `lanes` only (all or none in practice: with no lane the
// instruction is a no-op, which lets straight-line code switch a copy off without a branch).
__device__ __forceinline__ void copy16_to_lds_sv_masked(const void* base, uint32_t byte_offset, uint32_t lds_addr, uint64_t lanes) {
  // `lanes` is wave-uniform by contract; say so to the compiler (the operand must be scalar)
  lanes = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(lanes >> 32)) << 32) | __builtin_amdgcn_readfirstlane((uint32_t)lanes);
  uint64_t saved;
  asm volatile("s_mov_b32 m0, %1\n\ts_and_saveexec_b64 %0, %4\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, %0"
               : "=&s"(saved) : "s"(lds_addr), "v"(byte_offset), "s"(base), "s"(lanes) : "memory", "scc", "m0");
}
// The 4-byte form of copy16_to_lds_sv_masked (256 bytes per wave).
__device__ __forceinline__ void copy4_to_lds_sv_masked(const void* base, uint32_t byte_offset, uint32_t lds_addr, uint64_t lanes) {
  // `lanes` is wave-uniform by contract; say so to the compiler (the operand must be scalar)
  lanes = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(lanes >> 32)) << 32) | __builtin_amdgcn_readfirstlane((uint32_t)lanes);
  uint64_t saved;
  asm volatile("s_mov_b32 m0, %1\n\ts_and_saveexec_b64 %0, %4\n\tglobal_load_lds_dword %2, %3\n\ts_mov_b64 exec, %0"
               : "=&s"(saved) : "s"(lds_addr), "v"(byte_offset), "s"(base), "s"(lanes) : "memory", "scc", "m0");
}
// Same as copy16_to_lds with 4 bytes per lane (256 bytes per wave).
__device__ __forceinline__ void copy4_to_lds(const void* gptr, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr), "v"(gptr) : "memory", "m0");
}
__device__ __forceinline__ void wait_all_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A [rows x kRowElems] bf16 tile in LDS, cut into 16-byte pieces and 256-byte lines.  Pieces
// are XOR-swizzled inside their line so that both access patterns used on a tile are free of
// bank conflicts: 128-bit reads of one piece column over 16 consecutive rows, and the 64-bit
// transposing reads (ds_read_b64_tr_b16) that touch 4 consecutive rows x 64 bytes.
template <int kRowElems>
struct SwzTile {
  static_assert(kRowElems == 64 || kRowElems == 128, "row of 128 or 256 bytes");
  static constexpr int kPieces = kRowElems / 8;
  __device__ static __forceinline__ int key(int line) {
    return kRowElems == 128 ? (((line & 3) << 2) | ((line >> 2) & 3)) : (((line & 1) << 2) | ((line >> 1) & 3));
  }
  // byte offset of piece p of row r
  __device__ static __forceinline__ int piece(int r, int p) {
    const int lin = r * kPieces + p;
    const int line = lin >> 4, slot = lin & 15;
    return (line << 8) + ((slot ^ key(line)) << 4);
  }
  // byte offset of element (r, c); c % 4 == 0 for the 8-byte accesses
  __device__ static __forceinline__ int elem(int r, int c) { return piece(r, c >> 3) + ((c & 7) << 1); }
  // (row, first element) of the source piece that belongs at linear LDS piece index `lin`
  __device__ static __forceinline__ void source_of(int lin, int& r, int& c) {
    const int line = lin >> 4, slot = lin & 15;
    const int src = (line << 4) + (slot ^ key(line));
    r = src / kPieces;
    c = (src % kPieces) * 8;
  }
};

// K8 tile: rows of 128 bytes = 8 pieces of 16 bytes, two rows per 256-byte line; pieces are
// XOR-swizzled inside their line so that the 128-bit reads of one piece column over 16
// consecutive rows touch 16 different 16-byte bank groups.
__device__ __forceinline__ int k8_piece(int r, int p) {
  const int lin = r * 8 + p;
  const int line = lin >> 4, slot = lin & 15;
  return (line << 8) + ((slot ^ (line & 7)) << 4);
}
// (row, piece) of the source that belongs at linear LDS piece index `lin`
__device__ __forceinline__ void k8_source_of(int lin, int& r, int& p) {
  const int line = lin >> 4, slot = lin & 15;
  const int src = (line << 4) + (slot ^ (line & 7));
  r = src >> 3;
  p = src & 7;
}

// Rows of 256 bytes in LDS, four at a time: a copy (1 KiB, 64 lanes x 16 bytes) fetches four rows, lanes 4j .. 4j + 3 of every 16 a 64-byte piece of
// row j, so that the rows lie in turn every 64 bytes, and 16 bytes lie between one four and the next.  Both access patterns, 128-bit reads of one
// 16-byte column over 16 consecutive rows and the transposing 64-bit reads of 4 consecutive rows x 64 bytes, are free of bank conflicts, as with the
// swizzle, but the pieces of a tile are at constant distances from one address per lane, which go into the instructions: no address
// arithmetic and no registers for addresses.
template <int D>
struct RowsTile {
  static_assert(D == 128, "rows of 256 bytes");
  static constexpr int kFourRows = 1024 + 16, kEightRows = 2 * kFourRows;
  // What a lane of a copy fetches: row of the four, element of the row, and its byte offset from the first row (stride sn elements).
  __device__ static __forceinline__ int source_row(int lane) { return lane >> 2 & 3; }
  __device__ static __forceinline__ int source_column(int lane) { return (lane >> 4) * 32 + (lane & 3) * 8; }
  __device__ static __forceinline__ uint32_t source_bytes(int lane, int64_t sn) { return (uint32_t)(source_row(lane) * (int32_t)sn + source_column(lane)) * 2u; }
  // An MFMA operand of 32 rows: this lane's 16 bytes of k-step 0, and the distance to k-step t of the tile-th 32 rows.
  __device__ static __forceinline__ uint32_t row_at(int lane) { return (lane >> 2 & 7) * kFourRows + (lane & 3) * 64 + (lane >> 5) * 16; }
  __device__ static constexpr int row_step(int tile, int t) { return tile * 8 * kFourRows + t / 2 * 256 + t % 2 * 32; }
  // One of 32 columns, by two transposing reads kEightRows apart: this lane's 8 bytes, and the distance to columns 32 * dt of rows 16 * step.
  __device__ static __forceinline__ uint32_t column_at(int lane) {
    return (lane >> 5) * kFourRows + (lane >> 2 & 3) * 64 + (lane >> 4 & 1) * 32 + (lane & 3) * 8;
  }
  __device__ static constexpr int column_step(int step, int dt) { return step * 4 * kFourRows + dt * 256; }
};

// Transposing LDS read: within each group of 16 lanes, lane i supplies the address of 4
// consecutive bf16 of row i/4 (columns 4*(i%4)..) and receives, for column i of that 16-wide
// patch, the values of the group's 4 rows.
__device__ __forceinline__ u32x2 lds_read_tr(const char* p) {
  const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_cast<s16x4>(p));
  return __builtin_bit_cast(u32x2, v);
}

// The value of x in lane e of this lane's row of 16; e is a constant once loops are unrolled.
template <int E>
__device__ __forceinline__ float row_lane_at(float x) {
  constexpr int kRowNewBcast = 0x150, kAll = 0xf;
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), kRowNewBcast + E, kAll, kAll, true));
}
__device__ __forceinline__ float row_lane(float x, int e) {
  switch (e) {
    case 0: return row_lane_at<0>(x);
    case 1: return row_lane_at<1>(x);
    case 2: return row_lane_at<2>(x);
    case 3: return row_lane_at<3>(x);
    case 4: return row_lane_at<4>(x);
    case 5: return row_lane_at<5>(x);
    case 6: return row_lane_at<6>(x);
    case 7: return row_lane_at<7>(x);
    case 8: return row_lane_at<8>(x);
    case 9: return row_lane_at<9>(x);
    case 10: return row_lane_at<10>(x);
    case 11: return row_lane_at<11>(x);
    case 12: return row_lane_at<12>(x);
    case 13: return row_lane_at<13>(x);
    case 14: return row_lane_at<14>(x);
    default: return row_lane_at<15>(x);
  }
}

// max(x, value of x in lane^32), exchanged in registers (v_permlane32_swap: the upper 32 lanes
// of the first operand trade places with the lower 32 lanes of the second).
__device__ __forceinline__ float max_with_other_half(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  // Copy the elements out before reinterpreting them: a bit_cast applied directly to
  // sw[1] reads element 0.
  const uint32_t first = sw[0], second = sw[1];
  return fmaxf(__builtin_bit_cast(float, first), __builtin_bit_cast(float, second));
}

// ---- results of several groups of waves on the same rows ----------------------------------------
// Where S groups share a list each holds a partial result for all rows; they meet in LDS once every stage buffer is
// consumed.  Every wave writes its accumulators there as 16-byte pieces (tile i, quarter e4, lane), and every wave then
// sums an S-th of the pieces over the groups and stores them.  With the waves of one group doing all of it, one other group
// after the other, the merge and the stores took 3900 cycles (four groups, D 64) to 6700 (two, D 128), a tenth of a launch of 64
// items; 96 to 126 items of block 128, training step: 67.8 / 66.1, 48.7 / 46.3, 233 / 231 us.
template <int S, int kWaves, int kTiles, int kBudget = 160 * 1024>
struct Merge {
  static constexpr int kPieces = 4 * kTiles;
  static constexpr int kStatBytes = S * kWaves * 512;  // m and l of every wave, 64 floats each
  static constexpr int kRounds = S * kWaves * kPieces * 1024 + kStatBytes <= kBudget ? 1 : 2;
  static constexpr int kRoundPieces = kPieces / kRounds;
  static constexpr int kOwned = (kRoundPieces + S - 1) / S;  // pieces of a round that one group sums
  static constexpr int kLdsBytes = S == 1 ? 0 : S * kWaves * kRoundPieces * 1024 + kStatBytes;
  static_assert(kLdsBytes <= kBudget, "the partial results of a round fit the LDS");

  // This wave's pieces of round r into LDS.
  __device__ static __forceinline__ void write(const f32x16 (&acc)[kTiles], int r, char* lds, int group, int wave, int lane) {
    char* dst = lds + (group * kWaves + wave) * kRoundPieces * 1024 + lane * 16;
#pragma unroll
    for (int p = 0; p < kPieces; ++p)
      if (p / kRoundPieces == r) {
        const int i = p >> 2, e = 4 * (p & 3);
        *lds_cast<f32x4>(dst + (p - r * kRoundPieces) * 1024) = f32x4{acc[i][e], acc[i][e + 1], acc[i][e + 2], acc[i][e + 3]};
      }
  }
  // Group `from`'s values of piece p of a round.
  __device__ static __forceinline__ f32x4 read(int p, int from, const char* lds, int wave, int lane) {
    return *lds_cast<const f32x4>(lds + ((from * kWaves + wave) * kRoundPieces + p) * 1024 + lane * 16);
  }
  __device__ static __forceinline__ char* stats(char* lds, int group, int wave, int lane) {
    return lds + S * kWaves * kRoundPieces * 1024 + (group * kWaves + wave) * 512 + lane * 4;
  }
  // Plain sums; store(p, sum) gets the pieces of this wave, p = 4 * tile + quarter.
  template <class Store>
  __device__ static __forceinline__ void add(const f32x16 (&acc)[kTiles], char* lds, int group, int wave, int lane, Store&& store) {
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      __syncthreads();
      write(acc, r, lds, group, wave, lane);
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kOwned; ++i) {
        const int p = group * kOwned + i;
        if (kRoundPieces % S != 0 && p >= kRoundPieces) break;
        f32x4 sum = read(p, 0, lds, wave, lane);
#pragma unroll
        for (int from = 1; from < S; ++from) sum += read(p, from, lds, wave, lane);
        store(r * kRoundPieces + p, sum);
      }
    }
  }
  // Online-softmax partials (running maximum m, this lane's share l of the row sum, O), c = softmax scale * log2 e:
  // returns the row's maximum and sum in m and l; store(p, normalised values).
  template <class Store>
  __device__ static __forceinline__ void softmax(const f32x16 (&acc)[kTiles], float& m, float& l, float c, char* lds, int group, int wave,
                                                 int lane, Store&& store) {
    float weight[S];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      __syncthreads();  // the last stages are consumed, or the last round is read
      write(acc, r, lds, group, wave, lane);
      if (r == 0) {
        *lds_cast<float>(stats(lds, group, wave, lane)) = m;
        *lds_cast<float>(stats(lds, group, wave, lane) + 256) = l;
      }
      __syncthreads();
      if (r == 0) {
        float ms[S];
#pragma unroll
        for (int from = 0; from < S; ++from) ms[from] = *lds_cast<const float>(stats(lds, from, wave, lane));
        m = ms[0];
#pragma unroll
        for (int from = 1; from < S; ++from) m = fmaxf(m, ms[from]);
        l = 0.f;
#pragma unroll
        for (int from = 0; from < S; ++from) {
          // a group without a visible key has m = -inf, l = 0, O = 0
          weight[from] = m > ms[from] ? __builtin_amdgcn_exp2f((ms[from] - m) * c) : 1.f;
          l += *lds_cast<const float>(stats(lds, from, wave, lane) + 256) * weight[from];
        }
        l += __shfl_xor(l, 32);
        const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
        for (int from = 0; from < S; ++from) weight[from] *= inv;
      }
#pragma unroll
      for (int i = 0; i < kOwned; ++i) {
        const int p = group * kOwned + i;
        if (kRoundPieces % S != 0 && p >= kRoundPieces) break;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int from = 0; from < S; ++from) {
          const f32x4 v = read(p, from, lds, wave, lane);
#pragma unroll
          for (int x = 0; x < 4; ++x) sum[x] = __builtin_fmaf(v[x], weight[from], sum[x]);
        }
        store(r * kRoundPieces + p, sum);
      }
    }
  }
};

// Work item `id`, a workgroup id where every workgroup takes one; false: none.  Consecutive workgroup ids go to different XCDs.
// By slices: the blocks are cut into 8 slices of equal list weight; for head bh, XCD x takes slice
// (x + bh) mod 8 and the XCDs move from head to head together, so all of them work on the same head
// at the same time (its K/V stay in the shared last-level cache), neighbouring workgroups of an XCD
// share K/V tiles in that XCD's L2, and every XCD gets every slice equally often (slices of equal
// weight do not take exactly equal time).
__host__ __device__ __forceinline__ bool work_item(const WorkMap& w, uint32_t id, int32_t& bh, int32_t& block) {
  const uint32_t n_sliced = 8u * (uint32_t)w.sliced * (uint32_t)w.max_slice;
  if (id >= n_sliced) {
    // By falling list length.  A window of 8 ranks of every head goes to the 8 XCDs at once; inside it an
    // XCD takes neighbouring (head, rank) pairs, head by head, so that it stays with the same
    // heads / 8 heads from window to window (their K/V are what its L2 sees).
    const uint32_t idx = id - n_sliced, heads = (uint32_t)w.ordered;
    const uint32_t window = idx / (8u * heads), j = idx - window * 8u * heads;
    uint32_t head, rank;
    if (8u * window + 8u <= (uint32_t)w.n_blocks) {
      const uint32_t pair = (j & 7u) * heads + (j >> 3);
      head = pair >> 3;
      rank = 8u * window + (pair & 7u);
    } else {  // the last n_blocks % 8 ranks
      rank = j / heads;
      head = j - rank * heads;
      rank += 8u * window;
    }
    bh = w.sliced + (int32_t)head;
    block = w.order[rank];
    return true;
  }
  const uint32_t idx = id >> 3;
  bh = (int32_t)(idx / (uint32_t)w.max_slice);
  const int32_t pos = (int32_t)(idx - (uint32_t)bh * (uint32_t)w.max_slice);
  const int32_t sl = ((int32_t)(id & 7) + bh) & 7;
  const int32_t s0 = w.slice[sl];
  block = s0 + pos;
  return pos < w.slice[sl + 1] - s0;
}

// Where the last `halved` items of a launch are taken in two halves: item and half of workgroup `id`.  Both halves of an item
// are on one XCD (8 workgroups apart) while 8 items are left.
__device__ __forceinline__ uint32_t halved_item(uint32_t id, uint32_t first, uint32_t halved, int32_t& part) {
  const uint32_t j = id - first, by8 = halved >> 3;
  if (j < 16u * by8) {
    part = (int32_t)(j >> 3) & 1;
    return first + (j >> 4) * 8u + (j & 7u);
  }
  const uint32_t rest = halved & 7u, k = j - 16u * by8;
  part = k >= rest ? 1 : 0;
  return first + 8u * by8 + (k >= rest ? k - rest : k);
}

// What workgroup `id` of a launch over pairs of query blocks takes (see TwoMap): both blocks of a pair, block `block` of it, or half of that.
struct TwoItem {
  enum Form { kPair, kBlock, kHalf } form;
  int32_t bh, pair, block, half;
  int64_t record;  // of a trace: of the block, or of a pair's first, whose second has the one 8 further; its index and the workgroup's are the same modulo 8, but for the
                   // last pairs in halves where their number is no multiple of 8
};

// Workgroup `id` of those that share `count` items, 1 << kLog of them each: item and part.  All parts of an item are on one XCD while 8
// items are left.
template <int kLog>
__host__ __device__ __forceinline__ uint32_t split_item(uint32_t id, uint32_t count, int32_t& part) {
  const uint32_t whole = count & ~7u;
  if (id < whole << kLog) {
    part = (int32_t)(id >> 3) & ((1 << kLog) - 1);
    return (id >> (3 + kLog)) * 8u + (id & 7u);
  }
  const uint32_t rest = count - whole, k = id - (whole << kLog);
  part = (int32_t)(k / rest);
  return whole + k % rest;
}

__host__ __device__ __forceinline__ bool two_item(const WorkMap& w, const TwoMap& m, uint32_t id, TwoItem& item) {
  item.form = TwoItem::kPair;
  item.block = item.half = 0;
  item.record = 16 * (int64_t)(id >> 3) + (id & 7u);
  uint32_t pair_id = id;
  if (id >= m.n_two) {
    const uint32_t single = id - m.n_two;
    int32_t part;
    uint32_t k;
    if (single < 2u * m.n_one) {
      item.form = TwoItem::kBlock;
      k = split_item<1>(single, m.n_one, part);
      item.block = part;
      item.record = 2 * (int64_t)m.n_two + single;
    } else {
      item.form = TwoItem::kHalf;
      k = m.n_one + split_item<2>(single - 2u * m.n_one, m.n_half, part);
      item.block = part >> 1;
      item.half = part & 1;
      const uint32_t at = k - m.n_one, eights = at & ~7u;
      item.record = 2 * (int64_t)(m.n_two + m.n_one + eights) + (uint32_t)item.block * (m.n_half - eights < 8u ? m.n_half - eights : 8u) + (at & 7u);
    }
    pair_id = m.n_two + k;
  }
  if (pair_id >= m.n_sliced) {
    if (!work_item(m.pairs, pair_id - m.n_sliced, item.bh, item.pair)) return false;
    item.bh += w.sliced;
  } else {
    // As in work_item, XCD x takes the pairs that start in slice (x + bh) mod 8 of head bh, but one head after the other without gaps: a head
    // whose slices differ in length would leave workgroups without work among the others (heads of 8 blocks: 1.39 of the time).  Over 8 heads
    // every XCD has each slice once.
    const uint32_t xcd = id & 7u, per_head = (uint32_t)m.pairs.n_blocks, eight = (id >> 3) / per_head;
    int32_t left = (int32_t)((id >> 3) - eight * per_head), first = 0;
    item.bh = (int32_t)(8u * eight);
    for (int t = 0;; ++t, ++item.bh) {
      if (t == 8 || item.bh >= w.sliced) return false;
      const int32_t sl = (int32_t)(xcd + t) & 7;
      first = (w.slice[sl] + 1) / 2;
      const int32_t n = (w.slice[sl + 1] + 1) / 2 - first;
      if (left < n) break;
      left -= n;
    }
    item.pair = first + left;
  }
  return 2 * item.pair + item.block < w.n_blocks;
}

// ---- token-level rule of the radial mask inside listed blocks ---------------------------------
// (Sec. 4.2 of the paper, formal definition, plus the attention sink of App. A.1.)

// For one (query frame i, key frame j) pair: the largest |k - l| a query position k may
// attend; -1 = nothing, >= s - 1 = the whole frame.
__host__ __device__ __forceinline__ int32_t radial_half_width(const TokenRule& rule, int32_t i, int32_t j) {
  if (j < rule.sink || i >= rule.frames || j >= rule.frames) return rule.s;  // sink, text tokens
  const int32_t d = i > j ? i - j : j - i;
  if (rule.half_width) return rule.half_width[d];  // banded pattern: table lookup (d <= frames)
  if (d < 2) return rule.s - 1;            // band 0: the whole frame, never scaled
  const int32_t r = 31 - __builtin_clz(d);       // floor(log2 d)
  const int32_t w = rule.w0 >> r;          // diagonal width floor(c*s / 2^r)
  if (w >= 1) return (w < rule.s ? w : rule.s) - 1;
  const int64_t b_den = (int64_t)rule.den << r;
  const int32_t stride = (int32_t)((b_den + rule.s_num - 1) / rule.s_num);
  return d % stride == 0 ? 0 : -1;         // sub-sampled single diagonals
}

// A stage is 64 (or 32) consecutive tokens (keys for the query-stationary kernels, queries for the
// key-stationary one) that start at (frame, pos).  With s >= 64 it touches at most the two
// frames `frame` and `frame + 1`.
struct StagePos {
  int32_t frame, pos;
};

// (frame, position) of token index `block_start` for every lane's list entry.
__host__ __device__ __forceinline__ StagePos block_pos(int32_t block_start, int32_t s) {
  StagePos r;
  r.frame = block_start / s;
  r.pos = block_start - r.frame * s;
  return r;
}

// The position `offset` tokens further on, 0 <= offset <= kMaxOffset (the last stage's place in a block).
// pos < s and s >= 64: up to 64 tokens cross at most one frame boundary, up to 128 at most two.
template <int kMaxOffset>
__host__ __device__ __forceinline__ StagePos advance(StagePos at, int32_t offset, int32_t s) {
  static_assert(kMaxOffset <= 128, "more tokens than two frames");
  at.pos += offset;
#pragma unroll
  for (int crossed = 0; crossed < (kMaxOffset > 64 ? 2 : 1); ++crossed)
    if (at.pos >= s) {
      at.pos -= s;
      at.frame += 1;
    }
  return at;
}

// The first `count` tokens of a stage (count >= 64: all of them): those that exist before N.
__device__ __forceinline__ uint64_t stage_prefix(int32_t count) {
  return count >= 64 ? ~0ull : (count <= 0 ? 0ull : ((1ull << count) - 1ull));
}

// An MFMA accumulator pair (two 32-token tiles of a stage) holds, in lane group g = lane/32,
// element e of tile kt for stage token 32kt + 8(e/4) + 4g + e%4.  From a mask over the 64 stage
// tokens this returns the lane's 32 bits in element order (bit 16kt + e): nibble g of every
// byte of the mask, packed.
__device__ __forceinline__ uint32_t lane_element_bits(uint64_t token_mask, int g) {
  uint64_t v = (token_mask >> (4 * g)) & 0x0F0F0F0F0F0F0F0Full;
  v = (v | (v >> 4)) & 0x00FF00FF00FF00FFull;
  v = (v | (v >> 8)) & 0x0000FFFF0000FFFFull;
  v = (v | (v >> 16));
  return (uint32_t)v;
}

// The same bits for the tokens from x + 4g on (all of them up to x = 0, none from 64 on), with fewer instructions.  Not for the end of the
// sequence where listed blocks are dense: the compiler takes the parts of it that do not change out of that rare branch, 4 to 10 registers
// of every stage (D 64, block 64, 64 items L 28: 10.60 / 10.69 us).
__host__ __device__ __forceinline__ uint32_t elements_from(int32_t x) {
  x = max(min(x, 64), -4);
  return (uint32_t)(~0ull << (4 * (x >> 3) + min(x & 7, 4)));
}

// The elements of a stage that starts at position pos of a frame which a token at position own of its frame does not see, in lane group g: hw0 and hw1
// are the half widths of the pairs (own frame, stage's first frame) and (own frame, the next).  Of the first frame it sees the positions pos + x, x
// in [0, min(split, kWidth)), within hw0 of its own, of the second x - split, x in [split, kWidth), within hw1.  The bounds straight as elements: by
// way of the two intervals the forward of 30 heads x 24 x 316 tokens takes 533 us instead of 526, 1 x 108 x 1010 backward 4333 instead of 4209.
// kWidth: tokens in the stage (64, or 32 for the kernels that walk half-size stages).
template <int kWidth>
__host__ __device__ __forceinline__ uint32_t hidden_elements(int32_t own, int32_t pos, int32_t hw0, int32_t hw1, int32_t s, int g) {
  const int32_t split = s - pos, own_g = own - 4 * g;
  uint32_t seen = elements_from(own_g - hw0 - pos) & ~elements_from(min(own_g + hw0 - pos + 1, min(split, kWidth) - 4 * g));
  if (split < kWidth) seen |= elements_from(max(own_g - hw1, -4 * g) + split) & ~elements_from(min(own_g + hw1 + split + 1, kWidth - 4 * g));
  return ~seen;
}

// own_is_query: the lane holds a query and the stage holds keys; otherwise the reverse.
__host__ __device__ __forceinline__ int32_t pair_half_width(const TokenRule& rule, int32_t own, int32_t other, bool own_is_query) {
  return own_is_query ? radial_half_width(rule, own, other) : radial_half_width(rule, other, own);
}

// What a wave's 32 consecutive tokens cover: positions lo .. hi of a frame and, with s >= 64, at most 0 .. hi2 of the next (hi2 < 0: none).
struct WaveSpan {
  int32_t frame, lo, hi, hi2;
};
// The 32 tokens from `first` on; those past N - 1 stand for token N - 1, as in the lanes.
__host__ __device__ __forceinline__ WaveSpan wave_span(int32_t first, int32_t N, int32_t s) {
  const StagePos at = block_pos(first < N ? first : N - 1, s);
  const int32_t last = at.pos + (first + 31 < N ? 31 : first < N ? N - 1 - first : 0);
  return WaveSpan{at.frame, at.pos, last < s ? last : s - 1, last - s};
}

// The rule between a span and one stage of kWidth tokens: whether all tokens of the span see all of the stage, whether none sees any, and the
// half widths of the pairs of frames, [of the span][of the stage].
struct SpanRule {
  bool all, none;
  int32_t hw[2][2];
};
template <int kWidth>
__host__ __device__ __forceinline__ SpanRule span_rule(const TokenRule& rule, const WaveSpan& span, StagePos stage, bool own_is_query) {
  SpanRule r = {true, true, {{0, 0}, {0, 0}}};
  const int32_t end = stage.pos + kWidth - 1;  // last token of the stage, as a position of its first frame
#pragma unroll 1  // one copy of the half width's arithmetic
  for (int k = 0; k < 4; ++k) {
    const int i = k >> 1, j = k & 1;
    const int32_t lo = i ? 0 : span.lo, hi = i ? span.hi2 : span.hi;
    const int32_t from = j ? 0 : stage.pos, to = j ? end - rule.s : min(end, rule.s - 1);
    const int32_t hw = pair_half_width(rule, span.frame + i, stage.frame + j, own_is_query);
    if (hi >= lo && to >= from) {
      r.all = r.all && hi - from <= hw && to - lo <= hw;
      r.none = r.none && (hw < 0 || lo - to > hw || from - hi > hw);
    }
    if (k == 0) r.hw[0][0] = hw;
    if (k == 1) r.hw[0][1] = hw;
    if (k == 2) r.hw[1][0] = hw;
    if (k == 3) r.hw[1][1] = hw;
  }
  return r;
}

// The token rule in a wave that walks a list.  Lane l looks at every 64th stage, l of each 64, so that a stage which the wave sees wholly or not at
// all costs a bit test, and one that it sees in part some thirty vector instructions for the mask of its elements.  Left to itself
// at every stage a lane needs two half widths, 64-bit masks and a change of order, 180 instructions, 100 of them in every stage, beside the 170 of
// the forward's softmax; at 21 x 1560 tokens 72 % of a wave's stages are seen wholly, 15 % in part, and 30 % of a workgroup's in part by some wave.
// Each lane for itself in every stage / so, us: forward, D 128, block 128, 5 heads x 21 x 1560 tokens 1830 / 1661, 3 x 33 x 3600 10107 / 9297, block 64, 4 x 21 x
// 1183 946 / 826, D 64, block 64, 30 x 24 x 316 601 / 525; backward (a common launch's with arguments shared by its parts) 5727 / 5509, 8 x 30 x 900 6113 / 5586, D 64 1 x 108 x 1010 4725 / 4209, block 64,
// 4 x 16 x 400 169 / 163.  The price is scalars (masks, span, the half widths' arithmetic): the forward's kernels hold 3 to 33 in vector lanes, those with
// halves 69 to 90, where they held 0 to 20 and 26 to 35.
template <int kWidth, int kBlock>
struct ListRule {
  static constexpr int kSubs = kBlock / kWidth;
  WaveSpan span;
  int32_t own;       // position of this lane's token in its frame
  uint64_t seconds;  // lanes whose token is in the span's second frame
  uint64_t all, none;  // stages of the 64 around the current one
  int32_t pos, hw[2][2];  // of this lane's stage of them: position in its first frame, half widths

  // first, N: as for wave_span.
  __device__ __forceinline__ void init(const TokenRule& rule, int32_t first, int32_t N, int lane) {
    span = wave_span(first, N, rule.s);
    const int32_t token = first + (lane & 31);
    const StagePos at = block_pos(token < N ? token : N - 1, rule.s);
    own = at.pos;
    seconds = __builtin_amdgcn_ballot_w64(at.frame != span.frame);
  }
  // The 64 stages from the first one of entry `entry` of the chunk of 64 list entries on; vec: this lane's entry of the chunk.
  __device__ __forceinline__ void look(const TokenRule& rule, int32_t vec, int32_t entry, int lane, bool own_is_query) {
    const int32_t block = __shfl(vec, entry + lane / kSubs);
    const StagePos stage = advance<kBlock - kWidth>(block_pos(block * kBlock, rule.s), lane % kSubs * kWidth, rule.s);
    const SpanRule r = span_rule<kWidth>(rule, span, stage, own_is_query);
    all = __builtin_amdgcn_ballot_w64(r.all);
    none = __builtin_amdgcn_ballot_w64(r.none);
    pos = stage.pos;
#pragma unroll
    for (int k = 0; k < 4; ++k) hw[k >> 1][k & 1] = r.hw[k >> 1][k & 1];
  }
  __device__ __forceinline__ bool sees_all(int32_t u) const { return all >> (u & 63) & 1; }
  __device__ __forceinline__ bool sees_none(int32_t u) const { return none >> (u & 63) & 1; }
  // The elements of stage u that this lane's token does not see.
  __device__ __forceinline__ uint32_t hidden(int32_t u, int32_t s, int g, int lane) const {
    const int32_t at = __builtin_amdgcn_readlane(pos, u & 63);
    int32_t hw0 = __builtin_amdgcn_readlane(hw[0][0], u & 63), hw1 = __builtin_amdgcn_readlane(hw[0][1], u & 63);
    if (span.hi2 >= 0) {
      const bool second = seconds >> lane & 1;
      const int32_t b0 = __builtin_amdgcn_readlane(hw[1][0], u & 63), b1 = __builtin_amdgcn_readlane(hw[1][1], u & 63);
      hw0 = second ? b0 : hw0;
      hw1 = second ? b1 : hw1;
    }
    return hidden_elements<kWidth>(own, at, hw0, hw1, s, g);
  }
};

}  // namespace radial

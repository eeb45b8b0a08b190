// The forward of radial_attn_fwd_kernel.h and that of radial_attn_fwd_fp8.hip (8-bit scores) for two neighbouring query blocks at a time: head
// dimension 128, blocks of 128, listed blocks dense, launches that fill the chip several times over.
//
// One workgroup of four waves takes the query blocks 2p and 2p + 1, and wave w of it owns 32 rows of either, so that a key block which both
// lists name is copied into LDS once for 256 query rows and every K and V fragment read from LDS feeds two MFMAs.  These kernels run at the
// chip's power cap, and both are energy that is no arithmetic, and cycles: with the copies and the LDS reads halved the clock rises and fewer cycles are
// needed, by much the same share.  24 heads x 118 800 tokens, one block / two in turn on one box, by the counters: radial lists 74.2 / 65.8 ms, 1.64 / 1.75 GHz, the
// matrix pipes 61.5 / 65.1 % busy; all-ones list 152.8 / 135.7 ms, 1.69 / 1.81 GHz, 64.0 / 67.4 %.  Two workgroups share a compute unit, the two waves of
// a SIMD belong to different ones and so drift into each other's gaps: as one workgroup of eight waves of 32 rows, tied by its barrier, the same
// sharing gained nothing, and so did 64 rows of one block per wave in workgroups of two waves (half the LDS reads, the same copies: 0.99).
//
// The union of two neighbouring lists is 5 to 20 % longer than either.  The softmax does not mind the order, so a pair is walked in three
// passes, the entries of both lists, then those of the first alone and those of the second alone: three loops of their own, of which the
// last two are one piece of code (the second set of rows moves into the registers of the first).  With one loop that branches at every
// entry the compiler moves accumulators between the branches and spills 800 bytes a lane.  A pass over one list alone works like the
// kernel for single blocks; lists that have little in common gain nothing, and short ones lose (takes_pairs in radial_internal.h).
//
// Registers are what limits it: 128 of O, 64 of Q, 32 of scores, 12 of fragments in flight, and 20 for all the rest.  So
// - K and V lie in LDS four rows at a time, rows in turn every 64 bytes, with 16 bytes between one four and the next: both kinds of reads are free of
//   bank conflicts, as with the swizzle, but all pieces of a tile are at constant distances from one address per lane (the conflicts that the counters show, 0.2 % of the LDS
//   instructions, are the bitmaps' atomics, up to 32 lanes to a word: four times as many on an all-ones list);
// - values of rare use (the lane's number, addresses of a ragged stage, the store) are worked out again where they are needed;
// - strides and pointers that only the store needs are loaded again there, and the three forms of the kernel load their arguments each for itself;
// - sums and packed P are pinned where they are written, or the compiler keeps the 32 values of P until it needs their sum.
// Forward, us, single blocks / this: 24 heads x 118 800 tokens 77.0 / 68.7 ms, x 464 400 618 / 551, 40 x 32 760 13.38 / 12.35, all-ones list 19.9 /
// 18.0, 12 x 64 500 16.0 / 15.0, 400 x 1536 613 / 535, 600 x 1152 643 / 480.
#pragma once

#include "radial_attn_fwd_kernel.h"

namespace radial {
namespace fwd {

template <bool kFp8>
struct TwoTile {
  static constexpr int kD = 128, kBlk = 128, kStageKeys = 64, kWaves = 4;
  static constexpr int kFourRows = 1024 + 16;  // bytes of four rows and the gap behind them
  static constexpr int kVBytes = kStageKeys / 4 * kFourRows, kKBytes = kFp8 ? kStageKeys * kD : kVBytes, kStageBytes = kKBytes + kVBytes;
  static constexpr int kVLoads = kStageKeys / 4 / kWaves, kKLoads = kFp8 ? kKBytes / 1024 / kWaves : kVLoads;  // copies per wave and tile
  static constexpr int kSteps = kFp8 ? kD / 64 : kD / 16, kDTiles = kD / 32;
  static constexpr int kNamedAt = 2 * kStageBytes, kNamedWords = kMaxOrdered / 32;  // which blocks either list names, a bit each
  static constexpr int kLdsBytes = kNamedAt + 2 * kNamedWords * 4;
  static_assert(2 * kLdsBytes <= 160 * 1024, "two workgroups per compute unit");
};

// Query blocks qb and qb + 1 (which may not exist).
template <bool kTrace, class Args>
__device__ __forceinline__ void two_body(const Args& a, int32_t bh, int32_t qb, float c, int64_t record, char* lds_all) {
  constexpr bool kFp8 = std::is_same_v<Args, Fp8FwdArgs>;
  using T = TwoTile<kFp8>;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 31, g = lane >> 5;
  uint64_t t_begin = kTrace ? __builtin_amdgcn_s_memrealtime() : 0;
  int32_t heads = a.H;
  if constexpr (!kFp8) asm("" : "+s"(heads) : "s"(a.q.ptr), "s"(a.k.ptr), "s"(a.row_ptr));
  const int32_t b = bh / heads, h = bh % heads;
  // rows of Q and K: bf16, or contiguous 8-bit codes
  const char *qp, *kp;
  int64_t q_row_bytes = T::kD, k_row_bytes = T::kD;
  if constexpr (kFp8) {
    qp = (const char*)a.q8 + (int64_t)bh * a.N * T::kD;
    kp = (const char*)a.k8 + (int64_t)bh * a.N * T::kD;
  } else {
    qp = (const char*)((const __bf16*)a.q.ptr + (int64_t)b * a.q.sb + (int64_t)h * a.q.sh);
    kp = (const char*)((const __bf16*)a.k.ptr + (int64_t)b * a.k.sb + (int64_t)h * a.k.sh);
    q_row_bytes = 2 * a.q.sn;
    k_row_bytes = 2 * a.k.sn;
  }
  const __bf16* vp = (const __bf16*)a.v.ptr + (int64_t)b * a.v.sb + (int64_t)h * a.v.sh;

  const int32_t lo0 = __builtin_amdgcn_readfirstlane(a.row_ptr[qb]), lo1 = __builtin_amdgcn_readfirstlane(a.row_ptr[qb + 1]);
  const int32_t hi1 = qb + 2 <= a.n_blocks ? __builtin_amdgcn_readfirstlane(a.row_ptr[qb + 2]) : lo1;
  const auto named = lds_cast<uint32_t>(lds_all + T::kNamedAt);  // by the first list, by the second
  {
    const int32_t words = (a.n_blocks + 31) >> 5;
    for (int32_t i = threadIdx.x; i < words; i += 256) named[i] = named[T::kNamedWords + i] = 0u;
    __syncthreads();
    for (int32_t i = threadIdx.x; i < hi1 - lo0; i += 256) {
      const int32_t e = a.col_idx[lo0 + i];
      __hip_atomic_fetch_or(&named[(i < lo1 - lo0 ? 0 : T::kNamedWords) + (e >> 5)], 1u << (e & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
  }
  // A walk over the entries of list `w` that the other list names too (shared) or does not.
  int32_t entry = 0;       // this lane's of 64
  float entry_scale = 1.f, q_scale[2] = {1.f, 1.f}, factor[2] = {1.f, 1.f}, factor_next[2] = {1.f, 1.f};  // 8-bit scores: of the entry, of the rows, both
  uint64_t left = 0;       // which of them are to be visited
  int32_t chunk = 0, w = 0;
  bool shared = true;
  auto take = [&]() __attribute__((always_inline)) -> int32_t {  // the next block, -1: none
    const int32_t list = w ? lo1 : lo0, size = w ? hi1 - lo1 : lo1 - lo0;
    while (left == 0) {
      if (chunk >= size) return -1;
      const int i = chunk + lane_again();
      entry = i < size ? a.col_idx[list + i] : 0;
      if constexpr (kFp8) entry_scale = a.k_scale[(int64_t)bh * a.n_blocks + entry];
      const bool in = named[(w ^ 1) * T::kNamedWords + (entry >> 5)] >> (entry & 31) & 1u;
      left = __builtin_amdgcn_ballot_w64(i < size && in == shared);
      chunk += 64;
    }
    const int i = __builtin_ctzll(left);
    left &= left - 1;
    if constexpr (kFp8) {
      const float k_scale = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, entry_scale), i));
#pragma unroll
      for (int set = 0; set < 2; ++set) factor_next[set] = q_scale[set] * k_scale;
    }
    return __builtin_amdgcn_readlane(entry, i);
  };

  // B operands of the first product: 16 bytes of each of this lane's rows for every k-step of 16, or 32 bytes of codes for every one of 64
  using Frag = std::conditional_t<kFp8, i32x8, bf16x8>;
  const int32_t q_first = qb * T::kBlk + wave * 32 + lq;
  Frag qf[2][T::kSteps];
#pragma unroll
  for (int set = 0; set < 2; ++set) {
    const int32_t q_row = q_first + T::kBlk * set;
    const bool q_ok = q_row < a.N;
    const char* src = qp + (int64_t)(q_ok ? q_row : a.N - 1) * q_row_bytes + sizeof(Frag) * g;
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) {
      u32x4 raw[sizeof(Frag) / 16];  // rows start at multiples of 16 bytes
#pragma unroll
      for (int i = 0; i < (int)sizeof(Frag) / 16; ++i) {
        raw[i] = *(const u32x4*)(src + 2 * sizeof(Frag) * t + 16 * i);
        if (!q_ok) raw[i] = u32x4{0u, 0u, 0u, 0u};
      }
      qf[set][t] = __builtin_bit_cast(Frag, raw);
    }
    if constexpr (kFp8) q_scale[set] = a.q_scale[(int64_t)bh * a.n_blocks + (qb + set < a.n_blocks ? qb + set : qb)];
  }

  // A copy takes four rows: lanes 4j .. 4j + 3 of every 16 fetch 64 bytes of row j, so that the rows lie in turn every 64 bytes.
  const uint32_t voff = (uint32_t)((lane >> 2 & 3) * (int32_t)a.v.sn) * 2u + (lane >> 4) * 64 + (lane & 3) * 16;
  uint32_t koff[kFp8 ? T::kKLoads : 1];
  if constexpr (kFp8) {  // 8 rows of codes, swizzled
#pragma unroll
    for (int i = 0; i < T::kKLoads; ++i) {
      int r, piece;
      k8_source_of((wave * T::kKLoads + i) * 64 + lane, r, piece);
      koff[i] = (uint32_t)(r * T::kD + piece * 16);
    }
  } else {
    koff[0] = (uint32_t)((lane >> 2 & 3) * (int32_t)k_row_bytes) + (lane >> 4) * 64 + (lane & 3) * 16;
  }
  const uint32_t lds0 = lds_address(lds_all);
  const int i16 = lane & 15, half16 = (lane >> 4) & 1;
  // K row lq, piece g (codes: the pieces of both k-steps), and the V rows and columns of a transposing read; the first stage goes to the
  // other buffer.
  uint32_t rows_at[kFp8 ? 4 : 1];
  if constexpr (kFp8) {
#pragma unroll
    for (int i = 0; i < 4; ++i) rows_at[i] = lds0 + T::kStageBytes + k8_piece(lq, i / 2 * 4 + 2 * g + i % 2);
  } else {
    rows_at[0] = lds0 + T::kStageBytes + (lq >> 2) * T::kFourRows + (lq & 3) * 64 + g * 16;
  }
  uint32_t cols_at = lds0 + T::kStageBytes + T::kKBytes + g * T::kFourRows + (i16 >> 2) * 64 + half16 * 32 + (i16 & 3) * 8;
  uint32_t copy_at = lds0;  // where the copies of the next stage go, and this wave's of them
  const uint32_t kcopies = wave * T::kKLoads * (kFp8 ? 1024 : T::kFourRows), vcopies = T::kKBytes + wave * T::kVLoads * T::kFourRows;
  uint32_t kcopy = 0, vcopy = 0;
  constexpr int kKStep = kFp8 ? 1024 : T::kFourRows;  // LDS bytes from one copy of K to the next

  // All of this wave's copies of a stage at once (first stage, ragged stages: rows past N-1 are clamped to N-1).
  auto issue_stage = [&](int32_t key0) __attribute__((always_inline)) {
    const int32_t last = a.N - 1 - key0;
    const int lane = lane_again();
#pragma unroll 1
    for (int i = 0; i < T::kVLoads; ++i) {
      int32_t r = (wave * T::kVLoads + i) * 4 + (lane >> 2 & 3);
      r = r < last ? r : last;
      const int col = (lane >> 4) * 32 + (lane & 3) * 8;
      if constexpr (!kFp8) copy16_to_lds(kp + ((int64_t)key0 + r) * k_row_bytes + 2 * col, kcopy + i * T::kFourRows);
      copy16_to_lds(vp + ((int64_t)key0 + r) * a.v.sn + col, vcopy + i * T::kFourRows);
    }
    if constexpr (kFp8) {
#pragma unroll 1
      for (int i = 0; i < T::kKLoads; ++i) {
        int r, piece;
        k8_source_of((wave * T::kKLoads + i) * 64 + lane, r, piece);
        r = r < last ? r : last;
        copy16_to_lds(kp + ((int64_t)key0 + r) * k_row_bytes + piece * 16, kcopy + i * kKStep);
      }
    }
  };

  f32x16 o[2][T::kDTiles];
#pragma unroll
  for (int set = 0; set < 2; ++set)
#pragma unroll
    for (int i = 0; i < T::kDTiles; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[set][i][e] = 0.f;
  float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f}, mc[2] = {0.f, 0.f};  // mc: maximum times c, 0 while there is none
  constexpr int kAhead = 2;  // LDS fragments are read this many MFMAs (of one set) before their use; the fences keep the written order
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  const char *kbase = kp, *vbase = (const char*)vp;  // this wave's first rows of the next stage
  uint64_t copy_lanes = 0;
  const int64_t kstep = 4 * k_row_bytes, vstep = 8 * a.v.sn;  // bytes of four rows
  constexpr int kCopies = T::kKLoads + T::kVLoads;
  auto spread_copy = [&](int j) __attribute__((always_inline)) {
    // K and V in turn; codes first
    const bool of_v = kFp8 ? j >= T::kKLoads : j % 2 == 1;
    const int i = kFp8 ? (of_v ? j - T::kKLoads : j) : j / 2;
    if (of_v) {
      copy16_to_lds_sv_masked(vbase, voff, vcopy + i * T::kFourRows, copy_lanes);
      vbase += vstep;
      asm("" : "+s"(vbase));  // or the compiler holds all multiples of the step
    } else {
      copy16_to_lds_sv_masked(kbase, koff[kFp8 ? i : 0], kcopy + i * kKStep, copy_lanes);
      if (!kFp8) kbase += kstep;
      if (!kFp8) asm("" : "+s"(kbase));
    }
  };
  auto read_k = [&](int kt, int t) __attribute__((always_inline)) -> Frag {
    if constexpr (kFp8) {
      const u32x4 x = *lds_pointer<const u32x4>(rows_at[2 * t] + kt * 32 * T::kD), y = *lds_pointer<const u32x4>(rows_at[2 * t + 1] + kt * 32 * T::kD);
      return Frag{(int)x[0], (int)x[1], (int)x[2], (int)x[3], (int)y[0], (int)y[1], (int)y[2], (int)y[3]};
    } else {
      return *lds_pointer<const bf16x8>(rows_at[0] + (kt * 8 * T::kFourRows + t / 2 * 256 + t % 2 * 32));
    }
  };
  auto score = [&](Frag k, Frag q, f32x16 s) __attribute__((always_inline)) -> f32x16 {
    // codes: formats 0 / 0 = E4M3 for both operands; scale exponents 127 = 2^0
    if constexpr (kFp8) return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(k, q, s, 0, 0, 0, 0x7F7F7F7F, 0, 0x7F7F7F7F);
    else return mfma32(k, q, s);
  };
  auto read_v = [&](int kt, int j) __attribute__((always_inline)) {  // j = 4 * 16-key step + d tile
    const uint32_t at = cols_at + (j % 4 * 256 + (kt * 8 + j / 4 * 4) * T::kFourRows);
    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_pointer<s16x4>(at));
    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_pointer<s16x4>(at + 2 * T::kFourRows));
    const u32x2 a0 = __builtin_bit_cast(u32x2, v0), a1 = __builtin_bit_cast(u32x2, v1);
    return as_bf16x8(a0[0], a0[1], a1[0], a1[1]);
  };
  // The running maximum of set `set` with the scores of some tiles.
  auto raise = [&](int set, const auto& tiles) __attribute__((always_inline)) {
    float mx = kFp8 ? tiles[0][0] : m_run[set];
#pragma unroll
    for (const f32x16& s : tiles)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[e]);
    mx = max_with_other_half(mx);
    if constexpr (kFp8) mx = fmaxf(m_run[set], mx * factor[set]);  // the scales are positive: they commute with the maximum
    if (__builtin_amdgcn_ballot_w64(mx > m_run[set]) != 0) {
      const float alpha = mx > m_run[set] ? __builtin_amdgcn_exp2f((m_run[set] - mx) * c) : 1.f;
      l_run[set] *= alpha;
#pragma unroll
      for (int i = 0; i < T::kDTiles; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[set][i][e] *= alpha;
      m_run[set] = mx;
      mc[set] = mx > -INFINITY ? mx * c : 0.f;  // a row may still have no score above -inf when another row of the wave has
    }
  };
  // Scores of keys past N - 1: `exist` of a tile's 32 do.
  auto hide = [&](f32x16& s, int32_t exist) __attribute__((always_inline)) {
    const uint32_t hidden = elements_from(exist - 4 * (lane_again() >> 5));
    float lowest;  // not a register of the whole kernel
    asm volatile("v_mov_b32 %0, 0xff800000" : "=v"(lowest));
#pragma unroll
    for (int e = 0; e < 16; ++e)
      if ((hidden >> e) & 1u) s[e] = lowest;
  };
  // Element pairs 2 * pair, 2 * pair + 1 of tile s: P as bf16, its sum.
  auto softmax_pair = [&](const f32x16& s, int pair, float multiplier, float maximum, uint32_t& packed, float& sum) __attribute__((always_inline)) {
    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * pair], multiplier, -maximum));
    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * pair + 1], multiplier, -maximum));
    sum += p0 + p1;
    packed = pack_bf16(p0, p1);
    asm volatile("" : "+v"(packed), "+v"(sum));
  };

  // Half kt of a stage, 32 keys, for both sets of rows.  The first 16 keys' P are ready before the second product begins, the others follow
  // between its MFMAs (all of them before it: 1 % slower).
  constexpr int kRead = kFp8 ? 1 : kAhead;  // a k-step of codes is 64 bytes of a row and two MFMAs of 64 cycles
  Frag ahead[kRead];                        // the first of the second half
  auto both = [&](int32_t key0, int kt) __attribute__((always_inline)) {
    constexpr int kTiles = 1;  // written as loops over tiles: the allocator spills 36 bytes a lane of the plain form, 10 % of the time
    f32x16 s[2][kTiles];
    Frag kf[T::kSteps];
    bf16x8 vf[8];
#pragma unroll
    for (int t = 0; t < kRead; ++t) kf[t] = kt == 0 ? read_k(0, t) : ahead[t];
    __builtin_amdgcn_s_setprio(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) {
      if (t + kRead < T::kSteps) kf[t + kRead] = read_k(kt, t + kRead);
      s[0][0] = score(kf[t], qf[0][t], t == 0 ? zero : s[0][0]);
      if (kt == 0) {
#pragma unroll
        for (int j = t * kCopies / T::kSteps; j < (t + 1) * kCopies / T::kSteps; ++j) spread_copy(j);
      }
      s[1][0] = score(kf[t], qf[1][t], t == 0 ? zero : s[1][0]);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
    const int32_t exist = a.N - key0 - 32 * kt;
    if (exist < 32 * kTiles) {
#pragma unroll
      for (int i = 0; i < kTiles; ++i)
#pragma unroll
        for (int set = 0; set < 2; ++set) hide(s[set][i], exist - 32 * i);
    }
    uint32_t pk[2][8];
#pragma unroll
    for (int set = 0; set < 2; ++set) raise(set, s[set]);
    float psum[2] = {0.f, 0.f};
    const float multiplier[2] = {c * factor[0], c * factor[1]};
    auto p_of = [&](int set, int pair) __attribute__((always_inline)) {
      softmax_pair(s[set][0], pair, multiplier[set], mc[set], pk[set][pair], psum[set]);
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int pair = 0; pair < 4; ++pair) {
      p_of(0, pair);
      p_of(1, pair);
      if (pair >= 2) vf[pair - 2] = read_v(kt, pair - 2);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (j + kAhead < 8) vf[j + kAhead] = read_v(kt, j + kAhead);
      else if (kt == 0 && j + kAhead - 8 < kRead) ahead[j + kAhead - 8] = read_k(1, j + kAhead - 8);
      const int t = j / 4, dt = j % 4;
#pragma unroll
      for (int set = 0; set < 2; ++set) {
        o[set][dt] = mfma32(vf[j], as_bf16x8(pk[set][4 * t], pk[set][4 * t + 1], pk[set][4 * t + 2], pk[set][4 * t + 3]), o[set][dt]);
        if (j < 4) p_of(set, 4 + j);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    l_run[0] += psum[0];
    l_run[1] += psum[1];
    asm volatile("" : "+v"(l_run[0]), "+v"(l_run[1]));
  };

  // A stage of 64 keys for the first set of rows.
  auto one = [&](int32_t key0) __attribute__((always_inline)) {
    constexpr int kFirst = 2 * T::kSteps;
    f32x16 s[2];
    Frag kf[kFirst];
    bf16x8 vf[16];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) kf[i] = read_k(i % 2, i / 2);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < kFirst; ++i) {
      if (i + kAhead < kFirst) kf[i + kAhead] = read_k((i + kAhead) % 2, (i + kAhead) / 2);
      const int kt = i % 2, t = i / 2;
      s[kt] = score(kf[i], qf[0][t], t == 0 ? zero : s[kt]);
#pragma unroll
      for (int j = i * kCopies / kFirst; j < (i + 1) * kCopies / kFirst; ++j) spread_copy(j);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (key0 + T::kStageKeys > a.N) {
      hide(s[0], a.N - key0);
      hide(s[1], a.N - key0 - 32);
    }
    uint32_t pk[2][8];
    raise(0, s);
    float psum = 0.f;
    const float multiplier = c * factor[0];
    auto p_of = [&](int pair) __attribute__((always_inline)) {
      softmax_pair(s[pair / 8], pair % 8, multiplier, mc[0], pk[pair / 8][pair % 8], psum);
    };
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int pair = 0; pair < 4; ++pair) {
      p_of(pair);
      if (pair >= 2) vf[pair - 2] = read_v(0, pair - 2);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (j + kAhead < 16) vf[j + kAhead] = read_v((j + kAhead) / 8, (j + kAhead) % 8);
      const int kt = j / 8, t = j / 4 % 2, dt = j % 4;
      o[0][dt] = mfma32(vf[j], as_bf16x8(pk[kt][4 * t], pk[kt][4 * t + 1], pk[kt][4 * t + 2], pk[kt][4 * t + 3]), o[0][dt]);
      if (j < 12) p_of(4 + j);
      __builtin_amdgcn_sched_barrier(0);
    }
    l_run[0] += psum;
    asm volatile("" : "+v"(l_run[0]));
  };

  // A stage opens with one barrier: its copies have landed for every wave, and the buffer that the next one's go to is consumed.
  int32_t towards = -T::kStageBytes;  // from the buffer that is read to the other one
  auto swap_buffers = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (uint32_t& at : rows_at) at += towards;
    cols_at += towards;
    copy_at -= towards;
    kcopy = __builtin_amdgcn_readfirstlane(copy_at + kcopies);  // wave-uniform by construction
    vcopy = __builtin_amdgcn_readfirstlane(copy_at + vcopies);
    towards = -towards;
  };
  auto walk = [&](auto stage) __attribute__((always_inline)) {
    left = 0;
    chunk = 0;
    int32_t block = take();
    if (block < 0) return;
    int32_t key0 = block * T::kBlk;
    kcopy = __builtin_amdgcn_readfirstlane(copy_at + kcopies);
    vcopy = __builtin_amdgcn_readfirstlane(copy_at + vcopies);
    issue_stage(key0);
    for (int32_t u = 0;; u ^= 1) {
      swap_buffers();
      int32_t key0_next = key0 + T::kStageKeys;
      bool has_next = true;
      if (kFp8 && !u) {
        factor[0] = factor_next[0];
        factor[1] = factor_next[1];
      }
      if (u) {
        block = take();
        has_next = block >= 0;
        key0_next = block * T::kBlk;
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      const bool spread = has_next && key0_next + T::kStageKeys <= a.N;
      if (has_next && !spread) issue_stage(key0_next);
      const uint32_t on = __builtin_amdgcn_readfirstlane(spread ? ~0u : 0u);
      copy_lanes = ((uint64_t)on << 32) | on;
      const int64_t from = spread ? key0_next : key0;
      kbase = kp + (kFp8 ? from : from + wave * 4 * T::kKLoads) * k_row_bytes;
      vbase = (const char*)(vp + (from + wave * 4 * T::kVLoads) * a.v.sn);
      stage(key0);
      if (!has_next) break;
      key0 = key0_next;
    }
  };
  walk([&](int32_t key0) __attribute__((always_inline)) {
    both(key0, 0);
    both(key0, 1);
  });
  shared = false;
#pragma unroll 1
  for (int set = 0; set < 2; ++set) {
    w = set;
    walk([&](int32_t key0) __attribute__((always_inline)) { one(key0); });
    // What only the store needs is not held in scalars meanwhile.
    const Args& late = own_args<Args>();
    const int lane2 = lane_again(), g2 = lane2 >> 5;
    const int32_t b2 = bh / late.H, h2 = bh % late.H;
    __bf16* op = (__bf16*)late.o.ptr + (int64_t)b2 * late.o.sb + (int64_t)h2 * late.o.sh;
    const int32_t q_row = (qb + set) * T::kBlk + wave * 32 + (lane2 & 31);
    const float l_tot = l_run[0] + __shfl_xor(l_run[0], 32);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    if (q_row < late.N) {
      __bf16* const dst = op + (int64_t)q_row * late.o.sn;
#pragma unroll
      for (int dt = 0; dt < T::kDTiles; ++dt)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          u32x2 x;
          x[0] = pack_bf16(o[0][dt][4 * e4] * inv, o[0][dt][4 * e4 + 1] * inv);
          x[1] = pack_bf16(o[0][dt][4 * e4 + 2] * inv, o[0][dt][4 * e4 + 3] * inv);
          *(u32x2*)(dst + 32 * dt + 8 * e4 + 4 * g2) = x;
        }
      if (late.lse && g2 == 0) late.lse[(int64_t)bh * late.N + q_row] = l_tot > 0.f ? m_run[0] * late.scale + __logf(l_tot) : -INFINITY;
    }
    if constexpr (kTrace)
      if (a.wg_trace != nullptr && threadIdx.x == 0 && qb + set < a.n_blocks) t_begin = write_trace(a, t_begin, record + 8 * set);
#pragma unroll
    for (int dt = 0; dt < T::kDTiles; ++dt) o[0][dt] = o[1][dt];
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) qf[0][t] = qf[1][t];
    m_run[0] = m_run[1];
    l_run[0] = l_run[1];
    mc[0] = mc[1];
    q_scale[0] = q_scale[1];
  }
}

template <bool kTrace>
__global__ void __launch_bounds__(256, 2) radial_fwd_two_kernel(const FwdArgs a, const TwoMap m) {
  constexpr int kBytes = TwoTile<false>::kLdsBytes;
  TwoItem item;
  if (!two_item(a.work, m, blockIdx.x, item)) return;
  const int32_t qb = 2 * item.pair + item.block;
  if (item.form == TwoItem::kPair) two_body<kTrace>(a, item.bh, qb, m.c, item.record, static_lds<FwdKey<128, 128, false, kTrace, kBytes>, kBytes>());
  else if (item.form == TwoItem::kBlock) fwd_body<128, 128, false, kTrace, 1, 1, kBytes>(own_args<FwdArgs>(), item.bh, qb, 0, item.record);
  else fwd_body<128, 128, false, kTrace, 2, 2, kBytes>(own_args<FwdArgs>(), item.bh, qb, item.half, item.record);
}

template <bool kTrace>
int launch_two(const FwdArgs& a, hipStream_t stream) {
  const TwoMap m = make_two_map(a.work, a.pair_order, a.scale, TwoWalk::kForward);
  radial_fwd_two_kernel<kTrace><<<dim3(m.n_two + 2 * m.n_one + 4 * m.n_half), dim3(256), 0, stream>>>(a, m);
  RADIAL_HIP_TRY(hipGetLastError());
  return RADIAL_OK;
}

}  // namespace fwd
}  // namespace radial

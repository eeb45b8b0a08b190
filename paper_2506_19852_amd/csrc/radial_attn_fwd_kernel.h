// Block-sparse attention forward kernel for gfx950 (template; instantiated by radial_attn_fwd.hip and,
// with per-workgroup trace records, by radial_diag.hip): Eq. 2 of the paper evaluated only on the key
// blocks that the block list names (Eq. 1 when the list names all of them).
//
// One workgroup = one (batch, head, query block), or half of one.  Wave w of a group of waves owns 32
// query rows; where a launch is small, several groups share the rows and take the list's entries in turn.  Everything
// that belongs to query row r lives in lanes r and r+32 of that wave, because both products
// are computed transposed on v_mfma_f32_32x32x16_bf16:
//     S^T[key, q] = K[key, :] . Q[q, :]      A = K tile (LDS),     B = Q^T (registers)
//     O^T[d,   q] = V^T[d, key] . P^T[key, q] A = V^T (LDS, transposing read), B = P^T (registers)
// The accumulator layout of the first product (column = lane%32, 16 rows per lane) is, 8
// rows at a time, exactly the B-operand layout of the second one, so P never leaves
// registers, row maxima and sums are in-lane reductions plus one exchange with lane^32, and
// the running rescale of O is a per-lane multiply.
//
// Key blocks are walked in stages of 64 keys (32 for head dimension 128 with 64-token blocks).  The K and V rows of a stage are copied
// HBM -> LDS by global_load_lds (no register staging) into one of two LDS stage buffers; the
// copy of stage u+1 is issued right after the barrier that opens stage u, so it overlaps
// the whole of stage u's arithmetic and a stage needs exactly one barrier.  The copies are
// issued from inline assembly and waited for explicitly (s_waitcnt vmcnt(0) before that
// barrier): otherwise the compiler orders every LDS read after all outstanding copies.
// 16-byte pieces are XOR-swizzled inside 256-byte LDS lines so that the 128-bit K reads and
// the 64-bit transposing V reads are bank-conflict free.
#pragma once

#include <type_traits>

#include "radial_internal.h"
#include "radial_tile.h"

namespace radial {
namespace fwd {

// S: groups of waves that share the query rows; group i walks the list entries i, i + S, ... on its
// own stage buffers and the groups' results are merged at the end.
// R: workgroups per query block, of kRows rows each.
template <int D, int BLK, int S, int R>
struct Tile {
  static constexpr int kRows = BLK / R;
  // Keys per pipeline stage.  Head dimension 128 with 64 rows walks half-size stages: two
  // 64-key stage buffers (64 KiB) per 2 waves would leave a compute unit with 4 waves.
  static constexpr int kStageKeys = (D == 128 && kRows == 64) || kRows == 32 || (S == 2 && R == 2) ? 32 : 64;
  static constexpr int kWaves = kRows / 32;        // one wave per 32 query rows
  static constexpr int kThreads = 64 * kWaves * S;
  static constexpr int kPiecesPerRow = D / 8;      // 16-byte pieces per K/V row
  static constexpr int kSubs = BLK / kStageKeys;   // stages per listed key block
  static constexpr int kStageBytes = kStageKeys * D * 2;            // one K (or V) stage tile
  static constexpr int kLoadsPerWave = kStageBytes / 1024 / kWaves; // 1 KiB copies per wave per tile
  static constexpr int kSteps = D / 16;            // MFMA k-steps of the S product
  static constexpr int kKeyTiles = kStageKeys / 32;
  static constexpr int kDTiles = D / 32;           // 32-wide d tiles of O
  // a wave's copies of the next stage, and the MFMAs of the first product that they are spread over
  static constexpr int kCopies = 2 * kLoadsPerWave, kCopyOver = kKeyTiles * kSteps;
  static constexpr int kGroupBytes = 4 * kStageBytes;               // [stage buffer][K, V]
  using Join = Merge<S, kWaves, kDTiles, S == 2 && R == 2 ? S * kGroupBytes : 160 * 1024>;  // (2, 2): beside whole blocks in one kernel
  static constexpr int kLdsBytes = S * kGroupBytes > Join::kLdsBytes ? S * kGroupBytes : Join::kLdsBytes;
};

// Swizzle key of a 256-byte LDS line (16 pieces of 16 bytes); pieces move inside their line only.
template <int D, bool kIsV>
__device__ __forceinline__ int swizzle_key(int line) {
  if (kIsV) return D == 128 ? ((line & 3) << 2) : ((line & 1) << 2);
  return D == 128 ? (line & 15) : (line & 7);
}

// LDS byte offset of 16-byte piece p of tile row r.
template <int D, bool kIsV>
__device__ __forceinline__ int piece_offset(int r, int p) {
  const int lin = r * (D / 8) + p;
  const int line = lin >> 4, slot = lin & 15;
  return (line << 8) + ((slot ^ swizzle_key<D, kIsV>(line)) << 4);
}

// The static stage buffers of a kernel (one array per Key, named where it is used and not through a pointer: its address is
// then a constant that the reads of the stage loop carry in their offsets).  As dynamic LDS, D 128, block 128: 225 registers
// instead of 205 and 6 waits more in two stages (token rule: 50 vector instructions more); 40 x 32 760 all-ones list 19.34 /
// 19.25 ms, 24 x 118 800 74.7 / 74.3, 40 x 32 760 token rule 14.51 / 14.16.
template <class Key, int kBytes>
__device__ __forceinline__ char* static_lds() {
  __shared__ __attribute__((aligned(1024))) char lds[kBytes];
  return lds;
}
template <int D, int BLK, bool kExact, bool kTrace, int kShared>
struct FwdKey {};

// One record per (head, query block), by the first thread of the workgroup with its first rows: begin, end, where it ran.  Returns the end.
__device__ __forceinline__ uint64_t write_trace(const FwdArgs& a, uint64_t begin, int64_t record) {
  // hardware id registers: which XCD, shader engine and compute unit this workgroup ran on
  constexpr int kHwId = 4, kXccId = 20, kAllBits = 31 << 11;
  const uint64_t where = ((uint64_t)__builtin_amdgcn_s_getreg(kXccId | kAllBits) << 32) | (uint32_t)__builtin_amdgcn_s_getreg(kHwId | kAllBits);
  uint64_t* rec = a.wg_trace + 3 * record;
  const uint64_t end = __builtin_amdgcn_s_memrealtime();
  rec[0] = begin;
  rec[1] = end;
  rec[2] = where;
  return end;
}

// One block of query rows, or part `part` of the R of one.
// kExact: apply the token-level rule of the radial mask inside the listed blocks.
// kTrace: also record begin, end and hardware ids of the workgroup (diagnostics build of the kernel;
// the library's radial_attn_fwd launches kTrace = false, which carries none of it).
// kShared: bytes of the static stage buffers of a kernel that has several forms, 0: this is its only one.
template <int D, int BLK, bool kExact, bool kTrace, int S, int R, int kShared>
__device__ __forceinline__ void fwd_body(const FwdArgs& a, int32_t bh, int32_t qb, int32_t part, int64_t record) {
  using T = Tile<D, BLK, S, R>;
  using Key = FwdKey<D, BLK, kExact, kTrace, kShared>;
  constexpr bool kStatic = S == 1 || kShared;
  constexpr int kStaticBytes = kShared ? kShared : T::kLdsBytes;
  static_assert(T::kLdsBytes <= kStaticBytes, "every form uses the stage buffers of the largest");
  // [group][stage buffer][K, V][T::kStageKeys x D bf16]
  extern __shared__ __attribute__((aligned(1024))) char lds_all[];

  const int lane = threadIdx.x & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = S == 1 ? 0 : wave_all / T::kWaves;
  const int wave = S == 1 ? wave_all : wave_all % T::kWaves;
  // Through a pointer in half blocks only, where the compiler's schedule is the better one (126 items, D 128: 56.4 us
  // against 57.9; two groups at 240 items 112.2 against 111.3).
  const char* const lds_group = lds_all + group * T::kGroupBytes;
  const auto lds_at = [&](int32_t offset) __attribute__((always_inline)) -> const char* {
    if constexpr (S == 1) return static_lds<Key, kStaticBytes>() + offset;
    else if constexpr (kStatic) return static_lds<Key, kStaticBytes>() + group * T::kGroupBytes + offset;
    else if constexpr (R == 1) return lds_all + group * T::kGroupBytes + offset;
    else return lds_group + offset;
  };
  const uint32_t lds_base = lds_address(lds_at(0));
  const int lq = lane & 31;   // query column / K row inside a 32-tile
  const int g = lane >> 5;    // which half of the 16-wide MFMA k-slice this lane feeds

  const uint64_t t_begin = kTrace ? __builtin_amdgcn_s_memrealtime() : 0;
  // The division by the number of heads waits for that argument; the tensors' arguments are asked for before it (left to itself
  // the compiler loads them after it, another 0.1 to 0.2 us: D 64, block 128, 288 items L 3 12.3 / 12.1 us, 640 items L 1 11.1 / 10.9).
  int32_t heads = a.H;
  asm("" : "+s"(heads) : "s"(a.q.ptr), "s"(a.k.ptr), "s"(a.row_ptr));
  const int32_t b = bh / heads, h = bh % heads;

  const __bf16* qp = (const __bf16*)a.q.ptr + (int64_t)b * a.q.sb + (int64_t)h * a.q.sh;
  const __bf16* kp = (const __bf16*)a.k.ptr + (int64_t)b * a.k.sb + (int64_t)h * a.k.sh;
  const __bf16* vp = (const __bf16*)a.v.ptr + (int64_t)b * a.v.sb + (int64_t)h * a.v.sh;
  __bf16* op = (__bf16*)a.o.ptr + (int64_t)b * a.o.sb + (int64_t)h * a.o.sh;

  const int32_t list_lo = __builtin_amdgcn_readfirstlane(a.row_ptr[qb]);
  const int32_t n_row = __builtin_amdgcn_readfirstlane(a.row_ptr[qb + 1]) - list_lo;
  const int32_t n_list = S == 1 ? n_row : (n_row - group + S - 1) / S;  // entries of this group
  const int32_t n_stage = n_list * T::kSubs;
  const int32_t q_row = qb * BLK + part * T::kRows + wave * 32 + lq;
  const bool q_ok = q_row < a.N;

  // Q^T fragments: for k-step t this lane holds Q[q_row, 16t + 8g .. +7].
  bf16x8 qf[T::kSteps];
  {
    const __bf16* src = qp + (int64_t)(q_ok ? q_row : a.N - 1) * a.q.sn + 8 * g;
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) {
      u32x4 raw = *(const u32x4*)(src + 16 * t);
      if (!q_ok) raw = u32x4{0u, 0u, 0u, 0u};
      qf[t] = __builtin_bit_cast(bf16x8, raw);
    }
  }

  // The list entries of this row, 64 at a time in one register per lane; cvec is the chunk
  // being walked, nvec the one after it.
  const int32_t* cols = a.col_idx + list_lo + group;
  int32_t cvec = lane < n_list ? cols[S * lane] : 0;
  int32_t nvec = 64 + lane < n_list ? cols[S * (64 + lane)] : 0;
  ListRule<T::kStageKeys, BLK> token;
  if (kExact) token.init(a.rule, qb * BLK + part * T::kRows + wave * 32, a.N, lane);

  // Which piece of a stage tile each of this lane's copies fetches (fixed for the kernel),
  // as a byte offset from the first row of the tile.
  int32_t krow[T::kLoadsPerWave], kcol[T::kLoadsPerWave], vrow_[T::kLoadsPerWave], vcol[T::kLoadsPerWave];
  uint32_t koff[T::kLoadsPerWave], voff[T::kLoadsPerWave];
#pragma unroll
  for (int i = 0; i < T::kLoadsPerWave; ++i) {
    const int lin = (wave * T::kLoadsPerWave + i) * 64 + lane;  // LDS piece this lane fills
    const int line = lin >> 4, slot = lin & 15;
    const int ksrc = (line << 4) + (slot ^ swizzle_key<D, false>(line));
    const int vsrc = (line << 4) + (slot ^ swizzle_key<D, true>(line));
    krow[i] = ksrc / T::kPiecesPerRow;
    kcol[i] = (ksrc % T::kPiecesPerRow) * 8;
    vrow_[i] = vsrc / T::kPiecesPerRow;
    vcol[i] = (vsrc % T::kPiecesPerRow) * 8;
    koff[i] = (uint32_t)(krow[i] * (int32_t)a.k.sn + kcol[i]) * 2u;
    voff[i] = (uint32_t)(vrow_[i] * (int32_t)a.v.sn + vcol[i]) * 2u;
  }
  // Copies the 64 K rows and V rows starting at key `key0` into stage buffer `buf`.
  // Rows past N-1 are clamped to N-1; their scores are masked before the softmax.
  auto issue_stage = [&](int32_t key0, int buf) {
    const uint32_t kdst = lds_base + buf * 2 * T::kStageBytes + wave * T::kLoadsPerWave * 1024;
    const uint32_t vdst = kdst + T::kStageBytes;
    const __bf16* kbase = kp + (int64_t)key0 * a.k.sn;  // wave-uniform
    const __bf16* vbase = vp + (int64_t)key0 * a.v.sn;
    if (key0 + T::kStageKeys <= a.N) {
#pragma unroll
      for (int i = 0; i < T::kLoadsPerWave; ++i) copy16_to_lds_sv(kbase, koff[i], kdst + i * 1024);
#pragma unroll
      for (int i = 0; i < T::kLoadsPerWave; ++i) copy16_to_lds_sv(vbase, voff[i], vdst + i * 1024);
    } else {  // ragged end of the sequence
      const int32_t last = a.N - 1 - key0;  // >= 0: a listed block starts below N; a stage past N reads row N-1
#pragma unroll
      for (int i = 0; i < T::kLoadsPerWave; ++i) {
        const int32_t r = krow[i] < last ? krow[i] : last;
        copy16_to_lds(kp + ((int64_t)key0 + r) * a.k.sn + kcol[i], kdst + i * 1024);
      }
#pragma unroll
      for (int i = 0; i < T::kLoadsPerWave; ++i) {
        const int32_t r = vrow_[i] < last ? vrow_[i] : last;
        copy16_to_lds(vp + ((int64_t)key0 + r) * a.v.sn + vcol[i], vdst + i * 1024);
      }
    }
  };

  f32x16 o[T::kDTiles];
#pragma unroll
  for (int i = 0; i < T::kDTiles; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[i][e] = 0.f;
  float m_run = -INFINITY;  // running row maximum of the raw (unscaled) scores
  float l_run = 0.f;        // this lane's share of the running row sum
  const float c = a.scale * 1.4426950408889634f;  // exp(scale*x) = exp2(c*x)

  int32_t key0 = 0;  // first key of the stage about to be computed
  if (n_stage > 0) {
    key0 = __builtin_amdgcn_readlane(cvec, 0) * BLK;
    issue_stage(key0, 0);
  }

  // One stage: scores of 64 keys, online softmax, O update.  partial: the token rule hides some pair of stage u.  spread_lanes (all or none): also issue this
  // wave's copies of the next stage between the MFMAs of the first product.
  auto stage_body = [&](int buf, int32_t u, int32_t key0, int32_t key0_next, bool partial, uint64_t spread_lanes) __attribute__((always_inline)) {
    const uint32_t kdst_next = lds_base + (buf ^ 1) * 2 * T::kStageBytes + wave * T::kLoadsPerWave * 1024;
    const uint32_t vdst_next = kdst_next + T::kStageBytes;
    const __bf16* kbase_next = kp + (int64_t)key0_next * a.k.sn;  // wave-uniform
    const __bf16* vbase_next = vp + (int64_t)key0_next * a.v.sn;
    const char* lds_k = lds_at(buf * 2 * T::kStageBytes);
    const char* lds_v = lds_k + T::kStageBytes;

    // ---- S^T = K Q^T -------------------------------------------------------------------
    f32x16 s[T::kKeyTiles];
#pragma unroll
    for (int kt = 0; kt < T::kKeyTiles; ++kt) {
#pragma unroll
      for (int e = 0; e < 16; ++e) s[kt][e] = 0.f;
#pragma unroll
      for (int t = 0; t < T::kSteps; ++t) {
        const bf16x8 kf = *lds_cast<const bf16x8>(lds_k + piece_offset<D, false>(kt * 32 + lq, 2 * t + g));
        s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[t], s[kt], 0, 0, 0);
        const int i = kt * T::kSteps + t;  // copies of stage u+1 after this MFMA
#pragma unroll
        for (int j = i * T::kCopies / T::kCopyOver; j < (i + 1) * T::kCopies / T::kCopyOver; ++j) {
          if (j < T::kLoadsPerWave) copy16_to_lds_sv_masked(kbase_next, koff[j], kdst_next + j * 1024, spread_lanes);
          else copy16_to_lds_sv_masked(vbase_next, voff[j - T::kLoadsPerWave], vdst_next + (j - T::kLoadsPerWave) * 1024, spread_lanes);
        }
      }
    }

    // ---- online softmax ------------------------------------------------------------------
    // s[kt][e] belongs to key key0 + 32kt + 8(e/4) + 4g + e%4 and query q_row.  Keys >= N do not
    // exist; under the token rule some keys are hidden from this lane's query.
    if (key0 + T::kStageKeys > a.N || (kExact && partial)) {
      uint32_t hidden = 0u;
      if (!kExact || key0 + T::kStageKeys > a.N) hidden = ~lane_element_bits(stage_prefix(a.N - key0), g);
      if (kExact && partial) hidden |= token.hidden(u, a.rule.s, g, lane);
      constexpr int kTogether = kExact ? 1 : T::kKeyTiles;  // key tiles looked at together: the edge of a diagonal is often in one
#pragma unroll
      for (int k0 = 0; k0 < T::kKeyTiles; k0 += kTogether)
        if (__builtin_amdgcn_ballot_w64((kTogether == T::kKeyTiles ? hidden : hidden >> (16 * k0) & 0xffffu) != 0u) != 0) {
#pragma unroll
          for (int kt = k0; kt < k0 + kTogether; ++kt)
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if ((hidden >> (16 * kt + e)) & 1u) s[kt][e] = -INFINITY;
        }
    }
    float mx = s[0][0];
#pragma unroll
    for (int kt = 0; kt < T::kKeyTiles; ++kt)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[kt][e]);
    mx = max_with_other_half(mx);  // the other 32 keys of the row's stage
    // A stage that lies entirely past N (second half of a ragged last block) has mx = -inf.
    const float m_new = fmaxf(m_run, mx);
    if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0) {  // some row of this wave got a new maximum
      const float alpha = m_new > m_run ? __builtin_amdgcn_exp2f((m_run - m_new) * c) : 1.f;
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < T::kDTiles; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[i][e] *= alpha;
      m_run = m_new;
    }
    const float mc = m_run == -INFINITY ? 0.f : m_run * c;
    float psum = 0.f;
    uint32_t pk[T::kKeyTiles][8];  // P^T as bf16 pairs: B operands of the second product
#pragma unroll
    for (int kt = 0; kt < T::kKeyTiles; ++kt)
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][e], c, -mc));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][e + 1], c, -mc));
        psum += p0 + p1;
        pk[kt][e >> 1] = pack_bf16(p0, p1);
      }
    l_run += psum;

    // ---- O^T += V^T P^T --------------------------------------------------------------------
#pragma unroll
    for (int kt = 0; kt < T::kKeyTiles; ++kt)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const u32x4 praw = {pk[kt][4 * t], pk[kt][4 * t + 1], pk[kt][4 * t + 2], pk[kt][4 * t + 3]};
        const bf16x8 pf = __builtin_bit_cast(bf16x8, praw);
#pragma unroll
        for (int dt = 0; dt < T::kDTiles; ++dt) {
          // Lanes 0-15 / 16-31 / 32-47 / 48-63 each transpose a 4-key x 16-d patch: lane i of
          // a group reads 4 d-contiguous values of key i/4 and receives the 4 keys of d column i.
          const int i16 = lane & 15;
          const int vrow = kt * 32 + 16 * t + 4 * g + (i16 >> 2);
          const int dcol = 32 * dt + 16 * ((lane >> 4) & 1) + 4 * (i16 & 3);
          const int off0 = piece_offset<D, true>(vrow, dcol >> 3) + ((dcol & 7) << 1);
          const int off1 = piece_offset<D, true>(vrow + 8, dcol >> 3) + ((dcol & 7) << 1);
          const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_cast<s16x4>(lds_v + off0));
          const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_cast<s16x4>(lds_v + off1));
          const u32x2 a0 = __builtin_bit_cast(u32x2, v0), a1 = __builtin_bit_cast(u32x2, v1);
          const u32x4 vraw = {a0[0], a0[1], a1[0], a1[1]};
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vraw), pf, o[dt], 0, 0, 0);
        }
      }
  };

  // Two stages per trip, so that the stage buffer of each half is a compile-time constant and the
  // LDS addresses of its reads are immediates.
  auto one_stage = [&](int32_t u, auto buf_c) __attribute__((always_inline)) {
    constexpr int buf = decltype(buf_c)::value;
    if (kExact && buf == 0 && (u & 63) == 0) token.look(a.rule, cvec, u / T::kSubs & 63, lane, true);
    const bool skip = kExact && token.sees_none(u);  // nothing in this stage for any row of this wave
    const bool partial = kExact && !token.sees_all(u);
    // First key of stage u+1.
    int32_t key0_next = 0;
    const bool has_next = u + 1 < n_stage;
    if (has_next) {
      const int32_t e1 = (u + 1) / T::kSubs;
      if ((u + 1) % T::kSubs == 0 && (e1 & 63) == 0) {  // entering the next chunk of the list
        cvec = nvec;
        nvec = e1 + 64 + lane < n_list ? cols[S * (e1 + 64 + lane)] : 0;
      }
      key0_next = __builtin_amdgcn_readlane(cvec, e1 & 63) * BLK + ((u + 1) % T::kSubs) * T::kStageKeys;
    }

    if (T::kWaves == 1) {  // nobody else reads or writes this group's stage buffers
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's copies of stage u have landed
      __syncthreads();                                  // ... and everyone's; stage u-1 is fully consumed
    }

    // The copies of stage u+1 are spread over the first product of stage u (a burst of copies
    // would hold the wave at the memory pipeline before it reaches its first MFMA); only a
    // ragged next stage, or a stage this wave skips, issues them in one go.
    const bool spread = has_next && !skip && key0_next + T::kStageKeys <= a.N;
    if (has_next && !spread) issue_stage(key0_next, buf ^ 1);
    if (!skip) {
      const uint32_t on = __builtin_amdgcn_readfirstlane(spread ? ~0u : 0u);  // wave-uniform by construction
      stage_body(buf, u, key0, spread ? key0_next : key0, partial, ((uint64_t)on << 32) | on);
    }
    key0 = key0_next;
  };
  for (int32_t u = 0; u < n_stage; u += 2) {
    one_stage(u, std::integral_constant<int, 0>{});
    if (u + 1 < n_stage) one_stage(u + 1, std::integral_constant<int, 1>{});
  }

  __bf16* const dst = op + (int64_t)q_row * a.o.sn;
  const auto store_lse = [&](float m, float l) __attribute__((always_inline)) {
    const int64_t idx = ((int64_t)b * a.H + h) * a.N + q_row;
    a.lse[idx] = l > 0.f ? m * a.scale + __logf(l) : -INFINITY;
  };

  // ---- several groups: merge and store ------------------------------------------------------
  if (S > 1) {
    if (T::kWaves > 1)  // a stage is a barrier: as many as group 0, which has most stages
      for (int32_t u = n_stage; u < (n_row + S - 1) / S * T::kSubs; ++u) __syncthreads();
    float m = m_run, l = l_run;
    T::Join::softmax(o, m, l, c, kStatic ? static_lds<Key, kStaticBytes>() : lds_all, group, wave, lane, [&](int p, f32x4 v) __attribute__((always_inline)) {
      if (q_ok) *(u32x2*)(dst + 8 * p + 4 * g) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    });
    if (q_ok && a.lse && g == 0 && group == 0) store_lse(m, l);
  } else {
    // ---- epilogue: O / l, LSE --------------------------------------------------------------
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    if (q_ok) {
#pragma unroll
      for (int dt = 0; dt < T::kDTiles; ++dt)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          // o[dt][4*e4 + x] is d = 32dt + 8*e4 + 4g + x
          u32x2 w;
          w[0] = pack_bf16(o[dt][4 * e4] * inv, o[dt][4 * e4 + 1] * inv);
          w[1] = pack_bf16(o[dt][4 * e4 + 2] * inv, o[dt][4 * e4 + 3] * inv);
          *(u32x2*)(dst + 32 * dt + 8 * e4 + 4 * g) = w;
        }
      if (a.lse && g == 0) store_lse(m_run, l_tot);
    }
  }
  if (kTrace && a.wg_trace != nullptr && threadIdx.x == 0 && part == 0) write_trace(a, t_begin, record);
}

template <int D, int BLK, bool kExact, bool kTrace, int S, int R>
// Two waves per SIMD: two 4-wave workgroups per compute unit (BLK = 128) or four 2-wave ones (BLK = 64)
// with S = R = 1.
__global__ void __launch_bounds__(2 * BLK / R * S, 2) radial_fwd_kernel(const FwdArgs a) {
  int32_t bh, qb;
  if (!work_item(a.work, blockIdx.x, bh, qb)) return;
  const int32_t part = R == 1 ? 0 : bh % R;  // with R > 1 the work map counts R heads for each
  if (R > 1) bh /= R;
  fwd_body<D, BLK, kExact, kTrace, S, R, 0>(a, bh, qb, part, R == 1 ? (int64_t)blockIdx.x : (int64_t)bh * a.n_blocks + qb);
}

// Whole blocks, and the last a.work.halved of the launch in halves of two groups.
template <int D, int BLK, bool kExact, bool kTrace>
__global__ void __launch_bounds__(2 * BLK, 2) radial_fwd_halves_kernel(const FwdArgs a) {
  int32_t bh, qb, part = 0;
  const uint32_t whole = gridDim.x - 2u * (uint32_t)a.work.halved;
  constexpr int kBytes = Tile<D, BLK, 1, 1>::kLdsBytes;
  if (blockIdx.x < whole) {
    if (!work_item(a.work, blockIdx.x, bh, qb)) return;
    fwd_body<D, BLK, kExact, kTrace, 1, 1, kBytes>(a, bh, qb, 0, (int64_t)blockIdx.x);
  } else {
    const uint32_t id = halved_item(blockIdx.x, whole, (uint32_t)a.work.halved, part);
    if (!work_item(a.work, id, bh, qb)) return;
    fwd_body<D, BLK, kExact, kTrace, 2, 2, kBytes>(a, bh, qb, part, (int64_t)id);
  }
}

template <int D, int BLK, bool kExact, bool kTrace, int S, int R>
int launch_split(FwdArgs a, hipStream_t stream) {
  using T = Tile<D, BLK, S, R>;
  const auto kernel = radial_fwd_kernel<D, BLK, kExact, kTrace, S, R>;
  if (S > 1 && T::kLdsBytes > 65536) {
    static DeviceOnce configured;
    if (int rc = allow_dynamic_lds(configured, (const void*)kernel, T::kLdsBytes)) return rc;
  }
  a.work.ordered *= R;  // R > 1 only up to kOneRound items, where all heads are taken by list length
  kernel<<<dim3((unsigned)work_grid(a.work, a.n_blocks)), dim3(T::kThreads), S == 1 ? 0 : T::kLdsBytes, stream>>>(a);
  RADIAL_HIP_TRY(hipGetLastError());
  return RADIAL_OK;
}

template <int D, int BLK, bool kExact, bool kTrace>
int launch_halves(const FwdArgs& a, hipStream_t stream) {
  radial_fwd_halves_kernel<D, BLK, kExact, kTrace><<<dim3((unsigned)(work_grid(a.work, a.n_blocks) + a.work.halved)), dim3(2 * BLK), 0, stream>>>(a);
  RADIAL_HIP_TRY(hipGetLastError());
  return RADIAL_OK;
}

template <bool kTrace>
int launch_two(const FwdArgs& a, hipStream_t stream);  // radial_attn_fwd_two.h

template <int D, int BLK, bool kExact, bool kTrace>
int launch(const FwdArgs& a, hipStream_t stream) {
  if (work_grid_bound(a.work) > 0x7fffffffLL) return fail(RADIAL_ESHAPE, "B*H*n_blocks is too large for one launch");
  const int64_t items = work_items(a.work, a.n_blocks);
  if (items == 0) return RADIAL_OK;
  const int groups = query_groups(D, BLK, a.work, items, true);
  if (single_waves(BLK, a.work, items)) return launch_split<D, BLK, kExact, kTrace, D == 64 ? 8 : 4, BLK / 32>(a, stream);
  if (groups == 4) return launch_split<D, BLK, kExact, kTrace, 4, BLK / 64>(a, stream);
  if (groups == 2) return launch_split<D, BLK, kExact, kTrace, 2, 1>(a, stream);
  if constexpr (D == 128 && BLK == 128 && !kExact)
    if (takes_pairs(a.work)) return launch_two<kTrace>(a, stream);
  if constexpr (BLK == 128)
    if (const int32_t halved = halved_items(a.work, items)) {
      FwdArgs h = a;
      h.work.halved = halved;
      return launch_halves<D, BLK, kExact, kTrace>(h, stream);
    }
  return launch_split<D, BLK, kExact, kTrace, 1, 1>(a, stream);
}

// Launches the kernel instance for (D, block, token rule); kTrace selects the diagnostics build.
template <int D, int BLK, bool kTrace>
int launch_tile(const FwdArgs& a, hipStream_t stream) {
  return a.rule.exact ? launch<D, BLK, true, kTrace>(a, stream) : launch<D, BLK, false, kTrace>(a, stream);
}

template <bool kTrace>
int launch_any(int D, int block, const FwdArgs& a, hipStream_t stream) {
  if (D == 128 && block == 128) return launch_tile<128, 128, kTrace>(a, stream);
  if (D == 64 && block == 128) return launch_tile<64, 128, kTrace>(a, stream);
  if (D == 128 && block == 64) return launch_tile<128, 64, kTrace>(a, stream);
  if (D == 64 && block == 64) return launch_tile<64, 64, kTrace>(a, stream);
  return fail(RADIAL_EUNSUPPORTED, "head dimension %d with block %d is not supported", D, block);
}

}  // namespace fwd
}  // namespace radial

// Block-sparse attention backward for gfx950: the gradient of Eq. 2 of the paper restricted to
// the listed block pairs,
//     P = exp(scale*Q K^T - LSE),  dV = P^T dO,  dP = dO V^T,  delta = rowsum(dO * O),
//     dS = P * (dP - delta),       dQ = scale * dS K,          dK = scale * dS^T Q.
//
// Three parts, no atomics (results are reproducible run to run); dkdv and dq are workgroups of one launch where either alone
// would leave the chip idle (backward_form), else kernels of their own:
//   prepare : delta[b,h,q] = sum_d dO*O;
//   dkdv    : one workgroup per (batch, head, key block) walks the transposed list (the query
//             blocks that list this key block) in stages of 64 query rows.  Wave w owns 32
//             keys; its K and V rows stay in registers, dK^T and dV^T accumulate in registers
//             (column = key = lane%32).  S and dP are computed with query rows as MFMA rows
//             so that P and dS come out with keys across lanes: 8 accumulator rows at a time
//             they are the B operands of dV^T += dO^T P and dK^T += Q^T dS, whose A operands
//             are transposing LDS reads of the dO and Q stage tiles (head dimension 128, blocks of 128: two waves
//             share 32 keys, see PairTile);
//   dq      : one workgroup per (batch, head, query block) walks the row list in stages of 64
//             keys, like the forward kernel: wave w owns 32 query rows whose Q and dO rows stay
//             in registers; S^T = K Q^T and dP^T = V dO^T come out with queries across lanes,
//             LSE and delta are per-lane scalars, and dS^T feeds dQ^T += K^T dS^T from registers
//             (A operand: transposing LDS reads of the K stage tile).  S and dP are recomputed
//             here (7 products in total instead of 5), which is cheaper than pushing every
//             listed pair's 64 KiB of dQ partial sums through memory atomics.
// Stage tiles are copied HBM -> LDS by global_load_lds, double buffered, one stage ahead.
#include <type_traits>

#include "radial_internal.h"
#include "radial_tile.h"

namespace radial {
namespace {

constexpr int kStageQ = 64;  // query rows per pipeline stage
constexpr float kLog2e = 1.4426950408889634f;

// S: groups of waves that share the keys (dq kernel: the query rows); group i walks the list entries
// i, i + S, ... on its own stage buffers and the groups' sums are added at the end.
// R: workgroups per block, of kRows keys (rows) each.
template <int D, int BLK, int S, int R>
struct BwdTile {
  static constexpr int kRows = BLK / R;
  static constexpr int kWaves = kRows / 32;  // one wave per 32 keys
  static constexpr int kThreads = 64 * kWaves * S;
  static constexpr int kSubs = BLK / kStageQ;  // stages per listed query block
  static constexpr int kSteps = D / 16;
  static constexpr int kDTiles = D / 32;
  static constexpr int kQBytes = kStageQ * D * 2;        // Q or dO stage tile
  static constexpr int kStatBytes = 2 * kStageQ * 4;     // LSE and delta of a stage
  static constexpr int kStageBytes = 2 * kQBytes + kStatBytes;
  static constexpr int kGroupBytes = 2 * kStageBytes;
  using Join = Merge<S, kWaves, kDTiles>;
  static constexpr int kLdsBytes = S * kGroupBytes > Join::kLdsBytes ? S * kGroupBytes : Join::kLdsBytes;
  static constexpr int kQLoadsPerWave = kQBytes / 1024 / kWaves;
  static constexpr int kStatLoads = kWaves == 1 ? 2 : 1;  // copies of LSE and delta: waves 0 and 1 take one each
};

template <int D>
__global__ void __launch_bounds__(256) bwd_prepare_kernel(const BwdArgs a) {
  constexpr int kLanesPerRow = D / 8;
  constexpr int kRowsPerBlock = 256 / kLanesPerRow;
  const int64_t rows = (int64_t)a.B * a.H * a.N;
  const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + threadIdx.x / kLanesPerRow;
  const int piece = threadIdx.x % kLanesPerRow;
  float sum = 0.f;
  if (row < rows) {
    const int32_t q = (int32_t)(row % a.N);
    const int32_t bh = (int32_t)(row / a.N);
    const int32_t b = bh / a.H, h = bh % a.H;
    const __bf16* o = (const __bf16*)a.o.ptr + (int64_t)b * a.o.sb + (int64_t)h * a.o.sh + (int64_t)q * a.o.sn + piece * 8;
    const __bf16* g = (const __bf16*)a.dout.ptr + (int64_t)b * a.dout.sb + (int64_t)h * a.dout.sh + (int64_t)q * a.dout.sn + piece * 8;
    const bf16x8 ov = *(const bf16x8*)o;
    const bf16x8 gv = *(const bf16x8*)g;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += (float)ov[i] * (float)gv[i];
  }
#pragma unroll
  for (int off = kLanesPerRow / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (row < rows && piece == 0) a.delta[row] = sum;
}

// acc (+)= a * b with the accumulator in ordinary vector registers.  In a kernel that uses both
// register files the compiler places every MFMA result in the accumulation file; S and dP are
// consumed by vector instructions, which cannot read that file, so each of their 64 values per stage
// would be copied out one register at a time (a third of the kernel's vector instructions).
// The instruction is opaque to the compiler's hazard tracking.  What the compiler would guarantee
// is arranged here or checked on the compiled code by tests/test_kernel_asm.py:
//   - the result registers of the first k-step overlap no operand (early clobber);
//   - no vector instruction writes an operand within two wait states before the MFMA (checked);
//   - before a vector instruction reads or writes acc the caller waits with mfma_results_settle(),
//     and nothing else names acc in between (checked);
//   - a second MFMA on the same accumulator follows after one other MFMA at the earliest.
__device__ __forceinline__ void mfma32_vgpr_first(f32x16& acc, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma32_vgpr(f32x16& acc, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
// 16 wait states: more than the 11 an 8-pass MFMA needs before a vector instruction touches its result.
// The accumulators are operands so that every later use of them stays behind the wait.
__device__ __forceinline__ void mfma_results_settle(f32x16& acc0, f32x16& acc1) {
  asm volatile("s_nop 15" : "+v"(acc0), "+v"(acc1));
}

// kExact (all three kernels' callers): apply the token-level rule inside the listed blocks.
// kTwoWaves: two waves per SIMD and the compiler's schedule instead of one wave and the hand-made one.  At head dimension
// 64 a stage has 32 MFMAs (1024 cycles) to 178 plain vector instructions and 32 exponentials (1220 cycles), so the vector
// unit is what bounds it and one wave cannot keep it busy: 2478 items of block 128 (10 x 17 000 tokens) 4.75 -> 4.1 ms, the
// step 9.34 -> 8.21 ms.  192 to 216 registers (222 to 235 in groups of one wave beside dQ); held to 168 for a third wave it spills 23 (block 128) to 45: 1-2 % slower, in
// blocks of 64 25 %.  Head dimension 128 needs 376 to 384 registers and has one wave.
template <int D, int BLK, bool kExact, int S, int R, bool kTwoWaves>
__device__ __forceinline__ void dkdv_body(const BwdArgs& a, uint32_t id) {
  using T = BwdTile<D, BLK, S, R>;
  using QT = SwzTile<D>;  // Q, dO tiles: rows of D elements
  static_assert(kTwoWaves == (D == 64), "the hand-made schedule deals the 8 softmax pairs of a half over the 8 k-steps of head dimension 128");
  extern __shared__ __attribute__((aligned(1024))) char lds_all[];

  const int lane = threadIdx.x & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = S == 1 ? 0 : wave_all / T::kWaves;
  const int wave = S == 1 ? wave_all : wave_all % T::kWaves;
  char* lds = lds_all + group * T::kGroupBytes;
  const uint32_t lds_base = lds_address(lds);
  const int lq = lane & 31;
  const int g = lane >> 5;
  const int i16 = lane & 15;
  const int half16 = (lane >> 4) & 1;

  int32_t bh, kb;
  if (!work_item(a.work_t, id, bh, kb)) return;
  const int32_t part = R == 1 ? 0 : bh % R;  // with R > 1 the work map counts R heads for each
  if (R > 1) bh /= R;
  const int32_t b = bh / a.H, h = bh % a.H;

  const __bf16* qp = (const __bf16*)a.q.ptr + (int64_t)b * a.q.sb + (int64_t)h * a.q.sh;
  const __bf16* kp = (const __bf16*)a.k.ptr + (int64_t)b * a.k.sb + (int64_t)h * a.k.sh;
  const __bf16* vp = (const __bf16*)a.v.ptr + (int64_t)b * a.v.sb + (int64_t)h * a.v.sh;
  const __bf16* gp = (const __bf16*)a.dout.ptr + (int64_t)b * a.dout.sb + (int64_t)h * a.dout.sh;
  const float* lsep = a.lse + (int64_t)bh * a.N;
  const float* deltap = a.delta + (int64_t)bh * a.N;

  const int32_t list_lo = __builtin_amdgcn_readfirstlane(a.col_ptr[kb]);
  const int32_t n_col = __builtin_amdgcn_readfirstlane(a.col_ptr[kb + 1]) - list_lo;
  const int32_t n_list = S == 1 ? n_col : (n_col - group + S - 1) / S;  // entries of this group
  const int32_t n_stage = n_list * T::kSubs;
  const int32_t key_row = kb * BLK + part * T::kRows + wave * 32 + lq;
  const bool key_ok = key_row < a.N;

  // K and V rows of this lane's key: B operands of S = Q K^T and dP = dO V^T.
  bf16x8 kf[T::kSteps], vf[T::kSteps];
  {
    const int64_t r = key_ok ? key_row : a.N - 1;
    const __bf16* ks = kp + r * a.k.sn + 8 * g;
    const __bf16* vs = vp + r * a.v.sn + 8 * g;
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) {
      u32x4 kr = *(const u32x4*)(ks + 16 * t), vr = *(const u32x4*)(vs + 16 * t);
      if (!key_ok) kr = vr = u32x4{0u, 0u, 0u, 0u};
      kf[t] = __builtin_bit_cast(bf16x8, kr);
      vf[t] = __builtin_bit_cast(bf16x8, vr);
    }
  }

  const int32_t* rows_list = a.row_idx + list_lo + group;
  int32_t cvec = lane < n_list ? rows_list[S * lane] : 0;
  int32_t nvec = 64 + lane < n_list ? rows_list[S * (64 + lane)] : 0;
  ListRule<kStageQ, BLK> token;
  if (kExact) token.init(a.rule, kb * BLK + part * T::kRows + wave * 32, a.N, lane);

  int32_t srow[T::kQLoadsPerWave], scol[T::kQLoadsPerWave];
#pragma unroll
  for (int i = 0; i < T::kQLoadsPerWave; ++i) QT::source_of((wave * T::kQLoadsPerWave + i) * 64 + lane, srow[i], scol[i]);

  uint32_t qoff[T::kQLoadsPerWave], goff[T::kQLoadsPerWave];  // byte offsets from the stage's first row
#pragma unroll
  for (int i = 0; i < T::kQLoadsPerWave; ++i) {
    qoff[i] = (uint32_t)(srow[i] * (int32_t)a.q.sn + scol[i]) * 2u;
    goff[i] = (uint32_t)(srow[i] * (int32_t)a.dout.sn + scol[i]) * 2u;
  }
  // Copies Q, dO (64 rows from q0) and their LSE / delta into stage buffer `buf`, all at once
  // (first stage, ragged stages; rows past N-1 are clamped to N-1).
  auto issue_stage = [&](int32_t q0, int buf) {
    const uint32_t qdst = lds_base + buf * T::kStageBytes + wave * T::kQLoadsPerWave * 1024;
    const uint32_t gdst = qdst + T::kQBytes;
#pragma unroll
    for (int i = 0; i < T::kQLoadsPerWave; ++i) {
      int32_t r = q0 + srow[i];
      r = r < a.N ? r : a.N - 1;
      copy16_to_lds(qp + (int64_t)r * a.q.sn + scol[i], qdst + i * 1024);
      copy16_to_lds(gp + (int64_t)r * a.dout.sn + scol[i], gdst + i * 1024);
    }
    if (wave < 2) {
      int32_t r = q0 + lane;
      r = r < a.N ? r : a.N - 1;
      const uint32_t sdst = lds_base + buf * T::kStageBytes + 2 * T::kQBytes + wave * kStageQ * 4;
      copy4_to_lds((wave == 0 ? lsep : deltap) + r, sdst);
      if (T::kStatLoads == 2) copy4_to_lds(deltap + r, sdst + kStageQ * 4);
    }
  };

  f32x16 dk[T::kDTiles], dv[T::kDTiles];
#pragma unroll
  for (int i = 0; i < T::kDTiles; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) dk[i][e] = dv[i][e] = 0.f;
  const float c = a.scale * kLog2e;

  int32_t q0 = 0;
  if (n_stage > 0) {
    q0 = __builtin_amdgcn_readlane(cvec, 0) * BLK;
    issue_stage(q0, 0);
  }

  for (int32_t u = 0; u < n_stage; ++u) {
    const int buf = u & 1;
    if (kExact && (u & 63) == 0) token.look(a.rule, cvec, u / T::kSubs & 63, lane, false);
    const bool partial = kExact && !token.sees_all(u);
    int32_t q0_next = 0;
    const bool has_next = u + 1 < n_stage;
    if (has_next) {
      const int32_t e1 = (u + 1) / T::kSubs;
      if ((u + 1) % T::kSubs == 0 && (e1 & 63) == 0) {
        cvec = nvec;
        nvec = e1 + 64 + lane < n_list ? rows_list[S * (e1 + 64 + lane)] : 0;
      }
      q0_next = __builtin_amdgcn_readlane(cvec, e1 & 63) * BLK + ((u + 1) % T::kSubs) * kStageQ;
    }

    if (T::kWaves == 1) {  // nobody else reads or writes this group's stage buffers
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    } else {
      wait_all_copies();  // stage u has landed
      __syncthreads();    // for every wave; stage u-1 is finished
    }
    // The copies of a full next stage are spread over the first MFMAs of this one (see below);
    // a ragged one is issued at once.
    // A wave that sees nothing of the stage skips it.  Backward pass, us: D 64, block 128, 10 x 17 000 tokens 2150 / 2045, 4 x 30 000
    // 2754 / 2607, blocks of 64 (fewer such stages) 910 / 911.  Not with the hand-made schedule: the second way round its
    // loop cost 15 to 18 % (D 128, block 64, 8 x 14 040 2502 / 2953).
    const bool skip = kExact && kTwoWaves && token.sees_none(u);
    const bool spread_next = has_next && !skip && q0_next + kStageQ <= a.N;
    if (has_next && !spread_next) issue_stage(q0_next, buf ^ 1);
    if (skip) {
      q0 = q0_next;
      continue;
    }

    const char* sq = lds + buf * T::kStageBytes;
    const char* sg = sq + T::kQBytes;
    const char* st = sg + T::kQBytes;  // 64 x LSE then 64 x delta
    const bool ragged_q = q0 + kStageQ > a.N;
    uint32_t hidden = 0u;
    if (ragged_q || partial) {  // query rows past N, rows the token rule hides from this key
      if (!kExact || ragged_q) hidden = ~lane_element_bits(stage_prefix(a.N - q0), g);
      if (kExact && partial) hidden |= token.hidden(u, a.rule.s, g, lane);
    }
    const bool any_hidden = __builtin_amdgcn_ballot_w64(hidden != 0u) != 0;
    // this wave's copies of the next stage, one or two per k-step of phase A
    const uint32_t on = __builtin_amdgcn_readfirstlane(spread_next ? ~0u : 0u);
    const uint64_t copy_lanes = ((uint64_t)on << 32) | on;
    const int32_t q_src = spread_next ? q0_next : q0;  // any valid row when the copies are switched off
    const __bf16* qbase_next = qp + (int64_t)q_src * a.q.sn;
    const __bf16* gbase_next = gp + (int64_t)q_src * a.dout.sn;
    const uint32_t qdst_next = lds_base + (buf ^ 1) * T::kStageBytes + wave * T::kQLoadsPerWave * 1024;
    const uint32_t gdst_next = qdst_next + T::kQBytes;
    auto spread_copy = [&](int j) {  // Q pieces, dO pieces, LSE and delta
      if (j < T::kQLoadsPerWave) {
        copy16_to_lds_sv_masked(qbase_next, qoff[j], qdst_next + j * 1024, copy_lanes);
      } else if (j < 2 * T::kQLoadsPerWave) {
        copy16_to_lds_sv_masked(gbase_next, goff[j - T::kQLoadsPerWave], gdst_next + (j - T::kQLoadsPerWave) * 1024, copy_lanes);
      } else {
        const int which = T::kStatLoads == 2 ? j - 2 * T::kQLoadsPerWave : wave & 1;
        const uint32_t sdst = lds_base + (buf ^ 1) * T::kStageBytes + 2 * T::kQBytes + which * kStageQ * 4;
        copy4_to_lds_sv_masked((which == 0 ? lsep : deltap) + q_src, (uint32_t)lane * 4u, sdst, wave < 2 ? copy_lanes : 0ull);
      }
    };

    // LSE and delta of either half: element e of the half is the value in lane e of this lane's row of 16.  As 16-byte reads of
    // the same values in all lanes they were a quarter (D 128: a fifth) of what the kernel reads from LDS, and 64 registers of the
    // hand-made schedule.  Backward pass, us: D 64, block 128, 10 x 17 000 tokens 2059 / 2028, block 64, 5 x 14 040 840 / 821; D 128, block 64,
    // 8 x 14 040 2320 / 2283, block 128, 100 items L 16 71.2 / 69.2.
    float lse[2], delta[2];
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
      const int ql = h2 * 32 + 8 * (i16 >> 2) + 4 * g + (i16 & 3);
      lse[h2] = *lds_cast<const float>(st + ql * 4) * kLog2e;
      delta[h2] = *lds_cast<const float>(st + (kStageQ + ql) * 4);
    }

    if constexpr (kTwoWaves) {
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        f32x16 s, dp;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = dp[e] = 0.f;
#pragma unroll
        for (int t = 0; t < T::kSteps; ++t) {
          const bf16x8 qfrag = *lds_cast<const bf16x8>(sq + QT::piece(h2 * 32 + lq, 2 * t + g));
          const bf16x8 gfrag = *lds_cast<const bf16x8>(sg + QT::piece(h2 * 32 + lq, 2 * t + g));
          s = mfma32(qfrag, kf[t], s);
          dp = mfma32(gfrag, vf[t], dp);
          if (h2 == 0) {
            constexpr int kCopies = 2 * T::kQLoadsPerWave + T::kStatLoads;
#pragma unroll
            for (int j = t * kCopies / T::kSteps; j < (t + 1) * kCopies / T::kSteps; ++j) spread_copy(j);
          }
        }
        if (any_hidden) {
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if ((hidden >> (16 * h2 + e)) & 1u) s[e] = -INFINITY;
        }
        uint32_t pp[8], dsp[8];
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {  // element 4*e4 + x: query row 32*h2 + 8*e4 + 4g + x of the stage
          float pr[4], dr[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            pr[x] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[4 * e4 + x], c, -row_lane(lse[h2], 4 * e4 + x)));
            dr[x] = pr[x] * (dp[4 * e4 + x] - row_lane(delta[h2], 4 * e4 + x));
          }
          pp[2 * e4] = pack_bf16(pr[0], pr[1]);
          pp[2 * e4 + 1] = pack_bf16(pr[2], pr[3]);
          dsp[2 * e4] = pack_bf16(dr[0], dr[1]);
          dsp[2 * e4 + 1] = pack_bf16(dr[2], dr[3]);
        }
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
          const bf16x8 pf = as_bf16x8(pp[4 * t2], pp[4 * t2 + 1], pp[4 * t2 + 2], pp[4 * t2 + 3]);
          const bf16x8 dsf = as_bf16x8(dsp[4 * t2], dsp[4 * t2 + 1], dsp[4 * t2 + 2], dsp[4 * t2 + 3]);
          const int r0 = h2 * 32 + 16 * t2 + 4 * g + (i16 >> 2);
#pragma unroll
          for (int dt = 0; dt < T::kDTiles; ++dt) {
            const int col = 32 * dt + 16 * half16 + 4 * (i16 & 3);
            const u32x2 g0 = lds_read_tr(sg + QT::elem(r0, col)), g1 = lds_read_tr(sg + QT::elem(r0 + 8, col));
            const u32x2 q0v = lds_read_tr(sq + QT::elem(r0, col)), q1v = lds_read_tr(sq + QT::elem(r0 + 8, col));
            dv[dt] = mfma32(as_bf16x8(g0[0], g0[1], g1[0], g1[1]), pf, dv[dt]);
            dk[dt] = mfma32(as_bf16x8(q0v[0], q0v[1], q1v[0], q1v[1]), dsf, dk[dt]);
          }
        }
      }
      q0 = q0_next;
      continue;
    }

    // The stage is two 32-row halves (h = 0, 1).  One wave per SIMD has nobody to hide its LDS
    // and VALU latencies behind, so the four products are software-pipelined by hand:
    //   A: S, dP of half 0                    B: S, dP of half 1   | P, dS of half 0
    //   C: dV, dK with half 0 | P, dS of half 1                    D: dV, dK with half 1
    // LDS fragments are read kAhead MFMAs before their use and the scheduling fences keep the
    // written order.
    f32x16 s[2], dp[2];
    uint32_t pp[2][8], dsp[2][8];
    // P and dS of elements 2*pair, 2*pair + 1 of half h2 (key = this lane's, queries as above)
    auto softmax_pair = [&](int h2, int pair) {
      const int e = 2 * pair;
      const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h2][e], c, -row_lane(lse[h2], e)));
      const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h2][e + 1], c, -row_lane(lse[h2], e + 1)));
      pp[h2][pair] = pack_bf16(p0, p1);
      dsp[h2][pair] = pack_bf16(p0 * (dp[h2][e] - row_lane(delta[h2], e)), p1 * (dp[h2][e + 1] - row_lane(delta[h2], e + 1)));
      // keeps this arithmetic where it is written (between two MFMAs) instead of next to its first use
      asm volatile("" : "+v"(pp[h2][pair]), "+v"(dsp[h2][pair]));
    };
    // Rows that do not exist (ragged end) or that the token rule hides get P = exp(-inf) = 0 and
    // dS = 0.  Bit 16*h2 + e of `hidden` marks element e of half h2 for this lane.
    auto hide = [&](int h2) {
      if (any_hidden) {
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if ((hidden >> (16 * h2 + e)) & 1u) s[h2][e] = -INFINITY;
      }
    };
    constexpr int kAhead = 2;  // in units of one k-step (two fragments) or of one transposed fragment pair
    bf16x8 qfr[2 * T::kSteps], gfr[2 * T::kSteps];
    auto read_qg = [&](int i) {  // i = h2 * kSteps + t
      const int h2 = i / T::kSteps, t = i % T::kSteps;
      qfr[i] = *lds_cast<const bf16x8>(sq + QT::piece(h2 * 32 + lq, 2 * t + g));
      gfr[i] = *lds_cast<const bf16x8>(sg + QT::piece(h2 * 32 + lq, 2 * t + g));
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) read_qg(i);
    __builtin_amdgcn_sched_barrier(0);
    // ---- A: S, dP of half 0
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) {
      read_qg(t + kAhead);  // runs into half 1
      if (t == 0) {
        mfma32_vgpr_first(s[0], qfr[t], kf[t]);
        mfma32_vgpr_first(dp[0], gfr[t], vf[t]);
      } else {
        mfma32_vgpr(s[0], qfr[t], kf[t]);
        mfma32_vgpr(dp[0], gfr[t], vf[t]);
      }
      constexpr int kCopies = 2 * T::kQLoadsPerWave + T::kStatLoads;
#pragma unroll
      for (int j = t * kCopies / T::kSteps; j < (t + 1) * kCopies / T::kSteps; ++j) spread_copy(j);
      __builtin_amdgcn_sched_barrier(0);
    }
    mfma_results_settle(s[0], dp[0]);
    hide(0);
    __builtin_amdgcn_sched_barrier(0);
    // ---- B: S, dP of half 1 | P, dS of half 0
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) {
      if (t + kAhead < T::kSteps) read_qg(T::kSteps + t + kAhead);
      if (t == 0) {
        mfma32_vgpr_first(s[1], qfr[T::kSteps + t], kf[t]);
        mfma32_vgpr_first(dp[1], gfr[T::kSteps + t], vf[t]);
      } else {
        mfma32_vgpr(s[1], qfr[T::kSteps + t], kf[t]);
        mfma32_vgpr(dp[1], gfr[T::kSteps + t], vf[t]);
      }
      softmax_pair(0, t);
      __builtin_amdgcn_sched_barrier(0);
    }
    mfma_results_settle(s[1], dp[1]);
    hide(1);
    // dV^T[d, key] += dO^T[d, q] P[q, key];  dK^T[d, key] += Q^T[d, q] dS[q, key]:
    // fragment pair j = ((h2 * 2 + t2) * kDTiles + dt): transposed reads of dO and Q
    constexpr int kPairs = 2 * 2 * T::kDTiles;
    u32x4 gtr[kPairs], qtr[kPairs];
    auto read_tr = [&](int j) {
      const int h2 = j / (2 * T::kDTiles), t2 = (j / T::kDTiles) % 2, dt = j % T::kDTiles;
      const int r0 = h2 * 32 + 16 * t2 + 4 * g + (i16 >> 2);  // stage row of the first 4-row patch
      const int col = 32 * dt + 16 * half16 + 4 * (i16 & 3);
      const u32x2 g0 = lds_read_tr(sg + QT::elem(r0, col)), g1 = lds_read_tr(sg + QT::elem(r0 + 8, col));
      const u32x2 q0v = lds_read_tr(sq + QT::elem(r0, col)), q1v = lds_read_tr(sq + QT::elem(r0 + 8, col));
      gtr[j] = u32x4{g0[0], g0[1], g1[0], g1[1]};
      qtr[j] = u32x4{q0v[0], q0v[1], q1v[0], q1v[1]};
    };
#pragma unroll
    for (int j = 0; j < kAhead; ++j) read_tr(j);
    __builtin_amdgcn_sched_barrier(0);
    // ---- C: dV, dK with half 0 | P, dS of half 1;   D: dV, dK with half 1
#pragma unroll
    for (int j = 0; j < kPairs; ++j) {
      if (j + kAhead < kPairs) read_tr(j + kAhead);
      const int h2 = j / (2 * T::kDTiles), t2 = (j / T::kDTiles) % 2, dt = j % T::kDTiles;
      const bf16x8 pf = as_bf16x8(pp[h2][4 * t2], pp[h2][4 * t2 + 1], pp[h2][4 * t2 + 2], pp[h2][4 * t2 + 3]);
      const bf16x8 dsf = as_bf16x8(dsp[h2][4 * t2], dsp[h2][4 * t2 + 1], dsp[h2][4 * t2 + 2], dsp[h2][4 * t2 + 3]);
      dv[dt] = mfma32(__builtin_bit_cast(bf16x8, gtr[j]), pf, dv[dt]);
      dk[dt] = mfma32(__builtin_bit_cast(bf16x8, qtr[j]), dsf, dk[dt]);
      if (h2 == 0) {  // the 8 softmax pairs of half 1 spread over the 2 * kDTiles steps of half 0
        const int n0 = j * 8 / (2 * T::kDTiles), n1 = (j + 1) * 8 / (2 * T::kDTiles);
#pragma unroll
        for (int pair = n0; pair < n1; ++pair) softmax_pair(1, pair);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    q0 = q0_next;
  }

  // ---- epilogue: dK = scale * dK^T, dV -----------------------------------------------------
  __bf16* dkd = (__bf16*)a.dk.ptr + (int64_t)b * a.dk.sb + (int64_t)h * a.dk.sh + (int64_t)key_row * a.dk.sn;
  __bf16* dvd = (__bf16*)a.dv.ptr + (int64_t)b * a.dv.sb + (int64_t)h * a.dv.sh + (int64_t)key_row * a.dv.sn;
  if (S > 1) {
    if (T::kWaves > 1)  // a stage is a barrier: as many as group 0, which has most stages
      for (int32_t u = n_stage; u < (n_col + S - 1) / S * T::kSubs; ++u) __syncthreads();
    T::Join::add(dk, lds_all, group, wave, lane, [&](int p, f32x4 v) __attribute__((always_inline)) {
      if (key_ok) *(u32x2*)(dkd + 8 * p + 4 * g) = u32x2{pack_bf16(v[0] * a.scale, v[1] * a.scale), pack_bf16(v[2] * a.scale, v[3] * a.scale)};
    });
    T::Join::add(dv, lds_all, group, wave, lane, [&](int p, f32x4 v) __attribute__((always_inline)) {
      if (key_ok) *(u32x2*)(dvd + 8 * p + 4 * g) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    });
  } else if (key_ok) {
#pragma unroll
    for (int dt = 0; dt < T::kDTiles; ++dt)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const int d0 = 32 * dt + 8 * e4 + 4 * g;
        *(u32x2*)(dkd + d0) = u32x2{pack_bf16(dk[dt][4 * e4] * a.scale, dk[dt][4 * e4 + 1] * a.scale),
                                    pack_bf16(dk[dt][4 * e4 + 2] * a.scale, dk[dt][4 * e4 + 3] * a.scale)};
        *(u32x2*)(dvd + d0) = u32x2{pack_bf16(dv[dt][4 * e4], dv[dt][4 * e4 + 1]),
                                    pack_bf16(dv[dt][4 * e4 + 2], dv[dt][4 * e4 + 3])};
      }
  }
}

template <int D, int BLK, bool kExact>
__global__ void __launch_bounds__(2 * BLK, 1) radial_bwd_dkdv_kernel(const BwdArgs a) {
  dkdv_body<D, BLK, kExact, 1, 1, false>(a, blockIdx.x);
}
template <int D, int BLK, bool kExact, int S, int R>
__global__ void __launch_bounds__(2 * BLK / R * S, 1) radial_bwd_dkdv_split_kernel(const BwdArgs a) {
  dkdv_body<D, BLK, kExact, S, R, false>(a, blockIdx.x);
}

template <int D, int BLK, bool kExact, int S, int R>
__global__ void __launch_bounds__(2 * BLK / R * S, 2) radial_bwd_dkdv_two_kernel(const BwdArgs a) {  // two waves per SIMD
  dkdv_body<D, BLK, kExact, S, R, true>(a, blockIdx.x);
}

// dK/dV of head dimension 128, two waves per SIMD: a pair of waves shares 32 keys.  One wave of each kind has K, S, P and dV, the
// other V, dP, dS and dK, so that either needs little more than half the registers of a wave that does all four products (376 to 384).
// The second wave needs P: the first leaves it in LDS in float32, lane by lane (both products come out in the same
// layout), and the second takes it a stage later, when every P of that stage is behind the barrier anyway:
//   stage u:  first wave   S(u), P(u) -> LDS, dV += P(u)^T dO(u)
//             second wave  dS(u - 1) = P(u - 1) * (dP(u - 1) - delta), dP(u), dK += dS(u - 1)^T Q(u - 1)
// so Q has three stage buffers and dO two, and the vector part of one wave falls on the matrix part of the other.
// Wave w and wave w + kPairs share keys: they are on one SIMD.  200 registers (228 under the token rule; beside dQ in one launch 250
// and 256), and a pair that sees nothing of a stage skips it, which one wave with four products had no registers for.
// The chip lowers its clock for the busier matrix pipes (8 x 126 360 tokens, radial lists: 46 % busy at 2.05 GHz -> 54 % at 1.87), so the large
// launches gain least.  Backward pass, one wave with four products / pairs: 8 x 126 360 tokens 82.5 / 80.3 ms, 5 x 14 040 1728 / 1653 us,
// 5 x 32 760 with the token rule 6284 / 5897, 12 x 3500 398 / 363; equal lists, 4096 blocks L 1 417 / 404, 256 L 32 254 / 242, 320 L 8
// 129 / 119, 1680 L 12 679 / 633, 8 L 1 23.9 / 22.9.  What bounds it is LDS traffic: without the exchange of P (16 of 81 KiB per stage
// and pair) it ran 9 % faster; LSE and delta are read once and broadcast in registers, as 16-byte reads in all lanes they took 16 KiB
// more (256 L 32: 252 us).  Priorities of either wave, fragments read three MFMAs ahead and P read two groups ahead: ties.
template <int D, int BLK>
struct PairTile {
  static constexpr int kPairs = BLK / 32;
  static constexpr int kThreads = 128 * kPairs;
  static constexpr int kSubs = BLK / kStageQ;
  static constexpr int kSteps = D / 16;
  static constexpr int kDTiles = D / 32;
  using Rows = RowsTile<D>;
  static constexpr int kTileBytes = kStageQ / 4 * Rows::kFourRows;  // Q or dO of a stage
  static constexpr int kStatBytes = 2 * kStageQ * 4;  // LSE and delta of a stage
  static constexpr int kPBytes = kStageQ * 32 * 4;    // P of a stage and a pair
  static constexpr int kGradAt = 3 * kTileBytes;      // [Q x 3][dO x 2][LSE, delta x 3][P x 2 x pairs]
  static constexpr int kStatAt = kGradAt + 2 * kTileBytes;
  static constexpr int kPAt = kStatAt + 3 * kStatBytes;
  static constexpr int kLdsBytes = kPAt + 2 * kPairs * kPBytes;
  static constexpr int kLoadsPerWave = kStageQ / 4 / (2 * kPairs);
  static constexpr int kCopies = 2 * kLoadsPerWave + 1;  // Q, dO, and LSE (wave 0) or delta (wave 1)
};

template <int D, int BLK, bool kExact>
__device__ __forceinline__ void pairs_body(const BwdArgs& a, int32_t bh, int32_t kb) {
  using T = PairTile<D, BLK>;
  using Rows = typename T::Rows;
  extern __shared__ __attribute__((aligned(1024))) char lds_all[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool second = wave >= T::kPairs;
  const int pair = second ? wave - T::kPairs : wave;
  const uint32_t lds_base = lds_address(lds_all);
  const int lq = lane & 31;
  const int g = lane >> 5;
  const int i16 = lane & 15;

  const int32_t b = bh / a.H, h = bh % a.H;
  const __bf16* qp = (const __bf16*)a.q.ptr + (int64_t)b * a.q.sb + (int64_t)h * a.q.sh;
  const __bf16* gp = (const __bf16*)a.dout.ptr + (int64_t)b * a.dout.sb + (int64_t)h * a.dout.sh;
  const float* statp = (wave == 0 ? a.lse : a.delta) + (int64_t)bh * a.N;  // what this wave copies of them

  const int32_t list_lo = __builtin_amdgcn_readfirstlane(a.col_ptr[kb]);
  const int32_t n_list = __builtin_amdgcn_readfirstlane(a.col_ptr[kb + 1]) - list_lo;
  const int32_t n_stage = n_list * T::kSubs;
  const int32_t key_row = kb * BLK + pair * 32 + lq;
  const bool key_ok = key_row < a.N;

  bf16x8 kv[T::kSteps];  // K (first wave) or V row of this lane's key: B operands of S = Q K^T or dP = dO V^T
  {
    const TensorArg& src = second ? a.v : a.k;
    const __bf16* row = (const __bf16*)src.ptr + (int64_t)b * src.sb + (int64_t)h * src.sh + (int64_t)(key_ok ? key_row : a.N - 1) * src.sn + 8 * g;
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) {
      u32x4 raw = *(const u32x4*)(row + 16 * t);
      if (!key_ok) raw = u32x4{0u, 0u, 0u, 0u};
      kv[t] = __builtin_bit_cast(bf16x8, raw);
    }
  }

  const int32_t* rows_list = a.row_idx + list_lo;
  int32_t cvec = lane < n_list ? rows_list[lane] : 0;
  int32_t nvec = 64 + lane < n_list ? rows_list[64 + lane] : 0;
  ListRule<kStageQ, BLK> token;
  if (kExact) token.init(a.rule, kb * BLK + pair * 32, a.N, lane);

  uint32_t qoff[T::kLoadsPerWave], goff[T::kLoadsPerWave];  // byte offsets from the stage's first row
#pragma unroll
  for (int i = 0; i < T::kLoadsPerWave; ++i) {
    qoff[i] = (uint32_t)(((wave * T::kLoadsPerWave + i) * 4) * (int32_t)a.q.sn) * 2u + Rows::source_bytes(lane, a.q.sn);
    goff[i] = (uint32_t)(((wave * T::kLoadsPerWave + i) * 4) * (int32_t)a.dout.sn) * 2u + Rows::source_bytes(lane, a.dout.sn);
  }
  // Stage buffers of stage u: Q and the row statistics go round three, dO and P round two.
  struct Bufs {
    int32_t q, grad, stat, p;  // byte offsets
  };
  const auto next_bufs = [](Bufs x) {
    return Bufs{x.q == 2 * T::kTileBytes ? 0 : x.q + T::kTileBytes, 2 * T::kGradAt + T::kTileBytes - x.grad,
                x.stat == T::kStatAt + 2 * T::kStatBytes ? T::kStatAt : x.stat + T::kStatBytes, 2 * T::kPAt + T::kPairs * T::kPBytes - x.p};
  };
  // All of this wave's copies of a stage at once (first stage, ragged stages: rows past N-1 are clamped to N-1).
  auto issue_stage = [&](int32_t q0, const Bufs& to) {
    const uint32_t qdst = lds_base + to.q + wave * T::kLoadsPerWave * Rows::kFourRows, gdst = lds_base + to.grad + wave * T::kLoadsPerWave * Rows::kFourRows;
#pragma unroll
    for (int i = 0; i < T::kLoadsPerWave; ++i) {
      int32_t r = q0 + (wave * T::kLoadsPerWave + i) * 4 + Rows::source_row(lane);
      r = r < a.N ? r : a.N - 1;
      copy16_to_lds(qp + (int64_t)r * a.q.sn + Rows::source_column(lane), qdst + i * Rows::kFourRows);
      copy16_to_lds(gp + (int64_t)r * a.dout.sn + Rows::source_column(lane), gdst + i * Rows::kFourRows);
    }
    if (wave < 2) {
      int32_t r = q0 + lane;
      r = r < a.N ? r : a.N - 1;
      copy4_to_lds(statp + r, lds_base + to.stat + wave * kStageQ * 4);
    }
  };

  f32x16 acc[T::kDTiles];  // dV^T or dK^T: column = this lane's key, rows = d
#pragma unroll
  for (int i = 0; i < T::kDTiles; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
  const float c = a.scale * kLog2e;

  int32_t q0 = 0, q0_next = 0;
  Bufs at = {0, T::kGradAt, T::kStatAt, T::kPAt};
  if (n_stage > 0) {
    q0 = __builtin_amdgcn_readlane(cvec, 0) * BLK;
    issue_stage(q0, at);
  }

  // Where the copies of the next stage go, and whether they are spread over this one's MFMAs.
  Bufs to = at;
  bool spread = false;
  uint64_t copy_lanes = 0;
  const __bf16 *qbase = qp, *gbase = gp;
  bool partial = false, skip = false;  // token rule: some row of the stage does not see some key of this pair; no row sees any
  auto open_stage = [&](int32_t u) __attribute__((always_inline)) {
    const bool has_next = u + 1 < n_stage;
    if (kExact) {
      if ((u & 63) == 0) token.look(a.rule, cvec, u / T::kSubs & 63, lane, false);
      skip = token.sees_none(u);
      partial = !token.sees_all(u);
    }
    to = next_bufs(at);
    if (has_next) {
      const int32_t e1 = (u + 1) / T::kSubs;
      if ((u + 1) % T::kSubs == 0 && (e1 & 63) == 0) {
        cvec = nvec;
        nvec = e1 + 64 + lane < n_list ? rows_list[e1 + 64 + lane] : 0;
      }
      q0_next = __builtin_amdgcn_readlane(cvec, e1 & 63) * BLK + ((u + 1) % T::kSubs) * kStageQ;
    }
    wait_all_copies();  // stage u has landed
    __syncthreads();    // for every wave; stage u-1 is finished and its P written
    spread = has_next && !skip && q0_next + kStageQ <= a.N;
    if (has_next && !spread) issue_stage(q0_next, to);
    const uint32_t on = __builtin_amdgcn_readfirstlane(spread ? ~0u : 0u);
    copy_lanes = ((uint64_t)on << 32) | on;
    const int32_t q_src = spread ? q0_next : q0;  // any valid row when the copies are switched off
    qbase = qp + (int64_t)q_src * a.q.sn;
    gbase = gp + (int64_t)q_src * a.dout.sn;
  };
  auto close_stage = [&]() __attribute__((always_inline)) {
    q0 = q0_next;
    at = to;
  };
  auto spread_copy = [&](int j) __attribute__((always_inline)) {
    int32_t wave_at = wave;
    asm volatile("" : "+s"(wave_at));  // worked out here, not held: scalars are what the common launches are short of
    if (j < T::kLoadsPerWave) {
      copy16_to_lds_sv_masked(qbase, qoff[j], lds_base + to.q + (wave_at * T::kLoadsPerWave + j) * Rows::kFourRows, copy_lanes);
    } else if (j < 2 * T::kLoadsPerWave) {
      const int i = j - T::kLoadsPerWave;
      copy16_to_lds_sv_masked(gbase, goff[i], lds_base + to.grad + (wave_at * T::kLoadsPerWave + i) * Rows::kFourRows, copy_lanes);
    } else {
      copy4_to_lds_sv_masked(statp + (spread ? q0_next : q0), (uint32_t)lane * 4u, lds_base + to.stat + (wave & 1) * kStageQ * 4, wave < 2 ? copy_lanes : 0ull);
    }
  };
  // LDS fragments of both products: step i = 8 * half + k-step of the first, pair j = (2 * half + 16-row step) * kDTiles + d tile of
  // the second, whose A operand is read transposed.
  const uint32_t rows_at = lds_base + Rows::row_at(lane), columns_at = lds_base + Rows::column_at(lane);
  auto read_rows = [&](int32_t tile, int i) __attribute__((always_inline)) -> bf16x8 {
    return *lds_pointer<const bf16x8>(rows_at + tile + Rows::row_step(i / T::kSteps, i % T::kSteps));
  };
  auto read_columns = [&](int32_t tile, int j) __attribute__((always_inline)) -> bf16x8 {
    const uint32_t at = columns_at + tile + Rows::column_step(j / T::kDTiles, j % T::kDTiles);
    const s16x4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_pointer<s16x4>(at));
    const s16x4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_pointer<s16x4>(at + Rows::kEightRows));
    const u32x2 lo = __builtin_bit_cast(u32x2, x0), hi = __builtin_bit_cast(u32x2, x1);
    return as_bf16x8(lo[0], lo[1], hi[0], hi[1]);
  };
  const auto p_at = [&](const Bufs& x, int w) __attribute__((always_inline)) -> char* {  // w = 4 * half + quarter
    return lds_all + x.p + pair * T::kPBytes + w * 1024 + lane * 16;
  };
  // LSE (which = 0) or delta of half h2: element e of the half is this value in lane e of this lane's row of 16.
  const uint32_t stat_at = lds_base + (8 * (i16 >> 2) + 4 * g + (i16 & 3)) * 4;
  const auto read_stat = [&](const Bufs& x, int which, int h2) __attribute__((always_inline)) -> float {
    return *lds_pointer<const float>(stat_at + x.stat + (which * kStageQ + h2 * 32) * 4);
  };
  const auto operand = [](const uint32_t (&w)[16], int j) __attribute__((always_inline)) {
    const int k = j / T::kDTiles * 4;
    return as_bf16x8(w[k], w[k + 1], w[k + 2], w[k + 3]);
  };
  constexpr int kAhead = 2;  // LDS fragments are read this many MFMAs before their use; the fences keep the written order
  constexpr int kFirst = 2 * T::kSteps, kSecond = 4 * T::kDTiles;  // MFMAs of either product
  static_assert(T::kSteps == 8 && T::kDTiles == 4, "the vector work is dealt over 16 + 16 MFMAs");
  auto spread_copies = [&](int i) __attribute__((always_inline)) {
    if (i < T::kSteps) {
#pragma unroll
      for (int j = i * T::kCopies / T::kSteps; j < (i + 1) * T::kCopies / T::kSteps; ++j) spread_copy(j);
    }
  };
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  if (!second) {
    for (int32_t u = 0; u < n_stage; ++u) {
      open_stage(u);
      if (!skip) {
        const int32_t tq = at.q, tg = at.grad;
        uint32_t hidden = 0u;
        if (q0 + kStageQ > a.N || partial) {  // query rows past N, rows the token rule hides from this key
          if (!kExact || q0 + kStageQ > a.N) hidden = ~lane_element_bits(stage_prefix(a.N - q0), g);
          if (kExact && partial) hidden |= token.hidden(u, a.rule.s, g, lane);
        }
        const bool any_hidden = __builtin_amdgcn_ballot_w64(hidden != 0u) != 0;
        f32x16 s[2];
        float lse[2];
        f32x4 p4;
        uint32_t pp[16];
        bf16x8 rows[kFirst], columns[kSecond];
        auto hide = [&](int h2) __attribute__((always_inline)) {
          if (any_hidden) {
#pragma unroll
            for (int e = 0; e < 16; ++e)
              if ((hidden >> (16 * h2 + e)) & 1u) s[h2][e] = -INFINITY;
          }
        };
        // P of elements 2 * k and 2 * k + 1 of the stage's 32
        auto softmax_pair = [&](int k) __attribute__((always_inline)) {
          const int h2 = k / 8, e = 2 * (k % 8);
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h2][e], c, -row_lane(lse[h2], e)));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[h2][e + 1], c, -row_lane(lse[h2], e + 1)));
          p4[e & 3] = p0;
          p4[(e & 3) + 1] = p1;
          pp[k] = pack_bf16(p0, p1);
          asm volatile("" : "+v"(pp[k]));  // stays between its MFMAs
          if (k & 1) *lds_cast<f32x4>(p_at(at, k / 2)) = p4;
        };
#pragma unroll
        for (int i = 0; i < kAhead; ++i) rows[i] = read_rows(tq, i);
        lse[0] = read_stat(at, 0, 0) * kLog2e;
        lse[1] = read_stat(at, 0, 1) * kLog2e;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kFirst; ++i) {
          if (i + kAhead < kFirst) rows[i + kAhead] = read_rows(tq, i + kAhead);
          else columns[i + kAhead - kFirst] = read_columns(tg, i + kAhead - kFirst);
          const int h2 = i / T::kSteps, t = i % T::kSteps;
          s[h2] = mfma32(rows[i], kv[t], t == 0 ? zero : s[h2]);
          spread_copies(i);
          if (h2 == 1) softmax_pair(t);
          __builtin_amdgcn_sched_barrier(0);
          if (t == T::kSteps - 1) hide(h2);
        }
#pragma unroll
        for (int j = 0; j < kSecond; ++j) {
          if (j + kAhead < kSecond) columns[j + kAhead] = read_columns(tg, j + kAhead);
          acc[j % T::kDTiles] = mfma32(columns[j], operand(pp, j), acc[j % T::kDTiles]);
          if (j < 8) softmax_pair(8 + j);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      close_stage();
    }
    if (n_stage > 0) __syncthreads();
  } else {
    f32x16 dp[2] = {zero, zero};
    Bufs last = at;     // of the stage before
    bool owed = false;  // its dS and dK are
    f32x4 p4[8];
    float delta[2];
    uint32_t ds[16];
    auto read_p = [&](int w) __attribute__((always_inline)) {
      if (w == 0) {
        delta[0] = read_stat(last, 1, 0);
        delta[1] = read_stat(last, 1, 1);
      }
      p4[w] = *lds_cast<const f32x4>(p_at(last, w));
    };
    // dS of elements 2 * k and 2 * k + 1 of the stage's 32
    auto weight_pair = [&](int k) __attribute__((always_inline)) {
      const int h2 = k / 8, e = 2 * (k % 8);
      const f32x4 p = p4[k / 2];
      ds[k] = pack_bf16(p[e & 3] * (dp[h2][e] - row_lane(delta[h2], e)), p[(e & 3) + 1] * (dp[h2][e + 1] - row_lane(delta[h2], e + 1)));
      asm volatile("" : "+v"(ds[k]));
    };
    for (int32_t u = 0; u < n_stage; ++u) {
      open_stage(u);
      const int32_t tg = at.grad, tq = last.q;
      bf16x8 rows[kFirst], columns[kSecond];
      if (!kExact || !skip) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) rows[i] = read_rows(tg, i);
        read_p(0);  // of the first stage: not used
        f32x16 next[2];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kFirst; ++i) {
          if (i + kAhead < kFirst) rows[i + kAhead] = read_rows(tg, i + kAhead);
          else columns[i + kAhead - kFirst] = read_columns(tq, i + kAhead - kFirst);
          if (i % 2 == 0 && i / 2 + 1 < 8) read_p(i / 2 + 1);
          const int h2 = i / T::kSteps, t = i % T::kSteps;
          next[h2] = mfma32(rows[i], kv[t], t == 0 ? zero : next[h2]);
          spread_copies(i);
          weight_pair(i);
          __builtin_amdgcn_sched_barrier(0);
        }
        dp[0] = next[0];
        dp[1] = next[1];
      } else if (owed) {
#pragma unroll
        for (int w = 0; w < 8; ++w) read_p(w);
#pragma unroll
        for (int i = 0; i < kFirst; ++i) weight_pair(i);
#pragma unroll
        for (int j = 0; j < kAhead; ++j) columns[j] = read_columns(tq, j);
      }
      if (owed) {
#pragma unroll
        for (int j = 0; j < kSecond; ++j) {
          if (j + kAhead < kSecond) columns[j + kAhead] = read_columns(tq, j + kAhead);
          acc[j % T::kDTiles] = mfma32(columns[j], operand(ds, j), acc[j % T::kDTiles]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      owed = !skip;
      last = at;
      close_stage();
    }
    if (n_stage > 0) __syncthreads();
    if (owed) {
#pragma unroll
      for (int w = 0; w < 8; ++w) read_p(w);
#pragma unroll
      for (int i = 0; i < kFirst; ++i) weight_pair(i);
#pragma unroll
      for (int j = 0; j < kSecond; ++j) acc[j % T::kDTiles] = mfma32(read_columns(last.q, j), operand(ds, j), acc[j % T::kDTiles]);
    }
  }

  if (key_ok) {  // dK = scale * dK^T, dV
    const TensorArg& to_tensor = second ? a.dk : a.dv;
    const float f = second ? a.scale : 1.f;
    __bf16* dst = (__bf16*)to_tensor.ptr + (int64_t)b * to_tensor.sb + (int64_t)h * to_tensor.sh + (int64_t)key_row * to_tensor.sn + 4 * g;
#pragma unroll
    for (int dt = 0; dt < T::kDTiles; ++dt)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)
        *(u32x2*)(dst + 32 * dt + 8 * e4) = u32x2{pack_bf16(acc[dt][4 * e4] * f, acc[dt][4 * e4 + 1] * f),
                                                  pack_bf16(acc[dt][4 * e4 + 2] * f, acc[dt][4 * e4 + 3] * f)};
  }
}

template <int D, int BLK, bool kExact>
__device__ __forceinline__ void pairs_item(const BwdArgs& a, uint32_t id) {
  int32_t bh, kb;
  if (work_item(a.work_t, id, bh, kb)) pairs_body<D, BLK, kExact>(a, bh, kb);
}

// Pairs of waves for two neighbouring key blocks: wave w and wave w + 4 share 32 keys of either.  A query block that both transposed lists name is
// copied once for 256 keys, and every fragment of Q and dO read from LDS feeds two MFMAs: 48 KiB of LDS traffic per 64 MFMAs of a pair, with the
// exchange of P, instead of 81, and half the copies.  Registers (128 of dV or dK, 64 of K or V) leave 32 of scores, so a stage is 32 query rows and
// the second wave does all of its work a stage later:
//   stage u:  first wave   S(u), P(u) -> LDS, dV += P(u)^T dO(u)
//             second wave  dP(u - 1), dS(u - 1) = P(u - 1) * (dP(u - 1) - delta), dK += dS(u - 1)^T Q(u - 1)
// and Q, dO and the row statistics go round three buffers.  The lists are walked in three passes, as in the forward over pairs of query blocks
// (radial_attn_fwd_two.h): entries of both, of the first alone, of the second alone; lists with too little in common are walked one after the other, each
// by the pairs of waves for one block, which also take the last blocks of a launch singly.  All loops are written out for either kind of wave and
// either set of keys: with accumulators that pass a branch or move between registers the compiler spilled 36 to 580 bytes a lane.  255 registers.
// 40 heads x 126 360 tokens, radial lists: 226.6 -> 207.9 ms, the matrix pipes 58 % busy at 1.91 GHz (one block 54 % at 1.87).  Training steps, one
// block / two, us: 3 x 118 800 tokens 40 240 / 39 100, 20 x 32 760 all-ones list 41 600 / 39 900, 10 x 25 600 narrow bands 13 240 / 12 630, 16 x 12 800 4370 / 4212, 400 x 1024 1136 /
// 1104, 800 x 512 997 / 808, 1000 x 256 742 / 463 (heads of few blocks: no workgroups without work); random lists of a quarter of the blocks 9085 / 9134.
struct TwoKeysTile {
  static constexpr int kD = 128, kBlk = 128, kPairs = 4, kStage = 32, kSubs = kBlk / kStage, kSteps = kD / 16, kDTiles = kD / 32;
  using Rows = RowsTile<kD>;
  static constexpr int kTileBytes = kStage / 4 * Rows::kFourRows, kGradAt = 3 * kTileBytes, kStatAt = 6 * kTileBytes;  // [Q x 3][dO x 3]
  static constexpr int kStatBytes = 512;                      // LSE and delta of a stage, 64 floats each
  static constexpr int kPAt = kStatAt + 3 * kStatBytes, kPBytes = 2 * kStage * 32 * 4;  // P of a stage and a pair, [set][4 x 1 KiB]
  static constexpr int kNamedAt = kPAt + 2 * kPairs * kPBytes, kNamedWords = kMaxOrdered / 32;
  static constexpr int kLdsBytes = kNamedAt + 2 * kNamedWords * 4;
};

// Key blocks kb and kb + 1 (which may not exist).  False: their lists have too little in common, and nothing is done.
__device__ __forceinline__ bool two_keys_body(const BwdArgs& a, int32_t bh, int32_t kb, float c) {
  using T = TwoKeysTile;
  using Rows = T::Rows;
  extern __shared__ __attribute__((aligned(1024))) char lds_all[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool second = wave >= T::kPairs;
  const int pair = second ? wave - T::kPairs : wave;
  const uint32_t lds_base = lds_address(lds_all);
  const int lq = lane & 31, g = lane >> 5;
  const int32_t b = bh / a.H, h = bh % a.H;
  const __bf16* qp = (const __bf16*)a.q.ptr + (int64_t)b * a.q.sb + (int64_t)h * a.q.sh;
  const __bf16* gp = (const __bf16*)a.dout.ptr + (int64_t)b * a.dout.sb + (int64_t)h * a.dout.sh;
  const float* statp = (wave == 0 ? a.lse : a.delta) + (int64_t)bh * a.N;  // what this wave copies of them

  const int32_t lo0 = __builtin_amdgcn_readfirstlane(a.col_ptr[kb]), lo1 = __builtin_amdgcn_readfirstlane(a.col_ptr[kb + 1]);
  const int32_t hi1 = kb + 2 <= a.n_blocks ? __builtin_amdgcn_readfirstlane(a.col_ptr[kb + 2]) : lo1;
  const auto named = lds_cast<uint32_t>(lds_all + T::kNamedAt);  // by the first list, by the second
  {
    const int32_t words = (a.n_blocks + 31) >> 5;
    for (int32_t i = threadIdx.x; i < words; i += 512) named[i] = named[T::kNamedWords + i] = 0u;
    __syncthreads();
    for (int32_t i = threadIdx.x; i < hi1 - lo0; i += 512) {
      const int32_t e = a.row_idx[lo0 + i];
      __hip_atomic_fetch_or(&named[(i < lo1 - lo0 ? 0 : T::kNamedWords) + (e >> 5)], 1u << (e & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    // A stage of one list's entry alone has half the MFMAs to a barrier (1.15 of the time that the pairs of waves for one block take for it, a common
    // one 0.86 to 0.97).
    int32_t common = 0;
    for (int32_t i = lane; i < words; i += 64) common += __builtin_popcount(named[i] & named[T::kNamedWords + i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) common += __shfl_xor(common, off);
    if (20 * __builtin_amdgcn_readfirstlane(common) < 7 * (hi1 - lo0)) return false;
  }
  // A walk over the entries of list `w` that the other list names too (shared) or does not.
  int32_t entry = 0;  // this lane's of 64
  uint64_t left = 0;  // which of them are to be visited
  int32_t chunk = 0, w = 0;
  bool shared = true;
  auto take = [&]() __attribute__((always_inline)) -> int32_t {  // the next block, -1: none
    const int32_t list = w ? lo1 : lo0, size = w ? hi1 - lo1 : lo1 - lo0;
    while (left == 0) {
      if (chunk >= size) return -1;
      const int i = chunk + lane_again();
      entry = i < size ? a.row_idx[list + i] : 0;
      const bool in = named[(w ^ 1) * T::kNamedWords + (entry >> 5)] >> (entry & 31) & 1u;
      left = __builtin_amdgcn_ballot_w64(i < size && in == shared);
      chunk += 64;
    }
    const int i = __builtin_ctzll(left);
    left &= left - 1;
    return __builtin_amdgcn_readlane(entry, i);
  };

  bf16x8 kv[2][T::kSteps];  // K (first wave) or V rows of this lane's keys: B operands of S = Q K^T or dP = dO V^T
  {
    const TensorArg& src = second ? a.v : a.k;
#pragma unroll
    for (int set = 0; set < 2; ++set) {
      const int32_t key_row = (kb + set) * T::kBlk + pair * 32 + lq;
      const bool key_ok = key_row < a.N;
      const __bf16* row = (const __bf16*)src.ptr + (int64_t)b * src.sb + (int64_t)h * src.sh + (int64_t)(key_ok ? key_row : a.N - 1) * src.sn + 8 * g;
#pragma unroll
      for (int t = 0; t < T::kSteps; ++t) {
        u32x4 raw = *(const u32x4*)(row + 16 * t);
        if (!key_ok) raw = u32x4{0u, 0u, 0u, 0u};
        kv[set][t] = __builtin_bit_cast(bf16x8, raw);
      }
    }
  }
  f32x16 acc[2][T::kDTiles];  // dV^T or dK^T: column = this lane's key, rows = d
#pragma unroll
  for (int set = 0; set < 2; ++set)
#pragma unroll
    for (int i = 0; i < T::kDTiles; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[set][i][e] = 0.f;

  // A wave copies four rows of Q and of dO, waves 0 and 1 the row statistics as well.
  const uint32_t qoff = Rows::source_bytes(lane, a.q.sn), goff = Rows::source_bytes(lane, a.dout.sn);
  int32_t ring = 0, parity = 0;  // the buffer of three (of Q, dO and the statistics) and of two (of P) that the current stage reads
  auto ring_after = [](int32_t r) { return r == 2 ? 0 : r + 1; };
  auto issue_stage = [&](int32_t q0, int32_t to) __attribute__((always_inline)) {  // at once, rows past N-1 clamped to N-1
    const int lane = lane_again();
    int32_t r = q0 + wave * 4 + Rows::source_row(lane);
    r = r < a.N ? r : a.N - 1;
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_base + to * T::kTileBytes + wave * Rows::kFourRows);
    copy16_to_lds(qp + (int64_t)r * a.q.sn + Rows::source_column(lane), dst);
    copy16_to_lds(gp + (int64_t)r * a.dout.sn + Rows::source_column(lane), dst + T::kGradAt);
    if (wave < 2) {
      int32_t s = q0 + (lane & 31);
      s = s < a.N ? s : a.N - 1;
      copy4_to_lds(statp + s, __builtin_amdgcn_readfirstlane(lds_base + T::kStatAt + to * T::kStatBytes + wave * 256));
    }
  };
  int32_t next_row = 0;     // of the next stage, or any row
  uint64_t copy_lanes = 0;  // all: its copies are spread over this stage's MFMAs
  uint32_t copy_at = 0, stat_copy_at = 0;
  auto spread_copy = [&](int j) __attribute__((always_inline)) {
    if (j == 0) copy16_to_lds_sv_masked(qp + (int64_t)(next_row + wave * 4) * a.q.sn, qoff, copy_at, copy_lanes);
    if (j == 2) copy16_to_lds_sv_masked(gp + (int64_t)(next_row + wave * 4) * a.dout.sn, goff, copy_at + T::kGradAt, copy_lanes);
    if (j == 4) copy4_to_lds_sv_masked(statp + next_row, (uint32_t)(lane_again() & 31) * 4u, stat_copy_at, wave < 2 ? copy_lanes : 0ull);
  };
  const uint32_t rows_at = lds_base + Rows::row_at(lane), columns_at = lds_base + Rows::column_at(lane);
  auto p_at = [&](int32_t p) __attribute__((always_inline)) -> uint32_t {
    return lds_base + T::kPAt + (p * T::kPairs + pair) * T::kPBytes + (uint32_t)lane_again() * 16u;
  };
  auto read_rows = [&](uint32_t at, int t) __attribute__((always_inline)) -> bf16x8 { return *lds_pointer<const bf16x8>(at + Rows::row_step(0, t)); };
  auto read_columns = [&](uint32_t at, int j) __attribute__((always_inline)) -> bf16x8 {  // j = 4 * 16-row step + d tile
    const s16x4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_pointer<s16x4>(at + Rows::column_step(j / 4, j % 4)));
    const s16x4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(lds_pointer<s16x4>(at + Rows::column_step(j / 4, j % 4) + Rows::kEightRows));
    const u32x2 lo = __builtin_bit_cast(u32x2, x0), hi = __builtin_bit_cast(u32x2, x1);
    return as_bf16x8(lo[0], lo[1], hi[0], hi[1]);
  };
  constexpr int kAhead = 2;  // LDS fragments are read this many MFMAs (of one set) before their use; the fences keep the written order
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  // The first product of a stage, S or dP, for kSets sets of keys; the first fragments of the second product are read behind it.
  auto first_product = [&](auto& s, uint32_t rows, bool copies, auto sets_c) __attribute__((always_inline)) {
    constexpr int kSets = decltype(sets_c)::value;  // a bit each
    bf16x8 f[T::kSteps];
#pragma unroll
    for (int t = 0; t < kAhead; ++t) f[t] = read_rows(rows, t);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) {
      if (t + kAhead < T::kSteps) f[t + kAhead] = read_rows(rows, t + kAhead);
#pragma unroll
      for (int set = 0; set < 2; ++set) {
        if (kSets >> set & 1) s[set] = mfma32(f[t], kv[set][t], t == 0 ? zero : s[set]);
        if (set == 0 && copies) spread_copy(t);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // The second product, whose B operands come from elements(set, pair of elements): those of the first 16 rows before it, the others between its MFMAs.
  auto second_product = [&](uint32_t columns, auto sets_c, auto&& elements, uint32_t (&x)[2][8]) __attribute__((always_inline)) {
    constexpr int kSets = decltype(sets_c)::value;  // a bit each
    bf16x8 f[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
      for (int set = 0; set < 2; ++set)
        if (kSets >> set & 1) elements(set, k);
      if (k >= 2) f[k - 2] = read_columns(columns, k - 2);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (j + kAhead < 8) f[j + kAhead] = read_columns(columns, j + kAhead);
      const int t2 = j / 4, dt = j % 4;
#pragma unroll
      for (int set = 0; set < 2; ++set) {
        if (!(kSets >> set & 1)) continue;
        acc[set][dt] = mfma32(f[j], as_bf16x8(x[set][4 * t2], x[set][4 * t2 + 1], x[set][4 * t2 + 2], x[set][4 * t2 + 3]), acc[set][dt]);
        if (j < 4) elements(set, 4 + j);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // LSE (which = 0) or delta of the stage: element e is this value in lane e of this lane's row of 16.
  auto stat = [&](int which, int32_t r) __attribute__((always_inline)) {
    const int l = lane_again();
    return *lds_pointer<const float>(lds_base + T::kStatAt + r * T::kStatBytes + which * 256 + (8 * (l >> 2 & 3) + 4 * (l >> 5) + (l & 3)) * 4);
  };

  // Stage with rows from q0 on in buffer `r`, P in buffer `p`.
  auto do_first = [&](int32_t q0, int32_t r, int32_t p, auto sets_c) __attribute__((always_inline)) {
    constexpr int kSets = decltype(sets_c)::value;  // a bit each
    f32x16 s[2];
    const float lse = stat(0, r) * kLog2e;
    first_product(s, rows_at + r * T::kTileBytes, true, sets_c);
    if (q0 + T::kStage > a.N) {  // query rows past N: P = exp(-inf) = 0
      const uint32_t hidden = elements_from(a.N - q0 - 4 * (lane_again() >> 5));
      float lowest;
      asm volatile("v_mov_b32 %0, 0xff800000" : "=v"(lowest));
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if ((hidden >> e) & 1u) {
#pragma unroll
          for (int set = 0; set < 2; ++set)
            if (kSets >> set & 1) s[set][e] = lowest;
        }
    }
    const uint32_t to = p_at(p);
    uint32_t pp[2][8];
    f32x4 p4[2];
    second_product(columns_at + T::kGradAt + r * T::kTileBytes, sets_c, [&](int set, int k) __attribute__((always_inline)) {
      const int e = 2 * k;
      const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[set][e], c, -row_lane(lse, e)));
      const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[set][e + 1], c, -row_lane(lse, e + 1)));
      p4[set][e & 3] = p0;
      p4[set][(e & 3) + 1] = p1;
      pp[set][k] = pack_bf16(p0, p1);
      asm volatile("" : "+v"(pp[set][k]));  // stays between its MFMAs
      if (k & 1) *lds_pointer<f32x4>(to + (set * 4 + k / 2) * 1024) = p4[set];
    }, pp);
  };
  auto do_second = [&](int32_t r, int32_t p, bool copies, auto sets_c) __attribute__((always_inline)) {
    constexpr int kSets = decltype(sets_c)::value;
    f32x16 dp[2];
    const float delta = stat(1, r);
    first_product(dp, rows_at + T::kGradAt + r * T::kTileBytes, copies, sets_c);
    const uint32_t from = p_at(p);
    uint32_t ds[2][8];
    f32x4 p4[2][2];  // of the current four elements and the next
    auto read_p = [&](int set, int four) __attribute__((always_inline)) {
      p4[set][four & 1] = *lds_pointer<const f32x4>(from + (set * 4 + four) * 1024);
    };
#pragma unroll
    for (int set = 0; set < 2; ++set)
      if (kSets >> set & 1) read_p(set, 0);
    second_product(columns_at + r * T::kTileBytes, sets_c, [&](int set, int k) __attribute__((always_inline)) {
      const int e = 2 * k;
      if (k % 2 == 0 && k / 2 + 1 < 4) read_p(set, k / 2 + 1);
      const f32x4 p = p4[set][k / 2 & 1];
      ds[set][k] = pack_bf16(p[e & 3] * (dp[set][e] - row_lane(delta, e)), p[(e & 3) + 1] * (dp[set][e + 1] - row_lane(delta, e + 1)));
      asm volatile("" : "+v"(ds[set][k]));
    }, ds);
  };

  // One pass over the lists, of either kind of wave: loops of their own, which branch nowhere that the accumulators pass.
  auto walk = [&](auto second_c, auto sets_c) __attribute__((always_inline)) {
    constexpr bool kSecond = decltype(second_c)::value;
    left = 0;
    chunk = 0;
    int32_t block = take();
    if (block < 0) return;
    int32_t q0 = block * T::kBlk, q0_next = 0, last_ring = 0, to = 0, u = 0;
    bool has_next = true;
    issue_stage(q0, ring);
    auto open_stage = [&]() __attribute__((always_inline)) {
      q0_next = q0 + T::kStage;
      if (u == T::kSubs - 1) {
        block = take();
        has_next = block >= 0;
        q0_next = block * T::kBlk;
      }
      to = ring_after(ring);
      wait_all_copies();
      __syncthreads();  // this stage's copies have landed for every wave, the last one's P is written and the one before it is consumed
      const bool spread = has_next && q0_next + T::kStage <= a.N;
      if (has_next && !spread) issue_stage(q0_next, to);
      const uint32_t on = __builtin_amdgcn_readfirstlane(spread ? ~0u : 0u);
      copy_lanes = ((uint64_t)on << 32) | on;
      next_row = spread ? q0_next : q0;
      copy_at = __builtin_amdgcn_readfirstlane(lds_base + to * T::kTileBytes + wave * Rows::kFourRows);
      stat_copy_at = __builtin_amdgcn_readfirstlane(lds_base + T::kStatAt + to * T::kStatBytes + (wave & 1) * 256);
    };
    auto close_stage = [&]() __attribute__((always_inline)) {
      last_ring = ring;
      ring = to;
      parity ^= 1;
      q0 = q0_next;
      u = (u + 1) & (T::kSubs - 1);
    };
    if constexpr (kSecond) {  // nothing to do yet but its copies
      open_stage();
#pragma unroll
      for (int j = 0; j < 8; ++j) spread_copy(j);
      close_stage();
    }
    while (has_next) {
      open_stage();
      if constexpr (kSecond) do_second(last_ring, parity ^ 1, true, sets_c);
      else do_first(q0, ring, parity, sets_c);
      close_stage();
    }
    __syncthreads();
    if constexpr (kSecond) do_second(last_ring, parity ^ 1, false, sets_c);
  };
  auto run = [&](auto second_c) __attribute__((always_inline)) {
    constexpr bool kSecond = decltype(second_c)::value;
    walk(second_c, std::integral_constant<int, 3>{});
    shared = false;
    auto finish = [&](auto set_c) __attribute__((always_inline)) {
      constexpr int set = decltype(set_c)::value;
      w = set;
      walk(second_c, std::integral_constant<int, 1 << set>{});
      const int lane2 = lane_again(), g2 = lane2 >> 5;
      const int32_t key_row = (kb + set) * T::kBlk + pair * 32 + (lane2 & 31);
      if (key_row < a.N) {  // dK = scale * dK^T, dV
        const TensorArg& to_tensor = kSecond ? a.dk : a.dv;
        const float f = kSecond ? a.scale : 1.f;
        __bf16* dst = (__bf16*)to_tensor.ptr + (int64_t)b * to_tensor.sb + (int64_t)h * to_tensor.sh + (int64_t)key_row * to_tensor.sn + 4 * g2;
#pragma unroll
        for (int dt = 0; dt < T::kDTiles; ++dt)
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4)
            *(u32x2*)(dst + 32 * dt + 8 * e4) = u32x2{pack_bf16(acc[set][dt][4 * e4] * f, acc[set][dt][4 * e4 + 1] * f),
                                                      pack_bf16(acc[set][dt][4 * e4 + 2] * f, acc[set][dt][4 * e4 + 3] * f)};
      }
    };
    finish(std::integral_constant<int, 0>{});
    finish(std::integral_constant<int, 1>{});
  };
  if (second) run(std::true_type{});
  else run(std::false_type{});
  return true;
}

__global__ void __launch_bounds__(512, 2) radial_bwd_two_keys_kernel(const BwdArgs a, const TwoMap m) {
  TwoItem item;
  if (!two_item(a.work_t, m, blockIdx.x, item)) return;
  int32_t kb = 2 * item.pair + item.block, n = 1;
  if (item.form == TwoItem::kPair) {
    if (two_keys_body(own_args<BwdArgs>(), item.bh, kb, m.c)) return;
    n = kb + 1 < a.n_blocks ? 2 : 1;
  }
#pragma unroll 1
  for (; n > 0; --n, ++kb) {
    if (item.form == TwoItem::kPair) __syncthreads();  // the LDS is consumed
    pairs_body<128, 128, false>(own_args<BwdArgs>(), item.bh, kb);
  }
}

// kBeside: in a launch with whole blocks of one group at head dimension 64, whose LDS two groups share on half-size stages.
template <int D, int BLK, int S, int R, bool kBeside = false>
struct DqTile {
  static constexpr int kRows = BLK / R;
  // Keys per stage of the dQ kernel.  Head dimension 128 with 64 rows walks half-size stages:
  // two 64-key stage buffers (64 KiB) per 2 waves would leave a compute unit with 4 waves.
  static constexpr int kStageKeys = (D == 128 && kRows == 64) || kRows == 32 || kBeside ? 32 : 64;
  static constexpr int kWaves = kRows / 32;  // one wave per 32 query rows
  static constexpr int kThreads = 64 * kWaves * S;
  static constexpr int kSubs = BLK / kStageKeys;
  static constexpr int kSteps = D / 16;
  static constexpr int kDTiles = D / 32;
  static constexpr int kTileBytes = kStageKeys * D * 2;  // one K (or V) stage tile
  static constexpr int kLoadsPerWave = kTileBytes / 1024 / kWaves;
  static constexpr int kGroupBytes = 4 * kTileBytes;     // [stage buffer][K, V]
  using Join = Merge<S, kWaves, kDTiles, kBeside ? S * kGroupBytes : 160 * 1024>;
  static constexpr int kLdsBytes = S * kGroupBytes > Join::kLdsBytes ? S * kGroupBytes : Join::kLdsBytes;
};

// Part `part` of the R of query block qb.
template <int D, int BLK, bool kExact, int S, int R, bool kBeside = false>
__device__ __forceinline__ void dq_body(const BwdArgs& a, int32_t bh, int32_t qb, int32_t part) {
  using T = DqTile<D, BLK, S, R, kBeside>;
  using SW = SwzTile<D>;
  // [group][stage buffer][K, V][kStageKeys x D bf16]; one group's are a static array, as in the forward
  __shared__ __attribute__((aligned(1024))) char lds_one[S == 1 ? T::kLdsBytes : 16];
  extern __shared__ __attribute__((aligned(1024))) char lds_all[];

  const int lane = threadIdx.x & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = S == 1 ? 0 : wave_all / T::kWaves;
  const int wave = S == 1 ? wave_all : wave_all % T::kWaves;
  const auto lds_at = [&](int32_t offset) __attribute__((always_inline)) -> const char* {
    if constexpr (S == 1) return lds_one + offset;
    else return lds_all + group * T::kGroupBytes + offset;
  };
  const uint32_t lds_base = lds_address(lds_at(0));
  const int lq = lane & 31;
  const int g = lane >> 5;
  const int i16 = lane & 15;
  const int half16 = (lane >> 4) & 1;

  const int32_t b = bh / a.H, h = bh % a.H;

  const __bf16* qp = (const __bf16*)a.q.ptr + (int64_t)b * a.q.sb + (int64_t)h * a.q.sh;
  const __bf16* kp = (const __bf16*)a.k.ptr + (int64_t)b * a.k.sb + (int64_t)h * a.k.sh;
  const __bf16* vp = (const __bf16*)a.v.ptr + (int64_t)b * a.v.sb + (int64_t)h * a.v.sh;
  const __bf16* gp = (const __bf16*)a.dout.ptr + (int64_t)b * a.dout.sb + (int64_t)h * a.dout.sh;

  const int32_t list_lo = __builtin_amdgcn_readfirstlane(a.row_ptr[qb]);
  const int32_t n_row = __builtin_amdgcn_readfirstlane(a.row_ptr[qb + 1]) - list_lo;
  const int32_t n_list = S == 1 ? n_row : (n_row - group + S - 1) / S;  // entries of this group
  const int32_t n_stage = n_list * T::kSubs;
  const int32_t q_row = qb * BLK + part * T::kRows + wave * 32 + lq;
  const bool q_ok = q_row < a.N;
  const int64_t q_clamped = q_ok ? q_row : a.N - 1;

  // Q and dO rows of this lane's query: B operands of S^T = K Q^T and dP^T = V dO^T.
  bf16x8 qf[T::kSteps], gf[T::kSteps];
  {
    const __bf16* qs = qp + q_clamped * a.q.sn + 8 * g;
    const __bf16* gs = gp + q_clamped * a.dout.sn + 8 * g;
#pragma unroll
    for (int t = 0; t < T::kSteps; ++t) {
      qf[t] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qs + 16 * t));
      gf[t] = __builtin_bit_cast(bf16x8, *(const u32x4*)(gs + 16 * t));
    }
  }
  const float lse2 = a.lse[(int64_t)bh * a.N + q_clamped] * kLog2e;  // rows past N: values unused
  const float dlt = a.delta[(int64_t)bh * a.N + q_clamped];

  const int32_t* cols = a.col_idx + list_lo + group;
  int32_t cvec = lane < n_list ? cols[S * lane] : 0;
  int32_t nvec = 64 + lane < n_list ? cols[S * (64 + lane)] : 0;
  ListRule<T::kStageKeys, BLK> token;
  if (kExact) token.init(a.rule, qb * BLK + part * T::kRows + wave * 32, a.N, lane);

  uint32_t koff[T::kLoadsPerWave], voff[T::kLoadsPerWave];
#pragma unroll
  for (int i = 0; i < T::kLoadsPerWave; ++i) {
    int r, col;
    SW::source_of((wave * T::kLoadsPerWave + i) * 64 + lane, r, col);
    koff[i] = (uint32_t)(r * (int32_t)a.k.sn + col) * 2u;
    voff[i] = (uint32_t)(r * (int32_t)a.v.sn + col) * 2u;
  }
  // Copies the 64 K rows and V rows starting at key `key0` into stage buffer `buf`; rows past
  // N-1 are clamped to N-1 (their P is forced to zero).
  auto issue_stage = [&](int32_t key0, int buf) {
    const uint32_t kdst = lds_base + buf * 2 * T::kTileBytes + wave * T::kLoadsPerWave * 1024;
    const uint32_t vdst = kdst + T::kTileBytes;
    if (key0 + T::kStageKeys <= a.N) {
      const __bf16* kbase = kp + (int64_t)key0 * a.k.sn;  // wave-uniform
      const __bf16* vbase = vp + (int64_t)key0 * a.v.sn;
#pragma unroll
      for (int i = 0; i < T::kLoadsPerWave; ++i) copy16_to_lds_sv(kbase, koff[i], kdst + i * 1024);
#pragma unroll
      for (int i = 0; i < T::kLoadsPerWave; ++i) copy16_to_lds_sv(vbase, voff[i], vdst + i * 1024);
    } else {
      const int32_t last = a.N - 1 - key0;  // a stage wholly past N reads row N-1 only
#pragma unroll
      for (int i = 0; i < T::kLoadsPerWave; ++i) {
        int r, col;
        SW::source_of((wave * T::kLoadsPerWave + i) * 64 + lane, r, col);
        r = r < last ? r : last;
        copy16_to_lds(kp + ((int64_t)key0 + r) * a.k.sn + col, kdst + i * 1024);
        copy16_to_lds(vp + ((int64_t)key0 + r) * a.v.sn + col, vdst + i * 1024);
      }
    }
  };

  f32x16 dq[T::kDTiles];  // dQ^T: column = this lane's query, rows = d
#pragma unroll
  for (int i = 0; i < T::kDTiles; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) dq[i][e] = 0.f;
  const float c = a.scale * kLog2e;

  int32_t key0 = 0;
  if (n_stage > 0) {
    key0 = __builtin_amdgcn_readlane(cvec, 0) * BLK;
    issue_stage(key0, 0);
  }
  for (int32_t u = 0; u < n_stage; ++u) {
    const int buf = u & 1;
    if (kExact && (u & 63) == 0) token.look(a.rule, cvec, u / T::kSubs & 63, lane, true);
    const bool skip = kExact && token.sees_none(u);  // no pair of this wave's queries with the stage's keys
    const bool partial = kExact && !token.sees_all(u);
    int32_t key0_next = 0;
    const bool has_next = u + 1 < n_stage;
    if (has_next) {
      const int32_t e1 = (u + 1) / T::kSubs;
      if ((u + 1) % T::kSubs == 0 && (e1 & 63) == 0) {
        cvec = nvec;
        nvec = e1 + 64 + lane < n_list ? cols[S * (e1 + 64 + lane)] : 0;
      }
      key0_next = __builtin_amdgcn_readlane(cvec, e1 & 63) * BLK + ((u + 1) % T::kSubs) * T::kStageKeys;
    }
    if (T::kWaves == 1) {  // nobody else reads or writes this group's stage buffers
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    } else {
      wait_all_copies();
      __syncthreads();
    }

    const char* lds_k = lds_at(buf * 2 * T::kTileBytes);
    const char* lds_v = lds_k + T::kTileBytes;
    const bool ragged = key0 + T::kStageKeys > a.N;
    // The copies of a full next stage are spread over the MFMAs of the first key tile (a burst
    // would hold the wave at the memory pipeline); a ragged next stage, or a stage this wave
    // skips, issues them at once.
    uint32_t hidden = 0u;  // bit 16kt + e: element e of key tile kt is past N or hidden by the token rule
    if (ragged || partial) {
      if (!kExact || ragged) hidden = ~lane_element_bits(stage_prefix(a.N - key0), g);
      if (kExact && partial) hidden |= token.hidden(u, a.rule.s, g, lane);
    }
    const bool any_hidden = __builtin_amdgcn_ballot_w64(hidden != 0u) != 0;
    const bool spread = has_next && !skip && key0_next + T::kStageKeys <= a.N;
    if (has_next && !spread) issue_stage(key0_next, buf ^ 1);
    if (skip) {
      key0 = key0_next;
      continue;
    }
    const uint32_t on = __builtin_amdgcn_readfirstlane(spread ? ~0u : 0u);
    const uint64_t copy_lanes = ((uint64_t)on << 32) | on;
    const int32_t key_src = spread ? key0_next : key0;  // any valid rows when the copies are switched off
    const __bf16* kbase_next = kp + (int64_t)key_src * a.k.sn;
    const __bf16* vbase_next = vp + (int64_t)key_src * a.v.sn;
    const uint32_t kdst_next = lds_base + (buf ^ 1) * 2 * T::kTileBytes + wave * T::kLoadsPerWave * 1024;
    const uint32_t vdst_next = kdst_next + T::kTileBytes;
#pragma unroll
    for (int kt = 0; kt < T::kStageKeys / 32; ++kt) {
      // S^T[key, q] and dP^T[key, q] for 32 keys x this wave's 32 queries
      f32x16 s, dp;
#pragma unroll
      for (int e = 0; e < 16; ++e) s[e] = dp[e] = 0.f;
#pragma unroll
      for (int t = 0; t < T::kSteps; ++t) {
        const bf16x8 kfrag = *lds_cast<const bf16x8>(lds_k + SW::piece(kt * 32 + lq, 2 * t + g));
        const bf16x8 vfrag = *lds_cast<const bf16x8>(lds_v + SW::piece(kt * 32 + lq, 2 * t + g));
        s = mfma32(kfrag, qf[t], s);
        dp = mfma32(vfrag, gf[t], dp);
        if (kt == 0) {  // 2 * kLoadsPerWave copies over the kSteps steps of the first key tile
          constexpr int kCopies = 2 * T::kLoadsPerWave;
#pragma unroll
          for (int j = t * kCopies / T::kSteps; j < (t + 1) * kCopies / T::kSteps; ++j) {
            if (j < T::kLoadsPerWave) copy16_to_lds_sv_masked(kbase_next, koff[j], kdst_next + j * 1024, copy_lanes);
            else copy16_to_lds_sv_masked(vbase_next, voff[j - T::kLoadsPerWave], vdst_next + (j - T::kLoadsPerWave) * 1024, copy_lanes);
          }
        }
      }
      // element e: key = key0 + 32kt + 8(e/4) + 4g + e%4, query = q_row (this lane)
      if (any_hidden) {  // hidden pairs: P = exp(-inf) = 0
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if ((hidden >> (16 * kt + e)) & 1u) s[e] = -INFINITY;
      }
      uint32_t dsp[8];
#pragma unroll
      for (int e = 0; e < 16; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], c, -lse2));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e + 1], c, -lse2));
        dsp[e >> 1] = pack_bf16(p0 * (dp[e] - dlt), p1 * (dp[e + 1] - dlt));
      }
      // dQ^T[d, q] += K^T[d, key] dS^T[key, q]
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2) {
        const bf16x8 dsf = as_bf16x8(dsp[4 * t2], dsp[4 * t2 + 1], dsp[4 * t2 + 2], dsp[4 * t2 + 3]);
        const int r0 = kt * 32 + 16 * t2 + 4 * g + (i16 >> 2);
#pragma unroll
        for (int dt = 0; dt < T::kDTiles; ++dt) {
          const int col = 32 * dt + 16 * half16 + 4 * (i16 & 3);
          const u32x2 k0 = lds_read_tr(lds_k + SW::elem(r0, col)), k1 = lds_read_tr(lds_k + SW::elem(r0 + 8, col));
          dq[dt] = mfma32(as_bf16x8(k0[0], k0[1], k1[0], k1[1]), dsf, dq[dt]);
        }
      }
    }
    key0 = key0_next;
  }

  __bf16* dst = (__bf16*)a.dq.ptr + (int64_t)b * a.dq.sb + (int64_t)h * a.dq.sh + (int64_t)q_row * a.dq.sn;
  if (S > 1) {
    if (T::kWaves > 1)  // a stage is a barrier: as many as group 0, which has most stages
      for (int32_t u = n_stage; u < (n_row + S - 1) / S * T::kSubs; ++u) __syncthreads();
    T::Join::add(dq, lds_all, group, wave, lane, [&](int p, f32x4 v) __attribute__((always_inline)) {
      if (q_ok) *(u32x2*)(dst + 8 * p + 4 * g) = u32x2{pack_bf16(v[0] * a.scale, v[1] * a.scale), pack_bf16(v[2] * a.scale, v[3] * a.scale)};
    });
  } else if (q_ok) {
#pragma unroll
    for (int dt = 0; dt < T::kDTiles; ++dt)
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4)  // dq[dt][4*e4 + x] is d = 32dt + 8*e4 + 4g + x
        *(u32x2*)(dst + 32 * dt + 8 * e4 + 4 * g) =
            u32x2{pack_bf16(dq[dt][4 * e4] * a.scale, dq[dt][4 * e4 + 1] * a.scale),
                  pack_bf16(dq[dt][4 * e4 + 2] * a.scale, dq[dt][4 * e4 + 3] * a.scale)};
  }
}

// Work item `id`; with R > 1 the work map counts R heads for each.
template <int D, int BLK, bool kExact, int S, int R>
__device__ __forceinline__ void dq_item(const BwdArgs& a, uint32_t id) {
  int32_t bh, qb;
  if (!work_item(a.work, id, bh, qb)) return;
  const int32_t part = R == 1 ? 0 : bh % R;
  if (R > 1) bh /= R;
  dq_body<D, BLK, kExact, S, R>(a, bh, qb, part);
}
template <int D, int BLK, bool kExact, int S, int R>
__global__ void __launch_bounds__(2 * BLK / R * S, 2) radial_bwd_dq_kernel(const BwdArgs a) {
  dq_item<D, BLK, kExact, S, R>(a, blockIdx.x);
}

// The kernel's BwdArgs (its first parameter), for one part of a kernel that has several.  Through one name the compiler loads what the parts have in
// common before they branch and keeps it: under the token rule up to 100 scalars in vector lanes, a part of them reloaded in every stage, and
// with halves of whole blocks on two groups 68 bytes of private memory per lane that nothing uses.  kOwn: asked for part by part, there are none of
// either (7 scalars in pairs of waves under the token rule, as where dK/dV is a launch of its own).  Elsewhere loads before the branch are the better
// ones.  Training step, us, shared / own: token rule, D 64, block 64, 8 frames of 333 tokens, 4 heads 71.3 / 69.2, 24 x 316, 8 heads 538 / 520, block
// 128, 9 x 310, 3 heads 76.5 / 72.8, 40 x 800, 4 heads 2757 / 2725, D 128, 6 x 427, 2 heads 110.8 / 109.1, 21 x 620, 3 heads 904 / 877; block-dense, halves of
// whole blocks on two groups, 8 x 333, 4 heads 57.7 / 57.6, D 128, 9 x 613, 3 heads 251.5 / 250.8.  Not taken: groups of one wave, 5 x 256, 1 head, token rule
// 26.36 / 26.55, block-dense 22.67 / 22.88; halves of half blocks, 9 x 310 57.7 / 58.1; one group, 20 x 410, 5 heads 446 / 451.
template <bool kOwn>
__device__ __forceinline__ const BwdArgs& part_args(const BwdArgs& a) {
  if constexpr (!kOwn) return a;
  using Args = const BwdArgs __attribute__((address_space(4)));
  Args* args = (Args*)__builtin_amdgcn_kernarg_segment_ptr();
  asm("" : "+s"(args));  // not known to be the same memory
  return *(const BwdArgs*)args;
}

// The query blocks of a common launch, workgroup `id` of n: by S groups of waves in R parts each; the last a.work.halved of those parts in
// two halves, of half the rows and twice the groups.
template <int D, int BLK, bool kExact, int S, int R>
__device__ __forceinline__ void dq_item_or_half(const BwdArgs& a, uint32_t id, uint32_t n) {
  const uint32_t whole = n - 2u * (uint32_t)a.work.halved;
  if (id < whole) {
    dq_item<D, BLK, kExact, S, R>(part_args<kExact || S * R == 2>(a), id);
    return;
  }
  const BwdArgs& b = part_args<kExact || S * R == 2>(a);
  int32_t bh, qb, half = 0;
  if (!work_item(b.work, halved_item(id, whole, (uint32_t)b.work.halved, half), bh, qb)) return;
  const int32_t part = R == 1 ? half : 2 * (bh % R) + half;
  dq_body<D, BLK, kExact, 2 * S, 2 * R, S == 1>(b, R == 1 ? bh : bh / R, qb, part);
}

// dK/dV and dQ in one launch (see both_groups): the first n_key workgroups take key blocks, the others query blocks; kHalves: the last
// of them in halves.
template <int D, int BLK, bool kExact, int S, int R, bool kHalves>
__global__ void __launch_bounds__(2 * BLK / R * S, 2) radial_bwd_both_kernel(const BwdArgs a, uint32_t n_key) {
  if (blockIdx.x < n_key) dkdv_body<D, BLK, kExact, S, R, true>(a, blockIdx.x);
  else if constexpr (kHalves) dq_item_or_half<D, BLK, kExact, S, R>(a, blockIdx.x - n_key, gridDim.x - n_key);
  else dq_item<D, BLK, kExact, S, R>(part_args<kExact && S < 4>(a), blockIdx.x - n_key);
}

template <int D, int BLK, bool kExact>
__global__ void __launch_bounds__(4 * BLK, 2) radial_bwd_dkdv_pairs_kernel(const BwdArgs a) {
  pairs_item<D, BLK, kExact>(a, blockIdx.x);
}
// The same at head dimension 128, blocks of 128: dK/dV in pairs of waves, dQ by two groups; kHalves: the last a.work.halved query blocks in
// two halves, of 64 rows and four groups each.
template <int D, int BLK, bool kExact, bool kHalves>
__global__ void __launch_bounds__(4 * BLK, 2) radial_bwd_both_pairs_kernel(const BwdArgs a, uint32_t n_key) {
  if (blockIdx.x < n_key) {
    pairs_item<D, BLK, kExact>(a, blockIdx.x);
    return;
  }
  if constexpr (kHalves) dq_item_or_half<D, BLK, kExact, 2, 1>(a, blockIdx.x - n_key, gridDim.x - n_key);
  else dq_item<D, BLK, kExact, 2, 1>(part_args<kExact>(a), blockIdx.x - n_key);
}
// With the hand-made schedule, one wave per SIMD: two groups of 64 rows each.
template <int D, int BLK, bool kExact>
__global__ void __launch_bounds__(256, 1) radial_bwd_both_hand_kernel(const BwdArgs a, uint32_t n_key) {
  if (blockIdx.x < n_key) dkdv_body<D, BLK, kExact, 2, BLK / 64, false>(a, blockIdx.x);
  else dq_item<D, BLK, kExact, 2, BLK / 64>(part_args<kExact>(a), blockIdx.x - n_key);
}

template <int D, int BLK, bool kExact, int S, int R, bool kTwoWaves = false>
int launch_dkdv(BwdArgs a, hipStream_t stream) {
  using T = BwdTile<D, BLK, S, R>;
  void (*kernel)(BwdArgs);
  if constexpr (kTwoWaves) kernel = radial_bwd_dkdv_two_kernel<D, BLK, kExact, S, R>;
  else if constexpr (S == 1) kernel = radial_bwd_dkdv_kernel<D, BLK, kExact>;
  else kernel = radial_bwd_dkdv_split_kernel<D, BLK, kExact, S, R>;
  static DeviceOnce configured;
  if (int rc = allow_dynamic_lds(configured, (const void*)kernel, T::kLdsBytes)) return rc;
  a.work_t.ordered *= R;  // R > 1 only up to kOneRound items, where all heads are taken by list length
  kernel<<<dim3((unsigned)work_grid(a.work_t, a.n_blocks)), dim3(T::kThreads), T::kLdsBytes, stream>>>(a);
  return RADIAL_OK;
}

int launch_dkdv_two(const BwdArgs& a, hipStream_t stream) {
  const TwoMap m = make_two_map(a.work_t, a.pair_order_t, a.scale, TwoWalk::kKeyGrad);
  constexpr int kBytes = TwoKeysTile::kLdsBytes > PairTile<128, 128>::kLdsBytes ? TwoKeysTile::kLdsBytes : PairTile<128, 128>::kLdsBytes;
  static DeviceOnce configured;
  if (int rc = allow_dynamic_lds(configured, (const void*)radial_bwd_two_keys_kernel, kBytes)) return rc;
  radial_bwd_two_keys_kernel<<<dim3(m.n_two + 2 * m.n_one), dim3(512), kBytes, stream>>>(a, m);
  return RADIAL_OK;
}

template <int BLK, bool kExact>
int launch_dkdv_pairs(const BwdArgs& a, hipStream_t stream) {
  if constexpr (BLK == 128 && !kExact)
    if (takes_key_pairs(a.work_t)) return launch_dkdv_two(a, stream);
  using T = PairTile<128, BLK>;
  const auto kernel = radial_bwd_dkdv_pairs_kernel<128, BLK, kExact>;
  static DeviceOnce configured;
  if (int rc = allow_dynamic_lds(configured, (const void*)kernel, T::kLdsBytes)) return rc;
  kernel<<<dim3((unsigned)work_grid(a.work_t, a.n_blocks)), dim3(T::kThreads), T::kLdsBytes, stream>>>(a);
  return RADIAL_OK;
}

template <int D, int BLK, bool kExact, int S, int R>
int launch_dq(BwdArgs a, hipStream_t stream) {
  using T = DqTile<D, BLK, S, R>;
  const auto kernel = radial_bwd_dq_kernel<D, BLK, kExact, S, R>;
  if (S > 1 && T::kLdsBytes > 65536) {
    static DeviceOnce configured;
    if (int rc = allow_dynamic_lds(configured, (const void*)kernel, T::kLdsBytes)) return rc;
  }
  a.work.ordered *= R;
  kernel<<<dim3((unsigned)work_grid(a.work, a.n_blocks)), dim3(T::kThreads), S == 1 ? 0 : T::kLdsBytes, stream>>>(a);
  return RADIAL_OK;
}

template <int BLK, bool kExact, int S, int R, bool kHalves = false>
int launch_both(BwdArgs a, hipStream_t stream) {
  constexpr int kKeyBytes = BwdTile<64, BLK, S, R>::kLdsBytes, kQueryBytes = DqTile<64, BLK, S, R>::kLdsBytes;
  constexpr int kStatic = S == 1 ? kQueryBytes : 0;  // one group's stage buffers in dQ
  constexpr int kBytes = S == 1 || kKeyBytes > kQueryBytes ? kKeyBytes : kQueryBytes;
  static_assert((S == 4 ? 1 : 2) * (kStatic + kBytes) <= 160 * 1024, "two workgroups per compute unit; groups of one wave have it to themselves");
  if constexpr (kHalves) {
    constexpr int kHalfBytes = DqTile<64, BLK, 2 * S, 2 * R, S == 1>::kLdsBytes;
    static_assert(kHalfBytes <= kBytes);
  }
  const auto kernel = radial_bwd_both_kernel<64, BLK, kExact, S, R, kHalves>;
  static DeviceOnce configured;
  if (int rc = allow_dynamic_lds(configured, (const void*)kernel, kBytes)) return rc;
  a.work.ordered *= R;  // at most kOneRound items, where all heads are taken by list length
  a.work_t.ordered *= R;
  const uint32_t n_key = (uint32_t)work_grid(a.work_t, a.n_blocks);
  kernel<<<dim3(n_key + (unsigned)(work_grid(a.work, a.n_blocks) + a.work.halved)), dim3(2 * BLK / R * S), kBytes, stream>>>(a, n_key);
  RADIAL_HIP_TRY(hipGetLastError());
  return RADIAL_OK;
}

template <bool kExact, bool kHalves>
int launch_both_pairs(const BwdArgs& a, hipStream_t stream) {
  constexpr int kKeyBytes = PairTile<128, 128>::kLdsBytes, kQueryBytes = DqTile<128, 128, 2, 1>::kLdsBytes;
  constexpr int kBytes = kKeyBytes > kQueryBytes ? kKeyBytes : kQueryBytes;
  static_assert(!kHalves || DqTile<128, 128, 4, 2>::kLdsBytes <= kBytes);
  const auto kernel = radial_bwd_both_pairs_kernel<128, 128, kExact, kHalves>;
  static DeviceOnce configured;
  if (int rc = allow_dynamic_lds(configured, (const void*)kernel, kBytes)) return rc;
  const uint32_t n_key = (uint32_t)work_grid(a.work_t, a.n_blocks);
  kernel<<<dim3(n_key + (unsigned)(work_grid(a.work, a.n_blocks) + a.work.halved)), dim3(512), kBytes, stream>>>(a, n_key);
  RADIAL_HIP_TRY(hipGetLastError());
  return RADIAL_OK;
}
template <int BLK, bool kExact>
int launch_both_hand(BwdArgs a, hipStream_t stream) {
  constexpr int kKeyBytes = BwdTile<128, BLK, 2, BLK / 64>::kLdsBytes, kQueryBytes = DqTile<128, BLK, 2, BLK / 64>::kLdsBytes;
  constexpr int kBytes = kKeyBytes > kQueryBytes ? kKeyBytes : kQueryBytes;
  const auto kernel = radial_bwd_both_hand_kernel<128, BLK, kExact>;
  static DeviceOnce configured;
  if (int rc = allow_dynamic_lds(configured, (const void*)kernel, kBytes)) return rc;
  a.work.ordered *= BLK / 64;  // at most kOneRound items, where all heads are taken by list length
  a.work_t.ordered *= BLK / 64;
  const uint32_t n_key = (uint32_t)work_grid(a.work_t, a.n_blocks);
  kernel<<<dim3(n_key + (unsigned)work_grid(a.work, a.n_blocks)), dim3(256), kBytes, stream>>>(a, n_key);
  RADIAL_HIP_TRY(hipGetLastError());
  return RADIAL_OK;
}

template <int D, int BLK, bool kExact>
int launch(const BwdArgs& a, hipStream_t stream) {
  const int64_t rows = (int64_t)a.B * a.H * a.N;
  const int rows_per_block = 256 / (D / 8);
  const int64_t prep_grid = (rows + rows_per_block - 1) / rows_per_block;
  if (prep_grid > 0x7fffffffLL || work_grid_bound(a.work_t) > 0x7fffffffLL || work_grid_bound(a.work) > 0x7fffffffLL)
    return fail(RADIAL_ESHAPE, "problem too large for one launch");
  bwd_prepare_kernel<D><<<dim3((unsigned)prep_grid), dim3(256), 0, stream>>>(a);
  const int64_t items = work_items(a.work, a.n_blocks);
  // dQ reads no rows of Q and dO but those it replaces, so dq may be either's memory; dK/dV has to be finished with them then.
  const bool apart = !may_overlap(a.B, a.H, a.N, D, a.dq, a.q) && !may_overlap(a.B, a.H, a.N, D, a.dq, a.dout);
  const BackwardForm form = backward_form(D, BLK, a.work, a.work_t, items, apart);
  int rc;
  if constexpr (D == 64) {
    if (form.kind == BackwardForm::kTogether) {
      BwdArgs both = a;
      both.work.halved = form.key == 4 ? 0 : halved_query_items_64(BLK, a.work, items);
      if (form.key == 4) return launch_both<BLK, kExact, 4, BLK / 32>(both, stream);
      if (form.key == 2) return both.work.halved ? launch_both<BLK, kExact, 2, BLK / 64, true>(both, stream) : launch_both<BLK, kExact, 2, BLK / 64>(both, stream);
      if constexpr (BLK == 128)  // the only ones of one group
        return both.work.halved ? launch_both<BLK, kExact, 1, 1, true>(both, stream) : launch_both<BLK, kExact, 1, 1>(both, stream);
    }
    rc = form.key == 2 ? launch_dkdv<64, BLK, kExact, 2, BLK / 64, true>(a, stream) : launch_dkdv<64, BLK, kExact, 1, 1, true>(a, stream);
  } else {
    if (form.kind == BackwardForm::kTogetherByHand) return launch_both_hand<BLK, kExact>(a, stream);
    if constexpr (BLK == 128) {
      if (form.kind == BackwardForm::kTogetherInPairs) {
        BwdArgs both = a;
        both.work.halved = halved_query_items(a.work, items);
        return both.work.halved ? launch_both_pairs<kExact, true>(both, stream) : launch_both_pairs<kExact, false>(both, stream);
      }
      rc = form.key == 2 ? launch_dkdv<D, BLK, kExact, 2, 2>(a, stream) : launch_dkdv_pairs<128, kExact>(a, stream);
    } else {
      rc = form.key == 2 ? launch_dkdv<D, BLK, kExact, 2, 1>(a, stream) : launch_dkdv<D, BLK, kExact, 1, 1>(a, stream);
    }
  }
  if (rc) return rc;
  rc = form.query == 4 ? launch_dq<D, BLK, kExact, 4, BLK / 64>(a, stream)
                       : form.query == 2 ? launch_dq<D, BLK, kExact, 2, 1>(a, stream) : launch_dq<D, BLK, kExact, 1, 1>(a, stream);
  if (rc) return rc;
  RADIAL_HIP_TRY(hipGetLastError());
  return RADIAL_OK;
}

template <int D, int BLK>
int launch(const BwdArgs& a, hipStream_t stream) {
  return a.rule.exact ? launch<D, BLK, true>(a, stream) : launch<D, BLK, false>(a, stream);
}

}  // namespace

int launch_bwd(int D, int block, const BwdArgs& a, hipStream_t stream) {
  if (D == 128 && block == 128) return launch<128, 128>(a, stream);
  if (D == 64 && block == 128) return launch<64, 128>(a, stream);
  if (D == 128 && block == 64) return launch<128, 64>(a, stream);
  if (D == 64 && block == 64) return launch<64, 64>(a, stream);
  return fail(RADIAL_EUNSUPPORTED, "head dimension %d with block %d is not supported", D, block);
}

}  // namespace radial

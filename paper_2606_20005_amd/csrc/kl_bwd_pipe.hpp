// Pipelined backward kernels: the separate dQ and dK kernels of kl_bwd.hpp in
// a form that keeps one wave per SIMD busy by itself. A wave owns RB blocks
// of 32 resident rows and has the whole register file (512 registers: the
// accumulators and logits in the upper half would otherwise not fit), and
// the tile loop overlaps the matrix and vector work of neighbouring tiles.
//
// What bounds it, and why this form (MI355X, 32 heads, 16K x 16K):
//  - The chip is power limited here: the kernels of kl_bwd.hpp clock down to
//    1.74-1.82 GHz of 2.4 with the matrix pipe busy for 57-65% of the cycles.
//    Removing a third of the dQ kernel's stall cycles alone gave 2%, so the
//    energy of a tile counts as much as its cycles. Of the dQ kernel's time
//    the direct-to-LDS loads of the streamed tiles cost 6%,
//    half of the operand reads from LDS 1-3% (timing variants without them).
//    With RB = 2 each operand read from LDS feeds two MFMAs and each streamed
//    tile 256 rows: both halve.
//  - An MFMA (32 cycles of the matrix pipe) holds up the vector pipe for 8
//    cycles only; beside it a wave can issue 24 cycles of vector work. So the
//    vector work of a tile is spread over the MFMAs that do not depend on it:
//      phase B: logits of the tile, first distribution (chain 1), with the
//               second half of the previous tile's logit gradients;
//      phase C: gradient MFMAs of the previous tile;
//      phase D: logits of the tile, second distribution (chain 2), with what
//               chain 1 alone determines (exponentials, or the teacher-side
//               part of the ratio), and the transpose reads that phase C of
//               the next tile needs.
//    Scheduling barriers pin this order: left to itself the compiler forms
//    all logits, then all vector work (7% slower).
//  - Measured against the kernels of kl_bwd.hpp (same box, ms, dQ and dK, 32
//    heads x 16384): d 128/128 student 5.59, 5.93 -> 5.34, 5.64; d 128/64 4.10,
//    4.39 -> 3.96, 4.07; teacher at 128/128 5.52, 5.88 -> 5.26, 5.52; all four
//    gradients (RB = 1: the accumulators of both pairs leave no room for two
//    blocks) 8.99, 10.31 -> 8.06, 8.89, causal 4.72, 5.47 -> 4.26, 4.73. The
//    outputs are the same bit for bit. pipe_blocks says where each form runs.
//    Counters at d 128/128: 1.85-1.93 GHz (two boxes), matrix pipe busy for
//    56-61% of the cycles, vector pipe 49-50%; 20 and 16 LDS instructions a
//    32 x 32 block (dK, dQ) instead of 41 and 32, 110 and 103 vector ones
//    instead of 96 and 94. So the gain is clock: fewer LDS reads for the same
//    MFMAs.
//
// Masked pairs: their raw logits are replaced by kBwdMaskedRaw, which gives
// P = 0 exactly and finite factors at the scales that pipe_scale admits, so
// their logit gradients are 0. Before the first tile the pipeline holds a
// neutral one (every pair masked, operands 0).
#pragma once

#include <type_traits>

#include "kl_bwd.hpp"

namespace streamkl {

constexpr float kBwdMaskedRaw = -1e30f;   // raw logit of a pair the mask excludes

// Head-dim pairs that each form is built for: those that compile without
// spilling (tests/test_bwd_pipe.py). Two row blocks need room for both
// blocks' resident rows and gradients; all four gradients (mode 3) leave room
// for one block up to d1 + d2 = 320 (dQ) and 256 (dK, which also holds the
// streamed statistics).
template <int DA, int DB, int MODE, int RB, bool DK>
constexpr bool kPipeBuilt = MODE == 3 ? RB == 1 && DA + DB <= (DK ? 256 : 320)
                            : RB == 1 ? true
                                      : DA + DB >= 192 && (MODE == 1 ? DB : DA) <= 128 &&
                                            DA + DB <= ((MODE == 1 ? DB : DA) == 64 ? 320 : 256);

template <int DA, int DB, int MODE, int RB_>
struct PipeCfg {
  static constexpr int RB = RB_;                          // 32-row blocks per wave
  static constexpr int BR = 128 * RB;                     // resident rows per workgroup
  static constexpr int BS = 32;                           // streamed rows per tile
  static constexpr int CA = DA / 8, CB = DB / 8;
  static constexpr int STAGE = BS * (CA + CB);
  static constexpr bool WANT_B = (MODE & 1) != 0, WANT_A = (MODE & 2) != 0;
  static constexpr int KA = DA / 16, KB = DB / 16;        // k-steps of the two logit chains
  // The student gradient takes the shorter chain first (less is left to
  // overlap with it); the teacher gradient needs b's logits before a's.
  static constexpr bool A1 = MODE == 1 && KA <= KB;
  static constexpr int K1 = A1 ? KA : KB, K2 = A1 ? KB : KA, KT = K1 + K2;
  static constexpr int NB = WANT_B ? DB / 32 : 0, NA = WANT_A ? DA / 32 : 0, NG = NA + NB;   // gradient columns / 32
  static constexpr int NU = 2 * RB;                       // units of 8 logit gradients per lane: (rows half s, block x)
  static constexpr int UB = RB;                           // units formed in phase B, the others in phase C
  static constexpr int LA = 4;                            // operand reads in flight ahead of their MFMA
};

// What the pipeline carries from a tile to the next.
template <class C>
struct PipeState {
  f32x16 s2[C::RB];                             // raw logits of chain 2
  float p1[C::RB][16];                          // modes 1, 3: P of chain 1's distribution
  float w1[C::WANT_A ? C::RB : 1][16];          // modes 2, 3: s_b raw_b + dl
  bf16x8 bop[2][C::NG];                         // streamed rows as gradient operands, per rows half
  __device__ __forceinline__ PipeState() {
#pragma unroll
    for (int x = 0; x < C::RB; ++x)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s2[x][i] = kBwdMaskedRaw;
        p1[x][i] = 0.f;
        if constexpr (C::WANT_A) w1[x][i] = 0.f;
      }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int n = 0; n < C::NG; ++n) bop[s][n] = __builtin_bit_cast(bf16x8, u32x4{0u, 0u, 0u, 0u});
  }
};

__device__ __forceinline__ void pin_order() { __builtin_amdgcn_sched_barrier(0); }

// One step of the pipeline for one wave: phases B and D of the tile in
// `stage` (not when LAST, which only drains), second half and phase C of the
// previous tile. st1(x, i), st2(x, i): statistics of element i of block x for
// chain 1 of this tile and for the previous tile. ok_prev(x, i): whether the
// element of the previous tile is an allowed pair, asked only if mask_prev;
// on_mask(n1): puts the stand-in into chain 1's raw logits of excluded pairs,
// called only if mask_cur (both uniform). before_c(), after_c(): called around
// phase C, for statistics that change with the tile.
template <int DA, int DB, int MODE, class C, bool LAST, typename St1, typename St2, typename MaskFn, typename OkP,
          typename BeforeC, typename AfterC>
__device__ __forceinline__ void pipe_step(const u32x4* stage, PipeState<C>& P, const bf16x8 (&ra_op)[C::RB][C::KA],
                                          const bf16x8 (&rb_op)[C::RB][C::KB],
                                          f32x16 (&ga)[C::RB][C::WANT_A ? DA / 32 : 1],
                                          f32x16 (&gb)[C::RB][C::WANT_B ? DB / 32 : 1], float ca, float cb, float sa,
                                          float sb, int lane, St1 st1, St2 st2, bool mask_cur, MaskFn on_mask,
                                          bool mask_prev, OkP ok_prev, BeforeC before_c, AfterC after_c,
                                          const TrOffsets<DA, DB, MODE>& to) {
  constexpr int RB = C::RB, K1 = C::K1, K2 = C::K2, KT = C::KT, NG = C::NG, NB = C::NB, NU = C::NU, UB = C::UB;
  constexpr int LA = C::LA;
  const int half = lane >> 5, r = lane & 31;
  const u32x4* t1 = C::A1 ? stage : stage + C::BS * C::CA;   // chain 1's rows of the tile, then chain 2's
  const u32x4* t2 = C::A1 ? stage + C::BS * C::CA : stage;
  constexpr int C1 = C::A1 ? C::CA : C::CB, C2 = C::A1 ? C::CB : C::CA;
  bf16x8 buf[KT];
  auto rd = [&](int j) { buf[j] = j < K1 ? lds_row8<C1>(t1, r, 2 * j + half) : lds_row8<C2>(t2, r, 2 * (j - K1) + half); };
  auto mm1 = [&](int x, int j, f32x16& acc) {
    if constexpr (C::A1) acc = mfma32(buf[j], ra_op[x][j < C::KA ? j : 0], acc);
    else acc = mfma32(buf[j], rb_op[x][j < C::KB ? j : 0], acc);
  };
  auto mm2 = [&](int x, int j, f32x16& acc) {
    if constexpr (C::A1) acc = mfma32(buf[K1 + j], rb_op[x][j < C::KB ? j : 0], acc);
    else acc = mfma32(buf[K1 + j], ra_op[x][j < C::KA ? j : 0], acc);
  };

  pin_order();
  if constexpr (!LAST) {
#pragma unroll
    for (int j = 0; j < LA; ++j) rd(j);
  }
  if (mask_prev) {
#pragma unroll
    for (int x = 0; x < RB; ++x)
#pragma unroll
      for (int i = 0; i < 16; ++i) P.s2[x][i] = ok_prev(x, i) ? P.s2[x][i] : kBwdMaskedRaw;
  }
  f32x16 n1[RB], n2[RB];
#pragma unroll
  for (int x = 0; x < RB; ++x) {
    n1[x] = zero16();
    n2[x] = zero16();
  }
  // second half of the previous tile's logit gradients: element e of unit v
  float dsa[RB][16], dsb[RB][16];
  auto second = [&](int v, int e) {
    const int x = v % RB, i = 8 * (v / RB) + e;
    const RowStats rs = st2(x, i);
    const float r2 = P.s2[x][i];
    const float p2 = C::A1 ? exp2_fast(__builtin_fmaf(r2, cb, -rs.lsb2)) : exp2_fast(__builtin_fmaf(r2, ca, -rs.lsa2));
    if constexpr (C::WANT_B) dsb[x][i] = C::A1 ? p2 - P.p1[x][i] : P.p1[x][i] - p2;
    if constexpr (C::WANT_A) dsa[x][i] = p2 * __builtin_fmaf(r2, sa, -P.w1[x][i]);
  };
  bf16x8 pa[C::WANT_A ? NU : 1], pb[C::WANT_B ? NU : 1];
  auto pack = [&](int v) {
    if constexpr (C::WANT_A) pa[v] = pack8(dsa[v % RB] + 8 * (v / RB));
    if constexpr (C::WANT_B) pb[v] = pack8(dsb[v % RB] + 8 * (v / RB));
  };
  pin_order();
  // B
#pragma unroll
  for (int j = 0; j < K1; ++j) {
    if constexpr (!LAST) {
      if (j + LA < KT) rd(j + LA);
#pragma unroll
      for (int x = 0; x < RB; ++x) mm1(x, j, n1[x]);
    }
#pragma unroll
    for (int e = 8 * UB * j / K1; e < 8 * UB * (j + 1) / K1; ++e) {
      second(e / 8, e % 8);
      if (e % 8 == 7) pack(e / 8);
    }
    pin_order();
  }
  before_c();
  pin_order();
  // C
#pragma unroll
  for (int v = 0; v < NU; ++v) {
    const int s = v / RB, x = v % RB;
#pragma unroll
    for (int n = 0; n < NG; ++n) {
      if constexpr (C::WANT_B) {
        if (n < NB) gb[x][n < NB ? n : 0] = mfma32(pb[v], P.bop[s][n], gb[x][n < NB ? n : 0]);
      }
      if constexpr (C::WANT_A) {
        if (n >= NB) ga[x][n >= NB ? n - NB : 0] = mfma32(pa[v], P.bop[s][n], ga[x][n >= NB ? n - NB : 0]);
      }
      if (v + UB < NU) {
#pragma unroll
        for (int e = 8 * n / NG; e < 8 * (n + 1) / NG; ++e) second(v + UB, e);
        if (n == NG - 1) pack(v + UB);
      }
      pin_order();
    }
  }
  if constexpr (!LAST) {
    after_c();
    if (mask_cur) on_mask(n1);
    pin_order();
    // D
#pragma unroll
    for (int j = 0; j < K2; ++j) {
      if (K1 + j + LA < KT) rd(K1 + j + LA);
#pragma unroll
      for (int x = 0; x < RB; ++x) mm2(x, j, n2[x]);
#pragma unroll
      for (int e = 16 * RB * j / K2; e < 16 * RB * (j + 1) / K2; ++e) {
        const int x = e / 16, i = e % 16;
        const RowStats rs = st1(x, i);
        if constexpr (C::A1) {
          P.p1[x][i] = exp2_fast(__builtin_fmaf(n1[x][i], ca, -rs.lsa2));
        } else {
          if constexpr (C::WANT_B) P.p1[x][i] = exp2_fast(__builtin_fmaf(n1[x][i], cb, -rs.lsb2));
          if constexpr (C::WANT_A) P.w1[x][i] = __builtin_fmaf(n1[x][i], sb, rs.dl);
        }
      }
#pragma unroll
      for (int q = 2 * NG * j / K2; q < 2 * NG * (j + 1) / K2; ++q) {
        const int s = q / NG, n = q % NG;
        if constexpr (C::WANT_B) {
          if (n < NB)
            P.bop[s][n] = cat8(lds_tr4_at(stage, to.b[n < NB ? n : 0][0] + 256 * C::CB * s),
                               lds_tr4_at(stage, to.b[n < NB ? n : 0][1] + 256 * C::CB * s));
        }
        if constexpr (C::WANT_A) {
          if (n >= NB)
            P.bop[s][n] = cat8(lds_tr4_at(stage, to.a[n >= NB ? n - NB : 0][0] + 256 * C::CA * s),
                               lds_tr4_at(stage, to.a[n >= NB ? n - NB : 0][1] + 256 * C::CA * s));
        }
      }
      pin_order();
    }
#pragma unroll
    for (int x = 0; x < RB; ++x) P.s2[x] = n2[x];
  }
}

template <int DA, int DB, class C>
__device__ __forceinline__ void zero_grads(f32x16 (&ga)[C::RB][C::WANT_A ? DA / 32 : 1],
                                           f32x16 (&gb)[C::RB][C::WANT_B ? DB / 32 : 1]) {
#pragma unroll
  for (int x = 0; x < C::RB; ++x) {
#pragma unroll
    for (int n = 0; n < (C::WANT_A ? DA / 32 : 1); ++n) ga[x][n] = zero16();
#pragma unroll
    for (int n = 0; n < (C::WANT_B ? DB / 32 : 1); ++n) gb[x][n] = zero16();
  }
}

// End of a tile step: the next tile's loads have landed and this wave's
// reads of the tile have returned (the transpose reads are consumed in the
// next step only), for every wave.
__device__ __forceinline__ void pipe_end_step() {
  wait_vmem();
  wait_lds();
  barrier_no_fence();
}

// ----------------------------------------------------------------------------
// dQ: workgroup = 128 RB query rows of one (batch, head), streams key tiles.
// ----------------------------------------------------------------------------
template <int DA, int DB, bool CAUSAL, int MODE, int RB>
__global__ void __launch_bounds__(kThreads, 1)
kl_bwd_dq_pipe_kernel(const uint16_t* __restrict__ Qa, const uint16_t* __restrict__ Ka,
                      const uint16_t* __restrict__ Qb, const uint16_t* __restrict__ Kb, int NQ, int NK, float sa,
                      float sb, const float* __restrict__ kl, const float* __restrict__ lse_a,
                      const float* __restrict__ lse_b, const float* __restrict__ g, void* __restrict__ dQa,
                      void* __restrict__ dQb, int bf16) {
  using C = PipeCfg<DA, DB, MODE, RB>;
  __shared__ u32x4 st0[C::STAGE];   // two arrays: see kl_bwd_dq_kernel
  __shared__ u32x4 st1[C::STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
  const int TQ = (NQ + C::BR - 1) / C::BR;
  int bh, qt;
  head_block<CAUSAL, 1>(TQ, bh, qt);
  if (CAUSAL) qt = TQ - 1 - qt;   // rank 0: the last rows, the longest
  const int q0 = qt * C::BR;
  const int off = NK - NQ;
  const int qw = q0 + 32 * RB * wave;
  const int wlast = min(qw + 32 * RB - 1, NQ - 1);
  const float ca = sa * kLog2e, cb = sb * kLog2e;

  int ntiles = (NK + C::BS - 1) / C::BS;
  if (CAUSAL) {
    const int kmax = min(q0 + C::BR, NQ) - 1 + off;
    ntiles = kmax < 0 ? 0 : min(ntiles, kmax / C::BS + 1);
  }

  RowStats rs[RB];
  float gsign[RB];
  bf16x8 qa[RB][C::KA], qb[RB][C::KB];
#pragma unroll
  for (int x = 0; x < RB; ++x) {
    const int myq = qw + 32 * x + (lane & 31);
    const RowStats r0 = load_row_stats(kl, lse_a, lse_b, g, (size_t)bh * NQ + myq, myq < NQ);
    gsign[x] = r0.g < 0.f ? -1.f : 1.f;
    rs[x] = fold_row_stats(r0);
    load_resident<DA>(qa[x], Qa, (size_t)bh * NQ, myq, NQ, half);
    load_resident<DB>(qb[x], Qb, (size_t)bh * NQ, myq, NQ, half);
  }
  wait_vmem();   // before the tile loop (see kl_bwd_dq_kernel)

  f32x16 dqa[RB][C::WANT_A ? DA / 32 : 1], dqb[RB][C::WANT_B ? DB / 32 : 1];
  zero_grads<DA, DB, C>(dqa, dqb);
  const rsrc_t rka = make_rsrc(Ka + (size_t)bh * NK * DA, (uint32_t)NK * DA * 2u);
  const rsrc_t rkb = make_rsrc(Kb + (size_t)bh * NK * DB, (uint32_t)NK * DB * 2u);
  const TileDma<C::BS, C::CA, C::CB> dma(tid);
  const TrOffsets<DA, DB, MODE> tro(lane);

  PipeState<C> P;
  int k_prev = 0;
  bool m_prev = false;   // the neutral tile is masked already
  auto stats = [&](int x, int) { return rs[x]; };
  auto ok_at = [&](int k0) {
    return [=](int x, int i) {
      const int k = k0 + 8 * (i >> 2) + 4 * half + (i & 3);
      return k < NK && (!CAUSAL || k <= qw + 32 * x + (lane & 31) + off);
    };
  };
  auto nothing = [] {};
  auto tile = [&](const u32x4* stage, int kt) {
    const int k0 = kt * C::BS;
    bool active = qw < NQ;
    bool need_mask = k0 + C::BS > NK;
    if (CAUSAL) {
      active = active && (k0 <= wlast + off);
      need_mask = need_mask || (k0 + C::BS - 1 > qw + off);
    }
    if (!active) return;
    const auto ok = ok_at(k0);
    auto on_mask = [&](f32x16 (&n1)[RB]) {
#pragma unroll
      for (int x = 0; x < RB; ++x)
#pragma unroll
        for (int i = 0; i < 16; ++i) n1[x][i] = ok(x, i) ? n1[x][i] : kBwdMaskedRaw;
    };
    pipe_step<DA, DB, MODE, C, false>(stage, P, qa, qb, dqa, dqb, ca, cb, sa, sb, lane, stats, stats, need_mask, on_mask,
                                      m_prev, ok_at(k_prev), nothing, nothing, tro);
    k_prev = k0;
    m_prev = need_mask;
  };

  if (ntiles > 0) dma.issue(rka, rkb, 0, st0, wave);
  pipe_end_step();
  auto step = [&](const u32x4* cur, u32x4* nxt, int kt) {
    if (kt + 1 < ntiles) dma.issue(rka, rkb, (kt + 1) * C::BS, nxt, wave);
    tile(cur, kt);
    pipe_end_step();
  };
  for (int kt = 0; kt < ntiles; kt += 2) {
    step(st0, st1, kt);
    if (kt + 1 < ntiles) step(st1, st0, kt + 1);
  }
  pipe_step<DA, DB, MODE, C, true>(st0, P, qa, qb, dqa, dqb, ca, cb, sa, sb, lane, stats, stats, false,
                                   [](f32x16 (&)[RB]) {}, m_prev,
                                   ok_at(k_prev), nothing, nothing, tro);

#pragma unroll
  for (int x = 0; x < RB; ++x) {
    float rsign[16];
#pragma unroll
    for (int i = 0; i < 16; ++i)
      rsign[i] = __int_as_float(
          __builtin_amdgcn_ds_bpermute(4 * (8 * (i >> 2) + 4 * half + (i & 3)), __float_as_int(gsign[x])));
    auto row_sign = [&](int i) { return rsign[i]; };
    const int row0 = qw + 32 * x;
    if constexpr (C::WANT_B)
      write_grad<DB>(dQb, bf16 & kBf16dQb, dqb[x], (size_t)bh * NQ, row0, NQ, sb, lane, DB, row_sign);
    if constexpr (C::WANT_A)
      write_grad<DA>(dQa, bf16 & kBf16dQa, dqa[x], (size_t)bh * NQ, row0, NQ, sa, lane, DA, row_sign);
  }
}

// ----------------------------------------------------------------------------
// dK: workgroup = 128 RB key rows of one (batch, head), streams query tiles
// with their prepared statistics (kl_bwd_rowstats_kernel). |g| is folded into
// the statistics; a workgroup that has a negative g ahead (a flag of 0) flips
// the signs of those rows' gradient operands instead of their logit gradients
// (both exact).
// ----------------------------------------------------------------------------
template <int DA, int DB, bool CAUSAL, int MODE, int RB>
__global__ void __launch_bounds__(kThreads, 1)
kl_bwd_dk_pipe_kernel(const uint16_t* __restrict__ Qa, const uint16_t* __restrict__ Ka,
                      const uint16_t* __restrict__ Qb, const uint16_t* __restrict__ Kb, int NQ, int NK, float sa,
                      float sb, void* __restrict__ dKa, void* __restrict__ dKb, int bf16,
                      const float* __restrict__ pstats, const int* __restrict__ ppositive) {
  using C = PipeCfg<DA, DB, MODE, RB>;
  static_assert(C::BS == kRowStatsTile, "prepared statistics come in tiles of the streamed rows");
  __shared__ u32x4 st0[C::STAGE];
  __shared__ u32x4 st1[C::STAGE];
  __shared__ f32x4 sstat[2][4][C::BS / 4];   // statistics of the stages: [lsa2, lsb2, g, dl][rows / 4]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
  const int TK = (NK + C::BR - 1) / C::BR;
  int bh, kblk;
  head_block<CAUSAL, 1>(TK, bh, kblk);   // causal rank 0: the first keys, seen by the most rows
  const int kb0 = kblk * C::BR;
  const int off = NK - NQ;
  const int kw = kb0 + 32 * RB * wave;
  const int wklast = min(kw + 32 * RB - 1, NK - 1);
  const float ca = sa * kLog2e, cb = sb * kLog2e;

  const int ntq = (NQ + C::BS - 1) / C::BS;
  int t_begin = 0;
  if (CAUSAL) {
    const int qmin = kb0 - off;   // first row that sees key kb0
    t_begin = qmin <= 0 ? 0 : min(ntq, qmin / C::BS);
  }

  bool mine = false;
  for (int t = t_begin + tid; t < ntq; t += kThreads) mine = mine || ppositive[(size_t)bh * ntq + t] == 0;
  const bool negative = __syncthreads_or(mine) != 0;

  bf16x8 ka[RB][C::KA], kb[RB][C::KB];
#pragma unroll
  for (int x = 0; x < RB; ++x) {
    const int myk = kw + 32 * x + (lane & 31);
    load_resident<DA>(ka[x], Ka, (size_t)bh * NK, myk, NK, half);
    load_resident<DB>(kb[x], Kb, (size_t)bh * NK, myk, NK, half);
  }
  wait_vmem();   // before the tile loop (see kl_bwd_dq_kernel)

  f32x16 dka[RB][C::WANT_A ? DA / 32 : 1], dkb[RB][C::WANT_B ? DB / 32 : 1];
  zero_grads<DA, DB, C>(dka, dkb);
  const rsrc_t rqa = make_rsrc(Qa + (size_t)bh * NQ * DA, (uint32_t)NQ * DA * 2u);
  const rsrc_t rqb = make_rsrc(Qb + (size_t)bh * NQ * DB, (uint32_t)NQ * DB * 2u);
  const TileDma<C::BS, C::CA, C::CB> dma(tid);
  const PreparedStatsDma pdma(pstats, ppositive, (size_t)bh * ntq, ntq);
  const TrOffsets<DA, DB, MODE> tro(lane);

  PipeState<C> P;
  int r_prev = 0;
  bool m_prev = false;   // the neutral tile is masked already
  // statistics in registers, element i at [i / 4][i % 4]: this tile's for
  // chain 1 (c1: exponent offset, cd: dl), read before phase C, and the
  // exponent offset p2 that the second half of the tile needs in the next
  // step, read after it
  f32x4 c1[4], cd[4], p2[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) p2[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto stats1 = [&](int, int i) {
    const float o = c1[i >> 2][i & 3];
    return RowStats{o, o, 1.f, C::WANT_A ? cd[i >> 2][i & 3] : 0.f};
  };
  auto stats2 = [&](int, int i) { return RowStats{p2[i >> 2][i & 3], p2[i >> 2][i & 3], 1.f, 0.f}; };
  auto ok_at = [&](int r0) {
    return [=](int x, int i) {
      const int q = r0 + 8 * (i >> 2) + 4 * half + (i & 3);
      return q < NQ && (!CAUSAL || kw + 32 * x + (lane & 31) <= q + off);
    };
  };
  // SIGN: some g of the rows ahead is negative
  auto tile = [&](auto SIGN, const u32x4* stage, int buf, int t) {
    const int r0 = t * C::BS;
    bool active = kw < NK;
    bool need_mask = r0 + C::BS > NQ;
    if (CAUSAL) {
      const int qlast = min(r0 + C::BS, NQ) - 1;
      active = active && (qlast + off >= kw);
      need_mask = need_mask || (wklast > r0 + off);
    }
    if (!active) return;
    const f32x4 (&st)[4][C::BS / 4] = sstat[buf];
    auto read_first = [&] {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (MODE != 2) c1[q] = st[C::A1 ? 0 : 1][2 * q + half];
        if (C::WANT_A) cd[q] = st[3][2 * q + half];
      }
    };
    auto read_second = [&] {
#pragma unroll
      for (int q = 0; q < 4; ++q) p2[q] = st[C::A1 ? 1 : 0][2 * q + half];
    };
    const auto ok = ok_at(r0);
    // A statistic that is not finite (a row with non-finite inputs) must stay
    // out of the keys the row does not see: in a tile with masked pairs such
    // a row takes the offset +inf (P = 0), and NaN logits where it does see
    // the key.
    auto on_mask = [&](f32x16 (&n1)[RB]) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float o1 = MODE != 2 ? c1[i >> 2][i & 3] : 0.f, o2 = p2[i >> 2][i & 3];
        const float dl = C::WANT_A ? cd[i >> 2][i & 3] : 0.f;
        const bool bad = !(o1 > kNegInf) || !(o2 > kNegInf) || !(fabsf(dl) < __builtin_inff());
        if (MODE != 2) c1[i >> 2][i & 3] = bad ? __builtin_inff() : o1;
        p2[i >> 2][i & 3] = bad ? __builtin_inff() : o2;
        if (C::WANT_A) cd[i >> 2][i & 3] = bad ? 0.f : dl;
#pragma unroll
        for (int x = 0; x < RB; ++x)
          n1[x][i] = !ok(x, i) ? kBwdMaskedRaw : bad ? __builtin_nanf("") : n1[x][i];
      }
    };
    pipe_step<DA, DB, MODE, C, false>(stage, P, ka, kb, dka, dkb, ca, cb, sa, sb, lane, stats1, stats2, need_mask,
                                      on_mask, m_prev, ok_at(r_prev), read_first, read_second, tro);
    if (SIGN) {
      // element e of operand half s is streamed row 16 s + 8 (e / 4) + 4 half + e % 4
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const f32x4 g0 = st[2][4 * s + half], g1 = st[2][4 * s + 2 + half];
        auto sign2 = [](float lo, float hi) { return (lo < 0.f ? 0x8000u : 0u) | (hi < 0.f ? 0x80000000u : 0u); };
        const u32x4 flip = {sign2(g0[0], g0[1]), sign2(g0[2], g0[3]), sign2(g1[0], g1[1]), sign2(g1[2], g1[3])};
#pragma unroll
        for (int n = 0; n < C::NG; ++n)
          P.bop[s][n] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, P.bop[s][n]) ^ flip);
      }
    }
    r_prev = r0;
    m_prev = need_mask;
  };

  auto load = [&](int t, u32x4* stage, int buf) {
    dma.issue(rqa, rqb, t * C::BS, stage, wave);
    if (wave == 0) pdma.issue_stats(t, reinterpret_cast<float*>(&sstat[buf][0][0]), lane);
  };
  auto stream = [&](auto SIGN) {
    if (t_begin < ntq) load(t_begin, st0, 0);
    pipe_end_step();
    auto step = [&](const u32x4* cur, u32x4* nxt, int t, int buf) {
      if (t + 1 < ntq) load(t + 1, nxt, buf ^ 1);
      tile(SIGN, cur, buf, t);
      pipe_end_step();
    };
    for (int t = t_begin; t < ntq; t += 2) {
      step(st0, st1, t, 0);
      if (t + 1 < ntq) step(st1, st0, t + 1, 1);
    }
  };
  // With RB = 2 the flips sit in a loop of their own: a uniform test of
  // `negative` per tile in one loop cost every tile 2-5%. With RB = 1 (all
  // four gradients) the second loop costs registers, and 12% causal.
  if constexpr (RB == 1) {
    stream(negative);
  } else {
    if (negative)
      stream(std::true_type{});
    else
      stream(std::false_type{});
  }
  pipe_step<DA, DB, MODE, C, true>(st0, P, ka, kb, dka, dkb, ca, cb, sa, sb, lane, stats1, stats2, false,
                                   [](f32x16 (&)[RB]) {}, m_prev, ok_at(r_prev), [] {}, [] {}, tro);

#pragma unroll
  for (int x = 0; x < RB; ++x) {
    const int row0 = kw + 32 * x;
    if constexpr (C::WANT_B) write_grad<DB>(dKb, bf16 & kBf16dKb, dkb[x], (size_t)bh * NK, row0, NK, sb, lane);
    if constexpr (C::WANT_A) write_grad<DA>(dKa, bf16 & kBf16dKa, dka[x], (size_t)bh * NK, row0, NK, sa, lane);
  }
}

}  // namespace streamkl

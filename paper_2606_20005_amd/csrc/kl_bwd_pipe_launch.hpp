// Launchers of the pipelined backward kernels and the rule that picks them.
#pragma once

#include "kl_bwd_pipe.hpp"
#include "kl_launch.hpp"

namespace streamkl {

// Scales that the finite stand-in for masked logits (kBwdMaskedRaw) serves:
// times the scale it must lie far below any real logit (|q.k| < 1e29) and the
// log2 |g| beside it, and two such products must add up within the float32
// range. A call with another scale takes the kernel of kl_bwd.hpp, which
// selects a zero for every masked pair.
inline bool pipe_scale(float s) { return s >= 0x1p-80f && s <= 0x1p26f; }

// Row blocks per wave of the pipelined kernel a call takes, or 0 for the
// kernel of kl_bwd.hpp. Measured on MI355X, same box, old against new, ms:
//  - Where the old kernel leaves one wave per SIMD, the pipelined one with one
//    block is faster (short streams apart, below), since that one wave overlaps
//    its own matrix and vector work: wide heads, whose registers allow no second
//    wave (16 heads x 8192, dQ and dK: d 192/128 1.22, 1.22 -> 1.06, 0.95;
//    256/256 1.80, 1.66 -> 1.50, 1.46; all four gradients at 128/64 1.14,
//    1.16 -> 1.02, 0.98), and grids of at most one workgroup per CU (8 heads
//    x 2048, 128/128: 0.064, 0.071 -> 0.058, 0.059).
//  - Causal grids are handed out longest block first, at most two workgroups
//    to a CU. The old kernel runs both at once, the pipelined one in turn: it
//    is done with its longest block if the blocks that follow each other are
//    hardly longer than that together (the middle of the ranks is the longest
//    such pair; a start counts as 256 rows). Kernel times over the old
//    kernel's, mean of the sweep by the length of that pair over the longest
//    block: below 0.5 0.84 (dK) and 0.90 (dQ), 0.5-1 0.86 and 0.87, 1-1.1 0.92
//    and 1.00 (16 heads x 4096, where it is 1: 0.275 -> 0.244 and 0.265 ->
//    0.244 a backward), 1.1-1.5 1.16 and 1.02, above 1.18 and 1.15 (blocks of
//    nearly one length: 12 heads, 5000 rows on 60000 keys, d 64/128, 4.19 ->
//    4.65).
//  - Larger grids give the old kernel two waves per SIMD, which beat one
//    block (32 x 8192, 128/128: 1.49 against 1.73), but two blocks halve the
//    operand and tile traffic. Their 256-row workgroups sit alone on a CU, so
//    nothing hides their start and end: they pay once a workgroup streams
//    enough rows. What they save is power as much as cycles, so each form was
//    timed over 80 ms of whole backward passes (1423 grids on two boxes; time
//    over the old kernels', mean and largest, by the head dim whose gradients
//    are formed and the other one):
//      no mask   64 and 128, 192, 256: 0.98, 0.97, 0.95 (1.01); 128 and 128
//                0.98 (1.02, and one of 1.18), 128 and 64 1.00 (1.05);
//      causal    64 and 128, 192, 256: 0.99, 0.99, 0.97 (1.03) with the rule
//                below (1196 grids on four boxes); 128 and 128 1.01 (1.07), 128
//                and 64 1.02 (1.09) with dK alone from 4096 rows on: not taken.
//    dK: from 4096 rows on, over two rounds of workgroups, causal four. Causal
//    squares stream from nothing to all rows and gain from 8192 on (4096 to
//    8192 with 64 and 128, 192: 1.00 (1.05)), unless the other dim is four
//    times as wide (0.98 (1.00)).
//    dQ without a mask: from 16384 rows on, over four rounds or on a grid that
//    fills its last one to 95% (below four rounds 0.98 (1.00) where it does,
//    1.05 (1.26) below 85%). dQ causal: from 6144 rows on, over four rounds.
//    Square heads of 6K to 12K streamed rows took 0.99 (1.05) with dK alone and
//    0.97 (1.03) with both on two of the boxes, 0.99 (1.03) either way on the
//    others; all heads of 2K to 6K 0.99 (1.04) and 1.00 (1.23).
//    dQ without dK lost 1.06 (64 heads, 4385 rows on 14421 keys, d 192/64), so
//    dQ goes by dK's limits too. So also where dQ's blocks are of nearly one length, fill their rounds and
//    dK takes two: the last rows of a long context, ms without, with dK, with
//    both: d 192/64, 8 heads, 8192 rows on 131072 keys 9.92, 9.62, 9.61; d
//    256/64 11.73, 11.22, 10.96; d 128/64 8.34, 8.23, 7.96; d 192/64, 16 x 8192
//    on 65536 9.60, 9.60, 9.33; 8 x 7936 on 98000 7.16, 7.43, 6.99; 4 x 16384 on
//    131072 9.94, 9.84, 9.55; 24 x 8192 on 65536 (three rounds) 14.34, 14.25,
//    14.42.
//  - One block starts and drains its pipeline around the stream (dK also looks
//    through the flags of its tiles), which a short stream does not pay back.
//    Kernel times over the old kernel's, mean of a random sweep of grids within
//    one round, by streamed rows: dK 64-127 1.12 causal, 1.03 not; 128-255
//    1.03, 0.99; 256-511 0.95, 0.93; 512-1023 0.88. dQ 64-127 1.01; 128-255
//    0.96, 0.98. Where the old kernel has one wave per SIMD: dK 64-127 1.06,
//    0.99; 128-255 0.94, 0.97; dQ 0.93 at most, however short. dQ of causal
//    heads with N_K < N_Q goes by the rows that see a key, the others end at
//    once: 128-255 1.01, 256 on 0.96 and 0.91 (1 head, 34688 rows on 1920 keys,
//    d 256/64: backward 0.132 -> 0.103).
// The rows a workgroup streams are the mean over the grid, a head's allowed
// pairs over its own rows. Under the causal mask with N_K < N_Q only the last
// N_K query rows see a key, so that a key streams N_K / 2 of them: two blocks
// took 1367 us where the old kernel takes 1232 (backward of 1024 heads x 8300
// rows on 290 keys, d 128/64).
template <int DA, int DB, int MODE, bool DK>
int pipe_blocks(const BwdArgs& a, bool causal) {
  if (!pipe_scale(a.sa) || !pipe_scale(a.sb)) return 0;
  const long long nq = a.NQ, nk = a.NK, own = DK ? nk : nq;
  const long long rows = causal && nk < nq ? nk : nq;   // query rows that see a key
  const long long pairs = causal ? rows * (2 * nk - rows + 1) / 2 : rows * nk;
  const long long streamed = own > 0 ? pairs / own : 0;
  if constexpr (kPipeBuilt<DA, DB, MODE, 2, DK>) {
    const long long wg = a.BH * ((own + 255) / 256);
    const bool even = 20 * wg >= 19 * ((wg + kCus - 1) / kCus * kCus);
    constexpr int formed = MODE == 1 ? DB : DA, other = MODE == 1 ? DA : DB;   // head dims (two blocks: modes 1 and 2)
    const bool flat = 10 * pairs >= 6 * nq * nk;   // key blocks of nearly one length, N_K well above N_Q
    const bool dk_causal = formed < other && a.BH * ((nk + 255) / 256) >= 4 * kCus &&
                           pairs >= (flat || other >= 4 * formed ? 4096 : 8192) * nk;
    if (DK       ? (causal ? dk_causal : streamed >= 4096 && wg >= 2 * kCus)
        : causal ? dk_causal && (wg >= 4 * kCus ? streamed >= 6144 : even && nk >= 8 * nq)
                 : streamed >= 16384 && (wg >= 4 * kCus || even))
      return 2;
  }
  if constexpr (kPipeBuilt<DA, DB, MODE, 1, DK>) {
    constexpr bool alone = BwdCfg<DA, DB, MODE>::MINB == 1;
    const long long least = DK ? (alone ? 128 : 256) : alone ? 0 : rows < nq ? 256 : 128;
    if ((DK || rows == 0 ? streamed : pairs / rows) < least) return 0;
    const long long wg = a.BH * ((own + 127) / 128);
    if (alone || wg <= kCus) return 1;
    if (causal && wg <= 2 * kCus) {
      const long long after = nk - 128 * (kCus / a.BH), cap = DK ? nq : nk;   // block that the first freed CU takes
      if (10 * (2 * (after < 0 ? 0 : after < cap ? after : cap) + 256) <= 11 * (nk < cap ? nk : cap)) return 1;
    }
  }
  return 0;
}

template <int DA, int DB, bool CAUSAL, int MODE, int RB, bool DK>
hipError_t run_pipe(const BwdArgs& a) {
  if constexpr (kPipeBuilt<DA, DB, MODE, RB, DK>) {
    const long long rows = PipeCfg<DA, DB, MODE, RB>::BR;
    const dim3 grid((unsigned)(a.BH * (((DK ? a.NK : a.NQ) + rows - 1) / rows)));
    if constexpr (DK)
      hipLaunchKernelGGL((kl_bwd_dk_pipe_kernel<DA, DB, CAUSAL, MODE, RB>), grid, dim3(kThreads), 0, a.stream, a.Qa,
                         a.Ka, a.Qb, a.Kb, a.NQ, a.NK, a.sa, a.sb, a.dKa, a.dKb, a.bf16, a.pstats, a.ppositive);
    else
      hipLaunchKernelGGL((kl_bwd_dq_pipe_kernel<DA, DB, CAUSAL, MODE, RB>), grid, dim3(kThreads), 0, a.stream, a.Qa,
                         a.Ka, a.Qb, a.Kb, a.NQ, a.NK, a.sa, a.sb, a.kl, a.lse_a, a.lse_b, a.g, a.dQa, a.dQb, a.bf16);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

// Launches the pipelined kernel if the rule picks one; taken says whether.
template <int MODE, bool DK>
hipError_t launch_pipe_unit(int da, int db, bool causal, const BwdArgs& a, bool* taken) {
  *taken = false;
#define STREAMKL_CASE(DA, DB)                                                                                        \
  if (da == DA && db == DB) {                                                                                        \
    const int rb = pipe_blocks<DA, DB, MODE, DK>(a, causal);                                                        \
    *taken = rb != 0;                                                                                                \
    if (rb == 2) return causal ? run_pipe<DA, DB, true, MODE, 2, DK>(a) : run_pipe<DA, DB, false, MODE, 2, DK>(a);   \
    if (rb == 1) return causal ? run_pipe<DA, DB, true, MODE, 1, DK>(a) : run_pipe<DA, DB, false, MODE, 1, DK>(a);   \
    return hipSuccess;                                                                                               \
  }
  STREAMKL_FOR_EACH_DIM_PAIR(STREAMKL_CASE)
#undef STREAMKL_CASE
  return hipErrorInvalidValue;
}

}  // namespace streamkl

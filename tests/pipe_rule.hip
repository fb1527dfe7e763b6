// Prints, for calls read from standard input, which form of a backward kernel
// the host's rule picks: 0 the kernel of kl_bwd.hpp, 1 or 2 the pipelined
// kernel with that many row blocks per wave. Host code only. Input lines:
//   dK(0/1) mode d_a d_b heads N_Q N_K causal(0/1) s_a s_b
#include <cstdio>

#include "kl_bwd_pipe_launch.hpp"

namespace streamkl {

template <int DA, int DB, int MODE>
int blocks(bool dk, const BwdArgs& a, bool causal) {
  return dk ? pipe_blocks<DA, DB, MODE, true>(a, causal) : pipe_blocks<DA, DB, MODE, false>(a, causal);
}

}  // namespace streamkl

int main() {
  int dk, mode, da, db, heads, nq, nk, causal;
  float sa, sb;
  while (std::scanf("%d %d %d %d %d %d %d %d %f %f", &dk, &mode, &da, &db, &heads, &nq, &nk, &causal, &sa, &sb) == 10) {
    streamkl::BwdArgs a{};
    a.BH = heads;
    a.NQ = nq;
    a.NK = nk;
    a.sa = sa;
    a.sb = sb;
    int n = -1;
#define CASE(DA, DB)                                                  \
  if (da == DA && db == DB)                                           \
    n = mode == 1   ? streamkl::blocks<DA, DB, 1>(dk, a, causal != 0) \
        : mode == 2 ? streamkl::blocks<DA, DB, 2>(dk, a, causal != 0) \
                    : streamkl::blocks<DA, DB, 3>(dk, a, causal != 0);
    STREAMKL_FOR_EACH_DIM_PAIR(CASE)
#undef CASE
    std::printf("%d\n", n);
  }
  return 0;
}

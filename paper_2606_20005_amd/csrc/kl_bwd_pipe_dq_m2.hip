// Instantiations of the pipelined query-owned dQ backward kernel for gradient mode 2
// (first-slot distribution (Setting 2)).
#include "kl_bwd_pipe_launch.hpp"

namespace streamkl {

hipError_t launch_bwd_pipe_dq_m2(int da, int db, bool causal, const BwdArgs& a, bool* taken) {
  return launch_pipe_unit<2, false>(da, db, causal, a, taken);
}

}  // namespace streamkl

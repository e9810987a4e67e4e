// The team kernels (plcg_team_kernels.h) for the Jacobi-scaled variable-coefficient
// stencils; a translation unit of its own so that the build stays parallel.
#include "plcg_team_kernels.h"

namespace plcg {

hipError_t launch_plcg_team_var(const TeamArgs &a, int l, bool d3, hipStream_t s) {
  return launch_plcg_team_of<true>(a, l, d3, s);
}

hipError_t launch_cg_team_var(const TeamArgs &a, bool d3, hipStream_t s) {
  return launch_cg_team_of<true>(a, d3, s);
}

}  // namespace plcg

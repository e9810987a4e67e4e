// The team kernels (plcg_team_kernels.h) for the constant stencils, and the launchers.
#include "plcg_team_kernels.h"

namespace plcg {

hipError_t launch_plcg_team(const TeamArgs &a, int l, bool d3, hipStream_t s) {
  return a.od.sx != nullptr ? launch_plcg_team_var(a, l, d3, s)
                            : launch_plcg_team_of<false>(a, l, d3, s);
}

hipError_t launch_cg_team(const TeamArgs &a, bool d3, hipStream_t s) {
  return a.od.sx != nullptr ? launch_cg_team_var(a, d3, s) : launch_cg_team_of<false>(a, d3, s);
}

}  // namespace plcg

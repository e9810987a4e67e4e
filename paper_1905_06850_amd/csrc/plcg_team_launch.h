// Arguments and launchers of the team kernels, and the workspace solve that lends them
// its mail.
#pragma once

#include "plcg_internal.h"
#include "plcg_team.h"

namespace plcg {

// Team solves (plcg_team.hip): a whole segment of Alg. 1, or all of classic CG, in one
// launch of one workgroup per tile.  Constant and Jacobi-scaled variable stencils, FP64.
struct TeamArgs {
  const double *z0;          // p(l)-CG: z_0 = u_0 / ||u_0||; CG: r_0
  const double *x;           // x at the segment start
  double *x_out;             // receives the last iterate (not x: a run may be lost)
  const DevState *st_in;
  DevState *st_out;
  HostStatus *hs;
  double *hist;              // [hist_cap][4] or NULL
  OpData od;                 // edge weights of the variable-coefficient stencil; else NULL
  void *mail, *post;         // team_mail_bytes(g), team_post_bytes()
  TeamGeom g;
  int32_t base;              // first tag of this run; tags base .. base + imax + 1 (CG: + 2 imax + 2)
  int32_t imax;              // p(l)-CG: last sweep index m + l; CG: maxit
};
hipError_t launch_plcg_team(const TeamArgs &a, int l, bool d3, hipStream_t s);
hipError_t launch_cg_team(const TeamArgs &a, bool d3, hipStream_t s);
// The same for a.od.sx != NULL (plcg_team_var.hip); the launchers above hand over to these.
hipError_t launch_plcg_team_var(const TeamArgs &a, int l, bool d3, hipStream_t s);
hipError_t launch_cg_team_var(const TeamArgs &a, bool d3, hipStream_t s);

// A whole solve (as plcg_create + plcg_solve) in ws_bytes of device memory at
// ws and kTeamWsBytes at team_ws, with no device or pinned host allocation; 2D and
// 3D stencil operators.
// check_workspace_solve makes the same argument checks without any HIP call.
int32_t check_workspace_solve(const plcg_operator_desc *op, const plcg_config *cfg,
                              size_t ws_bytes);
constexpr size_t kTeamWsBytes = team_post_bytes() + kTeamMailMax;
int32_t solve_in_workspace(const plcg_operator_desc *op, const plcg_config *cfg, void *ws,
                           size_t ws_bytes, void *team_ws, const double *d_b, double *d_x,
                           double tol, int32_t maxit, void *stream, plcg_result *out);

}  // namespace plcg

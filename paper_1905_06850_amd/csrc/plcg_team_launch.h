// Arguments and launchers of the team kernels, and the workspace solve that lends them
// its mail.
#pragma once

#include <mutex>
#include <vector>

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
inline int team_grid(const TeamArgs &a) { return team_tiles(a.g) * (a.g.near ? kXcds : 1); }
hipError_t launch_plcg_team(const TeamArgs &a, int l, bool d3, hipStream_t s);
hipError_t launch_cg_team(const TeamArgs &a, bool d3, hipStream_t s);
// The same for a.od.sx != NULL (plcg_team_var.hip); the launchers above hand over to these.
hipError_t launch_plcg_team_var(const TeamArgs &a, int l, bool d3, hipStream_t s);
hipError_t launch_cg_team_var(const TeamArgs &a, bool d3, hipStream_t s);
// p(l)-CG for a.od.ell_k > 0, g from team_rows_plan (plcg_team_csr.hip).
hipError_t launch_plcg_team_csr(const TeamArgs &a, int l, hipStream_t s);

// A batched system's tiles in a team launch of several systems.
struct TeamSlot {
  TeamGeom g;
  int32_t slot, first;       // slot of the batch; its tile 0's place in the launch
  int32_t mail;              // its faces' mail: byte offset
  int32_t pad;
};

// Sweeps of all the systems of one launch (plcg_team_batch.hip): those of the
// Jacobi-scaled variable-coefficient operator, FP64, l = 2 or 3.
struct TeamSlotsArgs {
  const TeamSlot *table;
  const int32_t *blocks;     // per place: entry of the table, or -1
  const SlotDesc *slots;
  BatchState *state;         // as BatchArgs, copy `par` is read and rewritten
  const double *part;
  int32_t *lost;
  char *mail, *post;
  int32_t par, base, sweeps, l;
};
// Unknowns per thread of those kernels.
constexpr int team_slot_v(int l, bool d3) { return team_vmax(1, l, d3, true); }
// Tags that a launch of `sweeps` sweeps uses at most.
constexpr int team_slot_tags(int sweeps) { return sweeps + 2 * kTeamLMax + 2; }
hipError_t launch_team_slots(const TeamSlotsArgs &a, bool d3, int places, int threads,
                             hipStream_t s);

// A team launch needs all its workgroups on the GPU at once, so two that do not fit
// there together would wait for each other: they take turns (within the process; across
// processes the kernels' bounded waits and the streaming sweeps take over).  A launch is made
// under the lock, between enter() and leave(), and is waited for by later ones on the GPU;
// the host waits for nothing but the lock.
static_assert(kTeamXcds == kXcds, "the plans' XCDs are the device's");
class TeamTurn {
 public:
  // Makes the stream wait until a launch of `tiles` workgroups can run; owner: what makes it
  // (a solve's or a batch's handle, which has one entry).  *near as planned on entry: a launch
  // that would have to wait for a place on one XCD spreads over all of them (the same tiles and
  // the same bits; 100 x 80 CG 3.98 us per iteration instead of 3.15).  A launch of one
  // workgroup waits for no other, but counts for those that come after it.
  hipError_t enter(const void *owner, int tiles, int cus, hipStream_t s, int32_t *near);
  // After the launches.  waits: the owner calls done() once it has waited for them.
  hipError_t leave(const void *owner, bool waits);
  void done(const void *owner);
  std::mutex mu;             // held by the caller from enter() to leave(), and around done()

 private:
  struct Run {
    const void *owner;
    int need;
    hipStream_t stream;
    // After the launches, once recorded: by leave(), or, if the owner waits, by the first that
    // has to wait for it (an event in every solve would cost it more than this list).
    hipEvent_t ev;
    bool recorded;
  };
  hipError_t after(Run &r);
  std::vector<Run> runs_;    // that may not have ended, oldest first
};
constexpr int kMaxDevices = 64;
TeamTurn &team_turn(int device);

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

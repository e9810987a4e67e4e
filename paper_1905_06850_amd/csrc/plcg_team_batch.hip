// Team launches for batched and served solves: the sweeps of many systems, each by
// its own team of workgroups (plcg_team_kernels.h), in one launch.
//
// In the ticks every system pays a launch per iteration, and reads and writes all its
// vectors in each.  Here a launch runs many sweeps of as many systems as have a CU for
// every tile, with their vectors in registers from the first sweep to the last.  The
// setup, the residuals and the reports stay with the ticks, and the state and the
// vectors of a system between launches are those that its ticks would have left.
//
// What bounds it: the exchange of faces and the owner's sum and scalar step of each
// sweep, 1.3 us with one tile, 1.9 with six, against 20 us of a tick over 24 systems.
//
// What a system's sweeps compute depends on its own tiles alone, and not on where a
// launch starts or ends: the products of a launch's last sweep are summed as within
// it and kept in the slot's state (BatchState::raw).
//
// A launch either advances a system by all of its sweeps or leaves it as it was: no tile
// stores its vectors, and tile 0 not the state, before it is sure that none gives the run up
// (`stands` in team_sweeps).
#include "plcg_batch_phase.h"
#include "plcg_team_kernels.h"

namespace plcg {

namespace {

// The sweeps of one slot: i0 .. the launch's last, t <= m.
struct SlotRun {
  static constexpr bool kSlot = true;
  const SlotDesc *S;
  BatchState *st;
  const double *part;
  int32_t *lost_word;
  int tile_, post_off, i0, m;

  __device__ inline int tile() const { return tile_; }
  __device__ inline int first() const { return i0; }
  __device__ inline int post_offset() const { return post_off; }
  __device__ inline int32_t *lost(const TeamArgs &) const { return lost_word; }
  __device__ inline double *vec(int k) const { return S->vec + (size_t)k * S->vstride; }

  // Coefficients of the sweeps t whose columns earlier launches finalised, as
  // engine_step formed them.
  template <int L>
  __device__ inline void resume(const DevState &s, SweepCoef *coef) const {
    const int t = i0 - L + (int)threadIdx.x;
    if (threadIdx.x >= L - 1 || t < 0) return;
    const int c = t & (kTRing - 1), b = (t >= 1 ? t - 1 : 0) & (kTRing - 1);
    coef[t & 3] = SweepCoef{s.gam[c], t >= 1 ? s.dlt[b] : 0.0, 1.0 / s.dlt[c], 1.0 / s.eta[c],
                            t >= 1 ? s.zeta[b] : 0.0};
  }
  // Products of sweep i0 - 1: a team launch's sums, or a tick's partial sums.
  template <int ND>
  __device__ inline void pending(double (&raw)[ND]) const {
    const int n = st->nparts, lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < ND; ++q) {
      double v = 0.0;
      for (int k = lane; k < n; k += 64) v += part[(size_t)q * kMaxStream + k];
      v = row_sum(v);
      v = swap_add<16>(v, v);
      v = swap_add<32>(v, v);
      raw[q] = n > 0 ? lane_value(v, 0) : st->raw[q];
    }
  }
  // The slot's state after the launch (tile 0's owner wave).
  template <int L>
  __device__ inline void leave(const DevState &s, int i, const double (&raw)[L + 1]) const {
    const int lane = threadIdx.x & 63;
    for (int k = lane; k < (int)(sizeof(DevState) / 8); k += 64)
      reinterpret_cast<double *>(&st->d)[k] = reinterpret_cast<const double *>(&s)[k];
    if (lane != 0) return;
    sweep_next<L>(*st, s, *S, i - 1);
    st->nparts = 0;
#pragma unroll
    for (int q = 0; q <= L; ++q) st->raw[q] = raw[q];
  }
  // Unknown p of the vectors, in the roles that the ticks give the slot's storage.
  template <int L, int R, int V>
  __device__ inline void load(bool in, int p, double (&zl)[R][V], double (&zk)[L][2][V],
                              double &pv, double &xv, int v) const {
    const int t = i0 - L;
#pragma unroll
    for (int h = 0; h < R; ++h) {
      const int j = i0 - h;
      zl[h][v] = in && j >= 0 ? vec(2 * L + j % R)[p] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < L; ++k) {
      const int cur = (t >= 0 ? t + k : k) & 1;
      zk[k][0][v] = in && (t >= 0 || k <= i0) ? vec(2 * k + cur)[p] : 0.0;
      zk[k][1][v] = in && t >= 1 ? vec(2 * k + (cur ^ 1))[p] : 0.0;
    }
    pv = in && t >= 1 ? vec(2 * L + R)[p] : 0.0;
    xv = in ? S->x[p] : 0.0;
  }
  // Before sweep i; over: only x is still needed.
  template <int L, int R, int V>
  __device__ inline void store(int i, bool over, int p, const double (&zl)[R][V],
                               const double (&zk)[L][2][V], double pv, double xv,
                               int v) const {
    S->x[p] = xv;
    if (over) return;
    const int t = i - L;
#pragma unroll
    for (int h = 0; h < R; ++h)
      if (i >= h) vec(2 * L + (i - h) % R)[p] = zl[h][v];
#pragma unroll
    for (int k = 0; k < L; ++k) {
      const int cur = (t >= 0 ? t + k : k) & 1;
      if (t >= 0 || k <= i) vec(2 * k + cur)[p] = zk[k][0][v];
      if (t >= 0) vec(2 * k + (cur ^ 1))[p] = zk[k][1][v];
    }
    if (t >= 0) vec(2 * L + R)[p] = pv;
  }
};

}  // namespace

template <int L, bool D3>
__global__ __launch_bounds__(64 * (kTeamWaves + 1)) void slots_team_kernel(TeamSlotsArgs b) {
  const int e = b.blocks[blockIdx.x];
  if (e < 0) return;
  const TeamSlot &ts = b.table[e];
  const SlotDesc &S = b.slots[ts.slot];
  BatchState *st = b.state + 2 * ts.slot + b.par;
  if (st->phase != kSweep || st->d.status != kRunning || st->solo != 0) return;
  const int line = kTeamProducts * kWordBytes;
  SlotRun run;
  run.S = &S;
  run.st = st;
  run.part = b.part + (size_t)(2 * ts.slot + b.par) * (L + 1) * kMaxStream;
  run.lost_word = b.lost + ts.slot;
  run.tile_ = blockIdx.x - ts.first;
  run.post_off = ts.first * line;
  run.i0 = st->i;
  run.m = st->m;
  TeamArgs a;
  a.st_in = &st->d;
  a.od = OpData{nullptr, nullptr, nullptr, nullptr, 0, 0, S.sx, S.sy, S.sz, nullptr};
  a.g = ts.g;
  a.mail = b.mail + ts.mail;
  a.post = b.post + run.post_off;
  a.base = b.base;
  const int last = run.i0 + b.sweeps - 1, end = run.m + L;
  a.imax = last < end ? last : end;
  a.hist = nullptr;
  team_sweeps<L, GridOp<team_slot_v(L, D3), D3, true>>(a, run);
}

template <int L, bool D3>
static hipError_t launch_of(const TeamSlotsArgs &a, int places, int threads, hipStream_t s) {
  hipLaunchKernelGGL((slots_team_kernel<L, D3>), dim3(places), dim3(threads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_team_slots(const TeamSlotsArgs &a, bool d3, int places, int threads,
                             hipStream_t s) {
  if (a.l == 2) return d3 ? launch_of<2, true>(a, places, threads, s)
                          : launch_of<2, false>(a, places, threads, s);
  if (a.l == 3) return d3 ? launch_of<3, true>(a, places, threads, s)
                          : launch_of<3, false>(a, places, threads, s);
  return hipErrorInvalidValue;
}

}  // namespace plcg

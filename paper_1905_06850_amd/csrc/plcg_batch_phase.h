// The end of a batched system's sweep, shared by the ticks and the team launches.
#pragma once

#include "plcg_internal.h"

namespace plcg {

// After sweep i, and column i of G where the solve still runs (d: the slot's scalar
// state): what the slot does next.
template <int L>
__device__ inline void sweep_next(BatchState &b, const DevState &d, const SlotDesc &S, int i) {
  // The next sweep has t' = i + 1 - l; stop once nothing is left to do.
  // FP32-refined: every end of the inner solve adds its correction
  // (kCorrect) and returns to the FP64 residual, where kStart decides.
  const int tn = i + 1 - L;
  const int done = S.mixed ? kCorrect : kFinal;
  int next = kSweep;
  if (d.status == kRunning) {
    if (tn > b.m) {
      b.total += b.m;
      b.reason = 2;
      next = done;
    }
  } else if (tn > d.last_t) {
    if (d.status == kConverged) {
      const int td = d.last_t < b.m ? d.last_t : b.m;
      b.total += td;
      b.reason = d.last_t <= b.m ? 1 : 2;
      next = done;
    } else {  // breakdown: restart from x_{t-1} (Sec. 2.2), keeping the reference norm
      b.total += d.last_t > 0 ? (d.last_t < b.m ? d.last_t : b.m) : 0;
      b.restarts += 1;
      if (b.restarts > S.max_restarts) {
        b.reason = 3;
        next = done;
      } else if (b.total >= S.maxit) {
        b.reason = 2;
        next = done;
      } else {
        next = S.mixed ? kCorrect : kResid;
      }
    }
  }
  b.phase = next;
  b.i = i + 1;
}

}  // namespace plcg

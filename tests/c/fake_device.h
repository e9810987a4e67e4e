// A GPU that is none: the HIP calls and the kernel launchers that the host side of libplcg
// (plcg_engine.cpp, plcg_batch.cpp, plcg_serve.cpp) makes, as ordinary functions on host
// memory, so that its paths can be driven on the CPU into states that a real GPU reaches
// seldom.  Work is queued and runs at the next wait.  The launchers move the scalar state
// and the phases as the kernels do, and compute nothing.
#pragma once

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <mutex>
#include <string>
#include <vector>

#include "plcg_internal.h"
#include "plcg_team_launch.h"

namespace fake {

using namespace plcg;
using Work = std::function<void()>;

inline std::recursive_mutex mu;
inline std::vector<Work> queue;                  // all streams, in the order of the calls
inline std::vector<std::string> log;             // launches, event records (of a timing event: time), waits
inline std::function<void(hipStream_t)> on_sync; // before a stream is waited for
inline std::function<bool(size_t)> refuse;       // allocations that fail
inline hipStream_t capturing = nullptr;          // the caller's stream in capture
inline std::vector<Work> captured;
inline int capture_faults = 0;                   // calls that a capture does not allow
inline hipStream_t own_capture = nullptr;        // the library's own capture of its ticks
inline std::vector<Work> *recording = nullptr;

// solves
inline bool lose_team = false;                   // team launches of solves are lost
inline int lost_status = kRunning;               // ... after a record of this status
inline int converge_t = 1 << 30;                 // solves converge at this t
inline int sweeps = 0;                           // streaming sweeps that did work

// batches
inline bool lose_slots = false;                  // team launches of batches are lost
inline int steps[64];                            // steps that each slot has made

inline void enqueue(hipStream_t s, Work w) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  if (capturing != nullptr && s == capturing)
    captured.push_back(std::move(w));
  else if (own_capture != nullptr && s == own_capture)
    recording->push_back(std::move(w));
  else
    queue.push_back(std::move(w));
}
inline void note(const char *what) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  log.push_back(what);
}
inline void drain() {
  std::lock_guard<std::recursive_mutex> lk(mu);
  std::vector<Work> q;
  q.swap(queue);
  for (Work &w : q) w();
}
inline bool not_in_capture() {
  if (capturing == nullptr) return true;
  ++capture_faults;
  return false;
}
inline void reset() {
  std::lock_guard<std::recursive_mutex> lk(mu);
  queue.clear();
  log.clear();
  captured.clear();
  on_sync = nullptr;
  refuse = nullptr;
  capturing = nullptr;
  capture_faults = 0;
  lose_team = lose_slots = false;
  lost_status = kRunning;
  converge_t = 1 << 30;
  sweeps = 0;
  memset(steps, 0, sizeof(steps));
}
inline int count(const char *what) {
  std::lock_guard<std::recursive_mutex> lk(mu);
  int n = 0;
  for (const std::string &s : log) n += s == what;
  return n;
}

// After a batched system's sweep b.i: the next, or, with m x-updates made, the end.
inline void sweep(BatchState &b, int l) {
  ++b.i;
  if (b.i - l > b.m) {
    b.total = b.m;
    b.phase = kFinal;
  }
}

inline void publish(const DevState &d, HostStatus *hs, double zeta) {
  hs->status = d.status;
  hs->last_t = d.last_t;
  hs->cols = d.cols;
  hs->zeta = zeta;
  hs->beta = d.beta;
  hs->rref = d.rref;
  hs->sumsq = d.sumsq;
}

}  // namespace fake

// ---- the HIP runtime ---------------------------------------------------------

using FakeGraph = std::vector<fake::Work>;

extern "C" {

hipError_t hipMalloc(void **p, size_t n) {
  if (!fake::not_in_capture()) return hipErrorStreamCaptureUnsupported;
  if (fake::refuse && fake::refuse(n)) return hipErrorOutOfMemory;
  *p = aligned_alloc(256, (n + 255) / 256 * 256);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
  fake::drain();
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  *p = aligned_alloc(256, (n + 255) / 256 * 256);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) {
  free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  fake::drain();
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t st) {
  std::vector<char> v((const char *)s, (const char *)s + n);
  fake::enqueue(st, [d, v]() { memcpy(d, v.data(), v.size()); });
  return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) {
  fake::drain();
  memset(d, v, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
  fake::enqueue(st, [d, v, n]() { memset(d, v, n); });
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  if (fake::capturing != nullptr && s == fake::capturing) {
    ++fake::capture_faults;
    return hipErrorStreamCaptureUnsupported;
  }
  if (fake::on_sync) fake::on_sync(s);
  fake::drain();
  return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) {
  fake::drain();
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned flags) {
  *e = reinterpret_cast<hipEvent_t>(new unsigned(flags));
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<unsigned *>(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  fake::note(*reinterpret_cast<unsigned *>(e) & hipEventDisableTiming ? "record" : "time");
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t) {
  std::lock_guard<std::recursive_mutex> lk(fake::mu);
  return fake::queue.empty() ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t) {
  fake::drain();
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = 1.f;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) {
  fake::note("wait");
  return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
  *v = 256;
  return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = reinterpret_cast<hipStream_t>(malloc(8));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
  free(s);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c) {
  *c = fake::capturing != nullptr && s == fake::capturing ? hipStreamCaptureStatusActive
                                                          : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  fake::own_capture = s;
  fake::recording = new FakeGraph;
  return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = reinterpret_cast<hipGraph_t>(fake::recording);
  fake::own_capture = nullptr;
  fake::recording = nullptr;
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(new FakeGraph(*reinterpret_cast<FakeGraph *>(g)));
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) {
  for (const fake::Work &w : *reinterpret_cast<FakeGraph *>(e)) fake::enqueue(s, w);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete reinterpret_cast<FakeGraph *>(g);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  delete reinterpret_cast<FakeGraph *>(e);
  return hipSuccess;
}

}  // extern "C"

// ---- the launchers -------------------------------------------------------------

namespace plcg {

int resident_width(int, int, int, int n) { return n <= 4800 ? 1 : 0; }
hipError_t launch_residual(const double *, const double *, double *, double *, int, int, int, int,
                           bool, const OpData &, const double *, int, int, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_start(const double *, int, DevState *st, HostStatus *hs, int mode, double tol,
                        double, double, hipStream_t s) {
  fake::enqueue(s, [=]() {
    st->sumsq = 1.0;
    if (mode != 2) {
      st->beta = st->rref = st->cg_rho = 1.0;
      st->abs_tol = tol;
      st->status = kRunning;
      st->last_t = -1;
      st->cols = 0;
    }
    fake::publish(*st, hs, 1.0);
  });
  return hipSuccess;
}
hipError_t launch_scale(const double *, double *, double *, double *, const DevState *, int,
                        hipStream_t) {
  return hipSuccess;
}
hipError_t launch_scale(const double *, float *, float *, float *, const DevState *, int,
                        hipStream_t) {
  return hipSuccess;
}
template <typename S>
hipError_t launch_x_step(S *, const S *, double, int, hipStream_t) {
  return hipSuccess;
}
template hipError_t launch_x_step<double>(double *, const double *, double, int, hipStream_t);
template hipError_t launch_x_step<float>(float *, const float *, double, int, hipStream_t);
hipError_t launch_add_correction(double *, const float *, int, hipStream_t) { return hipSuccess; }
hipError_t launch_apply(const double *, double *, int, int, int, int, bool, const OpData &,
                        hipStream_t) {
  return hipSuccess;
}
hipError_t launch_copy(const double *, double *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_jacobi_in(const double *, const double *, double *, double *, int, hipStream_t) {
  return hipSuccess;
}
hipError_t launch_jacobi_out(double *, const double *, int, hipStream_t) { return hipSuccess; }

// A sweep of p(l)-CG: carries the state, converges at t = converge_t.
template <typename S>
static hipError_t fake_sweep(const SweepArgsT<S> &a, hipStream_t s) {
  fake::note("sweep");
  fake::enqueue(s, [a]() {
    DevState d = *a.st_in;
    if (d.status == kRunning) {
      ++fake::sweeps;
      d.cols = a.i;
      if (a.i - 1 >= fake::converge_t) {
        d.status = kConverged;
        d.last_t = a.i - 1;
      }
    }
    *a.st_out = d;
    fake::publish(d, a.hs, 1.0);
  });
  return hipSuccess;
}
hipError_t launch_plcg_sweep(const SweepArgsT<double> &a, hipStream_t s) { return fake_sweep(a, s); }
hipError_t launch_plcg_sweep(const SweepArgsT<float> &a, hipStream_t s) { return fake_sweep(a, s); }
hipError_t plcg_sweep_occupancy(const SweepArgsT<double> &, int *n) {
  *n = 4;
  return hipSuccess;
}
hipError_t plcg_sweep_occupancy(const SweepArgsT<float> &, int *n) {
  *n = 4;
  return hipSuccess;
}
hipError_t launch_cg_sweep_a(const CgArgs &a, hipStream_t s) {
  fake::note("sweep");
  fake::enqueue(s, [a]() {
    DevState d = *a.st_in;
    if (d.status == kRunning) {
      fake::sweeps += a.work;
      d.cols = d.last_t = a.k;
      if (a.k >= fake::converge_t) d.status = kConverged;
    }
    *a.st_out = d;
    fake::publish(d, a.hs, 1.0);
  });
  return hipSuccess;
}
hipError_t launch_cg_sweep_b(const CgArgs &a, hipStream_t s) {
  fake::enqueue(s, [a]() { *a.st_out = *a.st_in; });
  return hipSuccess;
}
static hipError_t fake_whole(const DevState *in, DevState *out, HostStatus *hs) {
  DevState d = *in;
  d.status = kConverged;
  d.last_t = d.cols = fake::converge_t;
  *out = d;
  fake::publish(d, hs, 1e-9);
  return hipSuccess;
}
hipError_t launch_plcg_resident(const ResArgs &a, int, int, hipStream_t s) {
  fake::note("resident");
  fake::enqueue(s, [a]() { fake_whole(a.st_in, a.st_out, a.hs); });
  return hipSuccess;
}
hipError_t launch_cg_resident(const ResArgs &a, int, hipStream_t s) {
  return launch_plcg_resident(a, 0, 0, s);
}
// (method, l, d3: what the launchers have a kernel for)
static hipError_t fake_team(const TeamArgs &a, bool built, hipStream_t s) {
  if (!built || a.g.wy * a.g.wz > kTeamWaves || team_tiles(a.g) > kTeamTiles ||
      team_mail_bytes(a.g) > kTeamMailMax)
    return hipErrorInvalidValue;
  fake::note("team");
  const bool lose = fake::lose_team;
  const int status = fake::lost_status;
  fake::enqueue(s, [a, lose, status]() {
    if (!lose) {
      fake_whole(a.st_in, a.st_out, a.hs);
      return;
    }
    a.hs->lost = a.base;
    a.hs->status = status;
    a.hs->last_t = 3;
  });
  return hipSuccess;
}
static bool fake_width(int method_plcg, int l, bool d3, const TeamArgs &a) {
  const int v = a.g.v;
  return v >= 2 && (v <= (method_plcg ? 6 : 8) || (!method_plcg && v == 10)) &&
         v <= team_vmax(method_plcg, l, d3, a.od.sx != nullptr);
}
hipError_t launch_plcg_team(const TeamArgs &a, int l, bool d3, hipStream_t s) {
  return fake_team(a, l >= 1 && l <= 3 && fake_width(1, l, d3, a), s);
}
hipError_t launch_cg_team(const TeamArgs &a, bool d3, hipStream_t s) {
  return fake_team(a, fake_width(0, 1, d3, a), s);
}
hipError_t launch_plcg_team_csr(const TeamArgs &a, int l, hipStream_t s) {
  return fake_team(a, l >= 1 && l <= 3 && ((a.g.v == 2 && a.od.ell_k <= kRowsShort) ||
                                           (a.g.v == 1 && a.od.ell_k <= kRowsLong)), s);
}

// ---- batches -------------------------------------------------------------------

// A tick moves each slot by one phase or sweep, but for the sweeps of team launches.
hipError_t launch_batch_tick(const BatchArgs &a, int blocks, hipStream_t s) {
  fake::note("tick");
  fake::enqueue(s, [a, blocks]() {
    for (int k = 0; k < blocks; ++k) {
      if (a.sched[k].y >= 0) continue;
      const int slot = a.sched[k].x, par = a.tick & 1;
      const SlotDesc &S = a.slots[slot];
      BatchState &b = a.state[2 * slot + par];
      b = a.state[2 * slot + (par ^ 1)];
      if (a.team != 0 && S.team != 0 && b.solo == 0 && b.phase == kSweep) {
        if (a.lost[slot] > 0) {
          a.lost[slot] = 0;
          b.solo = 1;
          a.reports[slot].solo = 1;
        }
        continue;
      }
      if (b.phase != kEmpty && b.phase != kDone) ++fake::steps[slot];
      switch (b.phase) {
        case kInit: b.phase = kResid; break;
        case kResid: b.phase = kStart; break;
        case kStart:
          b.m = S.maxit;
          b.phase = b.m > 0 ? kScale : kFinal;
          break;
        case kScale:
          b.phase = kSweep;
          b.i = 0;
          break;
        case kSweep: fake::sweep(b, a.l); break;
        case kFinal: b.phase = kFinal2; break;
        case kFinal2: b.phase = kReport; break;
        case kReport: {
          b.phase = kDone;
          SlotReport &r = a.reports[slot];
          r.iters = b.total;
          r.reason = PLCG_REASON_MAXIT;
          r.ticket = a.tickets[slot];
          r.phase = kDone;
          break;
        }
        default: break;
      }
    }
  });
  return hipSuccess;
}

hipError_t launch_team_slots(const TeamSlotsArgs &a, bool, int places, int, hipStream_t s) {
  fake::note("slots");
  const bool lose = fake::lose_slots;
  fake::enqueue(s, [a, places, lose]() {
    for (int k = 0; k < places; ++k) {
      const TeamSlot &ts = a.table[a.blocks[k]];
      if (k != ts.first) continue;
      BatchState &b = a.state[2 * ts.slot + a.par];
      if (b.phase != kSweep || b.solo != 0) continue;
      a.lost[ts.slot] = lose ? a.base : -a.base;
      for (int n = 0; !lose && n < a.sweeps && b.phase == kSweep; ++n) {
        ++fake::steps[ts.slot];
        fake::sweep(b, a.l);
      }
    }
  });
  return hipSuccess;
}

}  // namespace plcg

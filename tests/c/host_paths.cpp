// Paths of the host side that a GPU reaches seldom, on the device of fake_device.h.
// Usage: host_paths <scenario>; prints what went wrong and returns 1, or "ok".
#include "fake_device.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <string>
#include <thread>

using namespace plcg;

namespace {

bool good = true;
#define EXPECT(cond, ...)                                   \
  do {                                                      \
    if (!(cond)) {                                          \
      good = false;                                         \
      printf("%s:%d: %s: ", __FILE__, __LINE__, #cond);     \
      printf(__VA_ARGS__);                                  \
      printf("\n");                                         \
    }                                                       \
  } while (0)

double *vec(size_t n) {
  void *p = nullptr;
  (void)hipMalloc(&p, n * sizeof(double));
  memset(p, 0, n * sizeof(double));
  return static_cast<double *>(p);
}

plcg_handle *solver(int nx, int ny, int method, int l, int check_every = 0) {
  plcg_operator_desc op{};
  op.kind = PLCG_OP_STENCIL2D5;
  op.nx = nx;
  op.ny = ny;
  op.nz = 1;
  plcg_config cfg{};
  cfg.method = method;
  cfg.l = l;
  cfg.lambda_max = 8.0;
  cfg.check_every = check_every;
  cfg.max_restarts = -1;
  plcg_handle *h = nullptr;
  const plcg_status e = plcg_create(&op, &cfg, &h);
  EXPECT(e == PLCG_OK, "plcg_create: %d %s", e, plcg_last_error());
  return h;
}

// A team launch of a solve is lost after it has written a record that says the solve broke
// down: the streaming run that follows starts from a running state and makes all its
// iterations.
void lost_record() {
  for (int method : {PLCG_METHOD_CG, PLCG_METHOD_PLCG})
    for (int check_every : {1, 64}) {
      fake::reset();
      plcg_handle *h = solver(200, 150, method, 2, check_every);
      double *b = vec(30000), *x = vec(30000);
      fake::lose_team = true;
      fake::lost_status = method == PLCG_METHOD_CG ? kCgBreak : kBroken;
      fake::converge_t = 500;
      plcg_result r{};
      EXPECT(plcg_solve(h, b, x, 1e-8, 100000, nullptr, &r) == PLCG_OK, "%s", plcg_last_error());
      EXPECT(fake::count("team") == 1, "%d team launches", fake::count("team"));
      EXPECT(r.reason == PLCG_REASON_CONVERGED && r.iters == 500,
             "method %d check_every %d: reason %d after %d iterations, %d sweeps", method,
             check_every, r.reason, r.iters, fake::sweeps);
      plcg_destroy(h);
    }
}

plcg_batch *make_batch(int l, int slots, int use_graph) {
  plcg_batch_config cfg{};
  cfg.l = l;
  cfg.max_slots = slots;
  cfg.arena_bytes = 64 << 20;
  cfg.max_restarts = -1;
  cfg.use_graph = use_graph;
  plcg_batch *b = nullptr;
  EXPECT(plcg_batch_create(&cfg, &b) == PLCG_OK, "%s", plcg_last_error());
  return b;
}

uint64_t add(plcg_batch *b, int nx, int ny, double *v, int maxit, hipStream_t s = nullptr) {
  plcg_system_desc d{};
  d.kind = PLCG_OP_STENCIL2D5;
  d.nx = nx;
  d.ny = ny;
  d.nz = 1;
  uint64_t t = 0;
  const plcg_status e = plcg_batch_add(b, &d, v, v, 1e-8, maxit, s, &t);
  EXPECT(e == PLCG_OK, "plcg_batch_add: %s", plcg_last_error());
  return t;
}

// Steps move every system by as many steps as they are asked for, or to its end, those that
// earlier ones made ahead of it included: systems
// that came with this step or an earlier one, that team launches sweep or ticks (lanes mostly
// idle: the narrow ones), alone or together.  lose: now and then all launches of a step are
// lost, and the systems that they were to sweep are swept by ticks from the next step on.
void step_counts(bool lose) {
  double *v = vec(40000);
  for (int seed = 0; seed < 300 && good; ++seed) {
    fake::reset();
    srand(seed);
    plcg_batch *b = make_batch(2 + seed % 2, 8, seed / 2 % 2);
    const bool narrow = seed / 4 % 2 != 0;
    uint64_t ticket[8] = {0};          // by slot: a system gets the first free one
    bool open[8] = {false};
    int asked[8], made[8];             // steps since it came
    int room = 8;
    for (int call = 0; call < 12 && good; ++call) {
      for (int want = rand() % 4; want > 0 && room > 0; --want, --room)
        for (int k = 0; k < 8; ++k) {
          if (open[k]) continue;
          const bool thin = narrow && rand() % 2 == 0;
          ticket[k] = add(b, thin ? 1 : 20 + rand() % 150, thin ? 3000 : 20 + rand() % 150, v,
                          rand() % 60);
          open[k] = true;
          asked[k] = made[k] = 0;
          break;
        }
      const int sizes[] = {1, 2, 3, 4, 5, 8, 15, 16, 17, 31, 40};
      const int ticks = sizes[rand() % 11];
      memset(fake::steps, 0, sizeof(fake::steps));
      fake::lose_slots = lose && rand() % 3 == 0;
      EXPECT(plcg_batch_step(b, ticks, nullptr) == PLCG_OK, "%s", plcg_last_error());
      (void)hipStreamSynchronize(nullptr);
      for (int k = 0; k < 8; ++k) {
        if (!open[k]) continue;
        plcg_result r{};
        const bool done = plcg_batch_poll(b, ticket[k], &r) == PLCG_OK;
        asked[k] += ticks;
        made[k] += fake::steps[k];
        if (fake::lose_slots) asked[k] = std::min(asked[k], made[k]);
        EXPECT(done || made[k] >= asked[k], "seed %d call %d: system %d made %d of %d steps", seed,
               call, k, made[k], asked[k]);
        if (done) {
          open[k] = false;
          ++room;
        }
      }
    }
    plcg_batch_destroy(b);
  }
}

// While a solve's team launch is on the GPU: a solve of one workgroup ends, a batch step
// returns, another solve that fits beside it waits for nothing, and one that does not is made
// to wait on the GPU, after the event of the first.
void turns() {
  fake::reset();
  fake::converge_t = 100;
  const hipStream_t slow = reinterpret_cast<hipStream_t>(vec(1));
  struct Solve {
    plcg_handle *h;
    double *b, *x;
    hipStream_t s;
    plcg_result r{};
    std::atomic<bool> done{false};
    std::thread th;
    void start() {
      th = std::thread([this]() {
        plcg_solve(h, b, x, 1e-8, 1000, s, &r);
        done = true;
      });
    }
  };
  auto make = [](Solve &v, int nx, int ny, int l, hipStream_t s) {
    v.h = solver(nx, ny, PLCG_METHOD_PLCG, l);
    v.b = vec((size_t)nx * ny);
    v.x = vec((size_t)nx * ny);
    v.s = s;
  };
  auto soon = [](const std::function<bool()> &f) {
    for (int k = 0; k < 2000 && !f(); ++k) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    return f();
  };
  Solve a, one, small, large;
  make(a, 1024, 1024, 1, slow);          // 224 tiles
  make(one, 60, 40, 2, nullptr);         // one
  make(small, 100, 80, 2, nullptr);
  make(large, 1024, 1000, 1, nullptr);
  double *v = vec(10000);
  plcg_batch *b = make_batch(2, 2, 0);
  add(b, 100, 100, v, 1000);
  plcg_batch_step(b, 4, nullptr);        // set up
  (void)hipStreamSynchronize(nullptr);
  // the slow stream's wait for its team launch does not end until it may
  std::atomic<bool> waiting{false}, may_end{false};
  fake::on_sync = [&](hipStream_t s) {
    if (s != slow || fake::count("team") == 0) return;
    waiting = true;
    while (!may_end) std::this_thread::sleep_for(std::chrono::milliseconds(1));
  };
  a.start();
  EXPECT(soon([&]() { return waiting.load(); }), "the first solve did not start");
  one.start();
  EXPECT(soon([&]() { return one.done.load(); }), "a solve of one workgroup waits");
  EXPECT(fake::count("wait") == 0, "%d waits", fake::count("wait"));
  std::atomic<bool> stepped{false};
  std::thread step([&]() {
    plcg_batch_step(b, 16, nullptr);
    stepped = true;
  });
  EXPECT(soon([&]() { return stepped.load(); }), "a batch step waits on the host");
  small.start();
  EXPECT(soon([&]() { return small.done.load(); }), "a small solve waits on the host");
  EXPECT(fake::count("wait") == 0, "%d waits", fake::count("wait"));
  large.start();
  EXPECT(soon([&]() { return large.done.load(); }), "a large solve waits on the host");
  EXPECT(fake::count("wait") >= 1, "%d waits", fake::count("wait"));
  may_end = true;
  a.th.join();
  one.th.join();
  small.th.join();
  large.th.join();
  step.join();
  for (Solve *s : {&a, &one, &small, &large})
    EXPECT(s->r.reason == PLCG_REASON_CONVERGED && s->r.iters == 100, "reason %d after %d",
           s->r.reason, s->r.iters);
  fake::on_sync = nullptr;
  plcg_batch_destroy(b);
  // of any launches that may run at once what they need fits, whatever came and went before
  srand(5);
  for (int round = 0; round < 20000; ++round) {
    int needs[8], n = rand() % 8, per = 1 + rand() % 32, need = 1 + rand() % 32;
    for (int k = 0; k < n; ++k) needs[k] = 1 + rand() % per;
    const int first = team_beside(needs, n, need, per);
    int sum = need;
    for (int k = first; k < n; ++k) sum += needs[k];
    EXPECT(first == n || sum <= per, "%d of %d", sum, per);
    EXPECT(first == 0 || sum + needs[first - 1] > per, "waits for one that fits");
  }
}

// A step of a few ticks costs a team launch beside its ticks: it makes more sweeps for them.
void few_ticks() {
  for (int ticks = 1; ticks <= 4; ++ticks) {
    fake::reset();
    double *v = vec(10000);
    plcg_batch *b = make_batch(2, 1, 0);
    add(b, 100, 80, v, 1000);
    plcg_batch_step(b, 4, nullptr);
    (void)hipStreamSynchronize(nullptr);
    fake::log.clear();
    memset(fake::steps, 0, sizeof(fake::steps));
    for (int k = 0; k < 10; ++k) plcg_batch_step(b, ticks, nullptr);
    (void)hipStreamSynchronize(nullptr);
    EXPECT(fake::steps[0] >= 20 * ticks, "%d sweeps in steps of %d ticks", fake::steps[0], ticks);
    plcg_batch_destroy(b);
  }
}

// In steps of a few ticks of a batch some of whose systems ticks sweep, the team launches of the
// others come once in sixteen ticks, and new systems are swept as soon as their setup is done.
void few_ticks_mixed() {
  for (int ticks : {1, 2, 4, 8}) {
    fake::reset();
    double *v = vec(20000);
    plcg_batch *b = make_batch(2, 3, 0);
    add(b, 1, 3000, v, 1000000);
    add(b, 100, 80, v, 1000000);
    plcg_batch_step(b, 4, nullptr);
    (void)hipStreamSynchronize(nullptr);
    fake::log.clear();
    for (int k = 0; k < 160; k += ticks) plcg_batch_step(b, ticks, nullptr);
    (void)hipStreamSynchronize(nullptr);
    const int slots = fake::count("slots");
    EXPECT(slots >= 9 && slots <= 11, "%d launches in 160 ticks, %d at a time", slots, ticks);
    EXPECT(fake::steps[1] >= 4 * 140, "%d sweeps", fake::steps[1]);
    plcg_batch_step(b, 1, nullptr);        // a launch may have been made just now
    add(b, 90, 70, v, 1000000);
    for (int k = 0; k < 6; ++k) plcg_batch_step(b, ticks, nullptr);
    (void)hipStreamSynchronize(nullptr);
    EXPECT(fake::steps[2] >= 64, "new system: %d steps", fake::steps[2]);
    plcg_batch_destroy(b);
  }
}

// How x was updated, as it is reported: on every iteration by a team launch, on every second
// one by CG's streaming sweeps, which make the run after a lost launch.
void x_updates() {
  for (bool lose : {false, true}) {
    fake::reset();
    fake::converge_t = 100;
    fake::lose_team = lose;
    plcg_handle *h = solver(200, 150, PLCG_METHOD_CG, 1);
    double *b = vec(30000), *x = vec(30000);
    plcg_result r{};
    EXPECT(plcg_solve(h, b, x, 1e-8, 1000, nullptr, &r) == PLCG_OK, "%s", plcg_last_error());
    EXPECT(r.x_update_every == (lose ? 2 : 1), "lost %d: %d", lose, r.x_update_every);
    EXPECT(r.launch_mode == PLCG_LAUNCH_STREAMING, "%d", r.launch_mode);
    plcg_destroy(h);
  }
}

// A solve of a stencil; nz 0: 2D; var: variable coefficients, Jacobi-scaled.
void solve_stencil(int nx, int ny, int nz, int method, int l, bool var) {
  static std::vector<double> edges((size_t)3 << 20, 1.0);
  fake::converge_t = 100;
  plcg_operator_desc op{};
  op.kind = nz ? PLCG_OP_STENCIL3D7 : PLCG_OP_STENCIL2D5;
  op.nx = nx;
  op.ny = ny;
  op.nz = nz ? nz : 1;
  if (var) op.cx = op.cy = edges.data();
  if (var && nz) op.cz = edges.data();
  op.jacobi = var;
  plcg_config cfg{};
  cfg.method = method;
  cfg.l = l;
  cfg.lambda_max = 12.0;
  cfg.max_restarts = -1;
  plcg_handle *h = nullptr;
  plcg_status e = plcg_create(&op, &cfg, &h);
  EXPECT(e == PLCG_OK, "%d x %d x %d: %s", nx, ny, nz, plcg_last_error());
  const size_t n = (size_t)nx * ny * op.nz;
  double *b = vec(n), *x = vec(n);
  plcg_result r{};
  e = plcg_solve(h, b, x, 1e-8, 1000, nullptr, &r);
  EXPECT(e == PLCG_OK, "%d x %d x %d method %d l %d var %d: %s", nx, ny, nz, method, l, var,
         plcg_last_error());
  plcg_destroy(h);
  free(b);
  free(x);
}

// The solves that the tests of team launches compare with the oracle and the streaming kernels
// do run in them, and the next ones that should not do not.
void which_team() {
  struct Case {
    int nx, ny, nz, method, l;
    bool var, team;
  };
  std::vector<Case> cases;
  const int dims[][3] = {{63, 61, 0}, {64, 75, 0}, {64, 76, 0}, {65, 45, 0},  {65, 61, 0},
                         {129, 91, 0}, {127, 46, 0}, {40, 300, 0}, {700, 20, 0}, {33, 17, 9},
                         {64, 16, 31}, {65, 9, 14}, {20, 64, 5}, {130, 7, 13}};
  for (const auto &d : dims)
    for (int l = 0; l <= 4; ++l)
      for (bool var : {false, true}) {
        const int n = d[0] * d[1] * (d[2] ? d[2] : 1);
        const int m = l == 0 ? PLCG_METHOD_CG : PLCG_METHOD_PLCG;
        // CG of a system that the resident kernels take too: only in one workgroup
        const bool one = l == 0 && !var && n <= PLCG_RESIDENT_MAX && d[0] > 64;
        cases.push_back({d[0], d[1], d[2], m, l ? l : 1, var, l < 4 && !one});
      }
  cases.push_back({20, 20, 0, PLCG_METHOD_PLCG, 2, false, false});       // resident
  cases.push_back({1, 4000, 0, PLCG_METHOD_PLCG, 2, false, false});
  cases.push_back({1, 5000, 0, PLCG_METHOD_PLCG, 2, false, true});
  cases.push_back({2048, 2048, 0, PLCG_METHOD_PLCG, 1, false, false});   // too large
  for (const Case &c : cases) {
    fake::reset();
    solve_stencil(c.nx, c.ny, c.nz, c.method, c.l, c.var);
    EXPECT((fake::count("team") > 0) == c.team, "%d x %d x %d method %d l %d var %d", c.nx, c.ny,
           c.nz, c.method, c.l, c.var);
  }
}

// Systems in 3D that one workgroup of the resident kernels solves sooner than a team stay there.
void resident_3d() {
  const struct {
    int nx, ny, nz, l;                // l = 0: CG
    bool team;
  } cases[] = {{33, 7, 7, 0, false},  {56, 14, 2, 0, false}, {64, 8, 8, 0, false},
               {16, 17, 17, 0, false}, {65, 9, 9, 0, true},  {16, 16, 16, 1, true},
               {16, 12, 8, 1, true},  {29, 7, 8, 2, false},  {18, 43, 2, 2, false},
               {16, 16, 8, 2, true},  {16, 127, 1, 2, false}, {89, 23, 1, 2, false},
               {45, 48, 1, 2, false}, {50, 60, 1, 2, true},  {20, 39, 4, 2, true},
               {16, 16, 16, 2, true}, {29, 7, 8, 3, true},   {18, 43, 2, 3, true}};
  for (const auto &c : cases) {
    fake::reset();
    solve_stencil(c.nx, c.ny, c.nz, c.l ? PLCG_METHOD_PLCG : PLCG_METHOD_CG, c.l ? c.l : 1, false);
    EXPECT((fake::count("team") > 0) == c.team, "%d x %d x %d l %d", c.nx, c.ny, c.nz, c.l);
  }
}

// Solves of grids in 3D that are thin along x and would send mostly empty mail stream.
void thin_3d() {
  const struct {
    int nx, ny, nz, l;                // l = 0: CG
    bool team;
  } cases[] = {{4, 60, 60, 0, true},    {4, 114, 114, 0, false}, {8, 126, 126, 0, false},
               {10, 143, 146, 0, false}, {16, 143, 146, 0, false}, {16, 114, 114, 0, true},
               {24, 143, 146, 0, true}, {146, 143, 10, 0, true}, {4, 114, 114, 1, false},
               {4, 95, 147, 2, false},  {8, 95, 147, 2, true},   {4, 100, 100, 2, true},
               {4, 114, 114, 3, true}};
  for (bool var : {false, true})
    for (const auto &c : cases) {
      if (var && c.ny * c.nz > 11000) continue;       // no team plan
      fake::reset();
      solve_stencil(c.nx, c.ny, c.nz, c.l ? PLCG_METHOD_PLCG : PLCG_METHOD_CG, c.l ? c.l : 1, var);
      EXPECT((fake::count("team") > 0) == c.team, "%d x %d x %d l %d var %d", c.nx, c.ny, c.nz,
             c.l, var);
    }
}

// Stencils of any size, method and pipeline length: none is given to a launcher that has no
// kernel for it.
void any_stencil() {
  srand(11);
  int team = 0;
  for (int k = 0; k < 1500; ++k) {
    fake::reset();
    const bool d3 = rand() % 2;
    auto side = [&](int hi) { return (int)exp(log((double)hi) * (rand() % 1000) / 999.0); };
    const int nx = side(d3 ? 130 : 1500), ny = side(d3 ? 130 : 1500), nz = d3 ? side(130) : 0;
    const int l = rand() % 9;
    solve_stencil(nx, ny, nz, l ? PLCG_METHOD_PLCG : PLCG_METHOD_CG, l ? l : 1, rand() % 2);
    team += fake::count("team") > 0;
  }
  EXPECT(team > 200, "%d of 1500 in team launches", team);
}

// CG without an iteration to make starts no team launch, which would cost it its set-up.
void no_iterations() {
  fake::reset();
  plcg_handle *h = solver(200, 150, PLCG_METHOD_CG, 1);
  double *b = vec(30000), *x = vec(30000);
  plcg_result r{};
  EXPECT(plcg_solve(h, b, x, 1e-8, 0, nullptr, &r) == PLCG_OK, "%s", plcg_last_error());
  EXPECT(r.iters == 0 && r.reason == PLCG_REASON_MAXIT, "%d %d", r.iters, r.reason);
  EXPECT(fake::count("team") == 0, "%d", fake::count("team"));
  plcg_destroy(h);
}

// The five-point matrix of a side x side grid, its rows shuffled within blocks of `block`
// (1: not): whether a solve runs in a team launch.
bool rows_team(int side, int block, int l) {
  const int n = side * side;
  std::vector<int> at(n);
  for (int k = 0; k < n; ++k) at[k] = k;
  for (int b0 = 0; b0 < n; b0 += block)
    for (int k = std::min(n, b0 + block) - 1; k > b0; --k) std::swap(at[k], at[b0 + rand() % (k - b0 + 1)]);
  std::vector<std::vector<int>> cols(n);
  for (int k = 0; k < n; ++k) {
    const int x = k % side, y = k / side;
    std::vector<int> &c = cols[at[k]];
    c.push_back(at[k]);
    if (x > 0) c.push_back(at[k - 1]);
    if (x < side - 1) c.push_back(at[k + 1]);
    if (y > 0) c.push_back(at[k - side]);
    if (y < side - 1) c.push_back(at[k + side]);
  }
  std::vector<int64_t> rp(1, 0);
  std::vector<int32_t> ci;
  std::vector<double> va;
  for (std::vector<int> &c : cols) {
    std::sort(c.begin(), c.end());
    for (int j : c) {
      ci.push_back(j);
      va.push_back(1.0);
    }
    rp.push_back((int64_t)ci.size());
  }
  fake::reset();
  fake::converge_t = 100;
  plcg_operator_desc op{};
  op.kind = PLCG_OP_CSR;
  op.nx = n;
  op.ny = op.nz = 1;
  op.nnz = (int64_t)ci.size();
  op.rowptr = rp.data();
  op.colind = ci.data();
  op.vals = va.data();
  plcg_config cfg{};
  cfg.method = PLCG_METHOD_PLCG;
  cfg.l = l;
  cfg.lambda_max = 8.0;
  cfg.max_restarts = -1;
  plcg_handle *h = nullptr;
  EXPECT(plcg_create(&op, &cfg, &h) == PLCG_OK, "%s", plcg_last_error());
  double *b = vec(n), *x = vec(n);
  plcg_result r{};
  EXPECT(plcg_solve(h, b, x, 1e-8, 1000, nullptr, &r) == PLCG_OK, "%s", plcg_last_error());
  plcg_destroy(h);
  return fake::count("team") > 0;
}

// Matrices whose rows are in an order that scatters their gathers stream where that is faster.
void rows_order() {
  const struct {
    int side, block, l;
    bool team;
  } cases[] = {{200, 1, 1, true},   {200, 1, 3, true},     {200, 64, 2, true},
               {200, 256, 2, true}, {200, 1024, 1, true},  {200, 1024, 2, false},
               {200, 1024, 3, false}, {200, 4096, 1, false}, {200, 40000, 1, false},
               {200, 40000, 2, false}, {150, 22500, 2, true}, {346, 1024, 2, false},
               {346, 1024, 1, true}, {346, 4096, 1, false}, {490, 240100, 1, true},
               {510, 260100, 2, true}};
  for (const auto &c : cases)
    EXPECT(rows_team(c.side, c.block, c.l) == c.team, "%d^2 rows shuffled within %d, p(%d): %s",
           c.side, c.block, c.l, c.team ? "streams" : "team launch");
}

// A step in a caller's capture: its replays move every system by as many steps, whether the
// batch replays groups of ticks from a graph of its own or not.
void capture() {
  double *v = vec(40000);
  for (int use_graph : {0, 1})
    for (int built : {0, 1}) {
      fake::reset();
      const hipStream_t s = reinterpret_cast<hipStream_t>(v);
      plcg_batch *b = make_batch(2, 4, use_graph);
      add(b, 100, 80, v, 1000, s);
      add(b, 1, 3000, v, 1000, s);
      plcg_batch_step(b, built ? 40 : 6, s);       // built: with its own graph in place
      (void)hipStreamSynchronize(s);
      fake::capturing = s;
      EXPECT(plcg_batch_step(b, 20, s) == PLCG_OK, "%s", plcg_last_error());
      fake::capturing = nullptr;
      EXPECT(fake::capture_faults == 0, "%d calls that a capture forbids", fake::capture_faults);
      for (int replay = 0; replay < 3; ++replay) {
        memset(fake::steps, 0, sizeof(fake::steps));
        for (fake::Work &w : fake::captured) w();
        for (int k = 0; k < 2; ++k)
          EXPECT(fake::steps[k] == 20, "use_graph %d: system %d made %d of 20 steps", use_graph, k,
                 fake::steps[k]);
      }
      plcg_batch_destroy(b);
    }
}

// The schedule's tuner times the launches that its candidates change and nothing else, and
// moves the systems that team launches sweep meanwhile.
void autotune() {
  fake::reset();
  double *v = vec(40000);
  plcg_batch *b = make_batch(2, 4, 0);
  add(b, 100, 80, v, 100000);
  add(b, 1, 3000, v, 100000);
  EXPECT(plcg_batch_autotune(b, 8, nullptr) == PLCG_OK, "%s", plcg_last_error());
  (void)hipStreamSynchronize(nullptr);
  bool timed = false;
  int trials = 0, slots = 0, ticks = 0;
  for (const std::string &s : fake::log) {
    if (s == "time") {
      timed = !timed;
      trials += timed;
    }
    if (timed) {
      slots += s == "slots";
      ticks += s == "tick";
    }
  }
  EXPECT(trials == 20 && ticks == 8 * trials, "%d trials, %d timed ticks", trials, ticks);
  EXPECT(slots == 0, "%d team launches within the timed ticks", slots);
  for (int k = 0; k < 2; ++k)
    EXPECT(fake::steps[k] >= trials * 10, "system %d made %d steps in %d trials of 8 + 2", k,
           fake::steps[k], trials);
  plcg_batch_destroy(b);
  // with nothing that ticks sweep there is nothing to choose
  fake::reset();
  b = make_batch(2, 2, 0);
  add(b, 100, 80, v, 100000);
  EXPECT(plcg_batch_autotune(b, 8, nullptr) == PLCG_OK, "%s", plcg_last_error());
  int32_t cpb[3] = {0, 0, 0};
  plcg_batch_get_schedule(b, cpb);
  EXPECT(cpb[0] == 4 && cpb[1] == 4 && cpb[2] == 4, "%d %d %d", cpb[0], cpb[1], cpb[2]);
  plcg_batch_destroy(b);
}

// On a device with no room for the mail of team launches, a solver is made, and streams (or runs
// resident), as it did before it had any.
void no_mail() {
  for (int n : {64, 200}) {
    fake::reset();
    fake::converge_t = 100;
    TeamGeom g;
    EXPECT(team_plan(1, 2, false, false, n, n, 1, 256, &g), "no plan");
    const size_t mail = team_post_bytes() + team_mail_bytes(g);
    fake::refuse = [mail](size_t bytes) { return bytes == mail; };
    plcg_handle *h = solver(n, n, PLCG_METHOD_PLCG, 2);
    if (h == nullptr) return;
    double *b = vec((size_t)n * n), *x = vec((size_t)n * n);
    plcg_result r{};
    EXPECT(plcg_solve(h, b, x, 1e-8, 1000, nullptr, &r) == PLCG_OK, "%s", plcg_last_error());
    EXPECT(r.iters == 100 && r.reason == PLCG_REASON_CONVERGED, "%d", r.iters);
    EXPECT(fake::count("team") == 0, "%d", fake::count("team"));
    plcg_destroy(h);
  }
}

}  // namespace

int main(int argc, char **argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  if (name == "lost_record") lost_record();
  else if (name == "step_counts") step_counts(false);
  else if (name == "turns") turns();
  else if (name == "capture") capture();
  else if (name == "no_mail") no_mail();
  else if (name == "rows_order") rows_order();
  else if (name == "no_iterations") no_iterations();
  else if (name == "which_team") which_team();
  else if (name == "resident_3d") resident_3d();
  else if (name == "thin_3d") thin_3d();
  else if (name == "any_stencil") any_stencil();
  else if (name == "x_updates") x_updates();
  else if (name == "few_ticks") few_ticks();
  else if (name == "few_ticks_mixed") few_ticks_mixed();
  else if (name == "autotune") autotune();
  else if (name == "step_counts_lost") step_counts(true);
  else {
    printf("unknown scenario %s\n", name.c_str());
    return 2;
  }
  if (good) printf("ok\n");
  return good ? 0 : 1;
}

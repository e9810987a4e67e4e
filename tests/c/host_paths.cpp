// Paths of the host side that a GPU reaches seldom, on the device of fake_device.h.
// Usage: host_paths <scenario>; prints what went wrong and returns 1, or "ok".
#include "fake_device.h"

#include <string>

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

}  // namespace

int main(int argc, char **argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  if (name == "lost_record") lost_record();
  else {
    printf("unknown scenario %s\n", name.c_str());
    return 2;
  }
  if (good) printf("ok\n");
  return good ? 0 : 1;
}

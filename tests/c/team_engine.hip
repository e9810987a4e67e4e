// Host replay of recorded dot-product streams through engine_gather / engine_step (the
// team kernels' scalar step, l <= 3) beside engine_column: the same state after every
// column, byte for byte, and the coefficients that read_coef would give.  Input
// as engine_replay.hip.  Prints "identical" or "MISMATCH" per case.
#include "plcg_device.h"
#include <cstdio>
#include <cstring>
#include <cmath>
using namespace plcg;

template <int L>
bool same(DevState &a, DevState &b, const double *raw, int c) {
  const EngineIn<L> in = engine_gather<L>(b, c);
  const SweepCoef cf = engine_step<L>(b, in, raw, c, nullptr);
  engine_column(a, raw, c, nullptr);
  if (memcmp(&a, &b, sizeof(DevState)) != 0) return false;
  const int t = c - 1;
  if (a.status == kBroken) return true;
  const double dm1 = t >= 1 ? a.dlt[(t - 1) % kTRing] : 0.0;
  const double zm1 = t >= 1 ? a.zeta[(t - 1) % kTRing] : 0.0;
  return cf.gam == a.gam[t % kTRing] && cf.dm1 == dm1 && cf.zm1 == zm1 &&
         cf.inv_del == 1.0 / a.dlt[t % kTRing] && cf.inv_eta == 1.0 / a.eta[t % kTRing];
}

int main(int argc, char **argv) {
  FILE *f = argc > 1 ? std::fopen(argv[1], "r") : nullptr;
  int n = 0;
  if (!f || std::fscanf(f, "%d", &n) != 1) return 2;
  bool all = true;
  for (int k = 0; k < n; ++k) {
    char name[64];
    int l, ncols;
    DevState a;
    std::memset(&a, 0, sizeof(a));
    if (std::fscanf(f, "%63s %d %d %lf %lf", name, &l, &ncols, &a.beta, &a.abs_tol) != 5) return 2;
    for (int i = 0; i < l; ++i)
      if (std::fscanf(f, "%lf", &a.sigma[i]) != 1) return 2;
    a.l = l;
    a.last_t = -1;
    a.g[0][2 * kLMax] = 1.0;
    DevState b = a;
    bool ok = true;
    for (int c = 0; c < ncols; ++c) {
      int col;
      double raw[kLMax + 1];
      if (std::fscanf(f, "%d", &col) != 1) return 2;
      for (int m = 0; m <= l; ++m)
        if (std::fscanf(f, "%lf", &raw[m]) != 1) return 2;
      if (!ok || a.status != kRunning) continue;
      ok = l == 1   ? same<1>(a, b, raw, col)
           : l == 2 ? same<2>(a, b, raw, col)
                    : same<3>(a, b, raw, col);
    }
    std::printf("%s %s status %d\n", name, ok ? "identical" : "MISMATCH", (int)a.status);
    all = all && ok;
  }
  return all ? 0 : 1;
}

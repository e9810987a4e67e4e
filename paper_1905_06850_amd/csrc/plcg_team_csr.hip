// Team launches of p(l)-CG for assembled matrices: the rows' values and column offsets
// stay in registers beside the vectors, and z_i travels whole, one word per unknown, so
// that a row gathers its neighbours from wherever they are.
//
// What bounds it: the round trip of the words (posted past the L2s, gathered by the
// rows' K loads per wave, 1.2 us) and the owner's sum of the products, one after the
// other at l = 1; in the streaming kernels it was the launch (300 x 201, five entries per
// row, us per iteration: p(1) 6.1 -> 3.0, p(2) 5.3 -> 2.7, p(3) 5.5 -> 2.4).
#include "plcg_team_kernels.h"

namespace plcg {

namespace {

// A wave of rows: 64 lanes x V rows of up to K entries (ELL copy).
// z_i's words lie in one of four copies: those of z_{i+1} may be posted once everybody
// has read the copy's last, z_{i-3}; the coefficients of sweep i, which z_{i+1} needs, come
// from products that all workgroups formed after that (l <= 3).
template <int V_, int K>
struct RowsOp {
  static constexpr int V = V_;
  static constexpr bool D3 = false;
  struct Shared {
    int none;
  };
  struct Words {
    word4 w[K];
  };
  int n, p0, copy_bytes;
  rsrc_t mail;
  int ci[V][K];                      // byte offsets of the entries' words
  double va[V][K];
  __device__ inline RowsOp(const TeamArgs &a, int tile, int, int sw, Shared &)
      : n(a.g.nx), p0((tile * a.g.wz + sw) * 64 * V + (int)(threadIdx.x & 63)),
        copy_bytes(a.g.gx * a.g.wz * 64 * V * kWordBytes),
        mail(mail_rsrc(a.mail, 4 * copy_bytes)) {}
  __device__ inline int at(int v) const { return p0 + 64 * v; }
  __device__ inline bool in(int v) const { return at(v) < n; }
  // entries beyond the row's are its own unknown times zero, as in the ELL copy
  __device__ inline void prepare(const TeamArgs &a) {
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (int k = 0; k < K; ++k) {
        ci[v][k] = at(v) * kWordBytes;
        va[v][k] = 0.0;
        if (in(v) && k < a.od.ell_k) {
          const size_t e = (size_t)k * a.od.ell_ld + at(v);
          ci[v][k] = a.od.ci[e] * kWordBytes;
          va[v][k] = a.od.va[e];
        }
      }
  }
  __device__ inline int copy(int i) const { return (i & 3) * copy_bytes; }
  __device__ inline void post(int i, unsigned tag, const double (&u)[V]) {
#pragma unroll
    for (int v = 0; v < V; ++v) word_post(mail, at(v) * kWordBytes, copy(i), u[v], tag);
  }
  __device__ inline void gather(int i, int v, Words &w) {
    fresh();
    if (in(v)) {
#pragma unroll
      for (int k = 0; k < K; ++k) w.w[k] = word_load(mail, ci[v][k], copy(i));
    }
  }
  __device__ inline void request(int i, Words &w) { gather(i, 0, w); }
  // (A z_i)_v, the entries added in the row's order; false: lost
  __device__ inline bool sums(int i, unsigned tag, const double (&)[V], Words &w, double (&s)[V],
                              Patience &pat) {
    bool ok = true;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if (v > 0) gather(i, v, w);
      while (true) {
        bool miss = false;
        if (in(v)) {
#pragma unroll
          for (int k = 0; k < K; ++k) miss = miss || !word_is(w.w[k], tag);
        }
        if (!__any(miss)) break;
        if (pat.over()) {
          ok = false;
          break;
        }
        fresh();
        if (miss) {
#pragma unroll
          for (int k = 0; k < K; ++k)
            if (!word_is(w.w[k], tag)) w.w[k] = word_load(mail, ci[v][k], copy(i));
        }
      }
      s[v] = 0.0;
      if (in(v)) {
#pragma unroll
        for (int k = 0; k < K; ++k) s[v] = fma(va[v][k], word_value(w.w[k]), s[v]);
      }
    }
    return ok;
  }
  __device__ inline double apply(double, double s) const { return s; }
};

}  // namespace

template <int L, int V, int K>
__global__ __launch_bounds__(64 * (kTeamWaves + 1)) void rows_team_kernel(TeamArgs a) {
  if (own_tile(a) < 0) return;
  team_sweeps<L, RowsOp<V, K>>(a, WholeRun{a});
}

template <int L>
static hipError_t launch_rows(const TeamArgs &a, hipStream_t s) {
  const dim3 grid(team_grid(a)), block(team_threads(a.g));
  if (a.g.v == 2 && a.od.ell_k <= kRowsShort)
    hipLaunchKernelGGL((rows_team_kernel<L, 2, kRowsShort>), grid, block, 0, s, a);
  else if (a.g.v == 1 && a.od.ell_k <= kRowsLong)
    hipLaunchKernelGGL((rows_team_kernel<L, 1, kRowsLong>), grid, block, 0, s, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_plcg_team_csr(const TeamArgs &a, int l, hipStream_t s) {
  switch (l) {
    case 1: return launch_rows<1>(a, s);
    case 2: return launch_rows<2>(a, s);
    case 3: return launch_rows<3>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace plcg

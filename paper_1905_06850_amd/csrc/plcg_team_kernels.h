// Team kernels of libplcg: a whole run of Alg. 1, or of classic CG, in ONE launch
// of up to one workgroup per CU, for systems that fit the chip's registers.
//
// What bounds an iteration of a system of ten thousand to a million unknowns
// in the streaming kernels is not its bytes but the launch: 2.4 us between
// dependent launches, then the ramp of the grid and one memory round trip for the
// scalar state, one for the vectors.  Here the vectors stay in registers (512 KB
// per CU) and the workgroups wait for each other inside the launch instead.
//
// Mail: a double travels as one 16-byte word {low half, tag, high half, tag},
// written and read past the XCDs' L2 caches (agent scope) with no fence at all.
// The reader polls the word until both tags are the awaited one; each 8-byte half
// is written by one access, so a half with the right tag holds the right data, and
// nothing needs to be ordered against anything else.  Tags grow by one per
// iteration and are never used twice by a handle, so the mail is not cleared between
// solves.  A release fence per iteration, by comparison, writes back an XCD's L2.
// Measured with 256 workgroups: 1.35 us for an exchange of faces with four neighbours,
// 1.85 us for the sum of one double over all workgroups (1.15 and 1.5 with 64).
//
// Every wait is bounded by time: a workgroup that waits too long (another process
// or a long kernel on another stream holds CUs, so that not all workgroups run at
// once) marks the run as lost and leaves; so do the others, and the host runs the
// segment with the streaming kernels.  x is written to a.x_out, which the host
// copies to the caller's x only after a run that was not lost.
//
// Tiles (plcg_team.h): a wave holds 64 columns x V rows, thread = column; the x
// neighbours come from the adjacent lanes, the rows above and below from the
// thread's own registers, from LDS where another wave holds them and from the mail
// where another workgroup does.  Columns and rows beyond the grid hold zeros, which
// are what the Dirichlet boundary reads there, and are posted like any others.
#pragma once

#include "plcg_device.h"
#include "plcg_team_launch.h"

namespace plcg {

namespace {

typedef unsigned int word4 __attribute__((ext_vector_type(4)));
using rsrc_t = __amdgpu_buffer_rsrc_t;

constexpr int kAgentScope = 16;              // cache policy bit sc1 of the buffer accesses
constexpr long long kStartTicks = 25000000;  // 0.25 s of the 100 MHz clock: first waits of a run
constexpr long long kWaitTicks = 200000000;  // 2 s: any later one
constexpr long long kLastTicks = 2000000000; // 20 s: one that all workgroups are known to answer
constexpr int kNever = 0x7fffffff;

__device__ inline rsrc_t mail_rsrc(void *p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, bytes, 0x00027000);
}
// A word at byte offset lane_off (per lane) + off (uniform in the wave: a scalar register).
__device__ inline word4 word_load(rsrc_t r, int lane_off, int off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, off, kAgentScope);
}
__device__ inline void word_post(rsrc_t r, int lane_off, int off, double v, unsigned tag) {
  word4 w;
  w.x = (unsigned)__double2loint(v);
  w.y = tag;
  w.z = (unsigned)__double2hiint(v);
  w.w = tag;
  // The whole offset goes into the lane's register and none into a scalar one: with a scalar
  // offset the compiler lets the next vector instruction overwrite the 16 bytes' registers
  // at once, and the store, which reads them over several cycles, then sent lanes 12 to
  // 15 of each row the new contents (words with one tag, which were waited for in vain).
  // Without one it keeps the wait states that such a store needs.
  __builtin_amdgcn_raw_buffer_store_b128(w, r, lane_off + off, 0, kAgentScope);
}
__device__ inline bool word_is(const word4 &w, unsigned tag) { return w.y == tag && w.w == tag; }
__device__ inline double word_value(const word4 &w) {
  return __hiloint2double((int)w.z, (int)w.x);
}
// Loads after this are new ones, whatever was loaded from there before.
__device__ inline void fresh() { asm volatile("" ::: "memory"); }

// The workgroup's tile, or -1.  Workgroups are dealt to the XCDs in turn, so that of a near
// launch, which has kXcds of them per tile, the tiles' ones share the first XCD.
__device__ inline int own_tile(const TeamArgs &a) {
  if (a.g.near == 0) return blockIdx.x;
  return blockIdx.x % kXcds == 0 ? (int)(blockIdx.x / kXcds) : -1;
}

// The time limit of a wait, and what ends it early: another workgroup's loss.
struct Patience {
  int32_t *lost;
  int base;
  long long t0, limit;
  int spins;
  bool gone;                     // a sum was given up
  __device__ inline void reset(bool start, long long later = kWaitTicks) {
    spins = 0;
    limit = start ? kStartTicks : later;
  }
  // after a poll that did not find its word
  __device__ inline bool over() {
    if ((++spins & 255) != 0) return false;
    const long long now = wall_clock64();
    if (spins == 256) {
      t0 = now;
      return false;
    }
    return now - t0 > limit ||
           __hip_atomic_load(lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == base;
  }
};

// Polls a word (already requested once into w) until it carries the tag.
__device__ inline bool word_wait(rsrc_t r, int lane_off, int off, unsigned tag, word4 &w,
                                 Patience &pat) {
  while (!word_is(w, tag)) {
    if (pat.over()) return false;
    fresh();
    w = word_load(r, lane_off, off);
  }
  return true;
}

__device__ inline double lane_value(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// ---- sums across the lanes of a wave --------------------------------------

// Sum over the 16 lanes of each row of the wave, in every lane of the row.
__device__ inline double row_sum(double v) {
  v += dpp_move<0x128, 0xF>(v);      // row_ror:8
  v += dpp_move<0x124, 0xF>(v);
  v += dpp_move<0x122, 0xF>(v);
  v += dpp_move<0x121, 0xF>(v);
  return v;
}
// a + b after the upper half (W = 32) or the odd rows (W = 16) of a were swapped with
// the lower half / the even rows of b: lanes of a's kept part sum a, the others b.
template <int W>
__device__ inline double swap_add(double a, double b) {
  unsigned al = (unsigned)__double2loint(a), ah = (unsigned)__double2hiint(a);
  unsigned bl = (unsigned)__double2loint(b), bh = (unsigned)__double2hiint(b);
  if constexpr (W == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  }
}
// Sums over the wave of ND <= 4 products at once: every lane of row m ends with
// product m (rows beyond ND: ND = 1, 2 repeat them, ND = 3 holds zero).  Folding the
// products into one register first takes 7 additions where a sum of its own for each
// takes 6 ND, and the lane moves that go with them.
template <int ND>
__device__ inline double products_sum(const double (&a)[ND]) {
  static_assert(ND >= 1 && ND <= 4, "up to four products");
  double s;
  if constexpr (ND == 1) {
    s = swap_add<16>(a[0], a[0]);
    s = swap_add<32>(s, s);
  } else if constexpr (ND == 2) {
    s = swap_add<16>(a[0], a[1]);
    s = swap_add<32>(s, s);
  } else {
    const double s02 = swap_add<32>(a[0], a[2]);
    const double s13 = swap_add<32>(a[1], ND == 4 ? a[ND - 1] : 0.0);
    s = swap_add<16>(s02, s13);
  }
  return row_sum(s);
}

// ---- sums across the workgroups --------------------------------------------

// The workgroup's products from the streaming waves' sums (zeros where there is no wave):
// product m in every lane of row m of the owner wave.
template <int ND>
__device__ inline double own_products(const double (*red)[4]) {
  const int lane = threadIdx.x & 63, k = lane & 15, row = lane >> 4;
  return row_sum(row < ND ? red[k][row] : 0.0);
}
// The entry beyond the last wave's makes them NaN.  A wave that loses its wait finishes its
// sweep, as the barriers need it, on words that were not the awaited ones; its workgroup's
// products are NaN then, and so is everybody's sum of them: nobody goes on, or ends its run as
// one that was not lost, on what came of those words.  (As a flag that the owner looks at before it
// posts them this cost 1 to 3 % of a p(2) sweep, as a NaN in the wave's own sums 1 %.)
__device__ inline void spoil_products(double (*red)[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) red[kTeamWaves][m] = __builtin_nan("");
}

// The owner wave posts its workgroup's products of column c.
template <int ND>
__device__ inline void post_products(rsrc_t post, double own, int c, int tile, unsigned tag) {
  const int lane = threadIdx.x & 63, row = lane >> 4;
  if ((lane & 15) == 0 && row < ND)
    word_post(post, row * kWordBytes,
              ((c & (kTeamRing - 1)) * kTeamTiles + tile) * kTeamProducts * kWordBytes, own, tag);
}

// Adds this lane's share of a column's posted products, PER words per lane at
// lane_off + off, off + step, ..., to s in this order.  They are polled in rounds: those
// that have not arrived are requested again, all of a round's requests in flight
// together (one after the other, the words of 256 workgroups took 3.9 us).  Only the
// last word of a lane may be missing from the share (apart > 0: those of the lane's words
// that lie beyond `left` are).  meanwhile() is run once, while the first round travels.
// pat.gone: lost.  (Kept there, as of a result `ok && share_sum(...)` over the cases
// below the compiler left ok undefined on the path of one case.)
template <int PER, typename F>
__device__ inline void share_sum(rsrc_t post, int lane_off, int off, int step, unsigned tag,
                                 bool has, bool last, double &s, Patience &pat, F meanwhile,
                                 int left = 0, int apart = 0) {
  word4 w[PER];
  bool miss[PER], mine[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j)
    miss[j] = mine[j] = apart > 0 ? has && left > j * apart : j < PER - 1 ? has : last;
  bool first = true;
  while (true) {
    fresh();
#pragma unroll
    for (int j = 0; j < PER; ++j)
      if (miss[j]) w[j] = word_load(post, lane_off, off + j * step);
    if (first) meanwhile();
    first = false;
    bool any = false;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      miss[j] = miss[j] && !word_is(w[j], tag);
      any = any || miss[j];
    }
    if (!__any(any)) break;
    if (pat.over()) {
      pat.gone = true;
      return;
    }
  }
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (mine[j]) s += word_value(w[j]);
}

// The owner wave's sum of the posted products of column c over all workgroups.
// Each row of 16 lanes takes one product (one of the rows that share it, when ND <= 2)
// and each lane of it every 16th tile of the row's share, in ascending order; then the
// lanes are added, so every workgroup gets the same bits.  out[m] is uniform in the
// wave.  own: this workgroup's products, which are the sum where it is alone.
// false: lost.
template <int ND, typename F>
__device__ inline bool team_sum(rsrc_t post, int c, unsigned tag, int tiles, double own,
                                double (&out)[ND], Patience &pat, F meanwhile) {
  if (tiles == 1) {
    meanwhile();
#pragma unroll
    for (int q = 0; q < ND; ++q) out[q] = lane_value(own, 16 * q);
    return true;
  }
  constexpr int G = ND == 1 ? 4 : ND == 2 ? 2 : 1;      // rows per product
  const int lane = threadIdx.x & 63, k = lane & 15, row = lane >> 4;
  const int m = G == 4 ? 0 : G == 2 ? (row & 1) : row;
  const int first = k + 16 * (G == 4 ? row : G == 2 ? (row >> 1) : 0);
  const int line = kTeamProducts * kWordBytes, step = 16 * G * line;
  const int lane_off = first * line + m * kWordBytes;
  int off = (c & (kTeamRing - 1)) * kTeamTiles * line;
  double s = 0.0;
  // up to eight words per lane at a time (their registers)
  const int per = tiles < 128 * G ? (tiles + 16 * G - 1) / (16 * G) : 8;
  const bool has = m < ND && first < tiles;
  const bool last = m < ND && first + 16 * G * (per - 1) < tiles;
  switch (per) {
    case 1: share_sum<1>(post, lane_off, off, step, tag, has, last, s, pat, meanwhile); break;
    case 2: share_sum<2>(post, lane_off, off, step, tag, has, last, s, pat, meanwhile); break;
    case 3: share_sum<3>(post, lane_off, off, step, tag, has, last, s, pat, meanwhile); break;
    case 4: share_sum<4>(post, lane_off, off, step, tag, has, last, s, pat, meanwhile); break;
    case 5: share_sum<5>(post, lane_off, off, step, tag, has, last, s, pat, meanwhile); break;
    case 6: share_sum<6>(post, lane_off, off, step, tag, has, last, s, pat, meanwhile); break;
    case 7: share_sum<7>(post, lane_off, off, step, tag, has, last, s, pat, meanwhile); break;
    default: share_sum<8>(post, lane_off, off, step, tag, has, last, s, pat, meanwhile); break;
  }
  // beyond 128 G tiles, four words at a time
  for (int t0 = 128 * G; t0 < tiles; t0 += 64 * G) {
    off += (t0 == 128 * G ? 8 : 4) * step;
    const int left = tiles - t0 - first;
    share_sum<4>(post, lane_off, off, step, tag, m < ND && left > 0, false, s, pat, []() {}, left, 16 * G);
  }
  s = row_sum(s);
  if constexpr (G == 4) s = swap_add<16>(s, s);
  if constexpr (G >= 2) s = swap_add<32>(s, s);
#pragma unroll
  for (int q = 0; q < ND; ++q) out[q] = lane_value(s, 16 * q);
  return !pat.gone;
}

__device__ inline void state_copy(const DevState *src, DevState *dst) {
  const double *s = reinterpret_cast<const double *>(src);
  double *d = reinterpret_cast<double *>(dst);
  for (int k = threadIdx.x; k < (int)(sizeof(DevState) / 8); k += blockDim.x) d[k] = s[k];
}

// ---- faces ------------------------------------------------------------------

// A streaming wave and its lane.
template <int V, bool D3>
struct Place : TeamPlace {
  int lane, lane16, nz;
  bool col;                          // the lane's column lies in the grid
  int p0, stride;                    // unknown v is p0 + v * stride
  int xin, xout;                     // the lane's word of the x faces
  __device__ inline Place(const TeamGeom &g, int tile, int sw)
      : TeamPlace(g, V, D3, tile, sw) {
    lane = threadIdx.x & 63;
    lane16 = lane * kWordBytes;
    nz = g.nz;
    col = x0 + lane < g.nx && y < g.ny;
    stride = g.nx * g.ny;
    p0 = x0 + lane + g.nx * y + z0 * stride;
    const int k = (lane & 31) * kWordBytes;
    xin = (lane < 32 ? in_w : in_e) + k;
    xout = (lane < 32 ? out_w : out_e) + k;
  }
  __device__ inline bool in(int v) const { return col && z0 + v < nz; }
  // the lane carries a word of an x face (V <= 32)
  __device__ inline bool xlane() const { return (lane & 31) < V && (lane < 32 ? west : east); }
  __device__ inline bool ymail() const { return D3 && (ylo || yhi); }
};

// Posts a wave's part of its tile's faces of u.  The x faces' values are first
// gathered from lanes 0 and 63 into one lane per row, so that they leave in one store.
template <int V, bool D3>
__device__ inline void halo_post(rsrc_t mail, const Place<V, D3> &pl, int copy, unsigned tag,
                                 const double (&u)[V]) {
  if (pl.zlo) word_post(mail, pl.lane16, copy + pl.out_zlo, u[0], tag);
  if (pl.zhi) word_post(mail, pl.lane16, copy + pl.out_zhi, u[V - 1], tag);
  if (pl.west || pl.east) {
    double xv = 0.0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const double w = lane_value(u[v], 0), e = lane_value(u[v], 63);
      xv = (pl.lane & 31) == v ? (pl.lane < 32 ? w : e) : xv;
    }
    if (pl.xlane()) word_post(mail, pl.xout, copy, xv, tag);
  }
  if constexpr (D3) {
    if (pl.ymail()) {
#pragma unroll
      for (int v = 0; v < V; ++v)
        word_post(mail, pl.lane16, copy + pl.out_y + v * 64 * kWordBytes, u[v], tag);
    }
  }
}

// The mailed neighbours of a wave's rows: x holds, in lanes v and 32 + v, the west
// and east neighbours of row v; zlo and zhi the rows below the first and above the
// last.  (Rows beyond a y side are taken one by one, halo_y.)
struct Halo {
  double x, zlo, zhi;
};
struct HaloWords {
  word4 x, lo, hi;
};

template <int V, bool D3>
__device__ inline void halo_request(rsrc_t mail, const Place<V, D3> &pl, int copy, HaloWords &w) {
  fresh();
  if (pl.xlane()) w.x = word_load(mail, pl.xin, copy);
  if (pl.zlo) w.lo = word_load(mail, pl.lane16, copy + pl.in_zlo);
  if (pl.zhi) w.hi = word_load(mail, pl.lane16, copy + pl.in_zhi);
}

// The requested words' values once they carry the tag (zero where no tile lies).
template <int V, bool D3>
__device__ inline bool halo_wait(rsrc_t mail, const Place<V, D3> &pl, int copy, unsigned tag,
                                 HaloWords &w, Halo &h, Patience &pat) {
  bool ok = true;
  h.x = h.zlo = h.zhi = 0.0;
  if (pl.xlane()) {
    ok = word_wait(mail, pl.xin, copy, tag, w.x, pat);
    h.x = word_value(w.x);
  }
  if (pl.zlo) {
    ok = ok && word_wait(mail, pl.lane16, copy + pl.in_zlo, tag, w.lo, pat);
    h.zlo = word_value(w.lo);
  }
  if (pl.zhi) {
    ok = ok && word_wait(mail, pl.lane16, copy + pl.in_zhi, tag, w.hi, pat);
    h.zhi = word_value(w.hi);
  }
  return ok;
}

// The rows beyond the wave's y side, f(v, value) for each, two words in flight.
template <int V, bool D3, typename F>
__device__ inline bool halo_y(rsrc_t mail, const Place<V, D3> &pl, int copy, unsigned tag,
                              Patience &pat, F f) {
  bool ok = true;
  if constexpr (D3) {
    if (pl.ymail()) {
      constexpr int C = 2;
#pragma unroll
      for (int v0 = 0; v0 < V; v0 += C) {
        word4 w[C];
        fresh();
#pragma unroll
        for (int k = 0; k < C; ++k)
          if (v0 + k < V)
            w[k] = word_load(mail, pl.lane16, copy + pl.in_y + (v0 + k) * 64 * kWordBytes);
#pragma unroll
        for (int k = 0; k < C; ++k)
          if (v0 + k < V) {
            ok = ok && word_wait(mail, pl.lane16, copy + pl.in_y + (v0 + k) * 64 * kWordBytes, tag,
                                 w[k], pat);
            f(v0 + k, word_value(w[k]));
          }
      }
    }
  }
  return ok;
}

// Rows a wave shares with the workgroup's other waves: all of them in 3D (the y
// neighbours read each), the first and the last in 2D.
template <int V, bool D3>
constexpr int shared_rows() { return D3 ? V : 2; }

template <int V, bool D3, int SR>
__device__ inline void rows_put(double (*rows)[SR][64], const Place<V, D3> &pl,
                                const double (&u)[V]) {
  if constexpr (D3) {
#pragma unroll
    for (int v = 0; v < V; ++v) rows[pl.sw][v][pl.lane] = u[v];
  } else {
    rows[pl.sw][0][pl.lane] = u[0];
    rows[pl.sw][SR - 1][pl.lane] = u[V - 1];
  }
}

// Edge weights of the variable-coefficient operator (VarOp's Jacobi-scaled form: unit
// diagonal) at a workgroup's unknowns, in LDS, read by every sweep: 580 doubles per wave at
// V = 4 in 2D, where registers would take 26 per thread.  x(v, k) is the edge west of
// lane k (64: east of lane 63), z(v) below row v (V: above the last), y(v, 0 / 1) below and
// above row v.  Edges that leave the grid are zero.  The constant stencil has none.
template <int V, bool D3, bool VAR>
struct Edges {
  __device__ inline void load(const OpData &, const Place<V, D3> &, const TeamGeom &) {}
  __device__ inline double x(const Place<V, D3> &, int, int) const { return 1.0; }
  __device__ inline double y(const Place<V, D3> &, int, int) const { return 1.0; }
  __device__ inline double z(const Place<V, D3> &, int) const { return 1.0; }
};
template <int V, bool D3>
struct Edges<V, D3, true> {
  double ex[kTeamWaves][V][65];
  double ez[kTeamWaves][V + 1][64];
  double ey[D3 ? kTeamWaves : 1][D3 ? V : 1][2][64];
  __device__ inline void load(const OpData &od, const Place<V, D3> &pl, const TeamGeom &g) {
    const int X = pl.x0 + pl.lane;
    const double *wz = D3 ? od.sz : od.sy;    // 2D: the z axis here is the grid's y
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int Z = pl.z0 + v, p = pl.p0 + v * pl.stride, row = pl.y + g.ny * Z;
      const int xe = row * (g.nx + 1) + X;
      const bool in = pl.in(v);
      ex[pl.sw][v][pl.lane] = in && X > 0 ? od.sx[xe] : 0.0;
      if (pl.lane == 63) ex[pl.sw][v][64] = in && X < g.nx - 1 ? od.sx[xe + 1] : 0.0;
      if (v == 0) ez[pl.sw][0][pl.lane] = in && Z > 0 ? wz[p] : 0.0;
      ez[pl.sw][v + 1][pl.lane] = in && Z < g.nz - 1 ? wz[p + pl.stride] : 0.0;
      if constexpr (D3) {
        const int ye = p + Z * g.nx;
        ey[pl.sw][v][0][pl.lane] = in && pl.y > 0 ? od.sy[ye] : 0.0;
        ey[pl.sw][v][1][pl.lane] = in && pl.y < g.ny - 1 ? od.sy[ye + g.nx] : 0.0;
      }
    }
  }
  __device__ inline double x(const Place<V, D3> &pl, int v, int k) const { return ex[pl.sw][v][k]; }
  __device__ inline double y(const Place<V, D3> &pl, int v, int side) const {
    return ey[pl.sw][v][side][pl.lane];
  }
  __device__ inline double z(const Place<V, D3> &pl, int v) const { return ez[pl.sw][v][pl.lane]; }
};
// s + c u, the neighbour u behind an edge of weight c (1 for the constant stencil).
template <bool VAR>
__device__ inline double edge_add(double c, double u, double s) {
  if constexpr (VAR) return fma(c, u, s);
  else return s + u;
}
// (A u) from u and its weighted neighbour sum.
template <bool D3, bool VAR>
__device__ inline double from_sum(double u, double s) {
  if constexpr (VAR) return u - s;
  else return fma(D3 ? 6.0 : 4.0, u, -s);
}

// Face-neighbour sums of a thread's V unknowns u: what the wave and the workgroup
// hold first, then (halo_add) what came by mail.
template <int V, bool D3, bool VAR, int SR>
__device__ inline void rows_sum(double (*rows)[SR][64], const Place<V, D3> &pl, const TeamGeom &g,
                                const Edges<V, D3, VAR> &ed, const double (&u)[V],
                                double (&s)[V]) {
#pragma unroll
  for (int v = 0; v < V; ++v) {
    if constexpr (VAR)
      s[v] = fma(ed.x(pl, v, pl.lane + 1), lane_next(u[v]), ed.x(pl, v, pl.lane) * lane_prev(u[v]));
    else
      s[v] = lane_prev(u[v]) + lane_next(u[v]);
  }
  if constexpr (D3) {
    if (pl.wyi > 0) {
#pragma unroll
      for (int v = 0; v < V; ++v)
        s[v] = edge_add<VAR>(ed.y(pl, v, 0), rows[pl.sw - 1][v][pl.lane], s[v]);
    }
    if (pl.wyi < g.wy - 1) {
#pragma unroll
      for (int v = 0; v < V; ++v)
        s[v] = edge_add<VAR>(ed.y(pl, v, 1), rows[pl.sw + 1][v][pl.lane], s[v]);
    }
  }
  const int up = D3 ? g.wy : 1;          // waves between z-adjacent rows
#pragma unroll
  for (int v = 1; v < V; ++v) s[v] = edge_add<VAR>(ed.z(pl, v), u[v - 1], s[v]);
  if (pl.wzi > 0) s[0] = edge_add<VAR>(ed.z(pl, 0), rows[pl.sw - up][SR - 1][pl.lane], s[0]);
#pragma unroll
  for (int v = 0; v < V - 1; ++v) s[v] = edge_add<VAR>(ed.z(pl, v + 1), u[v + 1], s[v]);
  if (pl.wzi < g.wz - 1)
    s[V - 1] = edge_add<VAR>(ed.z(pl, V), rows[pl.sw + up][0][pl.lane], s[V - 1]);
}

template <int V, bool D3, bool VAR>
__device__ inline void halo_add(const Place<V, D3> &pl, const Edges<V, D3, VAR> &ed, const Halo &h,
                                double (&s)[V]) {
  if (pl.west || pl.east) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const double w = lane_value(h.x, v), e = lane_value(h.x, 32 + v);
      const double u = pl.lane == 0 ? w : pl.lane == 63 ? e : 0.0;
      s[v] = edge_add<VAR>(ed.x(pl, v, pl.lane == 0 ? 0 : 64), u, s[v]);
    }
  }
  s[0] = edge_add<VAR>(ed.z(pl, 0), h.zlo, s[0]);
  s[V - 1] = edge_add<VAR>(ed.z(pl, V), h.zhi, s[V - 1]);
}

// A streaming wave's part of the operator, as team_sweeps uses it: its unknowns, the
// posting of z_i (tag: of sweep i) and A z_i in two steps, the neighbours' request and
// their sum.  This one: the stencils.
template <int V_, bool D3_, bool VAR>
struct GridOp {
  static constexpr int V = V_;
  static constexpr bool D3 = D3_;
  static constexpr int SR = shared_rows<V, D3>();
  struct Shared {
    double rows[2][kTeamWaves][SR][64];            // z_i rows by sweep parity
    Edges<V, D3, VAR> edges;
  };
  using Words = HaloWords;
  const Place<V, D3> pl;
  const TeamGeom &g;
  Shared &sh;
  const int copy_bytes;
  const rsrc_t mail;
  __device__ inline GridOp(const TeamArgs &a, int tile, int tiles, int sw, Shared &s)
      : pl(a.g, tile, sw), g(a.g), sh(s), copy_bytes(tiles * a.g.words * kWordBytes),
        mail(mail_rsrc(a.mail, 2 * copy_bytes)) {}
  __device__ inline bool in(int v) const { return pl.in(v); }
  __device__ inline int at(int v) const { return pl.p0 + v * pl.stride; }
  __device__ inline void prepare(const TeamArgs &a) { sh.edges.load(a.od, pl, a.g); }
  __device__ inline int copy(int i) const { return (i & 1) * copy_bytes; }
  __device__ inline void post(int i, unsigned tag, const double (&u)[V]) {
    halo_post<V, D3>(mail, pl, copy(i), tag, u);
    rows_put<V, D3, SR>(sh.rows[i & 1], pl, u);
  }
  __device__ inline void request(int i, Words &w) { halo_request<V, D3>(mail, pl, copy(i), w); }
  // neighbour sums of z_i, from the wave, the workgroup and the mail; false: lost
  __device__ inline bool sums(int i, unsigned tag, const double (&u)[V], Words &w, double (&s)[V],
                              Patience &pat) {
    Halo hal;
    rows_sum<V, D3, VAR, SR>(sh.rows[i & 1], pl, g, sh.edges, u, s);
    bool ok = halo_wait<V, D3>(mail, pl, copy(i), tag, w, hal, pat);
    halo_add<V, D3, VAR>(pl, sh.edges, hal, s);
    return halo_y<V, D3>(mail, pl, copy(i), tag, pat, [&](int v, double y) {
             s[v] = edge_add<VAR>(sh.edges.y(pl, v, pl.ylo ? 0 : 1), y, s[v]);
           }) && ok;
  }
  __device__ inline double apply(double u, double s) const { return from_sum<D3, VAR>(u, s); }
};

}  // namespace

// One run of Alg. 1, sweeps i = 0 .. imax, with the per-unknown arithmetic of the
// streaming kernels (Sweep<L>) and their scalar engine.
//
// Wave 0 of every workgroup is an owner: it posts the workgroup's products of sweep
// i-1, adds up everybody's and finalises a column of G, the same bits in every
// workgroup.  Waves 1 .. wy*wz stream.  One workgroup barrier per sweep (two for
// l = 1), and between workgroups only the mail:
//   l = 1   sweep i needs column i: the streaming waves collect their faces of
//           z_i and form A z_i while the owner waits for the products;
//   l = 2   column i is finalised during sweep i, as in the resident kernel;
//   l = 3   there is one sweep more to spare: column i-1 is finalised during
//           sweep i, its words have arrived by then and the sweep is as long as
//           the exchange of faces, not as the reduction and the scalar step.
// Within a sweep the faces are requested first, everything that does not need
// A z_i (bases, p, x) is computed while they travel (l >= 2), and z_{i+1}'s faces
// are posted before the products are formed.
//
// RUN is WholeRun, or SlotRun for the sweeps of a batched system: those from i0 on to
// iend, or to the stop if that is known by then, from the slot's vectors and state and back.
template <int L, typename OP, typename RUN>
__device__ __forceinline__ void team_sweeps(const TeamArgs &a, const RUN &run) {
  constexpr int ND = L + 1;
  constexpr int R = L - 1 > 2 ? L - 1 : 2;
  constexpr bool SLOT = RUN::kSlot;
  constexpr int LAG = L >= 3 && !SLOT ? 1 : 0;
  constexpr int V = OP::V;
  constexpr bool D3 = OP::D3;
  // (also a batched system's x at l = 3, for the registers)
  constexpr bool XL = team_x_in_lds(L, V, D3) || (SLOT && L == 3 && !D3);
  constexpr bool PL = team_p_in_lds(L, V, D3);
  constexpr bool Z1 = !SLOT && team_z1_in_lds(L, V);
  constexpr int NT = kTeamWaves * 64;
  __shared__ double xs[XL ? V : 1][XL ? NT : 1], ps[PL ? V : 1][PL ? NT : 1];
  __shared__ double z1s[Z1 ? V : 1][Z1 ? NT : 1];
  __shared__ double red[2][kTeamWaves + 1][4];     // wave sums by sweep parity
  __shared__ typename OP::Shared ops;
  __shared__ DevState sh;
  __shared__ SweepCoef coef[4];                    // of sweep t, at t & 3
  // The first sweep that does not run: set before a barrier that comes before that
  // sweep's look at it, to a later sweep than any that a wave may be about to look
  // for, so all waves (and, from the same products, all workgroups) leave together.
  __shared__ int stop_at;
  __shared__ int gone;                             // SLOT: this workgroup lost the run
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = SLOT ? a.g.wy * a.g.wz : (blockDim.x >> 6) - 1;
  const int tile = run.tile(), tiles = team_tiles(a.g);
  const int i0 = run.first();
  const unsigned base = (unsigned)(a.base - i0);   // the tag of sweep i is base + i
  int32_t *const lost = run.lost(a);
  Patience pat{lost, a.base, 0, 0, 0, false};

  state_copy(a.st_in, &sh);
  if (threadIdx.x < 2 * (kTeamWaves + 1) * 4) (&red[0][0][0])[threadIdx.x] = 0.0;
  if (threadIdx.x == 0) {
    stop_at = kNever;
    if constexpr (SLOT) gone = 0;
  }
  __syncthreads();
  auto lose = [&](int at) {
    atomicMin(&stop_at, at);
    if constexpr (L >= 2) {                  // l = 1: all leave before the sweep's products
      spoil_products(red[0]);
      spoil_products(red[1]);
    }
    if constexpr (SLOT) gone = 1;
    __hip_atomic_store(lost, a.base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  };
  // Whether sweep i does not run.  A batched system's launch ends after sweep iend, but
  // not between the column that stops the solve and its last sweep.
  auto ended = [&](int i) {
    const int at = stop_at;
    return at <= i || (SLOT && i > a.imax && at == kNever);
  };

  // SLOT: whether the run surely stands once it has ended before sweep i, for everybody, so
  // that a workgroup may store its vectors at once.  It does after two sums of the launch:
  // every workgroup has made the first then, so all are on the GPU, and the waits after it end
  // for no time that they take, only if the run is lost already.  Otherwise everybody waits for
  // the products of the last sweep: a workgroup that gave up before has not posted any, and
  // if one has not begun, its neighbours wait for its faces in vain.
  auto stands = [&](int i) {
    const int at = stop_at;
    return tiles == 1 || (at - L < i - 1 ? at - L : i - 1) - i0 >= 2;
  };
  constexpr long long kLater = SLOT ? kLastTicks : kWaitTicks;

  if (wave == 0) {
    const rsrc_t post = mail_rsrc(a.post, (int)(team_post_bytes() - run.post_offset()));
    double *const hist = tile == 0 ? a.hist : nullptr;
    bool running = true;
    double own = 0.0, own_before = 0.0;   // this workgroup's products, this column's and the last's
    // column c from everybody's products; at: the sweep that a loss ends.  The entries of
    // the state it needs are gathered while the first poll travels (l = 3: before it, whose
    // words and entries together would not fit the registers).
    auto column = [&](int c, int at, bool over) {
      EngineIn<L> in;
      double raw[ND];
      if constexpr (L >= 3) in = engine_gather<L>(sh, c);
      if (!team_sum<ND>(post, c, base + (unsigned)c, tiles, LAG ? own_before : own, raw, pat, [&]() {
            if constexpr (L < 3) in = engine_gather<L>(sh, c);
          })) {
        if (lane == 0) lose(over ? kNever : at);
        running = false;
        return;
      }
      if constexpr (SLOT) {
        if (over && tile == 0) run.template leave<L>(sh, c, raw);
      }
      if (!over) {
        if (lane == 0) {
          coef[(c - 1) & 3] = engine_step<L>(sh, in, raw, c, hist);
          // the stop: x_{last_t} is formed by sweep last_t + L
          if (sh.status != kRunning) atomicMin(&stop_at, sh.last_t + L + 1);
        }
        running = __builtin_amdgcn_readfirstlane(sh.status) == kRunning;
      }
    };
    if constexpr (SLOT) {
      run.template resume<L>(sh, coef);
      if (i0 >= 1) {
        double raw[ND];
        run.template pending<ND>(raw);
        if (lane == 0) {
          coef[(i0 - 1) & 3] = engine_step<L>(sh, engine_gather<L>(sh, i0), raw, i0, nullptr);
          if (sh.status != kRunning) stop_at = sh.last_t + L + 1;
        }
        running = __builtin_amdgcn_readfirstlane(sh.status) == kRunning;
      }
    }
    __syncthreads();
    int i = i0;
    for (; SLOT || i <= a.imax; ++i) {
      // SLOT, over: everybody posts the products of the last sweep, of which the next
      // launch makes column i, and tile 0 collects them, so that it rewrites the state
      // only after all the others have read it; all do where the run may not stand.
      const bool over = SLOT && ended(i), ask = over && !stands(i);
      pat.reset(!over && i - i0 <= 1 + LAG, kLater);
      if (i >= (SLOT ? i0 + 1 : 1) && (running || (over && !gone))) {
        own_before = own;
        own = own_products<ND>(red[(i - 1) & 1]);
        if (tiles > 1) post_products<ND>(post, own, i, tile, base + (unsigned)i);
        if (i > LAG && (!over || ask || tile == 0)) column(i - LAG, L == 1 ? i : i + 1, over);
      }
      if (SLOT && over) {
        if (ask) __syncthreads();
        break;
      }
      if (L == 1) __syncthreads();
      if (!SLOT && stop_at <= i) break;
      __syncthreads();
    }
    // the last posted column, where it is finalised a sweep late
    if (LAG && i > a.imax && i >= 2 && running && stop_at > i) {
      own_before = own;
      column(a.imax, 0, false);
    }
  } else if (SLOT && wave > nw) {
    // waves that this system does not need keep the barriers
    __syncthreads();
    int i = i0;
    for (; !ended(i); ++i) __syncthreads();
    if (!stands(i)) __syncthreads();
  } else {
    OP op(a, tile, tiles, wave - 1, ops);
    static_assert(R == 2, "z_i and z_{i-1}");
    double zl[Z1 ? 1 : R][V], zk[L][2][V], pr[PL ? 1 : V], xr[XL ? 1 : V];
    // p, x and z_{i-1} are touched at most twice a sweep: the widest kernels keep them in LDS
    const int slot = threadIdx.x - 64;
    auto x = [&](int v) -> double & {
      if constexpr (XL) return xs[v][slot];
      else return xr[v];
    };
    auto p = [&](int v) -> double & {
      if constexpr (PL) return ps[v][slot];
      else return pr[v];
    };
    auto z1 = [&](int v) -> double & {
      if constexpr (Z1) return z1s[v][slot];
      else return zl[R - 1][v];
    };
    double sig[L];
#pragma unroll
    for (int k = 0; k < L; ++k) sig[k] = lane_value(sh.sigma[k], 0);
    if constexpr (SLOT) {
#pragma unroll
      for (int v = 0; v < V; ++v)
        run.template load<L, R>(op.in(v), op.at(v), zl, zk, p(v), x(v), v);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const double z0 = op.in(v) ? a.z0[op.at(v)] : 0.0;
        zl[0][v] = z0;
        z1(v) = 0.0;
#pragma unroll
        for (int k = 0; k < L; ++k) {
          zk[k][0][v] = k == 0 ? z0 : 0.0;
          zk[k][1][v] = 0.0;
        }
        p(v) = 0.0;
        x(v) = op.in(v) ? a.x[op.at(v)] : 0.0;
      }
    }
    op.prepare(a);
    op.post(i0, base + (unsigned)i0, zl[0]);
    __syncthreads();
    int i = i0;
    for (; SLOT || i <= a.imax; ++i) {
      const int t = i - L;
      const unsigned tag = base + (unsigned)i;
      SweepCoef cf;
      typename OP::Words words;
      double s[V];
      if (L >= 2 && ended(i)) break;
      pat.reset(i - i0 <= 1, kLater);
      op.request(i, words);
      auto neighbours = [&]() {
        if (!op.sums(i, tag, zl[0], words, s, pat)) lose(L == 1 ? i : i + 1);
      };
      // bases k = l-1 .. 0, p_t and x_t: nothing here needs A z_i.  (t = 0: the
      // previous vectors are zero, and so are their coefficients.)
      auto recurrences = [&]() {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          double above = zl[0][v];
#pragma unroll
          for (int k = L - 1; k >= 0; --k) {
            const double ck = zk[k][0][v];
            const double sk = sig[k] - cf.gam;
            const double nk = fma(-cf.dm1, zk[k][1][v], fma(sk, ck, above)) * cf.inv_del;
            zk[k][1][v] = ck;
            zk[k][0][v] = nk;
            above = ck;
          }
          const double pv = p(v);
          x(v) = fma(cf.zm1, pv, x(v));
          p(v) = fma(-cf.dm1, pv, zk[0][1][v]) * cf.inv_eta;
        }
      };
      if constexpr (L == 1) {
        neighbours();
        __syncthreads();
        if (stop_at <= i) break;
      }
      cf = coef[t & 3];
      if constexpr (L >= 2) {
        if (t >= 0) recurrences();
        neighbours();
      }
      // z_{i+1} into s
      if (t >= 0) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const double zc = zl[0][v];
          const double w = op.apply(zc, s[v]);
          const double zn = fma(-cf.dm1, z1(v), fma(-cf.gam, zc, w)) * cf.inv_del;
          s[v] = op.in(v) ? zn : 0.0;
        }
      } else {
        const double sigma_i = sh.sigma[i];
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const double w = op.apply(zl[0][v], s[v]);
          const double zn = fma(-sigma_i, zl[0][v], w);
          s[v] = op.in(v) ? zn : 0.0;
        }
      }
      op.post(i + 1, tag + 1, s);
      if constexpr (L == 1) {
        if (t >= 0) recurrences();
      }
      double acc[ND];
#pragma unroll
      for (int m = 0; m < ND; ++m) acc[m] = 0.0;
      if (t >= 0) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const double zn = s[v];
          acc[0] = fma(zn, zk[0][0][v], acc[0]);
          acc[L] = fma(zn, zn, acc[L]);
          if constexpr (L >= 2) acc[L - 1] = fma(zn, zl[0][v], acc[L - 1]);
          if constexpr (L >= 3) acc[L - 2] = fma(zn, z1(v), acc[L - 2]);
        }
      } else {
        // start-up: z_{i+1} is also the first vector of basis i+1
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const double zn = s[v];
#pragma unroll
          for (int m = 1; m <= L - 2; ++m) {
            const int h = L - 1 - m;
            if (h <= i) acc[m] = fma(zn, h == 0 ? zl[0][v] : z1(v), acc[m]);
          }
          if (i == L - 1) acc[0] = fma(zn, zk[0][0][v], acc[0]);
#pragma unroll
          for (int k = 1; k < L; ++k)
            if (i == k - 1) zk[k][0][v] = zn;
          acc[L] = fma(zn, zn, acc[L]);
          if constexpr (L >= 2) acc[L - 1] = fma(zn, zl[0][v], acc[L - 1]);
        }
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        z1(v) = zl[0][v];
        zl[0][v] = s[v];
      }
      const double q = products_sum<ND>(acc);
      if ((lane & 15) == 0 && (lane >> 4) < ND) red[i & 1][wave - 1][lane >> 4] = q;
      __syncthreads();
    }
    if constexpr (SLOT) {
      if (!stands(i)) __syncthreads();     // it does now, or it is lost
      if (!gone) {
        const bool over = stop_at <= i || i - L > run.m;
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (op.in(v))
            run.template store<L, R>(i, over, op.at(v), zl, zk, p(v), x(v), v);
      }
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (op.in(v)) a.x_out[op.at(v)] = x(v);
    }
  }
  if constexpr (SLOT) return;
  __syncthreads();
  if (tile == 0) {
    state_copy(&sh, a.st_out);
    // The record holds all that the host asks of the run, with the residual norm of the
    // iterate that x_out holds (run_segment's t_done): it need not fetch the state.
    if (threadIdx.x == 0) {
      const int m = a.imax - L, t = sh.last_t > 0 ? sh.last_t : 0;
      const int done = sh.status == kRunning || t > m ? m : t;
      publish(sh, a.hs, done == 0 ? sh.beta : fabs(sh.zeta[done % kTRing]), sh.cols);
    }
  }
}

// A whole segment of a solve: the launch's workgroups are the system's tiles.
struct WholeRun {
  static constexpr bool kSlot = false;
  const TeamArgs &a;
  __device__ inline int tile() const { return own_tile(a); }
  __device__ inline int first() const { return 0; }
  __device__ inline int post_offset() const { return 0; }
  __device__ inline int32_t *lost(const TeamArgs &a) const { return &a.hs->lost; }
};

template <int L, int V, bool D3, bool VAR>
__global__ __launch_bounds__(64 * (kTeamWaves + 1)) void plcg_team_kernel(TeamArgs a) {
  if (own_tile(a) < 0) return;
  team_sweeps<L, GridOp<V, D3, VAR>>(a, WholeRun{a});
}

// Classic CG (Sec. 2.1), iterations k = 0 .. imax - 1 and the stopping test of
// iterate imax, with the arithmetic of the resident kernel.  Two exchanges per
// iteration: r_k's faces and (r_k, r_k), then (p_k, A p_k).  p_k is formed from the
// faces of r_k by their reader too (p = r + beta p with the owner's roundings), so
// beta does not have to travel before them.  All threads form the scalars
// themselves from the same sums.
//
// 2D: the rows of r_k shared with other waves stand beside the mailed ones, and their
// p is kept the same way.  3D: every wave's p rows are shared through LDS, and the p
// beyond a y side lies there too.  x is touched once per iteration: where V
// unknowns per thread leave no room for it in registers (XL) it lies in LDS, and
// q = A p is then formed a second time for r -= alpha q instead of being held.
template <int V, bool D3, bool VAR>
__global__ __launch_bounds__(64 * (kTeamWaves + 1)) void cg_team_kernel(TeamArgs a) {
  if (own_tile(a) < 0) return;
  constexpr int SR = shared_rows<V, D3>();
  constexpr bool XL = D3 ? V > 5 : V > 6;
  constexpr bool QK = !XL && !(D3 && V > 4);    // q held
  __shared__ double rows[kTeamWaves][SR][64];   // 2D: r rows; 3D: p rows
  __shared__ double py[D3 ? kTeamWaves : 1][D3 ? V : 1][64];   // 3D: p beyond the y side
  __shared__ double xl[XL ? V : 1][XL ? kTeamWaves * 64 : 1];
  __shared__ double red[kTeamWaves + 1][4];
  __shared__ Edges<V, D3, VAR> edges;
  __shared__ double total[2];                   // (r, r), (p, A p)
  __shared__ DevState sh;
  // Whether this workgroup lost a wait, by the product it was on the way to: [0] is written
  // between the last barrier of an iteration and that before (r, r) is looked at, [1] from
  // there to the barrier before (p, A p) is, and each is looked at by all waves right after
  // its barrier, while none may write it.
  __shared__ int lost[2];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = own_tile(a), tiles = team_tiles(a.g);
  const unsigned base = (unsigned)a.base;
  Patience pat{&a.hs->lost, a.base, 0, 0, 0, false};

  state_copy(a.st_in, &sh);
  if (threadIdx.x < (kTeamWaves + 1) * 4) (&red[0][0])[threadIdx.x] = 0.0;
  if (threadIdx.x == 0) lost[0] = lost[1] = 0;
  __syncthreads();
  double rho = sh.cg_rho, beta = 0.0;
  const double abs_tol = sh.abs_tol;
  int status = sh.status, last_t = sh.last_t, cols = sh.cols;
  auto lose = [&](int q) {
    lost[q] = 1;
    spoil_products(red);
    __hip_atomic_store(&a.hs->lost, a.base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  };
  // After (r_k, r_k) is known: false when iteration k does not run.
  auto next = [&](int k) {
    if (k >= 1) {
      const double rr = total[0];
      cols = k;
      last_t = k;
      if (!isfinite(rr)) {
        status = kCgBreak;
        return false;
      }
      beta = rr / rho;
      rho = rr;
      if (sqrt(rho) < abs_tol) {
        status = kConverged;
        return false;
      }
    }
    return k < a.imax;
  };
  auto curvature_ok = [&](int k) {
    const double pq = total[1];
    if (isfinite(pq) && pq > 0.0) return true;
    status = kCgBreak;
    last_t = k;
    return false;
  };

  if (status != kRunning) {
    // nothing to do: the caller's test of x_0 already stopped the solve
  } else if (wave == 0) {
    const rsrc_t post = mail_rsrc(a.post, (int)team_post_bytes());
    // a reduction: column 2k is (r_k, r_k), 2k+1 is (p_k, A p_k)
    auto reduce = [&](int c) {
      const double own = own_products<1>(red);
      if (tiles > 1) post_products<1>(post, own, c, tile, base + (unsigned)c);
      double t[1];
      const bool ok = team_sum<1>(post, c, base + (unsigned)c, tiles, own, t, pat, []() {});
      if (lane == 0) {
        total[c & 1] = t[0];
        if (!ok) lose(c & 1);
      }
    };
    __syncthreads();                       // the streaming waves' r_0 rows
    for (int k = 0;; ++k) {
      pat.reset(k == 0);
      if (k >= 1) reduce(2 * k);
      __syncthreads();                     // (r, r), and the faces of r_k
      if (lost[0] || !next(k)) break;
      if (D3) __syncthreads();             // p rows
      __syncthreads();                     // wave sums of (p, A p)
      reduce(2 * k + 1);
      __syncthreads();                     // (p, A p)
      if (lost[1] || !curvature_ok(k)) break;
      __syncthreads();                     // wave sums of (r, r), r rows
    }
  } else {
    const Place<V, D3> pl(a.g, tile, wave - 1);
    const int copy_bytes = tiles * a.g.words * kWordBytes;
    const rsrc_t mail = mail_rsrc(a.mail, 2 * copy_bytes);
    double r[V], p[V], x[XL ? 1 : V], q[QK ? V : 1];
    Halo ph{0.0, 0.0, 0.0};                // p beyond the wave, as halo_wait lays it out
#pragma unroll
    for (int v = 0; v < V; ++v) {
      r[v] = pl.in(v) ? a.z0[pl.p0 + v * pl.stride] : 0.0;
      p[v] = 0.0;
      const double xv = pl.in(v) ? a.x[pl.p0 + v * pl.stride] : 0.0;
      if constexpr (XL) xl[v][threadIdx.x - 64] = xv;
      else x[v] = xv;
      if constexpr (D3) py[pl.sw][v][lane] = 0.0;
    }
    edges.load(a.od, pl, a.g);
    halo_post<V, D3>(mail, pl, 0, base, r);
    if constexpr (!D3) rows_put<V, D3, SR>(rows, pl, r);
    __syncthreads();
    // (A p)_v from the registers and ph; 3D reads the other waves' rows as well
    auto apply = [&](int v) {
      double s;
      if constexpr (VAR)
        s = fma(edges.x(pl, v, lane + 1), lane_next(p[v]), edges.x(pl, v, lane) * lane_prev(p[v]));
      else
        s = lane_prev(p[v]) + lane_next(p[v]);
      if (pl.west || pl.east) {
        const double w = lane_value(ph.x, v), e = lane_value(ph.x, 32 + v);
        s = edge_add<VAR>(edges.x(pl, v, lane == 0 ? 0 : 64), lane == 0 ? w : lane == 63 ? e : 0.0,
                          s);
      }
      if constexpr (D3) {
        s = edge_add<VAR>(edges.y(pl, v, pl.wyi > 0 || pl.ylo ? 0 : 1),
                          pl.wyi > 0 ? rows[pl.sw - 1][v][lane] : py[pl.sw][v][lane], s);
        if (pl.wyi < a.g.wy - 1)
          s = edge_add<VAR>(edges.y(pl, v, 1), rows[pl.sw + 1][v][lane], s);
        else if (pl.wyi > 0)
          s = edge_add<VAR>(edges.y(pl, v, 1), py[pl.sw][v][lane], s);
      }
      const double below = v > 0                ? p[v > 0 ? v - 1 : 0]
                           : D3 && pl.wzi > 0 ? rows[pl.sw - a.g.wy][SR - 1][lane]
                                              : ph.zlo;
      s = edge_add<VAR>(edges.z(pl, v), below, s);
      const double above = v < V - 1                      ? p[v < V - 1 ? v + 1 : 0]
                           : D3 && pl.wzi < a.g.wz - 1 ? rows[pl.sw + a.g.wy][0][lane]
                                                       : ph.zhi;
      s = edge_add<VAR>(edges.z(pl, v + 1), above, s);
      const double w = from_sum<D3, VAR>(p[v], s);
      return pl.in(v) ? w : 0.0;
    };
    for (int k = 0;; ++k) {
      const int copy = (k & 1) * copy_bytes, copy_next = copy_bytes - copy;
      const unsigned tag = base + (unsigned)k;
      // the faces of r_k
      HaloWords hw;
      Halo rh;
      pat.reset(k == 0);
      halo_request<V, D3>(mail, pl, copy, hw);
      if (!halo_wait<V, D3>(mail, pl, copy, tag, hw, rh, pat)) lose(0);
      if constexpr (!D3) {
        if (pl.wzi > 0) rh.zlo = rows[pl.sw - 1][SR - 1][lane];
        if (pl.wzi < a.g.wz - 1) rh.zhi = rows[pl.sw + 1][0][lane];
      }
      __syncthreads();
      if (lost[0] || !next(k)) break;
      // beta = 0 and p = 0 in iteration 0
#pragma unroll
      for (int v = 0; v < V; ++v) p[v] = fma(beta, p[v], r[v]);
      ph.x = fma(beta, ph.x, rh.x);
      ph.zlo = fma(beta, ph.zlo, rh.zlo);
      ph.zhi = fma(beta, ph.zhi, rh.zhi);
      if constexpr (D3) {
        rows_put<V, D3, SR>(rows, pl, p);
        if (!halo_y<V, D3>(mail, pl, copy, tag, pat, [&](int v, double u) {
              double &w = py[pl.sw][v][lane];
              w = fma(beta, w, u);
            }))
          lose(1);
        __syncthreads();
      }
      double acc[1] = {0.0};
#pragma unroll
      for (int v = 0; v < V; ++v) {
        if constexpr (XL) __builtin_amdgcn_sched_barrier(0);   // one row's values live at a time
        const double w = apply(v);
        if constexpr (QK) q[v] = w;
        acc[0] = fma(p[v], w, acc[0]);
      }
      {
        const double s = products_sum<1>(acc);
        if (lane == 0) red[wave - 1][0] = s;
      }
      __syncthreads();
      __syncthreads();
      if (lost[1] || !curvature_ok(k)) break;
      const double alpha = rho / total[1];
#pragma unroll
      for (int v = 0; v < V; ++v) {
        double w;
        if constexpr (XL) __builtin_amdgcn_sched_barrier(0);
        if constexpr (QK) w = q[v];
        else w = apply(v);
        r[v] = fma(-alpha, w, r[v]);
      }
      halo_post<V, D3>(mail, pl, copy_next, tag + 1, r);
      if constexpr (!D3) rows_put<V, D3, SR>(rows, pl, r);
      acc[0] = 0.0;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        if constexpr (XL) {
          double &xv = xl[v][threadIdx.x - 64];
          xv = fma(alpha, p[v], xv);
        } else {
          x[v] = fma(alpha, p[v], x[v]);
        }
        acc[0] = fma(r[v], r[v], acc[0]);
      }
      {
        const double s = products_sum<1>(acc);
        if (lane == 0) red[wave - 1][0] = s;
      }
      __syncthreads();
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (pl.in(v)) {
        if constexpr (XL) a.x_out[pl.p0 + v * pl.stride] = xl[v][threadIdx.x - 64];
        else a.x_out[pl.p0 + v * pl.stride] = x[v];
      }
  }
  __syncthreads();
  if (tile == 0) {
    if (threadIdx.x == 0) {
      sh.status = status;
      sh.last_t = last_t;
      sh.cols = cols;
      sh.cg_rho = rho;
      sh.cg_beta = beta;
    }
    __syncthreads();
    state_copy(&sh, a.st_out);
    if (threadIdx.x == 0) publish(sh, a.hs, sqrt(rho), 2 * cols);
  }
}

// ---- launchers, instantiated by plcg_team.hip (constant stencils) and plcg_team_var.hip ----

template <bool VAR, int L, int V, bool D3>
hipError_t launch_plcg_team_lv(const TeamArgs &a, hipStream_t s) {
  if constexpr (V <= team_vmax(1, L, D3, VAR)) {
    hipLaunchKernelGGL((plcg_team_kernel<L, V, D3, VAR>), dim3(team_grid(a)),
                       dim3(team_threads(a.g)), 0, s, a);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <bool VAR, int L, bool D3>
hipError_t launch_plcg_team_l(const TeamArgs &a, hipStream_t s) {
  switch (a.g.v) {
    case 2: return launch_plcg_team_lv<VAR, L, 2, D3>(a, s);
    case 3: return launch_plcg_team_lv<VAR, L, 3, D3>(a, s);
    case 4: return launch_plcg_team_lv<VAR, L, 4, D3>(a, s);
    case 5: return launch_plcg_team_lv<VAR, L, 5, D3>(a, s);
    case 6: return launch_plcg_team_lv<VAR, L, 6, D3>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <bool VAR>
hipError_t launch_plcg_team_of(const TeamArgs &a, int l, bool d3, hipStream_t s) {
  switch (l) {
    case 1:
      return d3 ? launch_plcg_team_l<VAR, 1, true>(a, s) : launch_plcg_team_l<VAR, 1, false>(a, s);
    case 2:
      return d3 ? launch_plcg_team_l<VAR, 2, true>(a, s) : launch_plcg_team_l<VAR, 2, false>(a, s);
    case 3:
      return d3 ? launch_plcg_team_l<VAR, 3, true>(a, s) : launch_plcg_team_l<VAR, 3, false>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <bool VAR, int V, bool D3>
hipError_t launch_cg_team_v(const TeamArgs &a, hipStream_t s) {
  if constexpr (V <= team_vmax(0, 1, D3, VAR)) {
    hipLaunchKernelGGL((cg_team_kernel<V, D3, VAR>), dim3(team_grid(a)),
                       dim3(team_threads(a.g)), 0, s, a);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <bool VAR, bool D3>
hipError_t launch_cg_team_d(const TeamArgs &a, hipStream_t s) {
  switch (a.g.v) {
    case 2: return launch_cg_team_v<VAR, 2, D3>(a, s);
    case 3: return launch_cg_team_v<VAR, 3, D3>(a, s);
    case 4: return launch_cg_team_v<VAR, 4, D3>(a, s);
    case 5: return launch_cg_team_v<VAR, 5, D3>(a, s);
    case 6: return launch_cg_team_v<VAR, 6, D3>(a, s);
    case 7: return launch_cg_team_v<VAR, 7, D3>(a, s);
    case 8: return launch_cg_team_v<VAR, 8, D3>(a, s);
    case 10: return launch_cg_team_v<VAR, 10, D3>(a, s);
    default: return hipErrorInvalidValue;
  }
}

template <bool VAR>
hipError_t launch_cg_team_of(const TeamArgs &a, bool d3, hipStream_t s) {
  return d3 ? launch_cg_team_d<VAR, true>(a, s) : launch_cg_team_d<VAR, false>(a, s);
}

}  // namespace plcg

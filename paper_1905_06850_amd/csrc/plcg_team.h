// Geometry and arguments of the team kernels (plcg_team.hip): how a grid is cut
// into tiles, one per workgroup, and where a tile's mail lies.  Plain C++ apart
// from the pointers, so that the host and the tests can check it.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <vector>

#if defined(__HIP__)
#define PLCG_HD __host__ __device__
#else
#define PLCG_HD
#endif

namespace plcg {

constexpr int kTeamWaves = 15;        // streaming waves per workgroup, beside one owner wave
constexpr int kTeamTiles = 256;       // tiles at most (one workgroup per CU)
constexpr int kTeamXcds = 8;          // XCDs that share the tiles of a launch
constexpr int kTeamRing = 16;         // slots of the posted products, by column
constexpr int kTeamProducts = 8;      // words of a workgroup's products of a column: a line
                                      // of 128 bytes of its own, l + 1 <= 4 of them used
constexpr int kTeamLMax = 3;          // deepest pipeline with a team kernel
constexpr size_t kTeamMailMax = (size_t)32 << 20;
constexpr int kWordBytes = 16;        // a posted double: {low, tag, high, tag}

// Words of a wave's row of an x face: its v words, in cache lines of their own.
PLCG_HD constexpr int team_xpitch(int v) { return (v + 7) / 8 * 8; }

// A grid of nx * ny * nz unknowns (x fastest) in the axes of the team kernels:
// x runs over the lanes of a wave, y over waves, z over waves and then over the V
// unknowns of a thread.  A 2D grid enters as (nx, 1, ny).  A tile is 64 x wy x
// (wz * v) unknowns, and the workgroup that holds it has wy * wz streaming waves.
struct TeamGeom {
  int32_t nx, ny, nz;
  int32_t gx, gy, gz;                 // tiles along each axis
  int32_t wy, wz, v;
  int32_t rx, ry, rz;                 // words of one x, y and z face of a tile
  int32_t words;                      // words of a tile's mail: two faces of each kind
  int32_t near;                       // the tiles' workgroups share an XCD
};

PLCG_HD inline int team_tiles(const TeamGeom &g) { return g.gx * g.gy * g.gz; }
PLCG_HD inline int team_threads(const TeamGeom &g) { return 64 * (g.wy * g.wz + 1); }
// Bytes of the face mail (two copies by parity) and of the posted products.
inline size_t team_mail_bytes(const TeamGeom &g) {
  return (size_t)2 * team_tiles(g) * g.words * kWordBytes;
}
constexpr size_t team_post_bytes() {
  return (size_t)kTeamRing * kTeamTiles * kTeamProducts * kWordBytes;
}

// CUs of one XCD that a launch may need: its tiles, if they share one, else an equal part of
// them on every XCD.
inline int team_need(int tiles, bool near) {
  return near ? tiles : (tiles + kTeamXcds - 1) / kTeamXcds;
}
// Of the n launches that may be on the GPU or waiting for it (what each needs, oldest
// first), the first that a new one of `need` can be beside, all later ones too: what they need
// together, on the XCD that they may share, is there.  The new one has to wait for those
// before it.  So of any launches that run at once the newest has counted all the others, and
// none of them waits for a CU that another holds while it waits itself.  (Which XCD
// a launch's first workgroup goes to differs by hardware queue and is not known here.)
inline int team_beside(const int *needs, int n, int need, int per_xcd) {
  int first = n, sum = need;
  while (first > 0 && sum + needs[first - 1] <= per_xcd) sum += needs[--first];
  return first;
}

// A streaming wave's place in the grid and its share of the mail, uniform in the wave:
// byte offsets within one parity copy, to which a lane adds 16 times its number (z and
// y faces; row v of a y face 64 v words on) or 16 times the row it stands for (x faces:
// lanes 0 .. v-1 carry the west side of rows 0 .. v-1, lanes 32 .. 32+v-1 the east side).
// Of the offsets only those are used whose neighbour tile exists and whose face the
// wave touches (the flags).
struct TeamPlace {
  int wyi, wzi, sw;
  bool west, east, zlo, zhi, ylo, yhi;   // a neighbour tile lies there and this wave touches it
  int in_w, in_e, in_zlo, in_zhi, in_y;          // where this wave reads
  int out_w, out_e, out_zlo, out_zhi, out_y;     // where it posts
  int x0, y, z0;                                 // lane 0's unknown of row 0

  PLCG_HD inline TeamPlace(const TeamGeom &g, int v, bool d3, int tile, int sw_) {
    sw = sw_;
    wyi = d3 ? sw % g.wy : 0;
    wzi = d3 ? sw / g.wy : sw;
    const int bx = tile % g.gx, byz = tile / g.gx;
    const int by = d3 ? byz % g.gy : 0, bz = d3 ? byz / g.gy : byz;
    const int gxy = g.gx * g.gy;
    west = bx > 0;
    east = bx < g.gx - 1;
    zlo = wzi == 0 && bz > 0;
    zhi = wzi == g.wz - 1 && bz < g.gz - 1;
    ylo = d3 && wyi == 0 && by > 0;
    yhi = d3 && wyi == g.wy - 1 && by < g.gy - 1;
    // mail of a tile: x faces (west, east), y faces (low, high), z faces (low, high)
    const int W = kWordBytes;
    const int fe = g.rx, fyl = 2 * g.rx, fyh = fyl + g.ry, fzl = fyh + g.ry, fzh = fzl + g.rz;
    const int row = (wyi * g.wz + wzi) * team_xpitch(v);
    const int mine = tile * g.words;
    in_w = (mine + row) * W;
    in_e = (mine + fe + row) * W;
    out_w = ((tile - 1) * g.words + fe + row) * W;
    out_e = ((tile + 1) * g.words + row) * W;
    in_zlo = (mine + fzl + wyi * 64) * W;
    in_zhi = (mine + fzh + wyi * 64) * W;
    out_zlo = ((tile - gxy) * g.words + fzh + wyi * 64) * W;
    out_zhi = ((tile + gxy) * g.words + fzl + wyi * 64) * W;
    in_y = (mine + (ylo ? fyl : fyh) + wzi * v * 64) * W;
    out_y = ((ylo ? (tile - g.gx) * g.words + fyh : (tile + g.gx) * g.words + fyl) +
             wzi * v * 64) * W;
    x0 = bx * 64;
    y = by * g.wy + wyi;
    z0 = (bz * g.wz + wzi) * v;
  }
};

// Unknowns per thread the team kernels are built for: those of kTeamWidths up to this, the
// largest that fits 128 registers (four waves per SIMD) without spilling and a CU's 160 KB
// of LDS.
// The variable-coefficient stencils' edge weights share the LDS.
constexpr int team_vmax(int method_plcg, int l, bool d3, bool var) {
  return method_plcg && l > kTeamLMax ? 0
         : var         ? (d3 ? (l == 3 ? 2 : 3) : !method_plcg ? 6 : l == 1 ? 4 : 3)
         : !method_plcg ? (d3 ? 6 : 10)
         : l == 1     ? (d3 ? 5 : 6)
         : l == 2     ? (d3 ? 4 : 5)
         : l == 3     ? 4
                      : 0;
}
// Whether a p(l)-CG team kernel keeps x, and p, in LDS.
constexpr bool team_x_in_lds(int l, int v, bool d3) {
  return v >= (l == 1 ? 6 : l == 2 && !d3 ? 5 : 4);
}
constexpr bool team_p_in_lds(int l, int v, bool d3) {
  return team_x_in_lds(l, v, d3) && !(d3 && l == 1);
}
// Whether it keeps z_{i-1} there too (l = 3: 8 of the 128 registers at v = 4, without which
// it spilled).  us per iteration, streaming -> team: 1000 x 901 p(3) 16.1 -> 4.1; 3D CG with
// v = 6, x in LDS, 128 x 101 x 97 18.3 -> 12.6.
constexpr bool team_z1_in_lds(int l, int v) { return l == 3 && v >= 4; }
constexpr int kTeamWidths[] = {2, 3, 4, 5, 6, 7, 8, 10};

// Cuts the grid into at most `tiles` tiles with v unknowns per thread: of the
// arrangements of up to kTeamWaves waves the one with the smallest faces, waves
// then evened out over the tiles.  false: it does not fit.
inline bool team_cut(int nx, int ny, int nz, int v, int tiles, TeamGeom *out) {
  const int gx = (nx + 63) / 64;
  long long best = -1;
  for (int wy = 1; wy <= kTeamWaves && wy <= ny; ++wy) {
    int wz = kTeamWaves / wy;
    const int zrows = (nz + v - 1) / v;              // z extent in units of v
    if (wz > zrows) wz = zrows;
    const int gy = (ny + wy - 1) / wy, gz = (zrows + wz - 1) / wz;
    if ((long long)gx * gy * gz > tiles) continue;
    // the same tile counts with the waves spread evenly
    const int ey = (ny + gy - 1) / gy, ez = (zrows + gz - 1) / gz;
    // a wave keeps the halo of one y side only
    if (gy > 1 && ey < 2) continue;
    const long long faces = (gx > 1 ? 2LL * ey * ez * v : 0) + (gy > 1 ? 128LL * ez * v : 0) +
                            (gz > 1 ? 128LL * ey : 0);
    if (best >= 0 && faces >= best) continue;
    best = faces;
    TeamGeom g{};
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.gx = gx;
    g.gy = gy;
    g.gz = gz;
    g.wy = ey;
    g.wz = ez;
    g.v = v;
    g.rx = gx > 1 ? ey * ez * team_xpitch(v) : 0;
    g.ry = gy > 1 ? 64 * ez * v : 0;
    g.rz = gz > 1 ? 64 * ey : 0;
    g.words = 2 * (g.rx + g.ry + g.rz);
    *out = g;
  }
  return best >= 0;
}

// The cut of a system the team kernels take.  More unknowns per thread mean fewer tiles,
// whose sums arrive sooner, and longer sweeps.  Measured (us per iteration, v = 1 .. 5):
//   p(2) 256^2 2.64 2.58 2.36 2.55 3.11, 512^2 - 3.23 2.84 2.74 3.17, 700 x 650 - 3.56
//        3.60 2.97 3.17, 64^3 - 3.93 3.78 2.97: the owner's chain sets the pace, so v >= 3
//        and few tiles, but x and p still in registers (v <= 4);
//   p(1) 256^2 2.94 2.89 3.02 3.12 3.38, 512^2 - 3.28 3.30 3.50 3.62, 64^3 - 3.61 3.72
//        3.40 3.46, p(3) 256^2 2.81 2.62 2.50, 512^2 - 3.26 2.77, 64^3 - 3.53 3.84:
//        flat once the tiles number 128 or less;
//   CG   256^2 4.47 4.35 4.65 4.86, 512^2 - 5.04 5.04 5.38: one product per sum, so tiles
//        cost little.
// One tile is best where one workgroup holds the system: no mail (64^2 p(1) v = 5 2.07
// against 2.28 with two tiles, 60 x 40 p(2) v = 4 1.73 against 1.92, CG v = 5 1.95 against
// 3.06), with the most unknowns per thread that stay in registers: fewer waves share the
// SIMDs and the barriers (37 x 53 CG v = 4 / 5 / 6 2.42 2.21 2.32, 64^2 - 2.44 2.28).
// Tiles of one XCD (up to 32 of 256) answer each other sooner, 1050 clocks from post to
// poll against 1570, so such launches put them there (near): 100 x 80 CG 3.98 -> 3.15, p(1)
// 2.55 -> 2.13, p(2) 2.01 -> 2.00, p(3) 1.91 -> 1.80; 24^3 CG 4.41 -> 4.01, p(1) 2.66 -> 2.52, but p(2)
// 2.57 -> 2.66.  In 2D where two exchanges follow each other, CG and p(1), it also pays to
// take more unknowns per thread for it: 300 x 200 CG 4.29 -> 3.83 (v = 2 -> 3), p(1) 2.85 ->
// 2.62 (3 -> 4), 400 x 300 CG 4.58 -> 4.45 (3 -> 5), but p(1) 2.97 -> 3.07 (4 -> 5); not in 3D,
// where a tile's faces grow with it: 36^3 CG 4.63 -> 5.43.
// So: one tile if it fits with v = one (CG also 6); else, in 2D, CG and p(1), the smallest v up
// to `near` with the tiles of one XCD; else the smallest v from `lo` up to `hi` with at
// most `cap` tiles, else hi, else the smallest larger v that fits at all.  false: the system is too large (or too narrow: the
// lanes of a wave lie along x), or its face mail would outgrow kTeamMailMax.
inline bool team_plan(int method_plcg, int l, bool d3, bool var, int nx, int ny, int nz, int tiles,
                      TeamGeom *out) {
  if (tiles > kTeamTiles) tiles = kTeamTiles;
  const int vmax = team_vmax(method_plcg, l, d3, var);
  const int lo = method_plcg && l == 2 ? 3 : 2;
  const int want = !method_plcg ? 2 : l == 3 ? 3 : 4, hi = want < vmax ? want : vmax;
  const int cap = !method_plcg ? kTeamTiles : l == 2 ? 64 : 128;
  const int one = !method_plcg || l == 1 ? 5 : l == 2 ? 4 : 3;
  for (int v = one; v <= vmax && v <= (method_plcg ? one : 6); ++v)
    if (team_cut(nx, d3 ? ny : 1, d3 ? nz : ny, v, 1, out) &&
        (v > one || method_plcg || out->wy * out->wz <= 11))
      return true;
  const int xcd = tiles / kTeamXcds, near = d3 ? 0 : !method_plcg ? 5 : l == 1 ? 4 : 0;
  for (int v : kTeamWidths)
    if (v <= near && v <= vmax && team_cut(nx, 1, ny, v, xcd, out)) {
      out->near = 1;
      return true;
    }
  for (int pass = 0; pass < 2; ++pass)
    for (int v : kTeamWidths) {
      if (v > vmax) break;
      if (pass == 0 ? (v < lo || v > hi) : v < hi) continue;
      if (team_cut(nx, d3 ? ny : 1, d3 ? nz : ny, v, pass == 0 && cap < tiles ? cap : tiles, out)) {
        out->near = team_tiles(*out) <= xcd && !(method_plcg && l == 2 && d3);
        return team_mail_bytes(*out) <= kTeamMailMax;
      }
    }
  return false;
}

// Whether a grid in 3D that the resident kernels do not take is faster in team launches than
// streaming.  A wave posts 64 lanes of a face however few of them are unknowns, so grids thin
// along x send mostly empty mail.  us per iteration of CG, team / streaming, by the words that
// the mail of a sweep has (k = 1024):
//   nx = 4   250 k 6.49 / 8.93, 394 k 8.23 / 9.31, 441 k 9.11 / 8.92, 494 k 9.27 / 9.16, 510 k
//            (v = 5) 10.67 / 8.92, 569 k 10.33 / 9.06, 656 k (v = 6) 12.22 / 9.17
//   nx = 8   441 k 9.15 / 9.26, 478 k 9.71 / 9.19, 510 k (v = 5) 10.62 / 9.17, 656 k 12.20 / 9.96
//   nx = 16  494 k 9.30 / 9.37, 510 k (v = 5) 10.65 / 9.83, 527 k (v = 4) 9.08 / 9.96, 656 k
//            12.19 / 11.12;   nx = 24  510 k 10.66 / 11.39, 656 k 12.21 / 13.46
// p(1) and p(2), with one exchange fewer, only at nx <= 4: p(1) 441 k 6.26 / 6.38, 478 k 6.59 /
// 6.42, 510 k 6.59 / 6.30, 527 k 6.01 / 6.39, p(2) 459 k 5.56 / 5.69, 478 k 6.12 / 5.71, 525 k
// 6.35 / 5.55, 527 k 5.67 / 5.74; p(3) never: 527 k 4.85 / 6.42.
inline bool team_grid_pays(int method_plcg, int l, bool d3, const TeamGeom &g) {
  if (!d3 || (long long)team_tiles(g) * g.words <= 470 * 1024) return true;
  return method_plcg ? l >= 3 || g.nx > 4 : g.nx > (g.v >= 5 ? 16 : 8);
}

// Assembled matrices (their ELL copy of k entries per row): entries per row that the
// kernels of two widths take, with as many rows per thread as their registers allow.
constexpr int kRowsShort = 5, kRowsLong = 9;
inline int team_rows_v(int k) { return k <= kRowsShort ? 2 : 1; }
// The cut of n rows: in order, wave by wave, over up to `tiles` workgroups.  Few tiles, as
// with the stencils, but the gathers of a workgroup share its CU's path to memory: 11
// streaming waves while there are tiles left, 15 with one row per thread (us per iteration,
// 11 / 15 waves of two rows, 15 of one: 300 x 201 p(1) 3.04 2.95 2.90, p(2) 2.74 2.98 2.95, p(3) 2.38
// 3.07 2.73; 400 x 300 p(2) 3.06 3.22 3.38; with 4 waves of one row 4.01 and 4.33;
// 60 x 50 x 40, seven entries, p(2) 4.36 with 15, 4.96 with 8).  On one XCD up to half its
// CUs' number of tiles: 100 x 77 p(1) 2.63 -> 2.36; with 30 tiles 2.75 -> 2.87.
inline bool team_rows_plan(int n, int k, int tiles, TeamGeom *out) {
  if (tiles > kTeamTiles) tiles = kTeamTiles;
  if (n < 1 || k < 1 || k > kRowsLong || tiles < 1) return false;
  const int v = team_rows_v(k), waves = (n - 1) / (64 * v) + 1;
  int wz = (waves - 1) / tiles + 1;
  const int want = v == 2 ? 11 : kTeamWaves;
  if (wz > kTeamWaves) return false;
  if (wz < want) wz = want;
  TeamGeom g{};
  g.nx = n;
  g.ny = g.nz = g.gy = g.gz = g.wy = 1;
  g.gx = (waves - 1) / wz + 1;
  g.wz = (waves - 1) / g.gx + 1;
  g.v = v;
  g.near = g.gx > 1 && g.gx <= tiles / (2 * kTeamXcds);
  g.words = 2 * g.wz * 64 * v;       // four copies of the unknowns' words, where faces have two
  *out = g;
  return team_mail_bytes(g) <= kTeamMailMax;
}

// Mean number of 128-byte lines of words that one gather of a wave touches, 64 rows' j-th
// entries (ELL: entry j of row p at j * ld + p): 8 where neighbours of consecutive rows are
// consecutive, 64 where the order of the rows says nothing.  From up to 256 waves.
inline double team_rows_lines(const int32_t *ci, int n, int k, int ld) {
  if (n < 1 || k < 1) return 0.0;
  const int waves = (n - 1) / 64 + 1, step = (waves - 1) / 256 + 1;
  std::vector<int32_t> seen((size_t)(n - 1) / 8 + 1, -1);
  int32_t gathers = 0;
  long long lines = 0;
  for (int w = 0; w < waves; w += step)
    for (int j = 0; j < k; ++j, ++gathers)
      for (int p = 64 * w; p < n && p < 64 * w + 64; ++p) {
        int32_t &s = seen[(size_t)ci[(size_t)j * ld + p] / 8];
        lines += s != gathers;
        s = gathers;
      }
  return (double)lines / gathers;
}
// Whether the team launches' gathers of words, twice as wide as the streaming kernels' and
// from beyond the L1 caches, leave them faster for rows of this order.  us per iteration,
// team / streaming, rows of a five-point grid shuffled within 256, 1024, 4096 rows and all
// (about 27, 43, 51 and 55 lines a gather; as the grid's, 9):
//   p(1)  40 000 3.8 / 6.2,  6.1 / 6.6, 7.4 / 6.8, 8.2 / 8.0;   119 700 -, 6.7 / 6.8, 7.9 / 7.0,
//         8.7 / 9.1;   240 100 -, 7.2 / 8.2, 8.5 / 8.9, 10.0 / 12.5
//   p(2)  22 500 -, 5.1 / 5.6, -, 6.2 / 6.9;   40 000 4.2 / 5.3, 6.7 / 5.7, 8.0 / 6.0, 8.8 / 7.1;
//         119 700 -, 7.3 / 6.1, -, 9.1 / 8.3;   230 400 5.6 / 7.2, 7.8 / 7.5, 8.5 / 8.0, 9.5 / 12.0;
//         260 100 5.6 / 8.1, 8.0 / 8.4, 8.6 / 8.9, 10.6 / 13.0
//   p(2), seven entries, 15 000 -, 5.6 / 6.3, -, 6.6 / 7.7;   27 000 -, 6.9 / 6.5, -, 8.6 / 8.1;
//         241 800 6.8 / 9.2, 9.3 / 9.4, 10.7 / 10.1, 10.6 / 14.9
// and p(3) as p(2).  The lines are drawn where rows shuffled within a part of the matrix, as an
// unstructured mesh numbers them, begin and cease to be slower.
inline bool team_rows_pays(int n, int l, double lines) {
  return l == 1 ? lines <= 47.0 || n < 24000 || n > 150000
                : lines <= 35.0 || n < 24000 || n > 250000;
}

}  // namespace plcg

// Host check of the team kernels' geometry: for every case the tiles cover each
// unknown once, every mailed word lies inside the mail, is posted by one lane and
// read by the one whose unknown is its face neighbour, and every neighbour that lies
// in another tile is read.  Input lines: method (1 p(l)-CG, 0 CG) l d3 var nx ny nz tiles.
// Prints "v tiles waves words" per case, or "none" where no plan fits; exit code 1
// on the first violation.
#include "plcg_team.h"
#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>
using namespace plcg;

static void need(bool ok, const char *what) {
  if (!ok) {
    std::printf("VIOLATION: %s\n", what);
    std::exit(1);
  }
}

int main() {
  int pl, l, d3, var, nx, ny, nz, tiles;
  while (std::scanf("%d %d %d %d %d %d %d %d", &pl, &l, &d3, &var, &nx, &ny, &nz, &tiles) == 8) {
    TeamGeom g;
    if (!team_plan(pl, l, d3 != 0, var != 0, nx, ny, nz, tiles, &g)) {
      std::printf("none\n");
      continue;
    }
    const int nt = team_tiles(g), nw = g.wy * g.wz, v = g.v;
    need(nt <= tiles && nt <= kTeamTiles && nw >= 1 && nw <= kTeamWaves, "tiles or waves");
    need(v <= 32 && v <= team_vmax(pl, l, d3 != 0, var != 0), "unknowns per thread");
    need(team_mail_bytes(g) <= kTeamMailMax, "mail size");
    const long long size = (long long)nt * g.words * kWordBytes;
    const int n = g.nx * g.ny * g.nz;
    std::vector<char> seen(n, 0);
    struct Cell { int x, y, z; };
    std::map<int, Cell> mail;
    auto post = [&](int off, int x, int y, int z) {
      need(off >= 0 && off + kWordBytes <= size && off % kWordBytes == 0, "post out of the mail");
      need(mail.emplace(off, Cell{x, y, z}).second, "two lanes post one word");
    };
    // f(place, lane, lane's x); the lane terms of the offsets as the kernels add them
    auto each = [&](auto f) {
      for (int t = 0; t < nt; ++t)
        for (int w = 0; w < nw; ++w) {
          const TeamPlace p(g, v, d3 != 0, t, w);
          for (int lane = 0; lane < 64; ++lane) f(p, lane, p.x0 + lane);
        }
    };
    const int W = kWordBytes;
    each([&](const TeamPlace &p, int lane, int x) {
      for (int k = 0; k < v; ++k) {
        const int z = p.z0 + k;
        if (x < g.nx && p.y < g.ny && z < g.nz) {
          const int q = x + g.nx * (p.y + g.ny * z);
          need(q < n && !seen[q], "unknown held twice");
          seen[q] = 1;
        }
        if (p.ylo || p.yhi) post(p.out_y + (lane + 64 * k) * W, x, p.y, z);
      }
      // lanes k and 32 + k carry the first and the last lane's values of row k
      const int k = lane & 31;
      if (k < v && lane < 32 && p.west) post(p.out_w + k * W, p.x0, p.y, p.z0 + k);
      if (k < v && lane >= 32 && p.east) post(p.out_e + k * W, p.x0 + 63, p.y, p.z0 + k);
      if (p.zlo) post(p.out_zlo + lane * W, x, p.y, p.z0);
      if (p.zhi) post(p.out_zhi + lane * W, x, p.y, p.z0 + v - 1);
      need(!(p.ylo && p.yhi), "a wave touches both y sides");
    });
    for (char c : seen) need(c, "unknown not held");
    size_t reads = 0;
    auto read = [&](int off, int x, int y, int z) {
      auto it = mail.find(off);
      need(it != mail.end(), "a word that nobody posts is awaited");
      need(it->second.x == x && it->second.y == y && it->second.z == z, "wrong neighbour read");
      ++reads;
    };
    each([&](const TeamPlace &p, int lane, int x) {
      const int k = lane & 31;
      if (k < v && lane < 32 && p.west) read(p.in_w + k * W, p.x0 - 1, p.y, p.z0 + k);
      if (k < v && lane >= 32 && p.east) read(p.in_e + k * W, p.x0 + 64, p.y, p.z0 + k);
      for (int r = 0; r < v; ++r) {
        if (p.ylo) read(p.in_y + (lane + 64 * r) * W, x, p.y - 1, p.z0 + r);
        if (p.yhi) read(p.in_y + (lane + 64 * r) * W, x, p.y + 1, p.z0 + r);
      }
      if (p.zlo) read(p.in_zlo + lane * W, x, p.y, p.z0 - 1);
      if (p.zhi) read(p.in_zhi + lane * W, x, p.y, p.z0 + v);
      // neighbours in another tile have a flag that makes the wave read them
      for (int r = 0; r < v; ++r) {
        const int z = p.z0 + r;
        if (!(x < g.nx && p.y < g.ny && z < g.nz)) continue;
        if (lane == 0) need((x > 0) == p.west, "west neighbour");
        if (lane == 63) need((x < g.nx - 1) == p.east, "east neighbour");
        if (r == 0 && p.wzi == 0) need((z > 0) == p.zlo, "z below");
        if (r == v - 1 && p.wzi == g.wz - 1) need(z >= g.nz - 1 || p.zhi, "z above");
        if (d3 && p.wyi == 0) need((p.y > 0) == p.ylo, "y below");
        if (d3 && p.wyi == g.wy - 1) need(p.y >= g.ny - 1 || p.yhi, "y above");
      }
    });
    need(reads == mail.size(), "a posted word is not read");
    std::printf("%d %d %d %d\n", v, nt, nw, g.words);
  }
  return 0;
}

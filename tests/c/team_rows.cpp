// Checks the cut of an assembled matrix's rows (plcg_team.h) as the row kernel places
// them: every row in one place, within the limits of a launch and of its mail.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "plcg_team.h"

using namespace plcg;

int main() {
  const int sizes[] = {1, 63, 64, 65, 128, 129, 1407, 1408, 1409, 4801, 60300, 245760, 245761,
                       262144, 360448, 360449, 491520, 491521, 2000000000};
  int taken = 0;
  for (int tiles : {1, 7, 256, 304})
    for (int k = 0; k <= kRowsLong + 1; ++k)
      for (int n : sizes) {
        TeamGeom g{};
        if (!team_rows_plan(n, k, tiles, &g)) {
          const long long room = 64LL * team_rows_v(k) * kTeamWaves * (tiles < kTeamTiles ? tiles : kTeamTiles);
          if (k >= 1 && k <= kRowsLong && n <= room) {
            std::printf("refused: n %d k %d tiles %d\n", n, k, tiles);
            return 1;
          }
          continue;
        }
        ++taken;
        const int cap = tiles < kTeamTiles ? tiles : kTeamTiles;
        if (k < 1 || k > kRowsLong || g.v != team_rows_v(k) || team_tiles(g) > cap ||
            g.wz < 1 || g.wz * g.wy > kTeamWaves || team_mail_bytes(g) > kTeamMailMax) {
          std::printf("limits: n %d k %d tiles %d\n", n, k, tiles);
          return 1;
        }
        // rows as RowsOp::at places them, and four copies of their words in the mail
        std::vector<char> seen(n, 0);
        const long long words = (long long)g.gx * g.wz * 64 * g.v;
        if (4 * words * kWordBytes != (long long)team_mail_bytes(g)) {
          std::printf("mail: n %d k %d tiles %d\n", n, k, tiles);
          return 1;
        }
        for (int tile = 0; tile < team_tiles(g); ++tile)
          for (int sw = 0; sw < g.wz; ++sw)
            for (int lane = 0; lane < 64; ++lane)
              for (int v = 0; v < g.v; ++v) {
                const long long p = (long long)(tile * g.wz + sw) * 64 * g.v + lane + 64 * v;
                if (p >= words) return 1;
                if (p < n && seen[p]++) {
                  std::printf("twice: row %lld of %d\n", p, n);
                  return 1;
                }
              }
        for (int p = 0; p < n; ++p)
          if (!seen[p]) {
            std::printf("missing: row %d of %d\n", p, n);
            return 1;
          }
      }
  std::printf("ok %d\n", taken);
  return taken > 100 ? 0 : 1;
}

// The chunks that the teams of a tap-chunk workgroup load (cci_chunks.hpp):
// every chunk of the reduction once, and uniform offsets inside the packed
// arrays of a single row (2 C bytes of values, C of indices).
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../paper_1910_11971_amd/csrc/cci_chunks.hpp"

int main() {
  for (int32_t C = 8; C <= 8192; C += 8)
    for (int32_t teams = 1; teams <= 2; ++teams) {
      const int32_t nch = (C + 63) / 64, n = cci::team_chunks(nch, teams);
      std::vector<int> seen(nch, 0);
      for (int32_t team = 0; team < teams; ++team)
        for (int32_t ch = 0; ch < n; ++ch) {
          const int32_t at = team * n + ch, l = cci::load_chunk(at, nch);
          if (at < nch && l != at) return printf("C %d: chunk %d loads %d\n", C, at, l), 1;
          if (at < nch) ++seen[at];
          if (l < 0 || 128 * l >= 2 * C || 64 * l >= C)
            return printf("C %d, %d teams: chunk %d at byte %d of %d\n", C, teams, at, 128 * l, 2 * C), 1;
        }
      for (int32_t c = 0; c < nch; ++c)
        if (seen[c] != 1) return printf("C %d: chunk %d loaded %d times\n", C, c, seen[c]), 1;
    }
  printf("chunk driver ok\n");
  return 0;
}

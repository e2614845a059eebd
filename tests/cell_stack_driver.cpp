// The check of the cell-lane tables on tables that break the rule its kernels rely
// on: they read the top stack entry one step ahead, so no step may take an entry
// that the step before left into.  Reads a forest (n, ncells, parent, cell_offsets),
// builds the tables, which must pass, then moves one flag so that a lane's stack
// stays balanced but an entry is left in the step before it is taken, or in the
// chunk boundary between the two.  Exit 0 if every such table is refused.
#include <cstdio>
#include <string>
#include <vector>

#include "../paper_1810_12742_amd/csrc/setup.hpp"

using namespace hines;

int main(int argc, char** argv) {
  FILE* f = argc == 2 ? std::fopen(argv[1], "rb") : nullptr;
  int64_t hdr[2];
  if (!f || std::fread(hdr, 8, 2, f) != 2) return 2;
  const int64_t n = hdr[0], nc = hdr[1];
  std::vector<int32_t> par(n);
  std::vector<int64_t> off(nc + 1);
  if ((int64_t)std::fread(par.data(), 4, n, f) != n || (int64_t)std::fread(off.data(), 8, nc + 1, f) != nc + 1) return 2;
  std::fclose(f);
  CellLanes C;
  std::string why;
  if (build_cell_lanes(par.data(), n, off.data(), nc, C, why) != OK || !check_cell_lanes(C, off.data(), nc, why)) {
    std::printf("sound tables refused: %s\n", why.c_str());
    return 3;
  }
  auto at = [&](int64_t w, int64_t q, int c) -> uint8_t& {
    return C.flags[cell_flag_index(C.waves[w].chunk_off + q / kCellChunk, c, (int)(q % kCellChunk))];
  };
  int tried = 0, across = 0;
  for (int64_t w = 0; w < C.nwaves; ++w)
    for (int c = 0; c < 64; ++c)
      for (int64_t q = 1; q < (int64_t)C.waves[w].nchunk * kCellChunk; ++q) {
        uint8_t &before = at(w, q - 1, c), &f0 = at(w, q, c);
        if (!(f0 & CF_POP) || (before & (CF_PUSH | CF_MERGE))) continue;
        if (q % kCellChunk == 0 ? across >= 50 : tried - across >= 200) continue;
        // the step before adds into the entry that this step takes: balanced as before
        before |= CF_MERGE;
        ++tried;
        across += q % kCellChunk == 0;
        const bool refused = !check_cell_lanes(C, off.data(), nc, why);
        before &= (uint8_t)~CF_MERGE;
        if (!refused || why.find("step after") == std::string::npos) {
          std::printf("wave %lld lane %d step %lld: accepted\n", (long long)w, c, (long long)q);
          return 4;
        }
      }
  std::printf("%d refused, %d of them across chunks\n", tried, across);
  return tried > 100 && across > 5 ? 0 : 5;
}

// Prints the block shape that the host's rules give each projection of a prompt or a step (test only).
// Arguments, five numbers each: epilogue (enum Epi), row tiles, column tiles, K chunks, bytes for the
// partial tiles of a K split; first argument "prompt" or "step".  One line "mr nc ks" per projection.
// First argument "nt": row tiles, blocks, d, FFN rows, vocabulary; 1 where the weights are nontemporal.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "tss_internal.h"

int main(int argc, char** argv) {
  if (argc < 2 || (argc - 2) % 5) return 2;
  const bool prompt = !std::strcmp(argv[1], "prompt");
  for (int i = 2; i + 4 < argc; i += 5) {
    if (!std::strcmp(argv[1], "nt")) {
      std::printf("%d\n", (int)tss::tile_weights_nt(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoi(argv[i + 2]),
                                                    std::atoi(argv[i + 3]), std::atoi(argv[i + 4])));
      continue;
    }
    const int epi = std::atoi(argv[i]), rt = std::atoi(argv[i + 1]), ct = std::atoi(argv[i + 2]);
    const int nkc = std::atoi(argv[i + 3]);
    const size_t parts = std::strtoull(argv[i + 4], nullptr, 10);
    const tss::TileShape t =
        prompt ? tss::prompt_tile(epi, rt, ct, nkc, parts) : tss::step_tile(epi, rt, ct, nkc, parts);
    std::printf("%d %d %d\n", t.mr, t.nc, t.ks);
  }
  return 0;
}

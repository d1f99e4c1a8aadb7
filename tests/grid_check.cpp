// Host-side check of the fp32 expert GEMMs' launch grids (gemm_pipe.h): for block counts on
// both sides of what one grid row holds, every block is there once, a row stays below 2^32
// threads and is a multiple of 8 blocks (the XCDs), only large grids have several rows, and
// the last row is not empty.  Prints "ok" and exits 0, else the first mismatch.
#include <cstdio>

#include "../paper_2609_05228_amd/csrc/gemm_pipe.h"

int main() {
  const unsigned threads = 512;
  const unsigned long long row = (1ull << 32) / threads;  // one block too many
  for (unsigned long long n : {8ull, 64ull, row - 8, row, row + 8, 2 * row - 8, 2 * row, 3 * row + 16, 1ull << 25})
    for (unsigned long long blocks = n; blocks <= n + 1024; blocks += 8) {
      const ace::PipeGrid g = ace::pipe_grid(blocks, threads);
      const unsigned long long all = static_cast<unsigned long long>(g.x) * g.y;
      const bool wrong = blocks < row ? g.y != 1 || g.x != blocks : g.x != 1u << ace::kPipeGridRow;
      if (wrong || g.x % 8 || static_cast<unsigned long long>(g.x) * threads >= (1ull << 32) || all < blocks ||
          all - blocks >= g.x) {
        std::printf("%llu blocks: grid %u x %u\n", blocks, g.x, g.y);
        return 1;
      }
    }
  std::printf("ok\n");
  return 0;
}

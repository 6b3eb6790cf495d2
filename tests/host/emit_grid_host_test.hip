// Host-side test of the pair emission's grid: this translation unit includes the
// binning source with kernel launches replaced by a record of their grids, and
// exports one entry point that the CPU test calls through ctypes.  Nothing is
// launched.
#include <hip/hip_runtime.h>

#include <stdio.h>

#include <algorithm>

static dim3 g_grid, g_block;
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kernel, grid, block, ...) (g_grid = (grid), g_block = (block))
#include "../../paper_2511_16144_amd/csrc/binning.hip"

// 0 if a launch for so many pairs and words to be zeroed has a thread for each
// 4 pairs and at most 16 words to a thread
extern "C" int lgs_emit_grid(int64_t pairs, int64_t words) {
  lgs::launch_emit(nullptr, nullptr, nullptr, nullptr, nullptr, pairs, pairs, 0, 0, nullptr, nullptr, nullptr, words,
                   nullptr);
  const int64_t threads = (int64_t)g_grid.x * g_block.x;
  const bool ok = g_grid.x >= 1 && threads * 4 >= pairs && threads * 16 >= words;
  if (!ok) fprintf(stderr, "%lld pairs, %lld words: %u blocks\n", (long long)pairs, (long long)words, g_grid.x);
  return !ok;
}

// Which (task, column tile) a wave of the WCSR tile kernels takes, and how many tasks a launch holds.
#pragma once

#include <algorithm>

#include "asp_internal.h"

namespace asp {

// The column tiles of a task go to neighbouring waves of a workgroup: a row of B or C whose width is no multiple of 128 bytes
// shares cache lines between its tiles, which then are read once and written whole.  (All tasks of one column tile
// first, i.e. the tiles a whole pass apart, bf16, band of 27, 500 000 rows, us: N = 200, heights 16 / 32 / 64 158 / 174 / 195
// against 123 / 118 / 128; N = 256, height 64 162 / 145.)
struct WaveTask {
    int task, tile;
};
__device__ __forceinline__ WaveTask wave_task(int n_tiles) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (n_tiles == 1) return {(int)blockIdx.x * 4 + wave, 0};
    const uint32_t group = blockIdx.x / (uint32_t)n_tiles, w = (blockIdx.x - group * n_tiles) * 4 + wave;  // 4 tasks
    const uint32_t t = w / (uint32_t)n_tiles;
    return {(int)(group * 4 + t), (int)(w - t * n_tiles)};
}

// HIP takes fewer than 2^32 threads a launch
inline int64_t tasks_per_launch(int64_t n_tiles) { return std::max<int64_t>(4, ((1 << 26) - 1) / n_tiles / 4 * 4); }
inline dim3 tile_grid(int64_t n_tasks, int64_t n_tiles) { return dim3((unsigned)ceil_div(n_tasks * n_tiles, 4)); }

}  // namespace asp

// Which (task, column tile) a wave of the WCSR tile kernels takes, and how many tasks a launch holds.
#pragma once

#include "asp_internal.h"

namespace asp {

// The column tiles of a task go to neighbouring waves of a workgroup: a row of B or C whose width is no multiple of 128 bytes
// shares cache lines between its tiles, which then are read once and written whole.  (All tasks of one column tile
// first, i.e. the tiles a whole pass apart, bf16, band of 27, 500 000 rows, us: N = 200, heights 16 / 32 / 64 158 / 174 / 195
// against 123 / 118 / 128; N = 256, height 64 162 / 145.)
// dealt: the list holds one range of tasks for each XCD, in groups of four (deal_to_xcds); workgroups go to the XCDs
// round-robin, so a group's workgroups are 8 apart.
// UNIFORM: the task counts as the same for the whole wave, and what it leads to is loaded by the scalar unit: 4 % faster in
// the bf16 kernel, 1-4 % slower in the fp32 ones except where it makes room for another wave (wcsr_spmm_launch).
struct WaveTask {
    int task, tile;
};
template <bool UNIFORM>
__device__ __forceinline__ WaveTask wave_task(int n_tiles, bool dealt) {
    const int wave = UNIFORM ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : (int)(threadIdx.x >> 6);
    if (n_tiles == 1) return {(int)blockIdx.x * 4 + wave, 0};
    const uint32_t xcd = dealt ? blockIdx.x & 7 : 0, local = dealt ? blockIdx.x >> 3 : blockIdx.x;
    const uint32_t round = local / (uint32_t)n_tiles, w = (local - round * n_tiles) * 4 + wave;
    const uint32_t t = w / (uint32_t)n_tiles;
    return {(int)((dealt ? round * 8 + xcd : round) * 4 + t), (int)(w - t * n_tiles)};
}

// HIP takes fewer than 2^32 threads a launch
inline int64_t tasks_per_launch(int64_t n_tiles) { return ((1 << 26) - 1) / n_tiles / 32 * 32; }  // n_tiles <= 65535
inline dim3 tile_grid(int64_t n_tasks, int64_t n_tiles, bool dealt) {
    return dim3((unsigned)(dealt ? ceil_div(n_tasks, 32) * 8 * n_tiles : ceil_div(n_tasks * n_tiles, 4)));
}

}  // namespace asp

// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <new>
#include <string>
#include <vector>

#include "asyncsparse.h"

namespace asp {

// thread-local detail string behind asp_last_error()
void set_error(const std::string &msg);
asp_status_t fail(asp_status_t s, const std::string &msg);

#define ASP_HIP_TRY(expr)                                                                        \
    do {                                                                                         \
        hipError_t e__ = (expr);                                                                 \
        if (e__ != hipSuccess)                                                                   \
            return ::asp::fail(e__ == hipErrorOutOfMemory ? ASP_ERR_OUT_OF_MEMORY : ASP_ERR_HIP, \
                               std::string(#expr) + ": " + hipGetErrorString(e__));             \
    } while (0)

// Benchmarking switches: environment variables that select among kernels and schedules which are all built and
// parity-tested, for the ladder and the tile-width study of bench.py.  Read once per process, in one place
// (asp_api.cpp); nothing else in the library looks at the environment.
struct Switches {
    int bcsr_bn;          // ASP_BCSR_BN=64|128|256: widest BCSR tile to consider (0: no cap)
    bool bcsr_regstage;   // ASP_BCSR_KERNEL=regstage: the synchronous register-staged kernel
    int bcsr_group_n;     // ASP_BCSR_GROUP_N=<n>: N-tiles walked together (0: the kernels' own rules)
    int bcsr_wgs_per_cu;  // ASP_BCSR_WGS_PER_CU=<n>: resident workgroups of the ring kernel (0: as many as LDS allows)
    int bcsr_workgroups;  // ASP_BCSR_WORKGROUPS=<n>: resident workgroups of the 128x512-tile kernel (0: one per compute unit)
    bool bcsr_xcd_aware;  // ASP_BCSR_XCD_AWARE=0: deal tiles without regard to XCDs
    bool bcsr_atomic;     // ASP_BCSR_SCHEDULE=atomic: tiles pulled from per-XCD atomic counters (ring kernel, 128x256)
    bool xt_generic;      // ASP_BCSR_XT=generic: asp_spmm_xt without matrix cores
    int bcsr_composite;   // ASP_BCSR_COMPOSITE=0|1: never / always keep the 128-row stacks of smaller blocks (-1: by fill)
    int wcsr_max_bn;      // ASP_WCSR_MAX_BN=64|128|256: widest fp32 WCSR wave tile to consider
};
const Switches &switches();

inline size_t dtype_size(int32_t dt) { return dt == ASP_DT_BF16 ? 2 : 4; }
constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// HIP takes fewer than 2^32 threads along a dimension of a launch
constexpr bool launch_fits(int64_t workgroups, int64_t threads) { return workgroups * threads < (1ll << 32); }

// ---- host-side converted forms -------------------------------------------------------------
// Zero-filled byte buffer taken from calloc: for gigabytes the pages arrive zeroed from the system and are first
// touched by the converter's worker threads, where a std::vector would fill them on one thread first.
class ZeroedBytes {
public:
    ZeroedBytes() = default;
    ZeroedBytes(const ZeroedBytes &) = delete;
    ZeroedBytes &operator=(const ZeroedBytes &) = delete;
    ZeroedBytes(ZeroedBytes &&o) noexcept : p_(o.p_), n_(o.n_) { o.p_ = nullptr, o.n_ = 0; }
    ZeroedBytes &operator=(ZeroedBytes &&o) noexcept {
        if (this != &o) {
            std::free(p_);
            p_ = o.p_, n_ = o.n_;
            o.p_ = nullptr, o.n_ = 0;
        }
        return *this;
    }
    ~ZeroedBytes() { std::free(p_); }
    void reset(size_t bytes) {
        std::free(p_);
        p_ = nullptr, n_ = 0;
        if (bytes == 0) return;
        p_ = (uint8_t *)std::calloc(bytes, 1);
        if (!p_) throw std::bad_alloc();
        n_ = bytes;
    }
    uint8_t *data() { return p_; }
    const uint8_t *data() const { return p_; }
    size_t size() const { return n_; }

private:
    uint8_t *p_ = nullptr;
    size_t n_ = 0;
};

struct HostBcsr {
    std::vector<int32_t> block_row_ptr;  // [n_brows + 1]
    std::vector<int32_t> block_col_idx;  // [nnz_blocks]
    std::vector<uint8_t> blocks;         // canonical [nnz_blocks][b_row][b_col], raw bytes
    std::vector<uint8_t> packed;         // same values in MFMA-fragment order (kernel-internal)
    // scheduling data of the main kernel: block-rows sorted by stored blocks (descending) and the
    // prefix sums of their tile weights (stored blocks + 1) in that order
    std::vector<int32_t> rank_info;            // [n_brows][4]
    std::vector<int64_t> sorted_weight_prefix; // [n_brows + 1]
    std::vector<int32_t> rank_info_32, rank_info_64;        // the same in 32 and 64 lists instead of 16 (Orders)
    std::vector<int64_t> weight_prefix_32, weight_prefix_64;
    std::vector<int32_t> by_length;            // bf16: block-rows, longest first,
    std::vector<int64_t> length_prefix;        // and the prefix sums of their weights
    int64_t n_nonempty = 0;                    // block-rows with at least one stored block (they come first)
    int64_t max_blocks = 0;                    // stored blocks of the longest block-row
    std::vector<int32_t> slice_rows;           // composite form only: [blocks][4] first row of B of each K slice
    std::vector<int32_t> piece_rows;           // composite form only: [super-rows][4] first row of C of each 32-row piece, -1 = none
};

// BCSR, 128 x 512 tiles: shares of 1 to 23 N-tiles (bcsr_build_shares); empty where block-rows are so many that whole rounds
// of them are even enough
struct BcsrShares {
    static constexpr int MAX_TILES = 23, WORKERS = 256, FIRST_PITCH = WORKERS + 1;
    static constexpr int64_t MAX_ROWS = 512;
    static constexpr int slot(int t) { return t - 1 - t / 8; }  // multiples of 8 are never shared
    // rank_info_32; [slot][n_nonempty][4] in its form, the block-rows list after list for 1, 2, ... tiles (together
    // `infos` entries); [slot][FIRST_PITCH] the first entry of every list
    std::vector<int32_t> lists;
    int64_t infos = 0;
    std::vector<int32_t> load;             // [slot][WORKERS] stored blocks + 2 per tile of every list
};

struct HostWcsr {
    std::vector<int32_t> window_row_ptr;  // [n_windows + 1]
    std::vector<int32_t> window_col_idx;  // [padded_cols]
    ZeroedBytes values;                   // [padded_cols / b_col][b_row][b_col], raw bytes
    std::vector<int32_t> tasks;           // [n_tasks][4]; filled on the host only in host-convert mode
    std::vector<int32_t> zero_windows;    // windows whose C rows must be cleared (empty or split)
    std::vector<int32_t> ws_slot;         // [n_windows] first scratch slot of a split window (one per task), -1 for the others
};

// How a WCSR product is dealt to kernels (wcsr_build_rows): windows whose rows share few columns are walked entry by
// entry (asp_wcsr_rows.hip), the others tile by tile.
struct HostRows {
    std::vector<int32_t> row_ptr;     // [m + 1] entries of the rows walked entry by entry, consecutive
    std::vector<std::pair<int64_t, int64_t>> runs;  // where those entries are in the CSR arrays
    int64_t n_entries = 0;
    std::vector<int32_t> tasks;       // [..][4] whole rows, see walk_rows (asp_wcsr_rows.hip); empty tasks fill up
    std::vector<int32_t> chunks;      // [..][4] a chunk of a long row each, see walk_rows; empty tasks fill up
    std::vector<int32_t> split;       // [..][4] = {row, first scratch row, scratch rows, 0} of rows longer than task_cols
    int64_t dense_len = INT64_MAX;    // rows of that many entries and more are nearly dense: cut at the same columns
    std::vector<int32_t> tile_tasks;  // [..][4] as the canonical tasks, of the other windows only; empty tasks fill up
    bool tiles_dealt = false;         // tile_tasks holds one range for each XCD (deal_to_xcds)
    std::vector<int32_t> tile_split;  // the split windows among those
};

// Nearly dense rows that meet in LDS (wcsr_build_dense, asp_wcsr_dense.hip), and the lists of HostRows without them.
struct HostDense {
    static constexpr int COLS = 256, ROWS = 64;  // columns of B at a time; rows to a workgroup, at most
    static constexpr int64_t RANGES = 256;       // of columns, at most
    int64_t ranges = 0, blocks = 0, per_pass = 0;  // ranges 0: the rest is not used; per_pass: rows to a workgroup
    int64_t meet_tenths = 0;                       // entries of a pass in a column in the mean, in tenths
    std::vector<int32_t> rows;                   // [..][4] = {row, first scratch row, 0, 0}
    std::vector<int32_t> ptr;                    // [rows][blocks + 1] first entry of each row from a block's first column on
    std::vector<int32_t> tasks, chunks, split;   // as in HostRows; split: the dense rows first
};

// Chunks of nearly dense rows for workgroups instead of waves, and the list of chunks without them (wcsr_build_teams).
struct HostWide {
    std::vector<int32_t> teams, chunks;
    int64_t count = 0, len = 0;  // of those chunks, and their entries in the mean
};

// Long rows of scattered entries that walk the columns of B together (wcsr_build_groups, asp_wcsr_groups.hip), and the
// lists of HostRows without them.
struct HostGroups {
    static constexpr int rows(size_t esize) { return esize == 2 ? 31 : 63; }  // pieces of rows to a task
    static constexpr int64_t RANGES = 8; // of columns, one to an XCD
    int64_t n_groups = 0;                // tasks of a range; 0: the rest is not used
    int64_t span = 0;                    // columns of the widest range
    static constexpr int32_t MANY_PIECES = 512;
    int64_t n_many = 0;                  // rows with more scratch rows than that: the first ones of `split`
    int64_t near_cols = 0;               // many entries whose rows meet in few columns at a time: that many, 0: they do not
    ZeroedBytes entries;                 // 8 bytes each, see wcsr_groups_kernel, as are:
    std::vector<int32_t> tasks, slots;
    std::vector<int32_t> row_tasks, chunks, split;  // as in HostRows
};

// converters (asp_convert.cpp); values are only bit-copied
void csr_to_bcsr(int64_t m, int64_t k, const int32_t *row_ptr, const int32_t *col_idx, const void *values,
                 size_t esize, int32_t b_row, int32_t b_col, HostBcsr &out);
enum class Orders { LENGTH, TILES, ROWS_128, ALL };
void bcsr_build_schedule(HostBcsr &b, Orders orders);
void bcsr_build_shares(const HostBcsr &b, BcsrShares &out);
double bcsr_build_composite(const HostBcsr &in, int64_t m, int64_t k, int32_t b, HostBcsr &out);
void bcsr_pack_fragments_bf16(const HostBcsr &in, int32_t b_row, int32_t b_col, std::vector<uint8_t> &packed);
void bcsr_pack_fragments_f32(const HostBcsr &in, int32_t b_row, int32_t b_col, std::vector<uint8_t> &packed);
bool csr_to_wcsr(int64_t m, int64_t k, const int32_t *row_ptr, const int32_t *col_idx, const void *values,
                 size_t esize, int32_t b_row, int32_t b_col, HostWcsr &out);
void wcsr_tasks_host(const std::vector<int32_t> &window_row_ptr, int32_t task_cols, std::vector<int32_t> &tasks);
void wcsr_build_rows(int64_t m, const int32_t *row_ptr, const int32_t *col_idx, size_t esize, int32_t b_row,
                     int32_t task_cols, const HostWcsr &in, HostRows &out);
void wcsr_build_groups(int64_t m, const int32_t *row_ptr, const int32_t *col_idx, const void *values, size_t esize,
                       int32_t b_row, int32_t task_cols, const HostWcsr &in, const HostRows &rows, HostGroups &out);
void wcsr_build_dense(int64_t m, const int32_t *row_ptr, const int32_t *col_idx, int32_t b_row, int32_t task_cols, const HostWcsr &in,
                      const HostRows &rows, HostDense &out);
void wcsr_build_teams(int64_t n_entries, const HostRows &rows, std::vector<int32_t> &chunks, std::vector<int32_t> &tasks,
                      std::vector<int32_t> &teams, HostWide &wide);
inline int64_t split_scratch_rows(const std::vector<int32_t> &split) {  // of a list of split rows, all together
    int64_t rows = 0;
    for (size_t i = 2; i < split.size(); i += 4) rows += split[i];
    return rows;
}
void wcsr_zero_windows(const std::vector<int32_t> &window_row_ptr, int32_t task_cols,
                       std::vector<int32_t> &zero_windows);
// returns empty string when the CSR arrays are valid, else a description of the first problem
std::string validate_csr(int64_t m, int64_t k, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx);

}  // namespace asp

// ---- the opaque handle ---------------------------------------------------------------------------
struct asp_handle {
    int64_t m = 0, k = 0, nnz = 0;
    int32_t format = 0, dtype = 0, b_row = 0, b_col = 0, task_cols = 0;
    uint32_t flags = 0;
    int device = -1;  // HIP device that owns the d_* arrays, -1 in host-convert mode
    int64_t n_brows = 0, n_units = 0, n_tasks = 0, n_zero_windows = 0;
    int64_t n_split_windows = 0;  // WCSR: windows with more than one task
    int64_t n_split_tasks = 0;    // WCSR: tasks of those windows = scratch slots

    asp::HostBcsr hb;  // BCSR: canonical arrays stay on the host for export
    // bf16 BCSR with 64x64 / 32x32 blocks: the composite form (128-row super-rows, asp_convert.cpp) when it was
    // judged worth it at creation; hc keeps its scheduling data, the packed values live on the device only
    asp::HostBcsr hc;
    bool has_comp = false;
    double comp_inflation = 0.0;    // composite work over stored-block work
    int64_t c_n_brows = 0, c_n_units = 0;  // super-rows, composite blocks
    int32_t *d_c_rank_info = nullptr;
    int32_t *d_c_rank_info_32 = nullptr;
    asp::BcsrShares shares;         // of hc, or of hb with 128-row blocks; its lists live on the device only
    int32_t *d_share_lists = nullptr;
    // asp_spmm / asp_spmm_xt by the ring kernel in 64-, 128- and 256-wide tiles, 1 to 128 of them: group_n + lists, 0 before the first
    mutable std::atomic<uint8_t> ring_walks[2][3][129] = {};
    // asp_spmm / asp_spmm_xt of 1 to 256 N-tiles: 1 + the number of shared ones, 0 before the first such call
    mutable std::atomic<uint8_t> n_shared[2][257] = {};
    int32_t *d_c_slice_rows = nullptr;     // [composite blocks][4]
    int32_t *d_c_piece_rows = nullptr;     // [super-rows][4]
    void *d_c_values = nullptr;
    asp::HostWcsr hw;  // WCSR: kept only in host-convert mode (device arrays are canonical)

    // device arrays
    int32_t *d_row_ptr = nullptr;   // block_row_ptr / window_row_ptr
    int32_t *d_col_idx = nullptr;   // block_col_idx / window_col_idx
    void *d_values = nullptr;       // BCSR: fragment-packed blocks; WCSR: canonical tiles
    int32_t *d_tasks = nullptr;     // WCSR tasks [n_tasks][4]
    int32_t *d_zero_windows = nullptr;
    int32_t *d_rank_info = nullptr; // BCSR: [n_brows][4] = {block-row, first block, stored blocks, block column of the first one}, heaviest first
    int32_t *d_rank_info_32 = nullptr, *d_rank_info_64 = nullptr;
    int32_t *d_by_length = nullptr;
    int n_cus = 0;                  // compute units of the owning device
    int32_t *d_sched = nullptr;     // BCSR: 8 tile counters of the dynamic-scheduling variant (a benchmarking switch)
    // WCSR: where the tasks of split windows put their partial tiles
    int32_t *d_ws_slot = nullptr;   // [n_windows] first scratch slot of a split window, -1 otherwise
    // WCSR: the kernels' work lists (HostRows) and the entries of the windows that are walked entry by entry
    int64_t n_row_tasks = 0, n_chunks = 0, n_split_rows = 0, n_tile_tasks = 0, n_tile_split = 0;
    bool tiles_dealt = false;
    int64_t n_teams = 0, scratch_rows = 0;  // (scratch_rows: that the split rows of the list add, here and in the lists below)
    int32_t *d_teams = nullptr;           // those that a workgroup takes instead of a wave (wcsr_build_teams)
    struct Wide {                         // HostWide; its teams stand before the others
        int64_t n_teams = 0, n_chunks = 0, count = 0, len = 0;
        int32_t *d_chunks = nullptr;
    } wide, d_wide;
    int32_t *d_row_tasks = nullptr, *d_chunks = nullptr, *d_split_rows = nullptr, *d_tile_tasks = nullptr, *d_tile_split = nullptr;
    int32_t *d_e_row_ptr = nullptr, *d_e_col = nullptr;
    void *d_e_val = nullptr;
    // WCSR: long rows in groups, and the lists of what is left beside them, for calls with scratch (HostGroups)
    int64_t n_groups = 0, group_span = 0, group_near_cols = 0, group_many = 0;
    int64_t n_g_row_tasks = 0, n_g_chunks = 0, n_g_split_rows = 0, n_g_teams = 0, g_scratch_rows = 0;
    int32_t *d_g_teams = nullptr;
    uint64_t *d_group_entries = nullptr;
    int32_t *d_group_tasks = nullptr, *d_group_slots = nullptr, *d_g_row_tasks = nullptr, *d_g_chunks = nullptr, *d_g_split_rows = nullptr;
    // WCSR: nearly dense rows over columns in LDS, and the lists of what is left beside them, for calls with scratch (HostDense)
    int64_t n_dense = 0, dense_ranges = 0, dense_blocks = 0, dense_per_pass = 0, dense_meet_tenths = 0;
    int64_t n_d_row_tasks = 0, n_d_chunks = 0, n_d_split_rows = 0, n_d_teams = 0, d_scratch_rows = 0;
    int32_t *d_dense_rows = nullptr, *d_dense_ptr = nullptr, *d_d_row_tasks = nullptr, *d_d_chunks = nullptr, *d_d_split_rows = nullptr,
            *d_d_teams = nullptr;
    float *d_ws = nullptr;          // fp32 scratch, one [b_row][N] tile per slot (asp_reserve)
    int64_t ws_floats = 0;          // its capacity
};

namespace asp {
// kernels' host launchers (asp_bcsr.hip / asp_wcsr.hip)
struct BcsrPlan {
    int32_t bn;
    int32_t n_tiles;
    int32_t vectorized;
    int64_t workgroups;
};
BcsrPlan bcsr_plan(const asp_handle *h, int64_t N, bool aligned);
// the 128x512-tile kernel can take this handle: 128x128 blocks with K % 128 == 0, or a composite form
inline bool bcsr_wide_capable(const asp_handle *h) { return h->has_comp || (h->b_row == 128 && h->k % 128 == 0); }
bool bcsr_dma_launch(const asp_handle *h, const void *B, void *C, int64_t N, const BcsrPlan &p, hipStream_t stream);
bool bcsr_dma_xt_launch(const asp_handle *h, const void *X, void *Y, int64_t N, const BcsrPlan &p, hipStream_t stream);
// the staged strips of asp_spmm_xt: 0, or their row tiles of 32 (asp_bcsr_xt.hip)
int bcsr_xt_staged_strips(const asp_handle *h, int64_t N);
void bcsr_wide_xt_launch(const asp_handle *h, const void *X, void *Y, int64_t N, hipStream_t stream);
bool bcsr_strip_launch(const asp_handle *h, const void *B, void *C, int64_t N, const BcsrPlan &p, hipStream_t stream);
// fp32, many 64 x 128 tiles: whether one wave takes a whole one (asp_bcsr_f32.hip)
bool bcsr_f32_one_wave(const asp_handle *h, int64_t N);
bool bcsr_f32_launch(const asp_handle *h, const void *B, void *C, int64_t N, hipStream_t stream);
bool bcsr_wide_launch(const asp_handle *h, const void *B, void *C, int64_t N, const BcsrPlan &p, hipStream_t stream);
// the tile width of the register-staged kernel where rows are not 16-byte aligned (asp_bcsr.hip)
int bcsr_unaligned_bn(const asp_handle *h, int64_t N);
asp_status_t bcsr_spmm_launch(const asp_handle *h, const void *B, void *C, int64_t N, hipStream_t stream);
asp_status_t bcsr_spmm_xt_launch(const asp_handle *h, const void *X, void *Y, int64_t N, hipStream_t stream);

struct WcsrPlan {
    int32_t bn;
    int32_t n_tiles;
    int32_t vectorized;
    int64_t workgroups;
};
WcsrPlan wcsr_plan(const asp_handle *h, int64_t N, bool aligned);
// columns of a lane in the tiles of heights 32 and 64, fp32
int wcsr_lane_columns(const asp_handle *h, int64_t N);
// ws / ws_floats: the fp32 buffer that takes the partial tiles of split windows and its capacity (the handle's
// reserved buffer, or the library's static one; nullptr / 0: none)
asp_status_t wcsr_spmm_launch(const asp_handle *h, const void *B, void *C, int64_t N, float *ws, int64_t ws_floats,
                              hipStream_t stream);
asp_status_t wcsr_bf16_spmm_launch(const asp_handle *h, const void *B, void *C, int64_t N, float *ws, int64_t ws_floats,
                                   hipStream_t stream);
// The library's static scratch array on `device` (which must be the current device): its device address, resolved
// once per device, and its capacity in floats.
asp_status_t wcsr_static_scratch(int device, float **ptr, int64_t *floats);
int64_t wcsr_scratch_floats(const asp_handle *h, int64_t N);  // fp32 scratch elements a call of width N uses
// windows that are walked entry by entry (empty ones among them), and the sums of their split rows
void wcsr_rows_launch(const asp_handle *h, const void *B, void *C, int64_t N, float *ws, hipStream_t stream);
void wcsr_rows_sum_launch(const asp_handle *h, void *C, int64_t N, const float *ws, hipStream_t stream);
// The walk by rows from wave `first` on, four to a workgroup, behind n_teams workgroups (a multiple of 8): where its launch ends.
constexpr int64_t rows_launch_end(int64_t waves, int64_t first, int64_t n_teams) {
    const int64_t most = first + (1 << 26) - 32 - 4 * n_teams;
    return waves < most ? waves : most;
}
static_assert(launch_fits(262144 + ceil_div(rows_launch_end(1ll << 31, 0, 262144), 4), 256), "one launch");
// whether workgroups share the chunks of nearly dense rows too: `count` of them, of `len` entries each
bool wcsr_share_chunks(const asp_handle *h, int64_t N, int64_t count, int64_t len);
// how many of the split rows (the first of the call's list) have their scratch rows added by many threads
int64_t wcsr_rows_sum_many(const asp_handle *h, int64_t N);
// the groups of long rows: whether calls of this width (with scratch) use them, and their kernel
bool wcsr_groups_apply(const asp_handle *h, int64_t N);
void wcsr_groups_launch(const asp_handle *h, const void *B, int64_t N, float *ws, hipStream_t stream);
// the nearly dense rows: whether calls of this width (with scratch) use them, and their kernel
bool wcsr_dense_apply(const asp_handle *h, int64_t N);
void wcsr_dense_launch(const asp_handle *h, const void *B, int64_t N, float *ws, hipStream_t stream);
// rows of split windows = sum of their tasks' partial tiles, in task order
void wcsr_sum_partial_tiles(const asp_handle *h, void *C, int64_t N, const float *ws, hipStream_t stream);
// GPU task partition: fills h->d_tasks / h->n_tasks from h->d_row_ptr (wavefront scans)
asp_status_t wcsr_build_tasks_device(asp_handle *h, hipStream_t stream);
}  // namespace asp

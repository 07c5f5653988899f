// WCSR x dense SpMM in fp32: a few nearly dense rows, over columns of B that a workgroup holds in LDS.
//
// Rows with a tenth of all columns meet in every column, and walked one by one (chunks in asp_wcsr_rows.hip) each of their entries
// pulls a row of B from L2, 15 TB/s.  Here a workgroup takes a range of the columns, 256 of them at a time: it reads these
// rows of B once, into LDS, and its 16 waves walk the entries of up to 64 rows against them, four rows to a wave, whose sums stay in
// registers for the whole range.  What bounds it is the one pass over B with the lines that the one workgroup on a compute unit
// has in flight (56 in the mean, 791 cycles each; 4.1 TB/s with the entries); LDS is busy for a quarter of that time, without bank conflicts.
// 64 rows of 200 000 entries over 2 000 000 columns, N = 64: 207 us in chunks, 150 here.
//
// A wave's 64 lanes are 4 groups of 16 that cover a row of B (64 columns, 4 to a lane) each and take every fourth entry: lane i of a
// group holds the group's i-th entry of up to 16, broadcast (row_newbcast) as it is used.  What fills up the last four adds 0 x 0 from a
// row of zeros: no row of A that does not store a column may see its values.  B and the entries of the next 256 columns are on their
// way while these are walked.  Sums are moved to a second register every 8 blocks, so that they stay short, and the ranges' sums go
// to rows of scratch memory, which wcsr_rows_sum_kernel adds up: a fixed order.
#include "asp_wcsr_rows.h"

namespace asp {

namespace {
constexpr int DENSE_COLS = HostDense::COLS, DENSE_WAVES = 16, DENSE_RPW = HostDense::ROWS / DENSE_WAVES;
}

// rows[r] = {row, first scratch row, -, -}; block_ptr[r * (n_blocks + 1) + b]: first entry of row r (a position of col / val) in the
// columns from b * 256 on, b = 0 .. n_blocks.  grid = (ranges, tiles of 64 columns of B, groups of per_pass <= 64 rows).  N >= 64.
__global__ __launch_bounds__(DENSE_WAVES * 64) void wcsr_dense_kernel(const int4 *__restrict__ rows, int n_rows, int per_pass,
                                                                     const int32_t *__restrict__ block_ptr, int n_blocks, int K,
                                                                     const int32_t *__restrict__ col, const float *__restrict__ val,
                                                                     const float *__restrict__ B, int64_t N, float *__restrict__ ws) {
    typedef float lds_vec_t __attribute__((ext_vector_type(4)));
    typedef float chunk_t __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int ROW = 64 * 4, CPR = ROW / 16, RPP = DENSE_WAVES * 64 / CPR, PASSES = DENSE_COLS / RPP;
    constexpr int STAGE = DENSE_COLS * ROW;
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * STAGE + ROW];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int group = lane >> 4, i16 = lane & 15;
    const int b0 = (int)((int64_t)n_blocks * blockIdx.x / gridDim.x), b1 = (int)((int64_t)n_blocks * (blockIdx.x + 1) / gridDim.x);
    const int64_t n0 = (int64_t)blockIdx.y * 64 < N - 64 ? (int64_t)blockIdx.y * 64 : N - 64;  // the last tile moves left
    int row_of[DENSE_RPW];  // of this wave; the last row again where there are fewer (not written)
    bool have[DENSE_RPW];
#pragma unroll
    for (int r = 0; r < DENSE_RPW; ++r) {
        const int i = r * DENSE_WAVES + wave, x = blockIdx.z * per_pass + i;
        have[r] = i < per_pass && x < n_rows;
        row_of[r] = have[r] ? x : n_rows - 1;
    }

    // B: thread t loads chunk t % CPR of rows t / CPR, + RPP, ...
    const int st_row = tid / CPR, st_chunk = tid % CPR;
    chunk_t staged[PASSES];
    auto load_b = [&](int b) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            const int k = b * DENSE_COLS + st_row + i * RPP;
            staged[i] = *(const chunk_t *)((const uint8_t *)(B + (int64_t)(k < K ? k : K - 1) * N + n0) + st_chunk * 16);
        }
    };
    auto store_b = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PASSES; ++i) {
            *(lds_vec_t *)(lds + buf * STAGE + (st_row + i * RPP) * ROW + st_chunk * 16) = staged[i];
        }
    };
    // the first entry of each of the wave's rows in blocks ptr_base + lane, 64 blocks at a time
    int ptr_base = b0, ptr[DENSE_RPW];
    auto load_ptr = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < DENSE_RPW; ++r) {
            const int at = ptr_base + lane < n_blocks ? ptr_base + lane : n_blocks;
            ptr[r] = block_ptr[(int64_t)row_of[r] * (n_blocks + 1) + at];
        }
    };
    // the wave's entries of a block, 64 of each row (what is past the end is dropped as they are used: no load has a condition, or
    // each would be waited for by itself)
    struct Entries {
        int first[DENSE_RPW], end[DENSE_RPW];
        int c[DENSE_RPW];
        float v[DENSE_RPW];
    };
    auto load_entry = [&](int first, int end, int &c, float &v) __attribute__((always_inline)) {
        const int e = min(first + 4 * i16 + group, max(end - 1, 0));
        c = col[e], v = val[e];
    };
    auto load_entries = [&](int b, Entries &e) __attribute__((always_inline)) {
        if (b + 1 - ptr_base >= 64) {
            ptr_base = b;
            load_ptr();
#pragma unroll
            for (int r = 0; r < DENSE_RPW; ++r) asm volatile("" : "+v"(ptr[r]));  // waited for here
        }
#pragma unroll
        for (int r = 0; r < DENSE_RPW; ++r) {
            e.first[r] = __builtin_amdgcn_readlane(ptr[r], b - ptr_base);
            e.end[r] = __builtin_amdgcn_readlane(ptr[r], b + 1 - ptr_base);
            load_entry(e.first[r], e.end[r], e.c[r], e.v[r]);
        }
    };

    float acc[DENSE_RPW][4], sum[DENSE_RPW][4];
#pragma unroll
    for (int r = 0; r < DENSE_RPW; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[r][i] = 0.f, sum[r][i] = 0.f;
    auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < DENSE_RPW; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[r][i] += acc[r][i], acc[r][i] = 0.f;
    };

    if (tid < ROW / 4) ((uint32_t *)(lds + 2 * STAGE))[tid] = 0u;
    if (b0 < b1) {
        Entries now, next;
        load_ptr();
        load_b(b0);
        load_entries(b0, now);
        store_b(0);
        __syncthreads();
        for (int b = b0; b < b1; ++b) {
            const int buf = (b - b0) & 1, bn = b + 1 < b1 ? b + 1 : b;
            load_b(bn);
            load_entries(bn, next);
#pragma unroll
            for (int r = 0; r < DENSE_RPW; ++r) {
                int c = now.c[r];
                float raw = now.v[r];
                for (int first = now.first[r]; first < now.end[r];) {
                    const int steps = (min(now.end[r] - first, 64) + 3) >> 2;
                    const bool in = first + 4 * i16 + group < now.end[r];
                    const int at = in ? buf * STAGE + (c - b * DENSE_COLS) * ROW : 2 * STAGE;  // where the entry's row of B is
                    const float v = in ? raw : 0.f;
#define ASP_STEP(j)                                                                                                       \
    do {                                                                                                                  \
        const int at_ = __builtin_amdgcn_mov_dpp(at, 0x150 + (j), 0xf, 0xf, true) + i16 * 16;          \
        const float f_ = __uint_as_float(__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x150 + (j), 0xf, 0xf, true)); \
        const lds_vec_t x_ = *(const lds_vec_t *)(lds + at_);                                                             \
        _Pragma("unroll") for (int q = 0; q < 4; ++q) acc[r][q] = __builtin_fmaf(f_, x_[q], acc[r][q]);         \
    } while (0)
#define ASP_STEPS(j)                                    \
    ASP_STEP(j); ASP_STEP((j) + 1); ASP_STEP((j) + 2); ASP_STEP((j) + 3)
                    ASP_STEPS(0);
                    if (steps > 4) {
                        ASP_STEPS(4);
                        if (steps > 8) {
                            ASP_STEPS(8);
                            if (steps > 12) {
                                ASP_STEPS(12);
                            }
                        }
                    }
#undef ASP_STEPS
#undef ASP_STEP
                    first += 64;
                    if (first < now.end[r]) load_entry(first, now.end[r], c, raw);
                }
            }
            if (((b - b0) & 7) == 7) flush();
            store_b(buf ^ 1);
            now = next;
            __syncthreads();
        }
    }
    flush();
#pragma unroll
    for (int r = 0; r < DENSE_RPW; ++r) {
        if (!have[r]) continue;
        typedef float out_t __attribute__((ext_vector_type(4), aligned(4)));
        out_t o;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float t = sum[r][i];
            t += __shfl_xor(t, 32);
            t += __shfl_xor(t, 16);
            o[i] = t;
        }
        if (group == 0) *(out_t *)(ws + ((int64_t)rows[row_of[r]].y + blockIdx.x) * N + n0 + i16 * 4) = o;
    }
}

// ---- host side ------------------------------------------------------------------------------------
// Where the pass over B costs less than the chunks' rows of B, which come faster where the memory-side cache holds it, where a row is
// walked by lane groups (N = 64) and where it is long and workgroups share the chunks (N > 128), and which have no columns to fill up.
// us, band of 9, 54 long rows / 64, chunks / here: N = 64, 600 000 rows (154 MB) 105 / 115, 114 / 119, 1 500 000 (384 MB) 306 / 278, 324 / 280;
// N = 72, 600 000 187 / 186, 206 / 186; N = 128, 300 000 (154 MB) 116 / 114, 122 / 114, 600 000 252 / 219, 269 / 221.  Shared, 54 of them: N = 130,
// 300 000 143 / 174, 600 000 319 / 338; N = 160 (192 columns walked), 300 000 142 / 164, 600 000 (384 MB) 324 / 321; N = 256, 300 000 (307 MB) 231
// / 238, 600 000 463 / 448; N = 200 (256 walked), 600 000 429 / 457.  Not shared, 64 of them, 600 000 rows: N = 130 333 / 342, N = 160 345 / 323, N =
// 200 457 / 461: even or faster here, and 1.6e-7 from the 64-bit sums instead of 2.7e-7 (shared 1.6e-7, lane groups 1.6e-7), with 4 entries a
// column walked and more; 54 of them, 1 500 000 rows, N = 130 770 / 796.  In two passes, 100 of them: 300 000 rows, N = 128 151 / 160, 600 000
// (307 MB) 335 / 313; 122, 600 000, N = 160 455 / 466, N = 200 596 / 677; 115, N = 192 493 / 485.  In bf16 chunks are always faster (600 000 rows 126 / 154).
bool wcsr_dense_apply(const asp_handle *h, int64_t N) {
    const int64_t bytes = h->k * N * 4, walked = 64 * ceil_div(N, 64);
    const bool one_pass = h->n_dense <= h->dense_per_pass;
    if (h->n_dense == 0 || N < 64 || bytes < ((N == 64 ? 224ll : one_pass ? 128ll : 160ll) << 20)) return false;
    if (N <= 128) return true;
    if (wcsr_share_chunks(h, N, h->wide.count, h->wide.len)) return bytes >= 352ll << 20 && 5 * walked <= 6 * N;
    return one_pass ? h->dense_meet_tenths * N >= 40 * walked : 20 * walked <= 21 * N;
}

void wcsr_dense_launch(const asp_handle *h, const void *B, int64_t N, float *ws, hipStream_t stream) {
    const dim3 grid((unsigned)h->dense_ranges, (unsigned)ceil_div(N, 64), (unsigned)ceil_div(h->n_dense, h->dense_per_pass));
    hipLaunchKernelGGL(wcsr_dense_kernel, grid, dim3(DENSE_WAVES * 64), 0, stream, (const int4 *)h->d_dense_rows, (int)h->n_dense,
                       (int)h->dense_per_pass, h->d_dense_ptr, (int)h->dense_blocks, (int)h->k, h->d_e_col, (const float *)h->d_e_val, (const float *)B, N, ws);
}

}  // namespace asp

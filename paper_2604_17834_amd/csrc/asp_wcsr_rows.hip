// WCSR x dense SpMM for row-windows whose rows share (almost) no columns: the entries are walked row by row.
//
// A window tile (paper, Section II-C) stores b_row values per packed column and pays off when several rows of the
// window meet in that column.  In graph-like matrices with scattered columns they do not: a packed column holds one
// entry, its tile is 64 (fp32, height 16) to 256 bytes of mostly zeros beside the 4 N bytes of the gathered row of B,
// and a window's tasks are as long as its longest row.  Such windows (wcsr_build_rows decides per window, at creation)
// run here from plain (column, value) entries, 6-8 bytes each.
//
// What bounds it: the gather.  Random rows of B that miss L2 arrive at 7.5 TB/s on this chip whatever the size of B
// (measured with rows of 128-512 bytes over 67 MB - 1 GB), so the design removes every other byte and keeps enough of
// those in flight: one wavefront walks a run of consecutive rows, 64 to 256 entries; columns and values are uniform
// for the wave and come through scalar loads (16 entries ahead), so an entry costs one vector load with a scalar base
// and E multiply-adds with a scalar factor; two batches of 8 rows of B are in flight per wave, up to 8 waves per SIMD.
// A row's entries are summed in fp32, in order where one wave walks them, by quarters where a workgroup does (wcsr_rows_kernel).  Rows
// longer than task_cols are cut into chunks (Section III-C) whose
// sums go to rows of scratch memory, which wcsr_rows_sum_kernel adds up.
//
// Order of the work: chunks of long rows are sorted by column and dealt to the XCDs in contiguous ranges, so that the
// chunks of different rows that cover the same columns run on one XCD at about the same time and find the rows of B in
// its L2 (64 rows of 200 000 entries over 2 000 000 columns, N = 64: 80 % of the line requests).
//
// Any N and any alignment: a lane owns E adjacent columns; the last lane of a row moves left so that it ends at N and
// computes some of its neighbour's columns a second time (the same bits), so that no access leaves the row.
#include <algorithm>

#include "asp_wcsr_rows.h"

namespace asp {

namespace {

__device__ __forceinline__ void narrow(float v, float &out) { out = v; }
__device__ __forceinline__ void narrow(float v, uint16_t &out) { out = __builtin_bit_cast(uint16_t, (__bf16)v); }  // to nearest even

// Entry positions go up to 2^31 - 1 and are ints, so nothing is added to an end.
// Batch of 8 from `base` (a multiple of 8): whether all of it, and whether its j-th entry, is in [e0, e1).
constexpr bool batch_inside(int base, int e0, int e1) { return base >= e0 && e1 - base >= 8; }
constexpr bool entry_inside(int base, int j, int e0, int e1) { return base + j >= e0 && j < e1 - base; }
// i-th entry of [e0, e1), the last one for those behind it
constexpr int entry_clamped(int e0, int e1, int i) { return e0 + (i < e1 - e0 ? i : e1 - e0 - 1); }
static_assert(!batch_inside(0x7ffffff8, 0, 0x7fffffff) && entry_inside(0x7ffffff8, 6, 0, 0x7fffffff) &&
                  !entry_inside(0x7ffffff8, 7, 0, 0x7fffffff) && entry_clamped(0x7ffffff0, 0x7fffffff, 63) == 0x7ffffffe,
              "the last entries of 2^31 - 1");

// The sum of a chunk {row, scratch row, -, -} at columns nc .. nc + E - 1 (the lane's own ones start at n): to its row of
// ws, or without ws (fp32 only) added to C with atomics.
template <typename T, int E>
__device__ __forceinline__ void put_chunk(int4 td, const float (&acc)[E], int64_t n, int64_t nc, int64_t N, T *C, float *ws) {
    if (ws) {
        float *dst = ws + (int64_t)td.y * N + nc;
#pragma unroll
        for (int i = 0; i < E; ++i) dst[i] = acc[i];
    } else if constexpr (sizeof(T) == 4) {
        float *dst = (float *)C + (int64_t)td.x * N + nc;
#pragma unroll
        for (int i = 0; i < E; ++i)
            if (nc + i >= n) unsafeAtomicAdd(dst + i, acc[i]);  // a column of two lanes is added by one of them
    }
}

// The sum of a whole row at columns nc .. nc + E - 1.
template <typename T, int E>
__device__ __forceinline__ void put_row(int row, const float (&acc)[E], int64_t nc, int64_t N, T *C) {
    T *dst = C + (int64_t)row * N + nc;
#pragma unroll
    for (int i = 0; i < E; ++i) narrow(acc[i], dst[i]);
}

}  // namespace

// tasks[t] = {first row, rows (1..63), first entry, end entry}: consecutive whole rows.  row_ptr / col / val: the entries
// of the rows handled here; col and val are readable up to the next multiple of 8 entries plus 8.
// CHUNK: the task is (part of) a chunk of a long row, {row, scratch row, first entry, end entry}; its sum stays in `acc`.
// One wave: task td, columns from blockIdx.y * 64 E.
template <typename T, int E, bool CHUNK>
__device__ __forceinline__ void walk_rows(const int4 td, const int32_t *__restrict__ row_ptr,
                                          const int32_t *__restrict__ col, const T *__restrict__ val,
                                          const T *__restrict__ B, T *__restrict__ C, int64_t N, float (&acc)[E]) {
    typedef typename RowVec<T, E>::type vec_t;
    const int lane = threadIdx.x & 63;
    const int64_t n = (int64_t)blockIdx.y * (64 * E) + lane * E;
    const int64_t nc = n < N - E ? n : N - E;  // N >= E
    const bool owner = n < N;
    const uint32_t voff = (uint32_t)(nc * (int64_t)sizeof(T)), row_bytes = (uint32_t)(N * (int64_t)sizeof(T));
    const int e0 = td.z, e1 = td.w;

#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.f;

    // batches of 8 entries, aligned; entries outside [e0, e1) read a row of B that the task reads anyway, and what they
    // add is dropped (no row of A that does not store a column may see its values: zero times Inf is NaN)
    struct Batch {
        int c[8];
        uint32_t v[8];  // fp32 bits (as integers, so that selections stay in scalar registers)
    };
    const int base0 = e0 & ~7, nb = e1 > e0 ? (e1 - base0 + 7) >> 3 : 0;
    const int c_any = nb > 0 ? col[e0] : 0;
    auto fetch = [&](int b, Batch &t) __attribute__((always_inline)) {
        const int base = base0 + 8 * b;
#pragma unroll
        for (int j = 0; j < 8; ++j) t.c[j] = col[base + j];
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int j = 0; j < 8; ++j) t.v[j] = __float_as_uint(widen(val[base + j]));
        } else {  // scalar loads are whole words
            const uint32_t *w = (const uint32_t *)(val + base);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t p = w[j];
                t.v[2 * j] = p << 16;
                t.v[2 * j + 1] = p & 0xffff0000u;
            }
        }
        if (!batch_inside(base, e0, e1))
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (!entry_inside(base, j, e0, e1)) t.c[j] = c_any;
    };
    auto gather = [&](const Batch &t, vec_t (&b)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const global_char *row = (const global_char *)B + (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(t.c[j]) * row_bytes;
            uint32_t off = voff;
            asm("" : "+s"(row), "+v"(off));  // scalar base + 32-bit offset, instead of a 64-bit vector address per row
            b[j] = *(const __attribute__((address_space(1))) vec_t *)(row + off);
        }
    };
    // Two batches in flight: while one is added, the next is on its way and the entries of the one after it are read.
    // (The loop issues without conditions -- otherwise the waits before the additions would have to assume that the
    // younger loads were not issued, and wait for them too.  The last batches are left to the code behind it.)
    auto walk = [&](auto add) __attribute__((always_inline)) {
        Batch t0, t1, t2;
        vec_t b0[8], b1[8];
        int b = 0;
        if (nb > 0) {
            fetch(0, t0);
            gather(t0, b0);
            if (nb > 1) fetch(1, t1);
        }
        for (; b + 3 < nb; b += 2) {
            gather(t1, b1);
            fetch(b + 2, t2);
            add(b, t0, b0);
            gather(t2, b0);
            t0 = t2;
            fetch(b + 3, t2);
            add(b + 1, t1, b1);
            t1 = t2;
        }
        if (b + 1 < nb) {
            gather(t1, b1);
            if (b + 2 < nb) fetch(b + 2, t2);
            add(b, t0, b0);
            if (b + 2 < nb) gather(t2, b0);
            add(b + 1, t1, b1);
            if (b + 2 < nb) add(b + 2, t2, b0);
        } else if (b < nb) {
            add(b, t0, b0);
        }
    };
    auto fma_entry = [&](const Batch &t, const vec_t (&bv)[8], int j) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < E; ++i) acc[i] = __builtin_fmaf(__uint_as_float(__builtin_amdgcn_readfirstlane(t.v[j])), widen((T)bv[j][i]), acc[i]);
    };

    if (CHUNK) {
        walk([&](int b, const Batch &t, const vec_t(&bv)[8]) __attribute__((always_inline)) {
            const int base = base0 + 8 * b;
            if (!batch_inside(base, e0, e1)) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (entry_inside(base, j, e0, e1)) fma_entry(t, bv, j);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) fma_entry(t, bv, j);
            }
        });
        return;
    }

    // lane i holds the end of the task's i-th row (-1: no entry is there).  Entries of the first batch before e0 count as a
    // row -1 that ends at e0 and is not stored.
    int ends = -1;
    if (lane < td.y) ends = row_ptr[td.x + lane + 1];
    int k = 0, end_k = __builtin_amdgcn_readlane(ends, 0);
    if (nb > 0 && base0 < e0) k = -1, end_k = e0;
    auto finish_row = [&]() __attribute__((always_inline)) {
        global_char *row = (global_char *)C + (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(td.x + k) * row_bytes;
        uint32_t off = voff;
        asm("" : "+s"(row), "+v"(off));
        vec_t v;
#pragma unroll
        for (int i = 0; i < E; ++i) {
            T o;
            narrow(acc[i], o);
            v[i] = o;
            acc[i] = 0.f;
        }
        if (owner && k >= 0) __builtin_nontemporal_store(v, (__attribute__((address_space(1))) vec_t *)(row + off));
        ++k;
        end_k = __builtin_amdgcn_readlane(ends, k);
    };
    walk([&](int b, const Batch &t, const vec_t(&bv)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            while (base0 + 8 * b + j == end_k) finish_row();
            fma_entry(t, bv, j);
        }
    });
    while (k < td.y) finish_row();  // the last row, and rows without entries behind it
}

// A chunk of a long row where walk_rows would load 4 bytes or less per lane.  Chunks of nearly dense rows find most of
// their rows of B in L2 and are bound by the address unit instead, and a 4-byte load per lane takes as long as a wider
// one.  So here L lanes cover a row of B with up to 16 bytes each, and the G = 64 / L lane groups of the wave take
// different entries.  A group's entries are loaded 16 at a time, lane i of every 16 lanes holding the i-th, and broadcast
// within the 16 lanes (row_newbcast) as they are used; the groups' sums are added at the end in a fixed order.
// (64 rows of 200 000 entries, N = 64, fp32: 0.236 -> 0.211 ms; 3.2e6 Zipf entries, N = 100, bf16: 0.146 -> 0.133 ms.
// At 8 bytes per lane walk_rows is the better one: 16.7e6 Zipf entries, N = 128, fp32: 1.255 against 1.208 ms.)
// (e0 < e1; every lane group ends with the whole sum in `acc`)
template <typename T, int E, int L>
__device__ __forceinline__ void walk_chunk(int e0, int e1, const int32_t *__restrict__ col,
                                           const T *__restrict__ val, const T *__restrict__ B, int64_t N, float (&acc)[E]) {
    typedef typename RowVec<T, E>::type vec_t;
    constexpr int G = 64 / L;
    const int lane = threadIdx.x & 63, g = lane / L, i16 = lane & 15;
    const int64_t n = (int64_t)blockIdx.y * (L * E) + (lane % L) * E;
    const int64_t nc = n < N - E ? n : N - E;  // N >= E
    const char *base = (const char *)B + nc * (int64_t)sizeof(T);
    const uint32_t row_bytes = (uint32_t)(N * (int64_t)sizeof(T));

#pragma unroll
    for (int i = 0; i < E; ++i) acc[i] = 0.f;
    // batch b: entries (b G + g) * 16 .. + 15 of the chunk for this group; past the end: the last entry, and nothing is added
    const int len = e1 - e0;
    auto fetch = [&](int b, int &c, float &v) __attribute__((always_inline)) {
        const int es = entry_clamped(e0, e1, (b * G + g) * 16 + i16);
        c = col[es];
        v = widen(val[es]);
    };
#define ASP_BCAST(x, i) __builtin_amdgcn_mov_dpp((int)(x), 0x150 + (i), 0xf, 0xf, true)  // row_newbcast: lane i of each 16
#define ASP_GATHER(dst, j, i) \
    dst[j] = *(const vec_t *)(base + (uint64_t)(uint32_t)ASP_BCAST(c, i) * row_bytes)
#define ASP_ADD(src, j, i)                                                                                  \
    do {                                                                                                    \
        const float f_ = __uint_as_float(ASP_BCAST(__float_as_uint(v), i));                                 \
        _Pragma("unroll") for (int q = 0; q < E; ++q) acc[q] = __builtin_fmaf(f_, widen((T)src[j][q]), acc[q]); \
    } while (0)
#define ASP_ADD_LAST(src, j, i)                                                                                    \
    do {                                                                                                           \
        const float f_ = __uint_as_float(ASP_BCAST(__float_as_uint(v), i));                                        \
        const bool in_ = ((nb - 1) * G + g) * 16 + (i) < len;                                                      \
        _Pragma("unroll") for (int q = 0; q < E; ++q) acc[q] = in_ ? __builtin_fmaf(f_, widen((T)src[j][q]), acc[q]) : acc[q]; \
    } while (0)
#define ASP_EIGHT(OP, x, o) \
    OP(x, 0, o + 0); OP(x, 1, o + 1); OP(x, 2, o + 2); OP(x, 3, o + 3); OP(x, 4, o + 4); OP(x, 5, o + 5); OP(x, 6, o + 6); OP(x, 7, o + 7)
    const int nb = (len + 16 * G - 1) / (16 * G);
    int c, cn;
    float v, vn;
    vec_t lo[8], hi[8];
    fetch(0, c, v);
    ASP_EIGHT(ASP_GATHER, lo, 0);
    for (int b = 0; b + 1 < nb; ++b) {  // eight gathers ahead of the additions
        ASP_EIGHT(ASP_GATHER, hi, 8);
        fetch(b + 1, cn, vn);
        ASP_EIGHT(ASP_ADD, lo, 0);
        c = cn;
        ASP_EIGHT(ASP_GATHER, lo, 0);
        ASP_EIGHT(ASP_ADD, hi, 8);
        v = vn;
    }
    ASP_EIGHT(ASP_GATHER, hi, 8);
    ASP_EIGHT(ASP_ADD_LAST, lo, 0);
    ASP_EIGHT(ASP_ADD_LAST, hi, 8);
#undef ASP_BCAST
#undef ASP_GATHER
#undef ASP_ADD
#undef ASP_ADD_LAST
#undef ASP_EIGHT
#pragma unroll
    for (int i = 0; i < E; ++i) {
        if (G >= 2) acc[i] += __shfl_xor(acc[i], 32);
        if (G >= 4) acc[i] += __shfl_xor(acc[i], 16);
    }
}

// One wave per chunk or task, the chunks first (they are the longest).  A wave covers 64 * E = CL * CE columns
// (CL = 64: walk_rows for the chunks too); grid.y = column tiles.
// Before those: teams[t] = {row, scratch row or -1: the row is here whole, first entry, end entry}, n_teams of them, a workgroup to
// each, whose waves take a quarter of the entries and add their sums in LDS, in order.  Where a launch is so small that its longest
// chunk or row sets its time (wcsr_build_teams): a wave takes 0.4 us for every 8 entries, 25 us for 512, however few others there are.
// (Whole rows are walked in the same order at every width unless the handle has groups, which the width decides on: a slice of B's
// columns gives a slice of C there, bit for bit.)
template <typename T, int E, int CE, int CL>
__global__ __launch_bounds__(256) void wcsr_rows_kernel(const int4 *__restrict__ teams, int n_teams,
                                                        const int4 *__restrict__ chunks, int n_chunks,
                                                        const int4 *__restrict__ tasks, int n_tasks,
                                                        const int32_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col, const T *__restrict__ val,
                                                        const T *__restrict__ B, T *__restrict__ C, int64_t N,
                                                        float *__restrict__ ws) {
    constexpr int SUMS = E > CE ? E : CE;
    __shared__ float part[4][SUMS][64];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const bool team = (int)blockIdx.x < n_teams;
    const int wave = ((int)blockIdx.x - n_teams) * 4 + w;
    // the waves' sums, in wave 0 (false elsewhere)
    auto gather_sums = [&](auto &acc) __attribute__((always_inline)) {
        constexpr int n = sizeof(acc) / 4;
#pragma unroll
        for (int i = 0; i < n; ++i) part[w][i][lane] = acc[i];
        __syncthreads();
        if (w != 0) return false;
#pragma unroll
        for (int i = 0; i < n; ++i) acc[i] = (acc[i] + part[1][i][lane]) + (part[2][i][lane] + part[3][i][lane]);
        return true;
    };
    if (team || wave < n_chunks) {
        int4 td = team ? teams[blockIdx.x] : chunks[wave];
        if (td.z >= td.w) return;  // fills up a list
        if (team) {
            const int quarter = ((td.w - td.z + 3) / 4 + 15) & ~15;
            const int lo = min(td.w - td.z, w * quarter), hi = min(td.w - td.z, (w + 1) * quarter);
            td.w = td.z + hi;
            td.z += lo;
        }
        if (team && td.y < 0) {
            float acc[E];
            walk_rows<T, E, true>(td, row_ptr, col, val, B, C, N, acc);
            if (!gather_sums(acc)) return;
            const int64_t n = (int64_t)blockIdx.y * (64 * E) + lane * E;
            if (n < N) put_row<T, E>(td.x, acc, n < N - E ? n : N - E, N, C);
            return;
        }
        float acc[CE];
        if (CL == 64) {
            walk_rows<T, CE, true>(td, row_ptr, col, val, B, C, N, acc);
        } else if (td.z < td.w) {
            walk_chunk<T, CE, CL>(td.z, td.w, col, val, B, N, acc);
        } else {
#pragma unroll
            for (int i = 0; i < CE; ++i) acc[i] = 0.f;
        }
        if (team && !gather_sums(acc)) return;
        const int64_t n = (int64_t)blockIdx.y * (CL * CE) + (lane % CL) * CE;
        if (lane < CL && n < N) put_chunk<T, CE>(td, acc, n, n < N - CE ? n : N - CE, N, C, ws);  // N >= CE
    } else if (wave - n_chunks < n_tasks) {
        float acc[E];
        walk_rows<T, E, false>(tasks[wave - n_chunks], row_ptr, col, val, B, C, N, acc);
    }
}

// Split rows: {row, first scratch row, scratch rows, -}: C[row] = sum of its scratch rows, rounded once.  A workgroup
// takes COLS columns; thread (j, c) adds the scratch rows j, j + J, ... of column c, and the J sums are added in order:
// a fixed order, bitwise reproducible.  <16, 64> for long lists (few rows: 64 rows of 3600 scratch rows, N = 64, take
// 12 us, with <64, 16> 19 us), <64, 4> for short ones (12 000 rows of 5 on average, N = 128: with <16, 64> most of a
// workgroup would have nothing to add).
template <typename T, int COLS, int J>
__global__ __launch_bounds__(COLS *J) void wcsr_rows_sum_kernel(const int4 *__restrict__ split, int n_split,
                                                                const float *__restrict__ ws, T *__restrict__ C, int64_t N) {
    __shared__ float part[J][COLS + 1];
    const int c = threadIdx.x % COLS, first = threadIdx.x / COLS;
    const int64_t n = (int64_t)blockIdx.y * COLS + c;
    for (int row = blockIdx.x; row < n_split; row += gridDim.x) {  // (once, but for millions of rows)
        const int4 s = split[row];
        float sum = 0.f;
        if (n < N) {
            const float *src = ws + (int64_t)s.y * N + n;
            int j = first;
            for (; j + J * 7 < s.z; j += J * 8) {
                float t[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = src[(int64_t)(j + J * e) * N];
                sum += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
            }
            for (; j < s.z; j += J) sum += src[(int64_t)j * N];
        }
        __syncthreads();  // `part` may still be read for the row before
        part[first][c] = sum;
        __syncthreads();
        if (first == 0 && n < N) {
            float t = 0.f;
#pragma unroll
            for (int e = 0; e < J; e += 4) t += (part[e][c] + part[e + 1][c]) + (part[e + 2][c] + part[e + 3][c]);
            T o;
            narrow(t, o);
            C[(int64_t)s.x * N + n] = o;
        }
    }
}

// ---- host side ------------------------------------------------------------------------------------
// Where a wave walks such a chunk an entry at a time (walk_rows), and not the 64 entries of the shortest: four waves are as much
// more to start as they are less to walk; and where their number leaves the chip waiting for the last ones, or the rows of B are long.
// us, band of 13 and long rows with a tenth of the columns, by a wave each / by four.  fp32, N = 128: 30 000 rows, 48 long ones, chunks of
// 128 23.4 / 21.6, 60 000 33.5 / 32.8, 250 000 (8900 of them) 108 / 112; 56, of 192, 30 000 22.5 / 20.5, 250 000 102 / 100 (N = 66 88 / 90);
// N = 256: 120 000 rows, 40, 96 / 84, 56 110 / 92; 100 000, 30, of 64 75 / 83.  bf16, N = 160: 30 000, 30, of 192 20.9 / 15.8, 250 000, 24, of 128
// (4500) 61 / 62, 26 61 / 64, 56, of 320, 88 / 83.  With up to 16 lanes to a row of B (walk_chunk) never: fp32, N = 20, 298 434 rows, 33, 43 / 51;
// bf16, N = 77, 198 717 rows, 53, of 320 55 / 64, N = 68, 736 246 rows, 48 133 / 150.
bool wcsr_share_chunks(const asp_handle *h, int64_t N, int64_t count, int64_t len) {
    const bool f32 = h->dtype == ASP_DT_F32;
    if (count == 0 || N <= (f32 ? 64 : 128)) return false;
    return count <= (len > 160 ? 5000 : 2500) || (f32 ? N > 128 : N > 160 || len > 160);
}

template <typename T>
static void launch_rows(const asp_handle *h, const void *B, void *C, int64_t N, float *ws, hipStream_t stream) {
    const bool groups = ws && wcsr_groups_apply(h, N);  // long rows run there: the lists without them
    const bool dense = ws && !groups && wcsr_dense_apply(h, N);  // nearly dense rows run there
    const int32_t *d_chunks = groups ? h->d_g_chunks : dense ? h->d_d_chunks : h->d_chunks;
    const int32_t *d_row_tasks = groups ? h->d_g_row_tasks : dense ? h->d_d_row_tasks : h->d_row_tasks;
    const int4 *d_teams = (const int4 *)(groups ? h->d_g_teams : dense ? h->d_d_teams : h->d_teams);
    int64_t n_chunks = groups ? h->n_g_chunks : dense ? h->n_d_chunks : h->n_chunks;
    const int64_t n_row_tasks = groups ? h->n_g_row_tasks : dense ? h->n_d_row_tasks : h->n_row_tasks;
    if (groups) wcsr_groups_launch(h, B, N, ws, stream);
    if (dense) wcsr_dense_launch(h, B, N, ws, stream);
    int64_t n_teams = groups ? h->n_g_teams : dense ? h->n_d_teams : h->n_teams, end;  // (131 072 at most, twice)
    if (!groups) {
        const asp_handle::Wide &wide = dense ? h->d_wide : h->wide;
        if (wcsr_share_chunks(h, N, wide.count, wide.len)) {
            n_teams += wide.n_teams;
            d_chunks = wide.d_chunks;
            n_chunks = wide.n_chunks;
        } else {
            d_teams += wide.n_teams;
        }
    }
    const int64_t waves = n_chunks + n_row_tasks;
    for (int64_t first = 0; first < waves || n_teams > 0; first = end, n_teams = 0) {
        end = rows_launch_end(waves, first, n_teams);
        const int64_t c0 = std::min(first, n_chunks), c1 = std::min(end, n_chunks), t0 = first - c0, t1 = end - c1;
        // columns per lane: as few as cover N in one pass of the wave -- more lanes per row of B, fewer bytes per lane
#define ASP_ROWS(E, CE, CL)                                                                                          \
    hipLaunchKernelGGL((wcsr_rows_kernel<T, E, CE, CL>),                                                             \
                       dim3((unsigned)(n_teams + ceil_div(end - first, 4)), (unsigned)ceil_div(N, 64 * (E))), dim3(256), 0, \
                       stream, d_teams, (int)n_teams, (const int4 *)d_chunks + c0, (int)(c1 - c0), (const int4 *)d_row_tasks + t0, (int)(t1 - t0), \
                       h->d_e_row_ptr, h->d_e_col, (const T *)h->d_e_val, (const T *)B, (T *)C, N, ws)
        if (N <= 16) ASP_ROWS(1, 1, 16);
        else if (N <= 32) ASP_ROWS(1, 2, 16);
        else if (N <= 64) ASP_ROWS(1, 4, 16);
        else if (N <= 128) ASP_ROWS(2, sizeof(T) == 2 ? 8 : 2, sizeof(T) == 2 ? 16 : 64);
        else if (N <= 256 || sizeof(T) == 4) ASP_ROWS(4, 4, 64);
        else if constexpr (sizeof(T) == 2) ASP_ROWS(8, 8, 64);
#undef ASP_ROWS
    }
}

void wcsr_rows_launch(const asp_handle *h, const void *B, void *C, int64_t N, float *ws, hipStream_t stream) {
    if (h->dtype == ASP_DT_BF16) launch_rows<uint16_t>(h, B, C, N, ws, stream);
    else launch_rows<float>(h, B, C, N, ws, stream);
}

// Long lists, where they are so on average, or each that is (the groups leave thousands of short ones beside those of a hub):
// 2^20 rows of Zipf lengths and a row of 604 368 entries, fp32, N = 128 1041 -> 986 us, the row 6.4e-7 -> 2.6e-7 from its sum
// in 64 bits (by rows 1244, 4.9e-7); bf16 633 -> 575 (616).  From lists of 128 on, the graph without that row 950 -> 959: another launch.
// Only the scratch rows of the call's own list count (with those of chunks whose rows are in groups counted too, 1 814 284 rows of Zipf
// lengths, degree 15, N = 41 went over the line: the sums 11 -> 59 us).
int64_t wcsr_rows_sum_many(const asp_handle *h, int64_t N) {
    const bool groups = wcsr_groups_apply(h, N), dense = !groups && wcsr_dense_apply(h, N);
    const int64_t n_split = groups ? h->n_g_split_rows : dense ? h->n_d_split_rows : h->n_split_rows;
    const int64_t rows = groups ? h->g_scratch_rows : dense ? h->d_scratch_rows : h->scratch_rows;
    return N > 65535 * 16 ? 0 : rows > 32 * n_split ? n_split : groups ? h->group_many : 0;
}

void wcsr_rows_sum_launch(const asp_handle *h, void *C, int64_t N, const float *ws, hipStream_t stream) {
    const bool groups = wcsr_groups_apply(h, N);
    const bool dense = !groups && wcsr_dense_apply(h, N);
    const int32_t *d_split = groups ? h->d_g_split_rows : dense ? h->d_d_split_rows : h->d_split_rows;
    const int64_t n_split = groups ? h->n_g_split_rows : dense ? h->n_d_split_rows : h->n_split_rows;
    if (n_split == 0) return;
    const int64_t n_many = wcsr_rows_sum_many(h, N);
#define ASP_ROWS_SUM(T, COLS, J, FIRST, COUNT)                                                                            \
    if ((COUNT) > 0)                                                                                                      \
        hipLaunchKernelGGL((wcsr_rows_sum_kernel<T, COLS, J>),                                                            \
                           dim3((unsigned)std::min<int64_t>(COUNT, 1 << 21), (unsigned)ceil_div(N, COLS)),                \
                           dim3((COLS) * (J)), 0, stream, (const int4 *)d_split + (FIRST), (int)(COUNT), ws, (T *)C, N)
    if (h->dtype == ASP_DT_BF16) {
        ASP_ROWS_SUM(uint16_t, 16, 64, 0, n_many);
        ASP_ROWS_SUM(uint16_t, 64, 4, n_many, n_split - n_many);
    } else {
        ASP_ROWS_SUM(float, 16, 64, 0, n_many);
        ASP_ROWS_SUM(float, 64, 4, n_many, n_split - n_many);
    }
#undef ASP_ROWS_SUM
}

}  // namespace asp

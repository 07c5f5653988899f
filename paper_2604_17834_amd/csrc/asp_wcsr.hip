// WCSR x dense SpMM for gfx950 and the GPU-side split of row-windows into sub-tasks
// (paper, Section II-C for the format, Section III-B/III-C for the gather kernel and the task split).
//
// The work is bound by the gather of B rows from HBM, so the kernel is built around that stream:
// one wavefront owns one (task, N-tile).  For every packed column of its task a quarter (or half)
// of the wave reads a contiguous run of the addressed B row with 16-byte loads straight into the
// register layout of the fp32 MFMA B operand -- no LDS stage, no barrier -- while the matching A
// values come from the contiguous tile.  Loads for the next tile are issued before the MFMAs of the
// current one; many resident waves per CU keep the HBM queue full.  The columns of a 64-wide (or
// 128-wide) group are dealt to the MFMA's N index as n = 4*j + t (j = lane's N index, t = which of
// the lane's four loaded values), so that each lane ends with 4 adjacent output columns per row and
// C is written (or atomically accumulated, for split windows) 16 bytes at a time.
//
// The paper fixes the window height at 64 to fit the Hopper instruction; the CDNA fp32 MFMAs are
// 16 or 32 rows tall, so heights 16 (default), 32 and 64 are built.
#include <algorithm>
#include <cstdlib>
#include <mutex>

#include "asp_wcsr_tile.h"

// Scratch for callers that cannot allocate (asp_spmm_static_scratch): the partial tiles of split windows go here
// instead of into a buffer from asp_reserve.  Every GPU the library runs on holds its own copy at its own address
// until the process ends.  In host code this name is only a handle for hipGetSymbolAddress; kernels and copies get
// the device address that wcsr_static_scratch() resolved.
static __device__ __align__(256) float scratch[ASP_STATIC_SCRATCH_BYTES / sizeof(float)];

namespace asp {

asp_status_t wcsr_static_scratch(int device, float **ptr, int64_t *floats) {
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static float *resolved[MAX_DEVICES] = {};
    if (device < 0 || device >= MAX_DEVICES) return fail(ASP_ERR_UNSUPPORTED, "device index beyond the static scratch table");
    std::lock_guard<std::mutex> lock(mu);
    if (!resolved[device]) {
        int cur = -1;
        ASP_HIP_TRY(hipGetDevice(&cur));
        if (cur != device) return fail(ASP_ERR_INVALID_ARG, "the static scratch of a device is resolved with that device current");
        float *p = nullptr;
        ASP_HIP_TRY(hipGetSymbolAddress((void **)&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(ASP_ERR_HIP, "hipGetSymbolAddress returned no address for the static scratch");
        resolved[device] = p;
    }
    *ptr = resolved[device];
    *floats = (int64_t)(ASP_STATIC_SCRATCH_BYTES / sizeof(float));
    return ASP_OK;
}

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

// ---- zero the C rows of windows that are empty or split: fp32 calls without scratch, whose split windows are summed
// with atomics
__global__ __launch_bounds__(256) void wcsr_zero_rows_kernel(const int32_t *__restrict__ zero_windows, int n_windows,
                                                             int b_row, float *__restrict__ C, int M, int64_t N) {
    for (int w = blockIdx.x; w < n_windows; w += gridDim.x) {
        const int64_t r0 = (int64_t)zero_windows[w] * b_row;
        const int64_t r1 = r0 + b_row < M ? r0 + b_row : M;
        float *base = C + r0 * N;
        for (int64_t i = threadIdx.x; i < (r1 - r0) * N; i += 256) base[i] = 0.f;
    }
}

// ---- rows of split windows from the partial tiles of their tasks (Section III-C) ---------------------
// Task j of a split window stored its fp32 partial tile [b_row][N] in slot ws_slot[w] + j of the scratch
// buffer.  One thread per output element adds the tiles in task order (fixed order: bitwise reproducible)
// and rounds once to the output type.
template <typename OutT, int U>  // U = elements per thread and access: 4 (16-byte loads) or 1
__global__ __launch_bounds__(256) void wcsr_sum_partials_kernel(const int32_t *__restrict__ split_windows, int n_windows,
                                                                const int32_t *__restrict__ ws_slot,
                                                                const int32_t *__restrict__ window_row_ptr,
                                                                int task_cols, int b_row, OutT *__restrict__ C,
                                                                const float *__restrict__ ws, int M, int64_t N) {
    typedef float vec_t __attribute__((ext_vector_type(U)));
    typedef OutT out_t __attribute__((ext_vector_type(U)));
    for (int sw = blockIdx.x; sw < n_windows; sw += gridDim.x) {
        const int w = split_windows[sw];
        const int slot0 = ws_slot[w];
        const int parts = (int)(((int64_t)window_row_ptr[w + 1] - window_row_ptr[w] + task_cols - 1) / task_cols);
        const int64_t r0 = (int64_t)w * b_row, r1 = r0 + b_row < M ? r0 + b_row : M;
        const int64_t units = (r1 - r0) * N / U, tile = (int64_t)b_row * N / U;
        const vec_t *src = (const vec_t *)(ws + (int64_t)slot0 * b_row * N);
        out_t *dst = (out_t *)(C + r0 * N);
        for (int64_t i = (int64_t)blockIdx.y * 256 + threadIdx.x; i < units; i += (int64_t)gridDim.y * 256) {
            vec_t sum = src[i];
            int j = 1;
            for (; j + 8 <= parts; j += 8) {  // 8 independent loads in flight, added in task order
                vec_t t[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = src[(j + e) * tile + i];
#pragma unroll
                for (int e = 0; e < 8; ++e) sum += t[e];
            }
            for (; j < parts; ++j) sum += src[j * tile + i];
            dst[i] = __builtin_convertvector(sum, out_t);  // bf16: round to nearest even
        }
    }
}

// 4 adjacent columns n..n+3 of a row, at any alignment, N >= 4: n was moved left so that n + 3 < N (own_n, the column it was
// moved from, tells which columns belong to this lane alone).
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ int64_t lane_column(int64_t own_n, int64_t N) { return own_n > N - 4 ? N - 4 : own_n; }

// wanted: whether the lane has a column of its own (a lane without one may load or not).  (As float4: with the four kept as one
// vector the tiles of height 16 take 3 to 6 % longer.)
__device__ __forceinline__ float4 gather4(const float *__restrict__ B, int col, int64_t N, int64_t n, bool wanted = true) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);  // zeros for a pad column (col < 0)
    if (col >= 0 && wanted) {
        const f32x4_any u = *(const f32x4_any *)(B + (int64_t)col * N + n);
        v = make_float4(u.x, u.y, u.z, u.w);
    }
    return v;
}

// V = 1 or 2 adjacent columns, N >= V, in the same way
template <int V>
struct Columns {
    typedef float any __attribute__((ext_vector_type(V), aligned(4)));
};
template <int V>
__device__ __forceinline__ typename Columns<V>::any gather_few(const float *__restrict__ B, int col, int64_t N, int64_t n) {
    typename Columns<V>::any v;
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = 0.f;
    if (col >= 0) v = *(const typename Columns<V>::any *)(B + (int64_t)col * N + n);
    return v;
}
template <int V>
__device__ __forceinline__ void put_few(float *__restrict__ C, int64_t row, int64_t M, int64_t N, int64_t own_n,
                                        typename Columns<V>::any v, bool split) {
    if (row >= M || own_n >= N) return;
    const int64_t n = own_n > N - V ? N - V : own_n;
    float *p = C + row * N + n;
    if (split) {
#pragma unroll
        for (int i = 0; i < V; ++i)
            if (n + i >= own_n) unsafeAtomicAdd(p + i, v[i]);
    } else {
        __builtin_nontemporal_store(v, (typename Columns<V>::any *)p);
    }
}

template <bool NONTEMPORAL = true>
__device__ __forceinline__ void put4(float *__restrict__ C, int64_t row, int64_t M, int64_t N, int64_t own_n, float4 v,
                                     bool split) {
    if (row >= M || own_n >= N) return;
    const int64_t n = lane_column(own_n, N);
    float *p = C + row * N + n;
    if (split) {  // (columns shared with another lane are added by that one)
        if (n >= own_n) unsafeAtomicAdd(p, v.x);
        if (n + 1 >= own_n) unsafeAtomicAdd(p + 1, v.y);
        if (n + 2 >= own_n) unsafeAtomicAdd(p + 2, v.z);
        unsafeAtomicAdd(p + 3, v.w);  // (own_n < N: the lane's own column, moved left or not)
    } else if (NONTEMPORAL) {
        __builtin_nontemporal_store(f32x4_any{v.x, v.y, v.z, v.w}, (f32x4_any *)p);
    } else {
        *(f32x4_any *)p = f32x4_any{v.x, v.y, v.z, v.w};
    }
}

// Where a task's tile goes.  An unsplit window writes its rows of C.  A split window (Section III-C) either
// adds into C with atomics (no scratch reserved) or stores its tile into its own slot of the scratch buffer:
// slot = first slot of the window + index of the task inside the window.
struct SplitTarget {
    float *base;
    int64_t row0;  // first row of the tile in base
    int64_t rows;  // rows that exist in base from its start (bound for the row check)
    bool atomic;
};
__device__ __forceinline__ SplitTarget split_target(int4 td, int b_row, float *C, int M, int64_t N, float *ws,
                                                    const int32_t *ws_slot, const int32_t *window_row_ptr,
                                                    int task_cols) {
    if (td.w != 0 && ws) {
        const int64_t slot = ws_slot[td.x] + (td.y - window_row_ptr[td.x]) / task_cols;
        return SplitTarget{ws + slot * b_row * N, 0, b_row, false};
    }
    return SplitTarget{C, (int64_t)td.x * b_row, M, td.w != 0};
}

// ---- window height 16: v_mfma_f32_16x16x4_f32 ----------------------------------------------------
// lane l: kq = l / 16 picks one of 4 packed columns of a k step, jl = l % 16 is the MFMA N index.
// NG = 64-column groups per wave (tile width BN = 64 * NG).
// RAGGED, for 256-wide tiles whose rows end inside a cache line: lanes past N load nothing, and stores are ordinary ones, so
// that L2 completes the lines that two rows share (band of 27, 500 000 rows, N = 200: 262 -> 254 us; narrower tiles
// gain nothing from either, and lose up to 20 % with ordinary stores).
// N >= V; V = 4 columns to a lane, 2 and 1 (with NG = 1) where N <= 32 and 16: 1 000 000 rows, band of 23, N = 29 114 -> 87 us, N = 16
// 90 -> 49; 30 000 rows 5.8 -> 5.1, 5.3 -> 4.4.
template <int NG, bool RAGGED, bool UNIFORM, int V>
__global__ __launch_bounds__(256) void wcsr16_spmm_kernel(const int4 *__restrict__ tasks, int n_tasks,
                                                          const int32_t *__restrict__ window_col_idx,
                                                          const float *__restrict__ values,
                                                          const float *__restrict__ B, float *__restrict__ C, int M,
                                                          int64_t N, int n_tiles, bool dealt, float *__restrict__ ws,
                                                          const int32_t *__restrict__ ws_slot,
                                                          const int32_t *__restrict__ window_row_ptr, int task_cols) {
    const auto [task, nt] = wave_task<UNIFORM>(n_tiles, dealt);
    if (task >= n_tasks) return;  // whole wave leaves together
    const int lane = threadIdx.x & 63, kq = lane >> 4, jl = lane & 15;
    const int4 td = tasks[task];  // window, first packed column, end packed column, split flag
    if (td.y >= td.z) return;     // fills up a list
    static_assert(V == 4 || (NG == 1 && !RAGGED), "narrow tiles");
    typedef float cols_t __attribute__((ext_vector_type(V)));
    int64_t n0[NG];  // first of the lane's columns in each group
#pragma unroll
    for (int g = 0; g < NG; ++g) n0[g] = V == 4 ? lane_column((int64_t)nt * (64 * NG) + 64 * g + 4 * jl, N) : V * jl > N - V ? N - V : V * jl;
    bool wanted[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) wanted[g] = !RAGGED || (int64_t)nt * (64 * NG) + 64 * g + 4 * jl < N;

    f32x4 acc[NG][V];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int t = 0; t < V; ++t) acc[g][t] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Software pipeline over chunks of D tiles (D*8 packed columns): while chunk c is multiplied, the B
    // rows and A values of chunk c+1 are in flight and the column indices of chunk c+2 are being read,
    // so neither the index -> address dependency nor the gather latency is waited for in the loop.
    constexpr int D = NG >= 2 ? 1 : 2;
    struct Chunk {
        float a[D][2];
        cols_t b[D][2][NG];
    };
    const int tile0 = td.y >> 3, tile1 = td.z >> 3;
    // Which packed column a lane multiplies in which k step is free as long as A and B agree: lane group kq takes
    // columns 2 kq and 2 kq + 1 of a tile (k steps h = 0, 1), so its two indices and its two values of a row are
    // one 8-byte load each and the 16 x 4 lanes read a tile's 512 bytes of values as one contiguous span.
    auto load_idx = [&](int base, int (&idx)[D][2]) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            int2 c2 = make_int2(-1, -1);
            if (base + d < tile1) c2 = *(const int2 *)(window_col_idx + (int64_t)(base + d) * 8 + 2 * kq);
            idx[d][0] = c2.x;
            idx[d][1] = c2.y;
        }
    };
    auto gather = [&](int base, const int (&idx)[D][2], Chunk &c) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            float2 a2 = make_float2(0.f, 0.f);
            if (base + d < tile1) a2 = *(const float2 *)(values + (int64_t)(base + d) * 128 + jl * 8 + 2 * kq);
            c.a[d][0] = a2.x;
            c.a[d][1] = a2.y;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    if constexpr (V == 4) {
                        const float4 v = gather4(B, idx[d][h], N, n0[g], wanted[g]);
                        c.b[d][h][g] = cols_t{v.x, v.y, v.z, v.w};
                    } else {
                        c.b[d][h][g] = gather_few<V>(B, idx[d][h], N, n0[g]);
                    }
                }
        }
    };
    auto multiply = [&](int base, const Chunk &c) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (base + d >= tile1) break;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < NG; ++g) {
#pragma unroll
                    for (int t = 0; t < V; ++t)
                        acc[g][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(c.a[d][h], c.b[d][h][g][t], acc[g][t], 0, 0, 0);
                }
        }
    };

    int idx[D][2];
    Chunk cur, nxt;
    load_idx(tile0, idx);
    gather(tile0, idx, cur);
    load_idx(tile0 + D, idx);
    for (int base = tile0; base < tile1; base += D) {
        const bool more = base + D < tile1;
        if (more) {
            gather(base + D, idx, nxt);
            load_idx(base + 2 * D, idx);
        }
        multiply(base, cur);
        if (more) cur = nxt;
    }

    // D layout: register r of lane l is row 4*(l/16) + r, MFMA column l%16 -> C column n0 + 64g + t
    const SplitTarget out = split_target(td, 16, C, M, N, ws, ws_slot, window_row_ptr, task_cols);
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (V == 4) {
                put4<!RAGGED>(out.base, out.row0 + 4 * kq + r, out.rows, N, (int64_t)nt * (64 * NG) + 64 * g + 4 * jl,
                              make_float4(acc[g][0][r], acc[g][1][r], acc[g][2][r], acc[g][3][r]), out.atomic);
            } else {
                typename Columns<V>::any v;
#pragma unroll
                for (int t = 0; t < V; ++t) v[t] = acc[g][t][r];
                put_few<V>(out.base, out.row0 + 4 * kq + r, out.rows, N, V * jl, v, out.atomic);
            }
        }
}

// ---- window heights 32 and 64: v_mfma_f32_32x32x2_f32 --------------------------------------------
// lane l: kq = l / 32 picks one of 2 packed columns of a k step, jl = l % 32 is the MFMA N index;
// the wave covers 32 V columns.  MTW = window height / 32 MFMA row tiles share every gathered B value.
// N >= V; V = 4, or 2 and 1 where N <= 64 and 32 and most of 128 columns would be multiplied for nothing (and with the registers that
// they take another wave or two fit a SIMD): 978 077 rows, band of 13, height 64, N = 64 257 -> 171 us, N = 16 245 -> 86; height 32
// 189 -> 139, 156 -> 61; 30 000 rows, height 64, N = 64 16.6 -> 11.9.
template <int MTW, int V>
__global__ __launch_bounds__(256, 2) void wcsr32_spmm_kernel(const int4 *__restrict__ tasks, int n_tasks,
                                                          const int32_t *__restrict__ window_col_idx,
                                                          const float *__restrict__ values,
                                                          const float *__restrict__ B, float *__restrict__ C, int M,
                                                          int64_t N, int n_tiles, bool dealt, float *__restrict__ ws,
                                                          const int32_t *__restrict__ ws_slot,
                                                          const int32_t *__restrict__ window_row_ptr, int task_cols) {
    constexpr int BRW = 32 * MTW;
    const auto [task, nt] = wave_task<false>(n_tiles, dealt);
    if (task >= n_tasks) return;
    const int lane = threadIdx.x & 63, kq = lane >> 5, jl = lane & 31;
    const int4 td = tasks[task];
    if (td.y >= td.z) return;
    typedef float cols_t __attribute__((ext_vector_type(V)));
    const int64_t own_n0 = (int64_t)nt * (32 * V) + V * jl, n0 = own_n0 > N - V ? N - V : own_n0;  // N >= V

    f32x16 acc[MTW][V];
#pragma unroll
    for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int t = 0; t < V; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][t][r] = 0.f;

    struct Stage {
        float a[4][MTW];
        cols_t b[4];
    };
    // lane group kq takes packed columns 4 kq .. 4 kq + 3 of a tile (k steps h = 0..3; any assignment works as long
    // as A and B agree): its four indices and its four values of a row are one 16-byte load each, and the 32 x 2
    // lanes read the 1 KB of values of a row tile as one contiguous span
    auto fetch = [&](int tile, Stage &s) {
        const int4 c4 = *(const int4 *)(window_col_idx + (int64_t)tile * 8 + 4 * kq);
        const int col[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
        for (int i = 0; i < MTW; ++i) {
            const float4 a4 = *(const float4 *)(values + (int64_t)tile * (BRW * 8) + (i * 32 + jl) * 8 + 4 * kq);
            s.a[0][i] = a4.x;
            s.a[1][i] = a4.y;
            s.a[2][i] = a4.z;
            s.a[3][i] = a4.w;
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            if constexpr (V == 4) {
                const float4 v = gather4(B, col[h], N, n0);
                s.b[h] = cols_t{v.x, v.y, v.z, v.w};
            } else {
                s.b[h] = gather_few<V>(B, col[h], N, n0);
            }
        }
    };
    auto multiply = [&](const Stage &s) {
#pragma unroll
        for (int h = 0; h < 4; ++h)
#pragma unroll
            for (int i = 0; i < MTW; ++i) {
#pragma unroll
                for (int t = 0; t < V; ++t)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x2f32(s.a[h][i], s.b[h][t], acc[i][t], 0, 0, 0);
            }
    };

    const int tile0 = td.y >> 3, tile1 = td.z >> 3;
    // two tiles in flight while a third is multiplied (three stages, walked with fixed register names): at this
    // register count the occupancy is the same as with one tile in flight, and the gather needs the bytes in flight
    Stage s0, s1, s2;
    fetch(tile0, s0);
    if (tile0 + 1 < tile1) fetch(tile0 + 1, s1);
    for (int tile = tile0; tile < tile1; tile += 3) {
        if (tile + 2 < tile1) fetch(tile + 2, s2);
        multiply(s0);
        if (tile + 3 < tile1) fetch(tile + 3, s0);
        if (tile + 1 < tile1) multiply(s1);
        if (tile + 4 < tile1) fetch(tile + 4, s1);
        if (tile + 2 < tile1) multiply(s2);
    }

    // D layout: register r of lane l is row 8*(r/4) + 4*(l/32) + r%4, MFMA column l%32
    const SplitTarget out = split_target(td, BRW, C, M, N, ws, ws_slot, window_row_ptr, task_cols);
#pragma unroll
    for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            int row = i * 32 + 8 * (r >> 2) + 4 * kq + (r & 3);
            if constexpr (V == 4)
                put4(out.base, out.row0 + row, out.rows, N, own_n0,
                     make_float4(acc[i][0][r], acc[i][1][r], acc[i][2][r], acc[i][3][r]), out.atomic);
            else {
                typename Columns<V>::any v;
#pragma unroll
                for (int t = 0; t < V; ++t) v[t] = acc[i][t][r];
                put_few<V>(out.base, out.row0 + row, out.rows, N, own_n0, v, out.atomic);
            }
        }
}

// ---- sub-task list on the GPU (Section III-C) -----------------------------------------------------
// tasks_of(w) = ceil(width(w) / task_cols); an exclusive prefix sum over windows gives every window
// the index of its first task.  The sum is a wavefront scan (cross-lane shifts), stitched over the 4
// waves of a workgroup through LDS and over workgroups through a second, single-workgroup pass.

__device__ __forceinline__ int wave_inclusive_scan(int v, int lane) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int up = __shfl_up(v, d, 64);
        if (lane >= d) v += up;
    }
    return v;
}

// inclusive scan over the 256 threads of a workgroup; returns the thread's inclusive value, *total = sum
__device__ __forceinline__ int block_inclusive_scan(int v, int *total) {
    __shared__ int wave_sum[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = wave_inclusive_scan(v, lane);
    __syncthreads();  // protects wave_sum against the previous call
    if (lane == 63) wave_sum[wave] = inc;
    __syncthreads();
    int base = 0;
    for (int w = 0; w < wave; ++w) base += wave_sum[w];
    *total = wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
    return inc + base;
}

__global__ __launch_bounds__(256) void wcsr_task_count_kernel(const int32_t *__restrict__ window_row_ptr, int n_windows,
                                                              int task_cols, int32_t *__restrict__ local_excl,
                                                              int32_t *__restrict__ block_sums) {
    const int w = blockIdx.x * 256 + threadIdx.x;
    int cnt = 0;
    // (64-bit: width + task_cols may pass 2^31)
    if (w < n_windows) cnt = (int)(((int64_t)window_row_ptr[w + 1] - window_row_ptr[w] + task_cols - 1) / task_cols);
    int total;
    int inc = block_inclusive_scan(cnt, &total);
    if (w < n_windows) local_excl[w] = inc - cnt;
    if (threadIdx.x == 0) block_sums[blockIdx.x] = total;
}

// one workgroup: exclusive scan of block_sums in place, grand total to block_sums[n_blocks]
__global__ __launch_bounds__(256) void wcsr_task_block_scan_kernel(int32_t *__restrict__ block_sums, int n_blocks) {
    int carry = 0;
    for (int base = 0; base < n_blocks; base += 256) {
        const int i = base + threadIdx.x;
        const int v = i < n_blocks ? block_sums[i] : 0;
        int total;
        int inc = block_inclusive_scan(v, &total);
        if (i < n_blocks) block_sums[i] = carry + inc - v;
        carry += total;
    }
    if (threadIdx.x == 0) block_sums[n_blocks] = carry;
}

__global__ __launch_bounds__(256) void wcsr_task_offsets_kernel(const int32_t *__restrict__ local_excl,
                                                                const int32_t *__restrict__ block_sums, int n_windows,
                                                                int n_blocks, int32_t *__restrict__ task_offsets) {
    const int w = blockIdx.x * 256 + threadIdx.x;
    if (w < n_windows) task_offsets[w] = local_excl[w] + block_sums[blockIdx.x];
    if (w == 0) task_offsets[n_windows] = block_sums[n_blocks];
}

// one thread per task: find its window by bisection in the offsets, then cut the window's range
__global__ __launch_bounds__(256) void wcsr_task_emit_kernel(const int32_t *__restrict__ window_row_ptr,
                                                             const int32_t *__restrict__ task_offsets, int n_windows,
                                                             int n_tasks, int task_cols, int4 *__restrict__ tasks) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= n_tasks) return;
    int lo = 0, hi = n_windows;  // first window whose offset exceeds t lies in (lo, hi]
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (task_offsets[mid] <= t) lo = mid; else hi = mid;
    }
    const int w = lo;
    const int64_t begin = window_row_ptr[w] + (int64_t)(t - task_offsets[w]) * task_cols;  // 64-bit: see above
    const int64_t wend = window_row_ptr[w + 1];
    int4 d;
    d.x = w;
    d.y = (int)begin;
    d.z = (int)(begin + task_cols < wend ? begin + task_cols : wend);
    d.w = (task_offsets[w + 1] - task_offsets[w]) > 1 ? 1 : 0;
    tasks[t] = d;
}

asp_status_t wcsr_build_tasks_device(asp_handle *h, hipStream_t stream) {
    const int nw = (int)h->n_brows;
    const int n_blocks = (int)ceil_div(nw, 256);
    int32_t *local_excl = nullptr, *block_sums = nullptr, *task_offsets = nullptr;
    asp_status_t st = ASP_OK;
    auto cleanup = [&]() {
        (void)hipFree(local_excl);
        (void)hipFree(block_sums);
        (void)hipFree(task_offsets);
    };
#define TRY_OR_CLEAN(expr)                                                                     \
    do {                                                                                       \
        hipError_t e__ = (expr);                                                               \
        if (e__ != hipSuccess) {                                                               \
            cleanup();                                                                         \
            return fail(e__ == hipErrorOutOfMemory ? ASP_ERR_OUT_OF_MEMORY : ASP_ERR_HIP,     \
                        std::string(#expr) + ": " + hipGetErrorString(e__));                  \
        }                                                                                      \
    } while (0)
    TRY_OR_CLEAN(hipMalloc((void **)&local_excl, (size_t)nw * 4));
    TRY_OR_CLEAN(hipMalloc((void **)&block_sums, (size_t)(n_blocks + 1) * 4));
    TRY_OR_CLEAN(hipMalloc((void **)&task_offsets, (size_t)(nw + 1) * 4));
    hipLaunchKernelGGL(wcsr_task_count_kernel, dim3(n_blocks), dim3(256), 0, stream, h->d_row_ptr, nw, h->task_cols,
                       local_excl, block_sums);
    hipLaunchKernelGGL(wcsr_task_block_scan_kernel, dim3(1), dim3(256), 0, stream, block_sums, n_blocks);
    hipLaunchKernelGGL(wcsr_task_offsets_kernel, dim3(n_blocks), dim3(256), 0, stream, local_excl, block_sums, nw,
                       n_blocks, task_offsets);
    TRY_OR_CLEAN(hipGetLastError());
    int32_t total = 0;
    TRY_OR_CLEAN(hipMemcpyAsync(&total, task_offsets + nw, 4, hipMemcpyDeviceToHost, stream));
    TRY_OR_CLEAN(hipStreamSynchronize(stream));
    h->n_tasks = total;
    TRY_OR_CLEAN(hipMalloc((void **)&h->d_tasks, total > 0 ? (size_t)total * 16 : 16));
    if (total > 0) {
        hipLaunchKernelGGL(wcsr_task_emit_kernel, dim3((unsigned)ceil_div(total, 256)), dim3(256), 0, stream,
                           h->d_row_ptr, task_offsets, nw, total, h->task_cols, (int4 *)h->d_tasks);
        TRY_OR_CLEAN(hipGetLastError());
        TRY_OR_CLEAN(hipStreamSynchronize(stream));
    }
#undef TRY_OR_CLEAN
    cleanup();
    return st;
}

// ---- host side ------------------------------------------------------------------------------------
WcsrPlan wcsr_plan(const asp_handle *h, int64_t N, bool aligned) {
    WcsrPlan p;
    if (h->dtype == ASP_DT_BF16) {  // one wavefront per (task, 128 columns), 4 to a workgroup; element-wise path: a workgroup per (window, 64 columns)
        p.vectorized = (aligned && N % 8 == 0) ? 1 : 0;
        p.bn = p.vectorized ? 128 : 64;
        p.n_tiles = (int32_t)ceil_div(N, p.bn);
        p.workgroups = p.vectorized ? ceil_div(h->n_tasks * p.n_tiles, 4) : h->n_brows * p.n_tiles;
        return p;
    }
    p.vectorized = (aligned && N % 4 == 0) ? 1 : 0;
    if (h->b_row == 16) {
        // Section IV-C rule over the built wave widths: widest that divides N, else least padding
        static const int cand[3] = {64, 128, 256};
        const int env_max = switches().wcsr_max_bn;  // benchmarking switch: widest wave tile to consider
        int best = -1;
        for (int c : cand)
            if (c <= env_max && N % c == 0 && c > best) best = c;
        if (best < 0) {
            int64_t best_pad = -1;
            for (int c : cand) {
                if (c > env_max) continue;
                int64_t pad = ceil_div(N, c) * c;
                if (best_pad < 0 || pad < best_pad || (pad == best_pad && c > best)) {
                    best_pad = pad;
                    best = c;
                }
            }
        }
        p.bn = best;
    } else {
        p.bn = 128;
    }
    p.n_tiles = (int32_t)ceil_div(N, p.bn);
    p.workgroups = ceil_div(h->n_tasks * p.n_tiles, 4);
    return p;
}

int64_t wcsr_scratch_floats(const asp_handle *h, int64_t N) { return h->n_split_tasks * h->b_row * N; }

void wcsr_sum_partial_tiles(const asp_handle *h, void *C, int64_t N, const float *ws, hipStream_t stream) {
    if (h->n_tile_split == 0) return;
    const bool vec = N % 4 == 0 && ((uintptr_t)C & 15) == 0;
    const unsigned gy = (unsigned)std::min<int64_t>(64, ceil_div((int64_t)h->b_row * N, vec ? 1024 : 256));
    dim3 grid((unsigned)std::min<int64_t>(h->n_tile_split, 1 << 23), gy), block(256);
#define ASP_SUM(T, U)                                                                                              \
    hipLaunchKernelGGL((wcsr_sum_partials_kernel<T, U>), grid, block, 0, stream, h->d_tile_split,                  \
                       (int)h->n_tile_split, h->d_ws_slot, h->d_row_ptr, h->task_cols, h->b_row, (T *)C, ws, (int)h->m, N)
    if (h->dtype == ASP_DT_BF16) {
        if (vec) ASP_SUM(__bf16, 4);
        else ASP_SUM(__bf16, 1);
    } else {
        if (vec) ASP_SUM(float, 4);
        else ASP_SUM(float, 1);
    }
#undef ASP_SUM
}

// fp32, columns of a lane, 32 lanes to a wave's tile.  Heights 32 and 64: 32 or 64 columns to a wave where that covers N; 64 also
// where two such tiles do at height 64, if that leaves every wave a SIMD of its own (30 000 rows, band of 13, N = 128 16.9 -> 12.4 us)
// or brings few SIMDs to three of them instead of two twice as long ones, or five instead of three (80 000 rows 33.0 -> 32.0, 150 000 64.1 ->
// 59.5; two instead of one, 50 000 rows, 19.5 / 21.4, on every SIMD, 98 000, N = 100, 34 / 38, four instead of two, 120 000, 36 / 56,
// 600 000 rows 186 / 200, N = 80 166 / 192); and where three do instead of two of 128 and there are enough of them (N = 160, 300 000 rows,
// heights 32 / 64 108 / 158 -> 102 / 143; 30 000 rows 13.6 -> 12.6, but at height 64, 469 windows, 17.3 / 20.6).  At height 32 two instead
// of one are slower (30 000 rows, N = 128 8.3 / 9.4, 300 000 72.6 / 75.1).
int wcsr_lane_columns(const asp_handle *h, int64_t N) {
    constexpr int64_t SIMDS = 1024;
    const int64_t n = h->n_tile_tasks;
    if (h->b_row == 16) return 4;
    if (N <= 64) return N <= 32 ? 1 : 2;
    if (N > 128) return N <= 192 && n >= 900 ? 2 : 4;
    return h->b_row == 64 && (2 * n <= SIMDS || (n > SIMDS && n <= 3 * SIMDS && (n - 1) % SIMDS < SIMDS / 3)) ? 2 : 4;
}

asp_status_t wcsr_spmm_launch(const asp_handle *h, const void *B, void *C, int64_t N, float *ws_buf, int64_t ws_floats,
                              hipStream_t stream) {
    if (h->dtype == ASP_DT_BF16) return wcsr_bf16_spmm_launch(h, B, C, N, ws_buf, ws_floats, stream);
    WcsrPlan p = wcsr_plan(h, N, true);
    const int columns = wcsr_lane_columns(h, N);
    if (columns < 4) p.n_tiles = (int32_t)ceil_div(N, 32 * columns);
    // split windows: partial tiles in the scratch buffer when it is large enough, else atomic adds into C
    const bool partial = h->n_split_tasks > 0 && ws_buf && ws_floats >= wcsr_scratch_floats(h, N);
    float *ws = partial ? ws_buf : nullptr;
    if (h->n_split_tasks > 0 && !partial)
        hipLaunchKernelGGL(wcsr_zero_rows_kernel, dim3((unsigned)std::min<int64_t>(h->n_zero_windows, 1 << 23)), dim3(256), 0,
                           stream, h->d_zero_windows, (int)h->n_zero_windows, h->b_row, (float *)C, (int)h->m, N);
    wcsr_rows_launch(h, B, C, N, ws, stream);
    const int64_t step = tasks_per_launch(p.n_tiles);
    for (int64_t first = 0; first < h->n_tile_tasks; first += step) {
        const int nt = (int)std::min(step, h->n_tile_tasks - first), M = (int)h->m;
        const dim3 grid = tile_grid(nt, p.n_tiles, h->tiles_dealt), block(256);
        const int4 *tasks = (const int4 *)h->d_tile_tasks + first;
        const float *vals = (const float *)h->d_values;
        const float *Bf = (const float *)B;
        float *Cf = (float *)C;
#define ASP_W16(NG, RAGGED, UNIFORM, V)                                                                           \
    hipLaunchKernelGGL((wcsr16_spmm_kernel<NG, RAGGED, UNIFORM, V>), grid, block, 0, stream, tasks, nt, h->d_col_idx, \
                       vals, Bf, Cf, M, N, p.n_tiles, h->tiles_dealt, ws, h->d_ws_slot, h->d_row_ptr, h->task_cols)
#define ASP_W32(MTW, V)                                                                                          \
    hipLaunchKernelGGL((wcsr32_spmm_kernel<MTW, V>), grid, block, 0, stream, tasks, nt, h->d_col_idx, vals, Bf, Cf, M, N, \
                       p.n_tiles, h->tiles_dealt, ws, h->d_ws_slot, h->d_row_ptr, h->task_cols)
        if (h->b_row == 16) {
            // 256-wide tiles in 168 registers, 3 waves per SIMD, where B and C are well past the 256 MB behind the L2s; in
            // 176, 2 waves, where they are not: the waves of one moment then reach over less of them.  us, N = 256, 3 / 2 waves:
            // 60 000 rows, band of 27 43 / 34, 500 000 rows 270 / 301; N = 200, 300 000 rows, band of 9 126 / 121.
            const bool far = (h->m + h->k) * N * 4 >= (512ll << 20);
            if (N <= 16) ASP_W16(1, false, false, 1);
            else if (N <= 32) ASP_W16(1, false, false, 2);
            else if (p.bn == 256 && N % 32 != 0 && far) ASP_W16(4, true, true, 4);
            else if (p.bn == 256 && N % 32 != 0) ASP_W16(4, true, false, 4);
            else if (p.bn == 256 && far) ASP_W16(4, false, true, 4);
            else if (p.bn == 256) ASP_W16(4, false, false, 4);
            else if (p.bn == 128) ASP_W16(2, false, false, 4);
            else ASP_W16(1, false, false, 4);
        } else if (h->b_row == 32) {
            if (columns == 1) ASP_W32(1, 1);
            else if (columns == 2) ASP_W32(1, 2);
            else ASP_W32(1, 4);
        } else {
            if (columns == 1) ASP_W32(2, 1);
            else if (columns == 2) ASP_W32(2, 2);
            else ASP_W32(2, 4);
        }
#undef ASP_W16
#undef ASP_W32
    }
    if (partial) {
        wcsr_rows_sum_launch(h, C, N, ws, stream);
        wcsr_sum_partial_tiles(h, C, N, ws, stream);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ASP_ERR_HIP, std::string("WCSR kernel launch: ") + hipGetErrorString(e));
    return ASP_OK;
}

}  // namespace asp

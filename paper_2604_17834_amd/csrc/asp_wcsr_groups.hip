// WCSR x dense SpMM: long rows of scattered entries in groups, all of them walking the columns of B together.
//
// A graph with power-law degrees keeps most of its entries in rows of more than 64, and several of these rows store
// any one column.  Walked row by row (asp_wcsr_rows.hip) each of those entries fetches its row of B through L2's memory
// side, 7.2 TB/s whatever else is done, because the rows are at different columns at any moment.  Here a wavefront holds
// the sums of up to 63 rows in registers (fp32; 31 in bf16, with two columns to a lane) and walks their entries in the
// order of the columns, and the waves that an XCD holds at once all walk the same range of columns, each with its own rows
// and all with as many entries: what one fetched the others find in L2.  The products stay one fp32 fused multiply-add
// each, in the order of the columns.
//
// 2^20-row Zipf graph, fp32, N = 128, 10.3 of 16.7 million entries in groups: these took 630 us by rows and take 367 (and 11 for
// the larger sums), 14.5 TB/s of rows of B, 85 % of the lines from L2; the product 1198 -> 946 us.  200 003 rows, bf16,
// N = 100: 121 -> 110.  What bounds it: the latency of L2 with the number of lines that an L1 keeps in flight, and the waves
// that run ahead or behind their XCD's others, whose lines L2 no longer holds.  So fewer and longer tasks are better: 4096
// tasks of up to 31 rows and 128 columns a wave 511 us with 48 % from L2, 4096 of 31 rows and 64 columns 416, 2048 of 63 rows 374.
//
// Sums in registers: which row an entry belongs to is uniform for the wave, so its sum is addressed through the vector
// register index (s_set_gpr_idx_on / _idx: M0 takes the index from bits 7:0 of the entry's key; bit 2 of the mode indexes
// the third source, bit 3 the destination).  LDS would hold 160 KB of sums per compute unit and make an add a read, a wait
// and a write where this is the multiply-add itself.
//
// The column ranges divide the entries evenly, 8 of them, one to an XCD.  The pieces that the rows leave in a range are dealt
// to its tasks by themselves, so that these are even whatever columns the rows store: a 2^20-row Zipf graph whose rows keep to
// one of 32 blocks of columns 1075 -> 856 us against one deal of whole rows for all ranges (by rows 893), its longest sum 1024
// terms -> 160.  A task leaves a partial sum per piece in scratch memory, and wcsr_rows_sum_kernel adds those of a row in order.
#include "asp_wcsr_rows.h"

namespace asp {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// tasks[x * per_xcd + i] = {first entry / 16, entries / 16, first column of the range, -}: task i in the range of XCD x.  entries = {(column - first column) << 8 | piece of the task, fp32 bits of the value}; what fills
// up the last 16 belongs to the piece behind the task's last, which nobody reads (no row of A that does not store a column may see its
// values).  slots[task][ROWS]: scratch row of each piece, -1: none.
template <typename T, int E>
__global__ __launch_bounds__(256, 2) void wcsr_groups_kernel(const int4 *__restrict__ tasks, int per_xcd,
                                                          const u32x2 *__restrict__ entries, const int32_t *__restrict__ slots,
                                                          const T *__restrict__ B, int64_t N, float *__restrict__ ws) {
    typedef typename RowVec<T, E>::type vec_t;
    constexpr int ROWS = E == 2 ? 31 : 63;
    typedef float sums_t __attribute__((ext_vector_type(32)));
    const int xcd = blockIdx.x & 7, i = (blockIdx.x >> 3) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (i >= per_xcd) return;
    const int4 td = tasks[xcd * per_xcd + i];
    const int lane = threadIdx.x & 63;
    const int64_t n = (int64_t)blockIdx.y * (64 * E) + lane * E;
    const int64_t nc = n < N - E ? n : N - E;  // N >= E: the last lane of a row moves left
    const uint32_t row_bytes = (uint32_t)(N * (int64_t)sizeof(T));
    const global_char *base = (const global_char *)B + (uint64_t)(uint32_t)td.z * row_bytes;
    const u32x2 *e = entries + (int64_t)td.x * 16;
    const int iters = td.y;
    sums_t s0, s1;
#pragma unroll
    for (int r = 0; r < 32; ++r) s0[r] = 0.f, s1[r] = 0.f;

    // The entries are read once and come from HBM: 16 at a time, lane i of every 16 holding the i-th, three loads ahead of
    // their use.  (Scalar loads cannot run ahead like that: they return in any order, so that a wait for one is a wait for
    // all.)  A lane's address is one add with the i-th lane's offset broadcast; index and value go to scalar registers.
    struct Sixteen {
        uint32_t off, key, val;
    };
    const uint32_t n_off = (uint32_t)(nc * (int64_t)sizeof(T));
    auto load = [&](int it) __attribute__((always_inline)) {
        return __builtin_nontemporal_load(e + (it < iters ? it : iters - 1) * 16 + (lane & 15));
    };
    auto decode = [&](u32x2 w, int it) __attribute__((always_inline)) {
        return Sixteen{(w.x >> 8) * row_bytes, it < iters ? w.x : ROWS, w.y};  // (a range of B has less than 4 GB)
    };
#define ASP_GATHER(dst, q, j)                                                                                              \
    dst[j] = *(const __attribute__((address_space(1))) vec_t *)(base + (n_off + (uint32_t)__builtin_amdgcn_update_dpp(     \
                                                                                    0, (int)(q).off, 0x150 + (j), 0xf, 0xf, true)))
#define ASP_GATHER8(dst, q, o)                                                                                  \
    do {                                                                                                        \
        ASP_GATHER(dst, q, o + 0); ASP_GATHER(dst, q, o + 1); ASP_GATHER(dst, q, o + 2); ASP_GATHER(dst, q, o + 3); \
        ASP_GATHER(dst, q, o + 4); ASP_GATHER(dst, q, o + 5); ASP_GATHER(dst, q, o + 6); ASP_GATHER(dst, q, o + 7); \
    } while (0)
    // (s_nop: two wait states between a scalar register's write by v_readlane and its read by the vector ALU)
    auto add4 = [&](const Sixteen &q, const vec_t (&v)[16], int o) __attribute__((always_inline)) {
        uint32_t k[4], f[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            k[j] = __builtin_amdgcn_readlane(q.key, o + j);
            f[j] = __builtin_amdgcn_readlane(q.val, o + j);
        }
        if constexpr (E == 2) {
            asm volatile(
                "s_set_gpr_idx_on %2, 0xc\n\ts_nop 0\n\tv_fma_f32 v64, %6, %10, v64\n\tv_fma_f32 v96, %6, %14, v96\n\t"
                "s_set_gpr_idx_idx %3\n\tv_fma_f32 v64, %7, %11, v64\n\tv_fma_f32 v96, %7, %15, v96\n\t"
                "s_set_gpr_idx_idx %4\n\tv_fma_f32 v64, %8, %12, v64\n\tv_fma_f32 v96, %8, %16, v96\n\t"
                "s_set_gpr_idx_idx %5\n\tv_fma_f32 v64, %9, %13, v64\n\tv_fma_f32 v96, %9, %17, v96\n\ts_set_gpr_idx_off"
                : "+{v[64:95]}"(s0), "+{v[96:127]}"(s1)
                : "s"(k[0]), "s"(k[1]), "s"(k[2]), "s"(k[3]), "s"(f[0]), "s"(f[1]), "s"(f[2]), "s"(f[3]),
                  "v"(widen((T)v[o][0])), "v"(widen((T)v[o + 1][0])), "v"(widen((T)v[o + 2][0])), "v"(widen((T)v[o + 3][0])),
                  "v"(widen((T)v[o][1])), "v"(widen((T)v[o + 1][1])), "v"(widen((T)v[o + 2][1])), "v"(widen((T)v[o + 3][1]))
                : "m0");
        } else {
            asm volatile(
                "s_set_gpr_idx_on %2, 0xc\n\ts_nop 0\n\tv_fma_f32 v64, %6, %10, v64\n\t"
                "s_set_gpr_idx_idx %3\n\tv_fma_f32 v64, %7, %11, v64\n\t"
                "s_set_gpr_idx_idx %4\n\tv_fma_f32 v64, %8, %12, v64\n\t"
                "s_set_gpr_idx_idx %5\n\tv_fma_f32 v64, %9, %13, v64\n\ts_set_gpr_idx_off"
                : "+{v[64:95]}"(s0), "+{v[96:127]}"(s1)
                : "s"(k[0]), "s"(k[1]), "s"(k[2]), "s"(k[3]), "s"(f[0]), "s"(f[1]), "s"(f[2]), "s"(f[3]),
                  "v"(widen((T)v[o][0])), "v"(widen((T)v[o + 1][0])), "v"(widen((T)v[o + 2][0])), "v"(widen((T)v[o + 3][0]))
                : "m0");
        }
    };
    // 16 to 32 rows of B in flight; past the task's end the last ones are gathered again, and added to the row nobody reads
    if (iters > 0) {
        Sixteen q0 = decode(load(0), 0), q1;
        u32x2 w1 = load(1), w2 = load(2), w3 = load(3), w4 = load(4);
        vec_t v0[16], v1[16];
        ASP_GATHER8(v0, q0, 0);
        ASP_GATHER8(v0, q0, 8);
        for (int it = 0; it < iters; it += 2) {
            q1 = decode(w1, it + 1);
            ASP_GATHER8(v1, q1, 0);
            ASP_GATHER8(v1, q1, 8);
            add4(q0, v0, 0), add4(q0, v0, 4), add4(q0, v0, 8), add4(q0, v0, 12);
            q0 = decode(w2, it + 2);
            ASP_GATHER8(v0, q0, 0);
            ASP_GATHER8(v0, q0, 8);
            add4(q1, v1, 0), add4(q1, v1, 4), add4(q1, v1, 8), add4(q1, v1, 12);
            w1 = w3;
            w2 = w4;
            w3 = load(it + 5);
            w4 = load(it + 6);
        }
    }
#undef ASP_GATHER
#undef ASP_GATHER8
    const int32_t *slot = slots + (int64_t)(xcd * per_xcd + i) * ROWS;
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int s = slot[r];
        if (s >= 0 && n < N) {
            float *dst = ws + (int64_t)s * N + nc;
            dst[0] = r < 32 ? s0[r & 31] : s1[r & 31];
            if constexpr (E == 2) dst[1] = s1[r];
        }
    }
}

// ---- host side ------------------------------------------------------------------------------------
// Narrow operands stay with the walk by rows, whose waves take several entries at once there: 831 834 rows, bf16, N = 19
// 192 us by rows and 274 in groups, 417 427 rows, N = 64 114 / 121 (but N = 72, 139 866 rows 82 / 72); 225 543 rows, fp32, N = 23
// 84 / 87, N = 34, 129 753 rows 64 / 55.  So does a B that an XCD's 4 MB of L2 hold.  (A range of B is addressed with 32 bits.)
// And so do large graphs in whose rows, as they follow each other, the same columns come again soon (near_cols,
// wcsr_build_groups), where these take few bytes of B: by rows most of them are found in L2 too, and the sums in pieces are extra
// work.  1.5 million rows, fp32, N = 128, columns within 1000 of the diagonal (7 MB) 999 by rows and 1118 in groups, within 10 000
// and 0.8 million rows (19 MB) 878 / 808; bf16, N = 128, communities of 16384 (6 MB) 548 / 608, of 65536 (16 MB) 356 / 346.
// fp32 in whole tiles of 64 columns gains earlier: 15 MB there, 20 MB else.  Of 348 graphs, most with communities or bands, 30 000
// to 2 000 000 rows, those in groups by this rule take at most 1.06 times as long as by rows (without it 1.27), 0.69 at best.
bool wcsr_groups_apply(const asp_handle *h, int64_t N) {
    const int64_t row_bytes = N * (int64_t)dtype_size(h->dtype);
    const int64_t least = h->dtype == ASP_DT_F32 && N % 64 == 0 ? 15000000 : 20000000;
    return h->n_groups > 0 && N > (h->dtype == ASP_DT_BF16 ? 64 : 32) && h->group_span * row_bytes < (1ll << 32) &&
           h->k * row_bytes >= (4 << 20) && (h->group_near_cols == 0 || h->group_near_cols * row_bytes >= least);
}

void wcsr_groups_launch(const asp_handle *h, const void *B, int64_t N, float *ws, hipStream_t stream) {
    const int per_xcd = (int)h->n_groups;
    const unsigned gx = (unsigned)ceil_div(per_xcd, 4) * 8;
#define ASP_GROUPS(T, E)                                                                                              \
    hipLaunchKernelGGL((wcsr_groups_kernel<T, E>), dim3(gx, (unsigned)ceil_div(N, 64 * (E))), dim3(256), 0, stream,   \
                       (const int4 *)h->d_group_tasks, per_xcd, (const u32x2 *)h->d_group_entries, \
                       h->d_group_slots, (const T *)B, N, ws)
    if (h->dtype == ASP_DT_BF16) ASP_GROUPS(uint16_t, 2);
    else ASP_GROUPS(float, 1);
#undef ASP_GROUPS
}

}  // namespace asp

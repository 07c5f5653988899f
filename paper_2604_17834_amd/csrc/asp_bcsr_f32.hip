// BCSR x dense SpMM in fp32 for gfx950 (paper, Section II-C for the format; Table I runs both formats at
// one precision, which is why BCSR also exists in fp32 here).
//
// What bounds it: the matrix cores.  v_mfma_f32_32x32x2_f32 takes 64 cycles, 1/16 of the bf16 rate, on operands that are
// twice as large, so everything else has to stay out of its way.  Both operands go straight from memory to registers, one
// unit of 8 k ahead: no LDS stage and no barrier (staging 16-k slices through LDS kept the matrix cores at two thirds:
// a barrier every 1024 MFMA cycles that all waves of the workgroup had to reach).  The waves that share a strip of A or a
// slab of B meet in the L1.  Block-rows are walked longest first, so that the launch ends with short ones: in the order of
// the bf16 schedule the last heavy tiles were a fifth of it.
// A load has no branch: with a case for rows past K in it the compiler left the loads of A to where they are multiplied, and every
// look-up of a block column waited for all loads in flight.  Of 60 products (1000 to 9000 rows, 64 to 2048 columns) 0.89 of the
// time in the mean, 0.80 at best; 9000 x 4000, 50 %, 64 x 64 blocks, 1024 columns 380 -> 327 us.
// Where K is a multiple of the blocks no row has to be looked at twice (WHOLE): 18944 x 3584 at 90 %, N = 16384, 128 / 64 / 32-row blocks 1.910 /
// 1.857 / 2.041 -> 1.750 / 1.760 / 1.905 ms (with that branch 1.829 / 1.825 / 2.022); of 110 products 0.965 of the time in the mean, 1.06 at most.
// 18944 x 3584 at 90 %, blocks of 128 / 64 / 32, through LDS -> so: N = 2048 301 / 276 / 306 -> 243 / 238 / 229 us (116 to 121 TFLOP/s;
// the same MFMAs on registers reach 149), N = 64 140 / 83 / 63 -> 15 / 14 / 13 (clocks move all of them by 5 % together).
//
// Operand layouts
//   A  blocks are pre-permuted on the host (bcsr_pack_fragments_f32): for every 32-row tile and group of
//      8 k, lane l holds 4 values A[l % 32][2t + l / 32], t = 0..3 -- the A operands of 4 consecutive MFMAs.
//   B  lane l = 32*kq + j reads V adjacent columns Vj .. Vj + V - 1 of row 2t + kq and feeds them to V MFMAs that share
//      the A value: MFMA v computes the columns n = Vj + v.  Every lane ends with V adjacent output columns per row.
// Any N and alignment: the last lane of a row moves left so that it ends at N and computes some of its neighbour's columns
// a second time (the same bits), so that no access leaves the row.
//
// A wave takes 32 MT rows x 32 V columns.  Launches with too few of those for the chip split the K loop: WK waves take
// contiguous parts of the stored blocks, and their sums are added through LDS in wave order (bitwise reproducible).
#include <algorithm>

#include "asp_internal.h"

namespace asp {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

namespace {

typedef __attribute__((address_space(1))) const char global_char;

template <int V>
struct Cols {
    typedef float type __attribute__((ext_vector_type(V), aligned(4)));
};
}  // namespace

// rank_info[r] = {block-row, first stored block, stored blocks, -}.  A workgroup is WM x WN x WK waves and computes 32 MT WM
// rows of a block-row x 32 V WN columns.  N >= V.  WHOLE: K % BR == 0, no unit has rows past K.
template <int BR, int MT, int V, int WM, int WN, int WK, bool WHOLE>
__global__ __launch_bounds__(64 * WM * WN * WK, MT *V > 4 ? 2 : 4) void bcsr_f32_spmm_kernel(
    const int4 *__restrict__ rank_info, const int32_t *__restrict__ block_col_idx, const float *__restrict__ a_packed,
    const float *__restrict__ B, float *__restrict__ C, int M, int K, int64_t N, int n_brows, int n_tiles, int xcd_cols) {
    typedef typename Cols<V>::type cols_t;
    constexpr int GROUPS = BR / (32 * MT * WM);  // workgroups per block-row
    constexpr int UPB = BR / 8;                  // units of 8 k per block
    static_assert(GROUPS * 32 * MT * WM == BR && (WK == 1 || WM * WN == 1), "shape of the workgroup");

    // Workgroups go to the 8 XCDs round-robin by flat id.  The XCDs form xcd_cols groups that share the column tiles out
    // between them, so that the tiles on one L2 read the same columns of B; the XCDs of a group share the block-rows.
    // An XCD walks the block-rows longest first, all its column tiles of each.
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, xn = xcd % xcd_cols, xr = xcd / xcd_cols;
    const int nt0 = (int)((int64_t)n_tiles * xn / xcd_cols), ntc = (int)((int64_t)n_tiles * (xn + 1) / xcd_cols) - nt0;
    const int in_tile = local / ntc * (8 / xcd_cols) + xr, nt = nt0 + local % ntc;
    if (in_tile >= n_brows * GROUPS) return;
    const int4 ri = rank_info[in_tile / GROUPS];
    const int br = ri.x, blk0 = ri.y, n_units = ri.z * UPB;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / (WM * WN), wm = wave / WN % WM, wn = wave % WN;
    const int kq = lane >> 5, jl = lane & 31;
    const int row0 = (in_tile % GROUPS * WM + wm) * MT;  // in 32-row tiles of the block-row
    const int64_t n0 = ((int64_t)nt * WN + wn) * (32 * V);
    if (WK == 1 && n0 >= N) return;
    const int64_t n = n0 + jl * V, nc = n < N - V ? n : N - V;
    const uint32_t row_bytes = (uint32_t)N * 4, coff = (uint32_t)nc * 4;  // N <= ASP_MAX_N: 8 rows take less than 2^32 bytes
    const int u0 = (int)((int64_t)n_units * wk / WK), u1 = (int)((int64_t)n_units * (wk + 1) / WK);

    f32x16 acc[MT][V];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][v][e] = 0.f;

    if (u0 < u1) {
        const float *a_tile = a_packed + (int64_t)blk0 * (BR * BR) + row0 * 512;
        // lane i holds the block column of the wave's i-th block, 64 at a time
        int col_base = u0 / UPB, cols;
        auto load_cols = [&]() __attribute__((always_inline)) {
            const int last = ri.z - 1, p = col_base + lane;
            cols = block_col_idx[blk0 + (p < last ? p : last)];
        };
        load_cols();
        struct Unit {
            f32x4 a[MT];
            cols_t b[4];
            int left;  // rows of B from the unit's first one on, or less than 1
        };
        auto load = [&](int u, Unit &f) __attribute__((always_inline)) {
            const int p = u / UPB, s = u % UPB;
            // (before the look-up: a wave's first columns are still on their way)  Blocks are [16 k][32-row tile][8 k][lane][4]
            global_char *a = (global_char *)(a_tile + (int64_t)p * (BR * BR) + (s >> 1) * (BR * 16) + (s & 1) * 256);
            uint32_t aoff = lane * 16;
            asm("" : "+s"(a), "+v"(aoff));
#pragma unroll
            for (int i = 0; i < MT; ++i) f.a[i] = *(const __attribute__((address_space(1))) f32x4 *)(a + i * 2048 + aoff);
            if (p - col_base >= 64) {
                col_base = p;
                load_cols();
                asm volatile("" : "+v"(cols));  // waited for here, or every look-up would wait for all loads in flight
            }
            const int k0 = __builtin_amdgcn_readlane(cols, p - col_base) * BR + s * 8;
            f.left = WHOLE ? 8 : K - k0;
            // past K, where a unit may also start: its last row, dropped when the unit is multiplied
            global_char *row = (global_char *)B + (uint64_t)(uint32_t)(WHOLE ? k0 : min(k0, K - 1)) * row_bytes;
            const int last = max(f.left - 1, 0);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t off = (uint32_t)(WHOLE ? 2 * t + kq : min(2 * t + kq, last)) * row_bytes + coff;
                asm("" : "+s"(row), "+v"(off));  // scalar base + 32-bit offset, instead of a 64-bit vector address per row
                f.b[t] = *(const __attribute__((address_space(1))) cols_t *)(row + off);
            }
            asm volatile("" ::: "memory");  // (the loads are issued here, not where the next unit is multiplied)
        };
        auto multiply = [&](Unit &f) __attribute__((always_inline)) {
            if (!WHOLE && f.left < 8)  // rows past K count as zeros
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int v = 0; v < V; ++v) f.b[t][v] = 2 * t + kq < f.left ? f.b[t][v] : 0.f;
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        acc[i][v] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[i][t], f.b[t][v], acc[i][v], 0, 0, 0);
        };
        Unit f0, f1;
        load(u0, f0);
        if constexpr (MT * V >= 4) {
            // one copy of the MFMAs: with two the accumulators are moved between them.  (The last round loads its own
            // unit again.)
#pragma unroll 1
            for (int u = u0; u < u1; ++u) {
                load(u + 1 < u1 ? u + 1 : u, f1);
                multiply(f0);
                f0 = f1;
            }
        } else {
            int u = u0;
            for (; u + 2 < u1; u += 2) {
                load(u + 1, f1);
                multiply(f0);
                load(u + 2, f0);
                multiply(f1);
            }
            if (u + 1 < u1) {
                load(u + 1, f1);
                multiply(f0);
                multiply(f1);
            } else {
                multiply(f0);
            }
        }
    }

    // D layout of the MFMA: register e of lane l is row 8*(e/4) + 4*(l/32) + e%4, column l%32 (= jl), and
    // MFMA v of a group holds output column V*jl + v: V adjacent columns per lane and row.
    if constexpr (WK == 1) {
        if (n >= N) return;
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int64_t row = (int64_t)br * BR + (row0 + i) * 32 + 8 * (e >> 2) + 4 * kq + (e & 3);
                cols_t c;
#pragma unroll
                for (int v = 0; v < V; ++v) c[v] = acc[i][v][e];
                if (row < M) __builtin_nontemporal_store(c, (cols_t *)(C + row * N + nc));  // C is write-once: keep B in L2
            }
    } else {
        // 16 rows at a time, so that the LDS leaves room for four workgroups of four waves on a compute unit
        constexpr int PITCH = 32 * V + 4;
        __shared__ __attribute__((aligned(16))) float part[WK][16][PITCH];
#pragma unroll
        for (int i = 0; i < 2 * MT; ++i) {
            if (i > 0) __syncthreads();
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                cols_t c;
#pragma unroll
                for (int v = 0; v < V; ++v) c[v] = acc[i >> 1][v][(i & 1) * 8 + e];
                *(cols_t *)&part[wk][8 * (e >> 2) + 4 * kq + (e & 3)][jl * V] = c;
            }
            __syncthreads();
            for (int x = tid; x < 16 * 32; x += 64 * WK) {
                const int lr = x >> 5, j = x & 31;
                const int64_t row = (int64_t)br * BR + row0 * 32 + i * 16 + lr, cn = n0 + j * V;
                cols_t s = *(const cols_t *)&part[0][lr][j * V];
#pragma unroll
                for (int w = 1; w < WK; ++w) s += *(const cols_t *)&part[w][lr][j * V];
                if (row < M && cn < N)
                    __builtin_nontemporal_store(s, (cols_t *)(C + row * N + (cn < N - V ? cn : N - V)));
            }
        }
    }
}

// ---- host side ------------------------------------------------------------------------------------
// false: too many threads for a launch
template <int BR, int MT, int V, int WM, int WN, int WK>
static bool launch_f32(const asp_handle *h, const void *B, void *C, int64_t N, hipStream_t stream) {
    const int64_t n_tiles = ceil_div(N, 32 * V * WN);
    // as many groups of XCDs as can share the column tiles out evenly (within an eighth)
    int xcd_cols = 8;
    while (xcd_cols > 1 && 8 * ceil_div(n_tiles, xcd_cols) * xcd_cols > 9 * n_tiles) xcd_cols /= 2;
    const int64_t per_xcd = ceil_div(h->n_brows * (BR / (32 * MT * WM)), 8 / xcd_cols) * ceil_div(n_tiles, xcd_cols);
    if (!launch_fits(8 * per_xcd, 64 * WM * WN * WK)) return false;
    dim3 grid((unsigned)(8 * per_xcd)), block(64 * WM * WN * WK);
#define ASP_F32(WHOLE)                                                                                                              \
    hipLaunchKernelGGL((bcsr_f32_spmm_kernel<BR, MT, V, WM, WN, WK, WHOLE>), grid, block, 0, stream, (const int4 *)h->d_rank_info, \
                       h->d_col_idx, (const float *)h->d_values, (const float *)B, (float *)C, (int)h->m, (int)h->k, N,             \
                       (int)h->n_brows, (int)n_tiles, xcd_cols)
    if (h->k % BR == 0) ASP_F32(true);
    else ASP_F32(false);
#undef ASP_F32
    return true;
}

// 64 x 128 tiles, where they are many: by two waves that divide the blocks (false), or by one, side by side for twice the columns.
// Two end long block-rows sooner (18944 x 3584 at 90 %, 2048 columns, 18 tiles to a compute unit, 128 / 64 / 32-row blocks 244 / 253 / 241 ->
// 244 / 242 / 235, geometric lengths 374 / 372 / 276 -> 238 / 231 / 215, before WHOLE), one starts and adds up less: from some 30 tiles to a unit on, but not
// where block-rows are long and alike (two / one: 15 260 x 3035 at 95 %, geometric, 64-row, 8192 columns 355 / 340, 13 202 x 2023 at 50 % 1698 /
// 1781), from fewer where all are short (12 034 x 1955 at 90 %, 128-row, 4096 columns 208 / 199, 12 567 x 4176 at 98 %, 8192 columns 188 / 172);
// with 32-row blocks, whose waves have half the sums, where they are alike too (10 094 x 3359 at 95 %, 8192 columns 281 / 274).  Of 230 products
// of 512 to 8192 columns 1.01 times faster in the mean than two everywhere, 1.06 than one.
bool bcsr_f32_one_wave(const asp_handle *h, int64_t N) {
    const int64_t cus = h->n_cus > 0 ? h->n_cus : 256, tall = h->n_brows * h->b_row / 64 * ceil_div(N, 128);
    const int64_t k_stored = h->n_units * h->b_row / h->n_brows;  // of a block-row in the mean
    auto longest_within = [&](int64_t times) { return h->hb.max_blocks * h->n_brows <= times * h->n_units; };
    if (h->b_row == 32) return tall >= 31 * cus || (longest_within(2) && k_stored <= 800);
    if (k_stored <= 256 && longest_within(5) && tall >= 23 * cus) return true;  // (geometric lengths: 5 to 7 times the mean)
    return tall >= 31 * cus && !longest_within(2);
}

// The largest wave tile that still gives the chip enough of them, and the narrower one where N would fill the wider one
// badly.  us at 90 %, 64 x 64 blocks, tiles of 64 x 128 / 64 x 128 by four waves / 32 x 64 by four / 32 x 32 by eight:
// 18944 x 3584 at 2048 columns 239 / 258 / 267 / -, at 1024 151 / 133 / 140 / 160, at 64 - / - / 19.5 / 16.2;
// 3584 x 9000 at 2048 163 / 124 / 128 / -, at 256 - / 42 / 29.6 / 29; 3000 x 3000 at 2048 - / 47 / 43 / 50, at 72 - / - / 12 / 9.
template <int BR>
static bool launch_f32_rows(const asp_handle *h, const void *B, void *C, int64_t N, hipStream_t stream) {
    constexpr int MT = BR >= 64 ? 2 : 1;
    const int64_t cus = h->n_cus > 0 ? h->n_cus : 256, n32 = ceil_div(N, 32), n64 = ceil_div(N, 64), n128 = ceil_div(N, 128);
    const int64_t tall = h->n_brows * BR / 64 * n128;  // tiles of 64 x 128 elements
    if (N >= 4 && 4 * n128 * 8 <= 2 * n64 * 9) {
        if (tall >= 16 * cus && bcsr_f32_one_wave(h, N)) return launch_f32<BR, MT, 4, BR / (32 * MT), 2, 1>(h, B, C, N, stream);
        if (tall >= 16 * cus) return launch_f32<BR, MT, 4, 1, 1, 2>(h, B, C, N, stream);
        if (tall >= 3 * cus) return launch_f32<BR, MT, 4, 1, 1, 4>(h, B, C, N, stream);
    }
    if (N >= 2 && 2 * n64 * 8 <= n32 * 9 && 2 * h->n_brows * (BR / 32) * n64 >= 5 * cus)
        return launch_f32<BR, 1, 2, 1, 1, 4>(h, B, C, N, stream);
    return launch_f32<BR, 1, 1, 1, 1, 8>(h, B, C, N, stream);
}

// Hundreds of millions of rows can take more threads than a launch has: then the shapes with the fewest threads
template <int BR>
static bool launch_f32_any(const asp_handle *h, const void *B, void *C, int64_t N, hipStream_t stream) {
    constexpr int MT = BR >= 64 ? 2 : 1;
    if (launch_f32_rows<BR>(h, B, C, N, stream)) return true;
    if (N >= 4) return launch_f32<BR, MT, 4, BR / (32 * MT), 2, 1>(h, B, C, N, stream);
    return launch_f32<BR, 1, 1, BR / 32, 1, 1>(h, B, C, N, stream);
}

// any N <= ASP_MAX_N and alignment; false: too many output tiles
bool bcsr_f32_launch(const asp_handle *h, const void *B, void *C, int64_t N, hipStream_t stream) {
    if (h->b_row == 128) return launch_f32_any<128>(h, B, C, N, stream);
    if (h->b_row == 64) return launch_f32_any<64>(h, B, C, N, stream);
    return launch_f32_any<32>(h, B, C, N, stream);
}

}  // namespace asp

// C = A x B for launches that are too small for the tile kernels, and for widths and alignments that do not allow 16-byte
// rows: strips of a block-row whose waves split the K loop.
//
// What bounds the tile kernels there: they walk a block-row slice by slice, every slice behind a barrier, at 0.4-0.7 us a
// slice when there is nothing else to run on the compute unit -- however far ahead they request (rings of 3 and of 8
// slices differ by 5 %).  58 us for the 15 blocks of a block-row of the 3584 x 18944 projection, at 64 columns as at 256.
// Here a workgroup takes 32 or 64 rows x 32 to 128 columns and its W waves each a contiguous part of the stored blocks,
// without a barrier in the loop: A comes from memory to registers in fragment order, B through registers into the wave's
// own piece of LDS, from where ds_read_b64_tr_b16 hands every lane 4 consecutive k of a column, one unit of 32 or 64 k
// ahead.  The waves' partial tiles meet in LDS once, are added in wave order (bitwise reproducible), rounded once, stored.
// us a call, before -> now: 1024 x 1024, 64 x 64 blocks, 256 columns 6.2 -> 3.7; 3584 x 18944 at 64 / 256 / 1024 columns
// 58 -> 6.6 / 58 -> 13 / 47 -> 34; 5003 x 3331 (80 %), 64 x 64 blocks, 1024 columns 42 -> 23.
// Rows at other alignments: 5003 x 3331 (80 %), 64 x 64 blocks, 1021 columns 26.8 -> 22.7 since the last column tile moves left
// instead of putting its lanes' loads together from a row's end (that tile alone had set the time of the launch).  Narrower than a tile single
// chunks move left: 26 713 x 852 (90 %), 128 x 128 blocks, 13 columns 11.9 -> 6.7, 68 784 x 862 (80 %), 64 x 64, 43 16.2 -> 11.1 (where a tile can
// move as a whole its 64 contiguous bytes are faster: 2012 x 7811 (80 %), 32 x 32, 61 columns 13.1 / 17.4).
// With more columns a strip's reads (B once per strip, A once per column tile) are so many more than the tile kernels' that
// these win.
#include <algorithm>

#include "asp_bcsr_pipe.h"

namespace asp {

// grid = units_m strips of 32 MT rows x column tiles of 32 NT; rank_info: {block-row, first block, blocks, -} in
// the schedule's order; col_idx / a_packed: the stored blocks,
// fragment-ordered; UKT: k per unit
enum StripRows { FEW, ANY, ALIGNED };  // N < 8; N >= 8; N % 8 == 0, B and C 16-byte aligned

template <int BR, int MT, int NT, int W, int UKT, StripRows ROWS>
__global__ __launch_bounds__(W * 64) void bcsr_strip_kernel(const int4 *__restrict__ rank_info,
                                                            const int32_t *__restrict__ col_idx,
                                                            const uint16_t *__restrict__ a_packed,
                                                            const uint16_t *__restrict__ B, uint16_t *__restrict__ C, int M,
                                                            int K, int N, int units_m) {
    constexpr int STRIPS = BR / (32 * MT);
    constexpr int UK = BR < UKT ? BR : UKT, KK = UK / 16, UPB = BR / UK;  // k of a unit, MFMA steps, units per block
    constexpr int LPR = NT * 4, RPI = 64 / LPR, BL = UK / RPI;  // lanes per row of B, rows per load, loads per unit
    constexpr int PB = NT * 64 + 64;          // LDS pitch of a row of B: the four rows of a transposing read share no bank
    constexpr int PITCH = 32 * NT + 4;        // floats per row of a partial tile
    constexpr int STAGE = UK * PB, PART = MT * 32 * PITCH * 4;
    __shared__ __attribute__((aligned(16))) uint8_t lds[W * (STAGE > PART ? STAGE : PART)];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // every XCD (workgroups go to them round-robin) takes a run of strips with all their column tiles, so that A stays in
    // its L2; the runs are cut from the schedule's lists (rank % 8), which have nearly the same number of blocks
    const int units_n = gridDim.x / units_m, xcd = blockIdx.x & 7, q = gridDim.x >> 3, r = gridDim.x & 7;
    const int id = xcd * q + (xcd < r ? xcd : r) + (blockIdx.x >> 3);
    const int un = id % units_n, um = id / units_n;
    const int n_brows = units_m / STRIPS, per = n_brows >> 3, more = n_brows & 7, at = um / STRIPS, strip = um % STRIPS;
    const int list = at < more * (per + 1) ? at / (per + 1) : more + (at - more * (per + 1)) / per;
    const int4 ri = rank_info[list + 8 * (at - list * per - (list < more ? list : more))];
    const int br = ri.x, blk0 = ri.y, n_units = ri.z * UPB;
    // Rows that are not 16-byte aligned: the last column tile moves left so that it ends at N.  Where N does not fill one tile, chunks of 8
    // columns that would pass N end there instead (those that start past it only feed columns that are never stored).
    const int n_own = un * (32 * NT), n0 = ROWS == ANY && N >= 32 * NT && n_own > N - 32 * NT ? N - 32 * NT : n_own;
    auto chunk_col = [&](int col) __attribute__((always_inline)) { return ROWS != FEW && col > N - 8 ? N - 8 : col; };
    auto chunk = [&](const uint16_t *row, int col) __attribute__((always_inline)) {
        if constexpr (ROWS == ALIGNED) return *(const u32x4 *)(row + col);
        else if constexpr (ROWS == ANY) return u32x4(*(const u32x4_a2 *)(row + col));
        else return load_tail8(row, col, N);
    };
    const int u0 = (int)((int64_t)n_units * wave / W), u1 = (int)((int64_t)n_units * (wave + 1) / W);

    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    if (u0 < u1) {
        uint8_t *sb = lds + wave * STAGE;
        const uint16_t *a_lane = a_packed + (int64_t)blk0 * (BR * BR) + strip * (MT * 512) + lane * 8;
        const int row_l = lane / LPR, col = chunk_col(n0 + (lane % LPR) * 8);
        uint8_t *st = sb + row_l * PB + (lane % LPR) * 16;
        // lane i holds the block column of the wave's i-th block, 64 at a time
        int col_base = u0 / UPB, cols;
        auto load_cols = [&]() __attribute__((always_inline)) {
            const int last = n_units / UPB - 1, p = col_base + lane;
            cols = col_idx[blk0 + (p < last ? p : last)];
        };
        load_cols();
        struct Unit {
            u32x4 a[MT][KK], b[BL];
        };
        auto load = [&](int u, Unit &f) __attribute__((always_inline)) {
            const int p = u / UPB, s = u % UPB;
            if (p - col_base >= 64) {
                col_base = p;
                load_cols();
                // Waited for here, or every look-up would wait for all loads in flight: of 85 products 0.987 of the time in the mean, 0.83 with
                // geometric lengths (5248 x 3072, 405 columns 16.8 -> 14.0 us), 1.06 at most.
                asm volatile("" : "+v"(cols));
            }
            const int k0 = __builtin_amdgcn_readlane(cols, p - col_base) * BR + s * UK;
            const u32x4 *a = (const u32x4 *)(a_lane + (int64_t)p * (BR * BR) + s * (UK * BR));
            if (k0 + UK <= K) {
                const uint16_t *src = B + (int64_t)(k0 + row_l) * N;
#pragma unroll
                for (int i = 0; i < BL; ++i) f.b[i] = chunk(src + (int64_t)(i * RPI) * N, col);
            } else {
#pragma unroll
                for (int i = 0; i < BL; ++i) {
                    const int k = k0 + row_l + i * RPI;
                    const uint16_t *row = B + (int64_t)(k < K ? k : K - 1) * N;
                    const u32x4 v = chunk(row, col);
                    f.b[i] = k < K ? v : u32x4{0u, 0u, 0u, 0u};
                }
            }
#pragma unroll
            for (int i = 0; i < KK; ++i)
#pragma unroll
                for (int g = 0; g < MT; ++g) f.a[g][i] = a[i * (BR * 2) + g * 64];
        };
        // transposing read: lane i of a 16-lane group addresses row i/4, 4 columns at 4*(i%4), and receives 4 rows of a column
        const uint8_t *tr = sb + (8 * (lane >> 5) + ((lane & 15) >> 2)) * PB + (16 * ((lane >> 4) & 1) + 4 * (lane & 3)) * 2;
        auto multiply = [&](const Unit &f) __attribute__((always_inline)) {
            // (LDS is in order within a wave: these writes come after the reads of the previous unit)
#pragma unroll
            for (int i = 0; i < BL; ++i) *(u32x4 *)(st + i * RPI * PB) = f.b[i];
#pragma unroll
            for (int i = 0; i < KK; ++i) {
                bf16x8 b[NT];
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const uint8_t *p0 = tr + i * 16 * PB + j * 64;
                    short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3))) *)(p0));
                    short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3))) *)(p0 + 4 * PB));
                    b[j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
#pragma unroll
                for (int g = 0; g < MT; ++g)
#pragma unroll
                    for (int j = 0; j < NT; ++j)  // operands swapped: a lane ends with 4 adjacent columns of a row
                        acc[g][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], __builtin_bit_cast(bf16x8, f.a[g][i]),
                                                                            acc[g][j], 0, 0, 0);
            }
        };
        Unit f0, f1;
        load(u0, f0);
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
    __syncthreads();  // the staging areas become partial tiles

    // lane l holds row l % 32, columns 8 q + 4 (l / 32) + 0..3
    float *part = (float *)lds;
#pragma unroll
    for (int g = 0; g < MT; ++g)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f32x4 v = {acc[g][j][4 * e], acc[g][j][4 * e + 1], acc[g][j][4 * e + 2], acc[g][j][4 * e + 3]};
                *(f32x4 *)&part[(wave * (MT * 32) + g * 32 + (lane & 31)) * PITCH + j * 32 + 8 * e + 4 * (lane >> 5)] = v;
            }
    __syncthreads();
    const int m0 = br * BR + strip * (32 * MT);
    for (int i = tid; i < MT * 32 * LPR; i += W * 64) {  // 8 adjacent columns of a row
        const int row = i / LPR, c = (i % LPR) * 8;
        f32x4 s0 = *(const f32x4 *)&part[row * PITCH + c], s1 = *(const f32x4 *)&part[row * PITCH + c + 4];
#pragma unroll
        for (int w = 1; w < W; ++w) {
            s0 += *(const f32x4 *)&part[(w * (MT * 32) + row) * PITCH + c];
            s1 += *(const f32x4 *)&part[(w * (MT * 32) + row) * PITCH + c + 4];
        }
        if (m0 + row >= M || n0 + c >= N || n0 + c + 8 <= n_own) continue;  // (a column of two tiles or chunks gets the same bits from both)
        const bf16x4 lo = __builtin_convertvector(s0, bf16x4), hi = __builtin_convertvector(s1, bf16x4);  // to nearest even
        const bf16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        const int col = chunk_col(n0 + c);
        uint16_t *dst = C + (int64_t)(m0 + row) * N + col;
        const short8v bits = __builtin_bit_cast(short8v, v);
        if constexpr (ROWS == ALIGNED) {
            *(u32x4 *)dst = __builtin_bit_cast(u32x4, v);
        } else if constexpr (ROWS == ANY) {
            *(u32x4_a2 *)dst = __builtin_bit_cast(u32x4, v);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (col + e < N) dst[e] = (uint16_t)bits[e];
        }
    }
}

// ---- host side ------------------------------------------------------------------------------------
// false: too many threads for a launch
template <int BR, int MT, int NT, int W, int UK, StripRows ROWS>
static bool launch_strip(const asp_handle *h, const void *B, void *C, int64_t N, hipStream_t stream) {
    const int units_m = (int)h->n_brows * (BR / 32 / MT);
    if (!launch_fits(units_m * ceil_div(N, 32 * NT), W * 64)) return false;
    dim3 grid((unsigned)(units_m * ceil_div(N, 32 * NT))), block(W * 64);
    hipLaunchKernelGGL((bcsr_strip_kernel<BR, MT, NT, W, UK, ROWS>), grid, block, 0, stream, (const int4 *)h->d_rank_info,
                       h->d_col_idx, (const uint16_t *)h->d_values, (const uint16_t *)B, (uint16_t *)C, (int)h->m,
                       (int)h->k, (int)N, units_m);
    return true;
}

// Shape of the wave tiles, the largest that still gives the chip enough of them.  At 90 %, us a call, 32 x 32 x 8 waves /
// 64 x 64 x 8 / 64 x 64 x 4: 3584 x 18944 at 64 columns 6.6 / 10.5 / 11, at 256 17.8 / 13.0 / 17, at 512 - / 22.6 / 20.8;
// 18944 x 3584, whose strips have too few units for 8 waves, at 64 columns 8.2 / 8.4 / 6.7, at 512 - / 45 / 25.6.
// 32-row blocks, 32 x 64 / 32 x 128: 3584 x 18944 at 512 columns 34 / 29, 18944 x 3584 27 / 23.5 (aligned rows only).
template <int BR, StripRows ROWS>
static bool launch_strips(const asp_handle *h, const void *B, void *C, int64_t N, hipStream_t stream) {
    const int64_t cus = h->n_cus > 0 ? h->n_cus : 256, n64 = ceil_div(N, 64);
    const bool short_rows = h->n_units * (BR / 32) < 14 * h->n_brows;
    if constexpr (ROWS != FEW && BR >= 64) {
        const int64_t tiles = h->n_brows * (BR / 64) * n64;
        if (2 * tiles >= cus) {
            if (2 * tiles >= 3 * cus || short_rows) return launch_strip<BR, 2, 2, 4, 32, ROWS>(h, B, C, N, stream);
            return launch_strip<BR, 2, 2, 8, 32, ROWS>(h, B, C, N, stream);
        }
    } else if constexpr (ROWS != FEW) {
        if constexpr (ROWS == ALIGNED)
            if (2 * h->n_brows * ceil_div(N, 128) >= 3 * cus) return launch_strip<BR, 1, 4, 2, 32, ROWS>(h, B, C, N, stream);
        if (2 * h->n_brows * n64 >= 3 * cus) return launch_strip<BR, 1, 2, 4, 64, ROWS>(h, B, C, N, stream);
    }
    if (short_rows) return launch_strip<BR, 1, 1, 4, 64, ROWS>(h, B, C, N, stream);
    return launch_strip<BR, 1, 1, 8, 64, ROWS>(h, B, C, N, stream);
}

template <int BR>
static bool launch_rows(const asp_handle *h, const void *B, void *C, int64_t N, bool vec, hipStream_t stream) {
    if (vec) return launch_strips<BR, ALIGNED>(h, B, C, N, stream);
    if (N >= 8) return launch_strips<BR, ANY>(h, B, C, N, stream);
    return launch_strips<BR, FEW>(h, B, C, N, stream);
}

// Whether strips are the faster choice: estimates in us, linear in the longest block-row (K slices of 32) and in the
// work, fitted to 3584 x 18944, 18944 x 3584, 4096 x 4096 (80 %), 1024 x 1024 and 5003 x 3331 (80 %) at 64 to 4096 columns.
// The crossing is near 500 columns for 18944 x 3584 and 1500 to 2000 for the others.  The ring kernel's costs are those of groups of
// four column tiles, and it is faster now: of 240 products (ten matrices, 128 to 3072 columns) the choice is in the mean 1.005
// (128-row), 1.02 (64) and 1.03 (32) times slower than the better kernel, at worst 1.43 (32-row, 2048 x 8192 at 80 %, 2048
// columns, strips 53, tiles 37 us).
static bool strips_win(const asp_handle *h, int64_t N, const BcsrPlan &p) {
    const double cus = h->n_cus > 0 ? h->n_cus : 256, b = h->b_row;
    const double work = (double)h->n_units * b * b * (double)N * 256 / cus;  // stored elements x columns
    const double longest = (double)h->hb.max_blocks * (b / 32), slices = (double)h->n_units * (b / 32);
    if (!p.vectorized) {
        // Against the register-staged kernel: of 90 products (1000 to 9000 rows, 64 to 9000 columns, half with
        // geometric block-row lengths) the choice is 1.007 times slower than the better one in the mean, 1.24 at most.  A block-row's strips run on
        // one XCD, so one that outweighs an eighth of the rest sets the time (1280 x 2112, geometric, 6183 columns 61 / 32).
        const double of_xcd = std::max(work, 8.0 * (double)h->hb.max_blocks * b * b * (double)N * 256 / cus);
        return 4 + (b == 32 ? 8e-9 : 6e-9) * of_xcd <
               3 + (b == 32 ? 0.3 : 0.33) * longest + (b == 32 ? 5.2e-9 : 2.5e-9) * work;
    }
    // with more of B than this in flight between the XCDs strips fall behind (1024 x 8192, 12 000 columns: 184 / 244 us)
    if ((double)h->k * (double)N * 2 > 64e6) return false;
    const double strips = 1.1 * (3 + (b == 32 ? 6.5e-9 : 4.6e-9) * work + 4e-7 * (double)h->m * (double)N * 256 / cus);  // (5 TB/s of C)
    const double tiles = (double)p.n_tiles / cus;
    if (p.bn == 512) {
        if (p.workgroups >= 2 * (int64_t)cus) return false;
        const double c_longest = h->has_comp ? (double)h->hc.max_blocks * 4 : longest;
        const double c_slices = h->has_comp ? (double)h->c_n_units * 4 : slices;
        return strips < 3 + 0.3 * c_longest + 0.9 * c_slices * tiles;
    }
    if (p.bn == 256) return strips < 1 + 0.72 * longest + 0.18 * slices * tiles;
    if (p.bn == 128) return strips < 1 + 0.57 * longest + 0.05 * slices * tiles;
    return strips < 1 + 0.45 * longest + 0.05 * slices * tiles;
}

// any block size, N < 2^25; p: the plan (p.vectorized: N % 8 == 0, B and C 16-byte aligned)
bool bcsr_strip_launch(const asp_handle *h, const void *B, void *C, int64_t N, const BcsrPlan &p, hipStream_t stream) {
    if (h->n_units == 0 || N >= (1ll << 25) || !strips_win(h, N, p)) return false;
    const bool vec = p.vectorized != 0;
    if (h->b_row == 128) return launch_rows<128>(h, B, C, N, vec, stream);
    if (h->b_row == 64) return launch_rows<64>(h, B, C, N, vec, stream);
    return launch_rows<32>(h, B, C, N, vec, stream);
}

}  // namespace asp

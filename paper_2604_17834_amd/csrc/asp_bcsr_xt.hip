// Y = X x A^T with K-contiguous activations (paper, Section IV-D's layout) for few tokens, and for any token count where
// the operands do not allow the 16-byte paths of the tile kernels: a decoded batch through a pruned projection.
//
// What bounds it: with a few tokens the product is one read of A (13.6 MB for the 18944 x 3584 projection at 90 %), and
// what costs time is not the bytes but that they be requested early and by the whole chip.  A 128 x 512 tile per
// workgroup, most of it padding, left 28 of 256 compute units working on the 28 block-rows of the down projection.
// So here the unit is a strip of 32 to 128 outputs x 32 or 64 tokens, and the W waves of a workgroup split the strip's K
// loop, every wave a contiguous part of the stored blocks.  A's fragment order and the K-contiguous X are what
// v_mfma_f32_32x32x16_bf16 wants in registers, so both operands go straight from memory to registers, 32 or 64 k at a
// time, one such unit ahead -- no LDS stage, no barrier in the loop.  The waves' partial tiles meet in LDS once and are
// added in wave order (bitwise reproducible), rounded once, and stored.
// us a call at 16 tokens, before (128 x 512 tiles) -> now: gate 26 -> 5.6, down 78 -> 6.4, down in 64 x 64 / 32 x 32
// blocks 122 -> 6.7 / 196 -> 5.8; down at 256 tokens 87.6 -> 18.5.  (The host takes 4.0 us to enqueue a call, 6.9 through
// SparseLinear; the gate and down kernels alone 6.5 and 7.5 in a trace: the chain block-row -> columns -> X of a wave.)
// With more tokens X goes through LDS (bcsr_xt_staged_kernel), and with many the ring kernel's larger tiles take over
// (bcsr_spmm_xt_launch).
//
// Any K, M, N and alignment (VEC = false): 16-byte loads of X at element alignment; elements past K count
// as zeros.
#include <algorithm>

#include "asp_bcsr_pipe.h"

namespace asp {

// grid = units_m strips of 32 MT rows x token tiles of 32 NT; rank_info: {block-row, first block, blocks, -} in
// the schedule's order; col_idx / a_packed: the stored blocks,
// fragment-ordered; UKT: k per unit
template <int BR, int MT, int NT, int W, int UKT, bool VEC>
__global__ __launch_bounds__(W * 64) void bcsr_xt_strip_kernel(const int4 *__restrict__ rank_info,
                                                               const int32_t *__restrict__ col_idx,
                                                               const uint16_t *__restrict__ a_packed,
                                                               const uint16_t *__restrict__ X, uint16_t *__restrict__ Y,
                                                               int M, int K, int64_t N, int units_m) {
    constexpr int STRIPS = BR / (32 * MT);
    constexpr int UK = BR < UKT ? BR : UKT, KK = UK / 16, UPB = BR / UK;  // k of a unit, MFMA steps, units per block
    constexpr int PITCH = 32 * MT + 4;                                          // floats per token of a partial tile
    __shared__ __attribute__((aligned(16))) float part[W][NT * 32][PITCH];

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
    const int64_t n0 = (int64_t)un * (32 * NT);
    const int u0 = (int)((int64_t)n_units * wave / W), u1 = (int)((int64_t)n_units * (wave + 1) / W);

    f32x16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    if (u0 < u1) {
        const int kl = 8 * (lane >> 5);  // this lane's 8 k inside an MFMA step
        const uint16_t *x[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int64_t t = n0 + j * 32 + (lane & 31);
            x[j] = X + (t < N ? t : N - 1) * K;  // tokens past N feed columns that are never stored
        }
        const uint16_t *a_lane = a_packed + (int64_t)blk0 * (BR * BR) + strip * (MT * 512) + lane * 8;
        // lane i holds the block column of the wave's i-th block, 64 at a time
        int col_base = u0 / UPB, cols;
        auto load_cols = [&]() __attribute__((always_inline)) {
            const int last = n_units / UPB - 1, p = col_base + lane;
            cols = col_idx[blk0 + (p < last ? p : last)];
        };
        load_cols();
        struct Unit {
            u32x4 a[MT][KK], x[NT][KK];
        };
        auto load = [&](int u, Unit &f) __attribute__((always_inline)) {
            const int p = u / UPB, s = u % UPB;
            if (p - col_base >= 64) {
                col_base = p;
                load_cols();
                // Waited for here, or every look-up would wait for all loads in flight: of 60 products of 17 to 600 tokens in a captured graph
                // 0.999 of the time in the mean, 0.93 (1088 x 16 768, geometric lengths, 533 tokens 26.2 -> 24.5 us) to 1.05.
                asm volatile("" : "+v"(cols));
            }
            const u32x4 *a = (const u32x4 *)(a_lane + (int64_t)p * (BR * BR) + s * (UK * BR));
#pragma unroll
            for (int i = 0; i < KK; ++i)
#pragma unroll
                for (int g = 0; g < MT; ++g) f.a[g][i] = a[i * (BR * 2) + g * 64];
            const int k0 = __builtin_amdgcn_readlane(cols, p - col_base) * BR + s * UK;
            if (k0 + UK <= K) {
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int i = 0; i < KK; ++i) {
                        const uint16_t *src = x[j] + k0 + i * 16 + kl;
                        f.x[j][i] = VEC ? *(const u32x4 *)src : *(const u32x4_a2 *)src;
                    }
            } else {
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int i = 0; i < KK; ++i) {
                        const int k = k0 + i * 16 + kl;
                        u32x4 v = {0u, 0u, 0u, 0u};
                        if (!VEC) v = load_tail8(x[j], k, K);
                        else if (k < K) v = *(const u32x4 *)(x[j] + k);  // K % 8 == 0
                        f.x[j][i] = v;
                    }
            }
        };
        auto multiply = [&](const Unit &f) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < KK; ++i)
#pragma unroll
                for (int g = 0; g < MT; ++g)
#pragma unroll
                    for (int j = 0; j < NT; ++j)
                        acc[g][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            __builtin_bit_cast(bf16x8, f.a[g][i]), __builtin_bit_cast(bf16x8, f.x[j][i]), acc[g][j], 0, 0, 0);
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

    // D of the MFMA: lane l holds token l % 32, rows 8 q + 4 (l / 32) + 0..3
#pragma unroll
    for (int g = 0; g < MT; ++g)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 v = {acc[g][j][4 * q], acc[g][j][4 * q + 1], acc[g][j][4 * q + 2], acc[g][j][4 * q + 3]};
                *(f32x4 *)&part[wave][j * 32 + (lane & 31)][g * 32 + 8 * q + 4 * (lane >> 5)] = v;
            }
    __syncthreads();
    const int m0 = br * BR + strip * (32 * MT);
    for (int i = tid; i < NT * 32 * 16 * MT; i += W * 64) {  // two adjacent outputs of a token
        const int t = i / (16 * MT), r = (i % (16 * MT)) * 2;
        float s0 = part[0][t][r], s1 = part[0][t][r + 1];
#pragma unroll
        for (int w = 1; w < W; ++w) {
            s0 += part[w][t][r];
            s1 += part[w][t][r + 1];
        }
        const uint32_t lo = __builtin_bit_cast(uint16_t, (__bf16)s0), hi = __builtin_bit_cast(uint16_t, (__bf16)s1);
        if (n0 + t < N) {
            uint16_t *dst = Y + (n0 + t) * M + m0 + r;
            if (VEC) {
                if (m0 + r < M) *(uint32_t *)dst = lo | (hi << 16);  // M % 8 == 0
            } else {
                if (m0 + r < M) dst[0] = (uint16_t)lo;
                if (m0 + r + 1 < M) dst[1] = (uint16_t)hi;
            }
        }
    }
}

// Strips of 64 or 128 outputs x 64 tokens for short prompts.  X goes through LDS here: an MFMA step wants 16 bytes of each of 32
// tokens, and a load with as many cache lines as lanes takes the L1 four times as long as one that reads whole lines.  So a
// wave reads 64 k of 8 tokens with an instruction, eight adjacent lanes to a token's 128 bytes, and leaves them in 8 KB of
// its own LDS, chunk c of token t at place c ^ (t % 8), which both the writes and the fragment reads meet without
// bank conflicts.  X is one unit of 64 k ahead in registers, A half a unit; a wave's LDS operations execute in order, so
// the loop has no barrier.  LDS and registers are for two workgroups on a compute unit (MT = 2: three): each fills the waits
// of the others.  us a call, straight to registers -> here: 3584 x 18944 at 90 %, 128-row blocks, 256 / 1024 / 2048 tokens 18.7 /
// 37.3 / 60.5 -> 12.9 / 28.6 / 54.7, 64-row blocks, 1024 tokens 46 -> 37; 18944 x 3584, 512 tokens 30 -> 22.  What bounds it: L2 misses on X
// (123 MB at 1024 tokens, the columns of different block-rows hardly meet) with one unit a wave ahead.
template <int BR, int MT>
__global__ __launch_bounds__(256, MT == 4 ? 2 : 3) void bcsr_xt_staged_kernel(const int4 *__restrict__ rank_info,
                                                                             const int32_t *__restrict__ col_idx,
                                                                             const uint16_t *__restrict__ a_packed,
                                                                             const uint16_t *__restrict__ X, uint16_t *__restrict__ Y,
                                                                             int M, int K, int64_t N, int units_m) {
    constexpr int STRIPS = BR / (32 * MT), UPB = BR / 64;
    __shared__ __attribute__((aligned(16))) union {
        u32x4 x[4][64][8];             // [wave][token][chunk of 8 k]
        f32x4 part[4][MT * 4][64];     // [wave][register / 4][lane]
    } lds;
    __shared__ __attribute__((aligned(16))) uint16_t out[64][16 * MT + 8];

    typedef __attribute__((address_space(1))) char global_char;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // as above: an XCD takes a run of strips with all their column tiles
    const int units_n = gridDim.x / units_m, xcd = blockIdx.x & 7, q = gridDim.x >> 3, r = gridDim.x & 7;
    const int id = xcd * q + (xcd < r ? xcd : r) + (blockIdx.x >> 3);
    const int un = id % units_n, um = id / units_n;
    const int n_brows = units_m / STRIPS, per = n_brows >> 3, more = n_brows & 7, at = um / STRIPS, strip = um % STRIPS;
    const int list = at < more * (per + 1) ? at / (per + 1) : more + (at - more * (per + 1)) / per;
    const int4 ri = rank_info[list + 8 * (at - list * per - (list < more ? list : more))];
    const int br = ri.x, blk0 = ri.y, n_units = ri.z * UPB;
    const int64_t n0 = (int64_t)un * 64;
    const int u0 = n_units * wave / 4, u1 = n_units * (wave + 1) / 4;

    f32x16 acc[MT][2];
    const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)  // 0 x 0 + 0 (copies of zeros would take a tile's registers more)
            asm volatile("s_nop 3\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %1, 0" : "=a"(acc[i][j]) : "v"(zero));

    if (u0 < u1) {
        const int chunk = lane & 7, row = lane >> 3, half = lane >> 5;
        // offsets of tokens; those past N feed columns that are never stored
        const uint32_t row_bytes = (uint32_t)K * 2, last_token = (N - n0 < 64 ? (uint32_t)(N - n0) - 1 : 63) * row_bytes;
        const uint32_t first_token = row * row_bytes < last_token ? row * row_bytes : last_token;
        const char *x0 = (const char *)(X + n0 * K);
        const char *a_base = (const char *)(a_packed + (int64_t)blk0 * (BR * BR) + strip * (MT * 512));
        const int last = u1 - 1;
        // (a block column is a vector load of one address, a unit ahead of the loads of X that need it: it is waited for in
        // order with them)
        auto column = [&](int u) __attribute__((always_inline)) {
            uint32_t zero = 0;
            asm("" : "+v"(zero));
            return col_idx[blk0 + (u < last ? u : last) / UPB + zero];
        };
        u32x4 xr[8], a0[MT][2], a1[MT][2];
        int k0;  // first k of the unit in xr
        auto load_x = [&](int u, int col) __attribute__((always_inline)) {
            k0 = __builtin_amdgcn_readfirstlane(col) * BR + (u % UPB) * 64;
            const uint32_t at = (uint32_t)(k0 + chunk * 8 < K ? k0 + chunk * 8 : K - 8) * 2;
            uint32_t token = first_token;
            asm("" : "+v"(token));  // (eight offsets kept through the loop are eight registers too many)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                xr[i] = *(const u32x4 *)(x0 + (token + at));
                token = token + 8 * row_bytes < last_token ? token + 8 * row_bytes : last_token;
            }
        };
        auto load_a = [&](int u, int h, u32x4 (&a)[MT][2]) __attribute__((always_inline)) {
            uint32_t at = lane * 16;
            asm("" : "+v"(at));
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const global_char *src = (const global_char *)a_base + (int64_t)u * (128 * BR) + h * (64 * BR) + i * (32 * BR);
                asm("" : "+s"(src));
#pragma unroll
                for (int g = 0; g < MT; ++g) a[g][i] = *(const __attribute__((address_space(1))) u32x4 *)(src + at + g * 1024);
            }
        };
        auto multiply = [&](int h, const u32x4 (&a)[MT][2]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                u32x4 x[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) x[j] = lds.x[wave][j * 32 + (lane & 31)][(4 * h + 2 * i + half) ^ (lane & 7)];
#pragma unroll
                for (int g = 0; g < MT; ++g)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        // (in place, accumulation registers: the compiler's own moves them around the loop)
                        asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc[g][j]) : "v"(a[g][i]), "v"(x[j]));
            }
        };
        load_x(u0, column(u0));
        int col = column(u0 + 1);
        load_a(u0, 0, a0);
        for (int u = u0; u < u1; ++u) {
#pragma unroll
            for (int i = 0; i < 8; ++i) lds.x[wave][i * 8 + row][chunk ^ (row & 7)] = xr[i];
            if (k0 + 64 > K && k0 + chunk * 8 >= K)  // K % 8 == 0
#pragma unroll
                for (int i = 0; i < 8; ++i) lds.x[wave][i * 8 + row][chunk ^ (row & 7)] = u32x4{0u, 0u, 0u, 0u};
            load_a(u, 1, a1);
            const int next = u < last ? u + 1 : u;  // (the last unit once more, instead of a loop body without loads)
            load_x(next, col);
            col = column(u + 2);
            __builtin_amdgcn_sched_barrier(0);
            multiply(0, a0);
            __builtin_amdgcn_sched_barrier(0);
            load_a(next, 0, a0);
            __builtin_amdgcn_sched_barrier(0);
            multiply(1, a1);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // The last products, before anything reads them: what does depends on this statement (the compiler does not see that the
    // accumulators were written by MFMAs, and would not wait by itself)
    if constexpr (MT == 2)
        asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[1][0]), "+a"(acc[1][1]));
    else
        asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[1][0]), "+a"(acc[1][1]),
                                              "+a"(acc[2][0]), "+a"(acc[2][1]), "+a"(acc[3][0]), "+a"(acc[3][1]));

    // Half of the row tiles at a time: every wave leaves its products, [(g 2 + j) 4 + e] the registers 4 e .. of row tile g and
    // tokens j, adds a quarter of all in wave order and rounds.  D of the MFMA: lane l holds token l % 32, rows
    // 8 e + 4 (l / 32) + 0..3.
    const int m0 = br * BR + strip * (32 * MT);
#pragma unroll
    for (int part = 0; part < 2; ++part) {
        __syncthreads();
#pragma unroll
        for (int g = 0; g < MT / 2; ++g)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const f32x16 &v = acc[part * (MT / 2) + g][j];
                    lds.part[wave][(g * 2 + j) * 4 + e][lane] = f32x4{v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]};
                }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int at = wave * MT + i;
            f32x4 v = lds.part[0][at][lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) v += lds.part[w][at][lane];
            uint32_t o[2];
#pragma unroll
            for (int c = 0; c < 2; ++c)
                o[c] = __builtin_bit_cast(uint16_t, (__bf16)v[2 * c]) | (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)v[2 * c + 1]) << 16;
            *(uint2 *)&out[at / 4 % 2 * 32 + (lane & 31)][at / 8 * 32 + at % 4 * 8 + 4 * (lane >> 5)] = uint2{o[0], o[1]};
        }
        __syncthreads();
        for (int i = tid; i < 64 * 2 * MT; i += 256) {  // eight adjacent outputs of a token
            const int t = i / (2 * MT), r = i % (2 * MT) * 8, m = m0 + part * (16 * MT) + r;
            if (n0 + t < N && m < M) *(u32x4 *)(Y + (n0 + t) * M + m) = *(const u32x4 *)&out[t][r];
        }
    }
}

// Up to 16 NT tokens, 16-byte aligned operands: strips of 16 rows on v_mfma_f32_16x16x32_bf16, otherwise as above.  What bounds a
// decoded batch is the time of a strip: the look-up of its row, of its block columns, A and X, the sum, each behind the other, with
// few lines on the way (18944 x 3584 at 90 %, 16 tokens: 2.5e5 lines of 551 cycles each in 4.9 us, 46 at a time to a compute unit in the mean;
// 3584 x 18944 2.2e5 of 442, 31).  Strips of 32 rows give each compute unit at most one of the 112 of a projection with 28 block-rows, and
// twice the bytes of its longest one.
template <int BR, int NT, int W>
__global__ __launch_bounds__(W * 64) void bcsr_xt_decode_kernel(const int4 *__restrict__ rank_info,
                                                                const int32_t *__restrict__ col_idx,
                                                                const uint16_t *__restrict__ a_packed,
                                                                const uint16_t *__restrict__ X, uint16_t *__restrict__ Y,
                                                                int M, int K, int N, int units_m) {
    constexpr int STRIPS = BR / 16, UK = BR < 64 ? BR : 64, KK = UK / 32, UPB = BR / UK;
    constexpr int PITCH = 20;  // floats per token of a partial tile
    __shared__ __attribute__((aligned(16))) float part[W][NT * 16][PITCH];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // (XCDs and lists as in the strips above)
    const int xcd = blockIdx.x & 7, q = gridDim.x >> 3, r = gridDim.x & 7;
    const int um = xcd * q + (xcd < r ? xcd : r) + (blockIdx.x >> 3);
    const int n_brows = units_m / STRIPS, per = n_brows >> 3, more = n_brows & 7, at = um / STRIPS, strip = um % STRIPS;
    const int list = at < more * (per + 1) ? at / (per + 1) : more + (at - more * (per + 1)) / per;
    const int4 ri = rank_info[list + 8 * (at - list * per - (list < more ? list : more))];
    const int br = ri.x, blk0 = ri.y, n_units = ri.z * UPB;
    const int u0 = n_units * wave / W, u1 = n_units * (wave + 1) / W;

    f32x4 acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (u0 < u1) {
        const int k_l = 8 * (lane >> 4);  // this lane's 8 k of 32
        const uint16_t *x[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            const int t = j * 16 + (lane & 15);
            x[j] = X + (int64_t)(t < N ? t : N - 1) * K;  // tokens past N feed columns that are never stored
        }
        // row 16 strip + lane % 16, k 8 (lane / 16) of 32: groups of 32 rows, 16 k at a time
        const uint16_t *a_lane = a_packed + (int64_t)blk0 * (BR * BR) + (lane >> 5) * (BR * 16) + (strip >> 1) * 512 +
                                 ((lane & 15) + 16 * (strip & 1) + 32 * ((lane >> 4) & 1)) * 8;
        // lane i holds the block column of the wave's i-th block, 64 at a time
        int col_base = u0 / UPB, cols;
        auto load_cols = [&]() __attribute__((always_inline)) {
            const int last = n_units / UPB - 1, p = col_base + lane;
            cols = col_idx[blk0 + (p < last ? p : last)];
        };
        load_cols();
        struct Unit {
            u32x4 a[KK], x[NT][KK];
        };
        auto load = [&](int u, Unit &f) __attribute__((always_inline)) {
            const int p = u / UPB, s = u % UPB;
            if (p - col_base >= 64) {
                col_base = p;
                load_cols();
                asm volatile("" : "+v"(cols));  // as above: of 60 products of 1 to 16 tokens 0.998 of the time in the mean, 0.98 to 1.04
            }
            const u32x4 *a = (const u32x4 *)(a_lane + (int64_t)p * (BR * BR) + s * (UK * BR));
#pragma unroll
            for (int i = 0; i < KK; ++i) f.a[i] = a[i * (BR * 4)];
            const int k0 = __builtin_amdgcn_readlane(cols, p - col_base) * BR + s * UK + k_l;
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
                for (int i = 0; i < KK; ++i) {
                    const int k = k0 + i * 32;  // K % 8 == 0; k past K count as zeros
                    const u32x4 v = *(const u32x4 *)(x[j] + (k < K ? k : 0));
                    f.x[j][i] = k < K ? v : u32x4{0u, 0u, 0u, 0u};
                }
        };
        auto multiply = [&](const Unit &f) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < KK; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.a[i]),
                                                                     __builtin_bit_cast(bf16x8, f.x[j][i]), acc[j], 0, 0, 0);
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

    // D: lane l holds token l % 16, rows 4 (l / 16) + 0..3
#pragma unroll
    for (int j = 0; j < NT; ++j) *(f32x4 *)&part[wave][j * 16 + (lane & 15)][4 * (lane >> 4)] = acc[j];
    __syncthreads();
    const int m0 = br * BR + strip * 16;
    for (int i = tid; i < NT * 16 * 8; i += W * 64) {  // two adjacent outputs of a token
        const int t = i / 8, c = i % 8 * 2;
        float s0 = part[0][t][c], s1 = part[0][t][c + 1];
#pragma unroll
        for (int w = 1; w < W; ++w) {
            s0 += part[w][t][c];
            s1 += part[w][t][c + 1];
        }
        const uint32_t lo = __builtin_bit_cast(uint16_t, (__bf16)s0), hi = __builtin_bit_cast(uint16_t, (__bf16)s1);
        if (t < N && m0 + c < M) *(uint32_t *)(Y + (int64_t)t * M + m0 + c) = lo | (hi << 16);  // M % 8 == 0
    }
}

// ---- host side ------------------------------------------------------------------------------------
// false: too many rows for a launch
template <int BR, int MT, int NT, int W, int UK>
static bool launch_strip(const asp_handle *h, const void *X, void *Y, int64_t N, bool vec, hipStream_t stream) {
    const int units_m = (int)h->n_brows * (BR / 32 / MT);
    if (!launch_fits(units_m, W * 64)) return false;
    // as many tokens at a time as the threads of a launch allow
    const int64_t step = ((1ll << 32) - 1) / ((int64_t)units_m * W * 64) * (32 * NT);
    for (int64_t first = 0; first < N; first += step) {
        const int64_t tokens = std::min(step, N - first);
        const uint16_t *x = (const uint16_t *)X + first * h->k;
        uint16_t *y = (uint16_t *)Y + first * h->m;
        dim3 grid((unsigned)(units_m * ceil_div(tokens, 32 * NT))), block(W * 64);
#define ASP_STRIP(VEC)                                                                                                       \
    hipLaunchKernelGGL((bcsr_xt_strip_kernel<BR, MT, NT, W, UK, VEC>), grid, block, 0, stream, (const int4 *)h->d_rank_info, \
                       h->d_col_idx, (const uint16_t *)h->d_values, x, y, (int)h->m, (int)h->k, tokens, units_m)
        if (vec) ASP_STRIP(true);
        else ASP_STRIP(false);
#undef ASP_STRIP
    }
    return true;
}

template <int BR, int NT, int W>
static bool launch_decode(const asp_handle *h, const void *X, void *Y, int64_t N, hipStream_t stream) {
    const int64_t units_m = h->n_brows * (BR / 16);
    if (!launch_fits(units_m, W * 64)) return false;
    hipLaunchKernelGGL((bcsr_xt_decode_kernel<BR, NT, W>), dim3((unsigned)units_m), dim3(W * 64), 0, stream,
                       (const int4 *)h->d_rank_info, h->d_col_idx, (const uint16_t *)h->d_values, (const uint16_t *)X,
                       (uint16_t *)Y, (int)h->m, (int)h->k, (int)N, (int)units_m);
    return true;
}

template <int BR, int MT>
static bool launch_staged(const asp_handle *h, const void *X, void *Y, int64_t N, hipStream_t stream) {
    const int64_t units_m = h->n_brows * (BR / 32 / MT), n64 = ceil_div(N, 64);
    if (!launch_fits(units_m * n64, 256) || h->k >= (1ll << 25)) return false;  // (offsets of 64 tokens are 32-bit)
    hipLaunchKernelGGL((bcsr_xt_staged_kernel<BR, MT>), dim3((unsigned)(units_m * n64)), dim3(256), 0, stream,
                       (const int4 *)h->d_rank_info, h->d_col_idx, (const uint16_t *)h->d_values, (const uint16_t *)X,
                       (uint16_t *)Y, (int)h->m, (int)h->k, N, (int)units_m);
    return true;
}

// Whether 16-byte aligned operands go through the staged strips, and how high these are: 0, or 2 or 4 row tiles.  Their start and
// end take 0.6 us more than those of the other strips, which wins from 7 pieces of 64 outputs x 64 k x 64 tokens to a compute unit on
// (counted in 32 tokens, what the other strips pad to): of 466 products of 64- and 128-row blocks at 80 to 95 %, 33 to 6000 tokens,
// timed in a captured graph, the 105 with less took 1.04 times as long in the mean, up to 1.21 (6656 x 2816, 71 tokens 5.4 / 6.5 us),
// the others 0.85.  Not below three 64-row strips to four compute units, where eight waves to a strip are the better ones
// (3584 x 18944, 90 %, 128-row blocks, 64 / 128 / 256 tokens 9.5 / 11.8 / 18.7 us, staged 11.4 / 11.6 / 12.9; 1664 x 3904, 80 %, 287
// tokens 9.4 / 10.6), and with less than three units of 64 k a block-row, where the ends of the strips are all there is (2944 x 1280,
// 90 %, 64-row blocks, 4185 tokens 18.8 / 21.5).  Nor where block-rows are about as long as each other and some compute units would
// take a second strip while the 32-token strips are no more than two to each: the launch is as long as those few (3520 x 6208,
// 80 %, 263 tokens, 280 strips 13.7 / 15.0 us, 90 % 9.5 / 10.3; 6336 x 10560, 143 tokens, 297 strips 17.9 / 18.6).  Of 600 products
// drawn after these lines were, 350 take these strips: 0.84 of the others' time in the mean, 1.10 at worst (4288 x 7424, 90 %,
// geometric rows, 150 tokens 9.0 / 9.9).
// Three 64-row strips fit a compute unit, two of 128 rows, which read X once instead of twice: better where rows are long
// enough (6 blocks) to be bound by that and there are more 64-row strips than places (3584 x 18944, 256 / 768 / 1024 / 2048 tokens,
// 64 and 128 rows 12.9 / 17.0, 28.9 / 30.8, 35.4 / 30.9, 67 / 55 us; 18944 x 3584, three blocks a row, 512 / 1024 tokens
// 22.3 / 22.8, 39.2 / 39.8).
int bcsr_xt_staged_strips(const asp_handle *h, int64_t N) {
    const int64_t cus = h->n_cus > 0 ? h->n_cus : 256, rows = h->n_brows * (h->b_row / 64);
    const int64_t strips = rows * ceil_div(N, 64), strips_32 = rows * ceil_div(N, 32);
    if (h->b_row < 64 || N <= 32 || 4 * strips < 3 * cus || h->n_units * (h->b_row / 64) < 3 * h->n_brows) return 0;
    if (h->n_units * (h->b_row / 64) * (h->b_row / 64) * ceil_div(N, 32) < 14 * cus) return 0;
    if (strips > cus && strips_32 <= 2 * cus && h->hb.max_blocks * h->n_brows <= 3 * h->n_units) return 0;
    return h->b_row == 128 && strips > 3 * cus && h->n_units >= 6 * h->n_brows ? 4 : 2;
}

// Whether up to 32 tokens go through the strips of 16 rows, and by how many waves each: 0, 4 or 8.  us in a captured graph, the other
// strips / 4 / 8 waves: 18944 x 3584, 90 %, 128-row blocks, 16 tokens 5.28 / 4.79 / 4.76, 1 token 4.79 / 3.53 / 4.02; 3584 x 18944,
// 16 tokens 6.9 / 5.5 / 5.35; geometric rows, 18944 x 9472, 16 tokens 14.1 / 12.0 / 10.4; of 77 products of 64- and 128-row blocks up to
// 16 tokens 0.84 in the mean.
// Eight waves where a block-row has 24 units of 64 k (80 %, 18944 x 3584, up to 20: 6.7 / 7.0) or strips are few.  Not with 32-row
// blocks and more than two strips to a compute unit: a 32-row block has a strip of its own already, and 16-row ones read X twice
// (18944 x 3584, 16 tokens 4.62 / 4.73).  Nor where block-rows are long and alike and some compute units have a strip more than the
// others (8960 x 18944, 80 %, 64-row, 560 strips on 256 units 14.4 / 15.9).  Above 16 tokens only where the others leave compute units
// idle (3584 x 18944, 32 tokens 8.8 / 8.0; 18944 x 3584 5.8 / 6.9).
static int decode_waves(const asp_handle *h, int64_t N) {
    const int64_t cus = h->n_cus > 0 ? h->n_cus : 256, strips = h->n_brows * (h->b_row / 16);
    if (N > 16) return h->b_row >= 64 && strips <= cus ? 8 : 0;
    if (h->b_row == 32) return strips <= 2 * cus ? 8 : 0;
    const bool alike = h->hb.max_blocks * h->n_brows <= 2 * h->n_units, long_rows = h->n_units * (h->b_row / 64) >= 24 * h->n_brows;
    if (strips > cus && alike && long_rows && 4 * ceil_div(strips, cus) * cus > 5 * strips) return 0;
    return h->hb.max_blocks * (h->b_row / 64) >= 24 || 4 * strips <= 5 * cus ? 8 : 4;
}

// Shape of the wave tiles of the other strips: the largest that still gives the chip enough of them, since a larger one reads fewer bytes
// per MFMA.  18944 x 3584 (gate) and 3584 x 18944 (down), 90 % sparse, us a call, tiles of 32 x 32 / 64 x 32 / 64 x 64 /
// 128 x 64: gate at 64 tokens 8.3 / 7.7 / 8.6 / 10.3, at 256 22 / 19 / 18 / 20; down at 64 tokens 9.3 / 10.9 / 17 / 21,
// at 256 22 / 18 / 19 / 23, at 768 52 / 39 / 43 / 33.  128 x 64 needs block-rows long enough that every wave of the
// workgroup gets blocks: 512 tokens 31 / 24 us (64 x 64 / 128 x 64) with 15 blocks a row, 29 / 34 us with 3.
template <int BR>
static bool launch_strips(const asp_handle *h, const void *X, void *Y, int64_t N, bool vec, hipStream_t stream) {
    const int64_t cus = h->n_cus > 0 ? h->n_cus : 256, n32 = ceil_div(N, 32), n64 = ceil_div(N, 64);
    if (vec && N <= 32) {
        const int waves = decode_waves(h, N);
        if (waves == 8 && N <= 16 && launch_decode<BR, 1, 8>(h, X, Y, N, stream)) return true;
        if constexpr (BR >= 64) {  // (32-row blocks: eight waves, up to 16 tokens)
            if (waves == 4 && launch_decode<BR, 1, 4>(h, X, Y, N, stream)) return true;
            if (waves == 8 && N > 16 && launch_decode<BR, 2, 8>(h, X, Y, N, stream)) return true;
        }
    }
    if constexpr (BR == 128) {
        const int staged = vec ? bcsr_xt_staged_strips(h, N) : 0;
        if (staged != 0 && (staged == 4 ? launch_staged<BR, 4>(h, X, Y, N, stream) : launch_staged<BR, 2>(h, X, Y, N, stream)))
            return true;
        // (or too many rows for a launch of 64-row strips)
        if ((h->n_units >= 8 * h->n_brows && h->n_brows * n64 >= cus * 3 / 4) || h->n_brows >= (1 << 23))
            return launch_strip<BR, 4, 2, 4, 32>(h, X, Y, N, vec, stream);
    }
    if constexpr (BR == 64) {
        if (vec && bcsr_xt_staged_strips(h, N) != 0 && launch_staged<BR, 2>(h, X, Y, N, stream)) return true;
    }
    if constexpr (BR >= 64) {
        const int64_t strips = h->n_brows * (BR / 64);
        if (strips * n64 >= 3 * cus) return launch_strip<BR, 2, 2, 4, 32>(h, X, Y, N, vec, stream);
        if (strips * n32 >= cus / 2) {
            if (strips * n32 >= cus * 5 / 4) return launch_strip<BR, 2, 1, 4, 64>(h, X, Y, N, vec, stream);
            return launch_strip<BR, 2, 1, 8, 64>(h, X, Y, N, vec, stream);
        }
    }
    if constexpr (BR == 32) {  // (with larger blocks there are fewer than 256 here)
        if (h->n_brows * n32 > 2 * cus) return launch_strip<BR, 1, 1, 4, 64>(h, X, Y, N, vec, stream);
    }
    return launch_strip<BR, 1, 1, 8, 64>(h, X, Y, N, vec, stream);
}

// any K, M, N <= ASP_MAX_N and alignment; vec: 16-byte aligned X and Y, K % 8 == 0, M % 8 == 0
static bool launch_any_strips(const asp_handle *h, const void *X, void *Y, int64_t N, bool vec, hipStream_t stream) {
    if (h->b_row == 128) return launch_strips<128>(h, X, Y, N, vec, stream);
    if (h->b_row == 64) return launch_strips<64>(h, X, Y, N, vec, stream);
    return launch_strips<32>(h, X, Y, N, vec, stream);
}

// Kernel without matrix cores (a benchmarking switch, for the comparison): one thread per (token, quarter of the
// block-row's outputs), fp32 multiply-adds over the stored blocks in order.  grid = (block-rows, ceil(N / 64)), 256 threads.
template <int BR>
__global__ __launch_bounds__(256) void bcsr_xt_generic_kernel(const int32_t *__restrict__ block_row_ptr,
                                                              const int32_t *__restrict__ block_col_idx,
                                                              const uint16_t *__restrict__ a_packed,
                                                              const uint16_t *__restrict__ X, uint16_t *__restrict__ Y,
                                                              int M, int K, int64_t N) {
    constexpr int RPT = BR / 4;  // outputs per thread
    const int br = blockIdx.x, rg = threadIdx.x >> 6;
    const int64_t n = (int64_t)blockIdx.y * 64 + (threadIdx.x & 63);
    if (n >= N) return;
    float acc[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) acc[r] = 0.f;
    const uint16_t *x = X + n * K;
    for (int p = block_row_ptr[br]; p < block_row_ptr[br + 1]; ++p) {
        const int k0 = block_col_idx[p] * BR;
        const uint16_t *blk = a_packed + (int64_t)p * BR * BR;
        for (int k = 0; k < BR && k0 + k < K; ++k) {
            const float xv = __uint_as_float((uint32_t)x[k0 + k] << 16);
#pragma unroll
            for (int r = 0; r < RPT; ++r) {
                const int row = rg * RPT + r;
                // fragment order: [16-wide k slice][group of 32 rows][lane = row % 32 + 32 * (k % 16 / 8)][k % 8]
                const int idx = (((k >> 4) * (BR / 32) + (row >> 5)) * 64 + (row & 31) + 32 * ((k & 15) >> 3)) * 8 + (k & 7);
                acc[r] = fmaf(__uint_as_float((uint32_t)blk[idx] << 16), xv, acc[r]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
        const int m = br * BR + rg * RPT + r;
        if (m < M) {
            // round to nearest even (inputs are finite sums; NaN payloads are not preserved)
            uint32_t u = __float_as_uint(acc[r]);
            u += 0x7FFFu + ((u >> 16) & 1u);
            Y[n * M + m] = (uint16_t)(u >> 16);
        }
    }
}

__global__ __launch_bounds__(256) void bcsr_fill_zero_kernel(uint16_t *__restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0;
}

// Which kernel: the one with the shortest estimate, in us on 256 compute units.  A ring kernel's launch takes as long as
// its longest block-row at the pace of a lone tile plus all its work at the pace of the full chip; the strip kernel,
// which splits the K loop, takes about 4 us plus its work.  Costs per K slice of 32, fitted to 18944 x 3584, 3584 x 18944
// and 4096 x 4096 at 90 %, 1 to 8192 tokens, when the ring kernel walked groups of four (128, 64) or two (32) column tiles.  Of
// 240 products of ten matrices, 128 to 3072 tokens, the choice is now in the mean 1.01 (128-row), 1.02 (64) and 1.06 (32)
// times slower than the better kernel, at worst 1.3, 1.2 and 1.9 (32-row, 1024 x 1024 at 80 %, 768 tokens, ring 8.2, strips 4.3 us):
struct XtCost {
    double slice_alone[3], slice[3];  // tiles 64, 128, 256 tokens wide
    double strip;                     // per stored element and token
};
static XtCost xt_cost(int b) {
    if (b == 128) return XtCost{{0.40, 0.53, 0.75}, {0.25, 0.30, 0.44}, 6.5e-9};
    if (b == 64) return XtCost{{0.44, 0.50, 0.61}, {0.14, 0.27, 0.41}, 6.5e-9};
    return XtCost{{0.38, 0.51, 0.70}, {0.13, 0.17, 0.37}, 12e-9};
}

asp_status_t bcsr_spmm_xt_launch(const asp_handle *h, const void *X, void *Y, int64_t N, hipStream_t stream) {
    const double cus = h->n_cus > 0 ? h->n_cus : 256;
    if (h->n_units == 0) {
        hipLaunchKernelGGL(bcsr_fill_zero_kernel, dim3(1024), dim3(256), 0, stream, (uint16_t *)Y, N * h->m);
    } else if (switches().xt_generic) {
        dim3 grid((unsigned)h->n_brows, (unsigned)ceil_div(N, 64)), block(256);
#define ASP_XT_GENERIC(BR)                                                                                          \
    hipLaunchKernelGGL(bcsr_xt_generic_kernel<BR>, grid, block, 0, stream, h->d_row_ptr, h->d_col_idx,              \
                       (const uint16_t *)h->d_values, (const uint16_t *)X, (uint16_t *)Y, (int)h->m, (int)h->k, N)
        if (h->b_row == 128) ASP_XT_GENERIC(128);
        else if (h->b_row == 64) ASP_XT_GENERIC(64);
        else ASP_XT_GENERIC(32);
#undef ASP_XT_GENERIC
    } else {
        const bool vec = (((uintptr_t)X | (uintptr_t)Y) & 15) == 0 && h->k % 8 == 0 && h->m % 8 == 0;
        const bool tiles_ok = vec && N < (1ll << 25) && h->k < (1ll << 22);
        // the kernel for 128 x 512 tiles, once there are 1.5 of them per compute unit (at 0.75 / 1 / 1.75 per unit: down
        // 95 / 89 / 127 us, the ring kernel 76 / 82 / 126)
        const int64_t wide_rows = !bcsr_wide_capable(h) ? 0 : h->has_comp ? h->hc.n_nonempty : h->hb.n_nonempty;
        if (tiles_ok && 2 * wide_rows * ceil_div(N, 512) >= 3 * (int64_t)cus) {
            bcsr_wide_xt_launch(h, X, Y, N, stream);
        } else {
            const XtCost c = xt_cost(h->b_row);
            const double slices = (double)h->n_units * (h->b_row / 32), longest = (double)h->hb.max_blocks * (h->b_row / 32);
            const double work = (double)h->n_units * h->b_row * h->b_row * (double)N * 256 / cus;
            double best = 4.0 + c.strip * work, ring_at_least = 0.0;
            int bn = 0;
            for (int i = 0; i < (h->b_row == 32 ? 2 : 3) && tiles_ok; ++i) {  // (256 wide never pays with 32 rows)
                const double alone = c.slice_alone[i] * longest, all = c.slice[i] * slices * (double)ceil_div(N, 64 << i) / cus;
                if (alone + all < best) best = alone + all, bn = 64 << i, ring_at_least = std::max(alone, all);
            }
            // The staged strips are up to 1.8 times faster than those that the estimate was fitted to.  Where the ring kernel
            // is said to be faster than those, it takes between the longer of its two terms and their sum, and stays where the
            // staged strips are not below the former (2688 x 4352, 80 %, geometric rows, 5994 tokens ring 54, staged 66 us).
            const int staged = vec ? bcsr_xt_staged_strips(h, N) : 0;
            const double per_strip = h->b_row == 64 ? 5.2e-9 : staged == 4 ? 4.0e-9 : 4.4e-9;
            if (staged && 4.0 + 4e-10 * (double)h->m * (double)N * 256 / cus + per_strip * work < ring_at_least) bn = 0;
            BcsrPlan p = {bn, bn ? (int32_t)ceil_div(N, bn) : 0, 1, 0};
            p.workgroups = h->n_brows * p.n_tiles;
            if (bn != 0 && p.workgroups * 8 < (1ll << 31)) bcsr_dma_xt_launch(h, X, Y, N, p, stream);
            else if (launch_any_strips(h, X, Y, N, vec, stream)) {}
            else if (tiles_ok && wide_rows > 0) bcsr_wide_xt_launch(h, X, Y, N, stream);
            else return fail(ASP_ERR_UNSUPPORTED, "too many output tiles");
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ASP_ERR_HIP, std::string("BCSR K-contiguous kernel launch: ") + hipGetErrorString(e));
    return ASP_OK;
}

}  // namespace asp

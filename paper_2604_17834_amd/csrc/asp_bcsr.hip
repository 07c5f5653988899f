// BCSR x dense SpMM for gfx950: dispatch (tile-width rule of the paper's Section IV-C) and the
// register-staged kernel.
//
// The register-staged kernel is the synchronous-copy design (the analogue of the paper's Section III-A
// kernel with cooperative loads, plus one slice of prefetch): global loads go to VGPRs, then to LDS.  It
// serves operands whose rows are not 16-byte aligned (16-byte accesses at element alignment, which a direct-to-LDS load
// does not take) and stays selectable for comparison runs; aligned operands take the direct-to-LDS ring kernel in
// asp_bcsr_dma.hip.
//
// One workgroup computes one (block-row, N-tile) output tile of b_row x BN: it walks the stored blocks
// of its block-row (Section II-C), and for each K slice of a block stages the A slice and the matching
// rows of B through LDS, double buffered, while the previous slice is multiplied on the matrix cores
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation).
//
// Operand layouts
//   A  blocks are pre-permuted on the host into MFMA fragment order, so a slice is one contiguous,
//      fully coalesced run in memory and in LDS (ds_read_b128, lane-linear).
//   B  is row-major K x N: a K slice lands in LDS row by row (pitch BN*2+64 bytes so the four rows of a
//      transposing read fall in disjoint banks) and is read with ds_read_b64_tr_b16, which hands every
//      lane 4 consecutive k of one column -- the K-contiguous operand the MFMA wants.
//   The MFMA is issued with the operands swapped (B fragment first), so each lane ends with 4
//   consecutive columns of one output row: the tile is rounded to bf16, passed through LDS and written
//   to C with 16-byte row-contiguous stores.
#include <cstdlib>
#include <cstring>

#include "asp_bcsr_pipe.h"

namespace asp {

template <int BR, int BC, int BN, int WM, int WN, bool VEC>
struct BcsrCfg {
    static constexpr int KS = 32;                  // k rows per pipeline stage
    static constexpr int NT = WM * WN * 64;        // threads
    static constexpr int TM = BR / WM;             // wave tile rows
    static constexpr int TN = BN / WN;             // wave tile columns
    static constexpr int MT = TM / 32;             // 32x32 MFMA tiles per wave, along M
    static constexpr int NTL = TN / 32;            //   and along N
    static constexpr int KK = KS / 16;             // MFMA k steps per stage
    static constexpr int SPB = BC / KS;            // stages per block
    static constexpr int A_STAGE = BR * KS * 2;    // bytes
    static constexpr int PB = BN * 2 + 64;         // LDS pitch of a B row, bytes
    static constexpr int B_STAGE = KS * PB;
    static constexpr int STAGE = A_STAGE + B_STAGE;
    static constexpr int A_CHUNKS = A_STAGE / 16;  // 16-byte units per stage
    static constexpr int B_CPR = BN / 8;           // 16-byte units per B row
    static constexpr int B_CHUNKS = KS * B_CPR;
    static constexpr int A_LD = (A_CHUNKS + NT - 1) / NT;
    static constexpr int B_LD = (B_CHUNKS + NT - 1) / NT;
    static constexpr int C_PITCH = TN * 2 + 16;    // epilogue staging pitch per wave, bytes
    static constexpr int C_WAVE = TM * C_PITCH;
    static constexpr int LDS_BYTES = (2 * STAGE > WM * WN * C_WAVE) ? 2 * STAGE : WM * WN * C_WAVE;
    static_assert(TM % 32 == 0 && TN % 32 == 0, "wave tile must be made of 32x32 MFMA tiles");
    static_assert(BC % KS == 0, "block width must be a multiple of the stage depth");
};

template <int BR, int BC, int BN, int WM, int WN, bool VEC>
__global__ __launch_bounds__(WM *WN * 64, 2) void bcsr_spmm_kernel(
    const int32_t *__restrict__ block_row_ptr, const int32_t *__restrict__ block_col_idx,
    const uint16_t *__restrict__ a_packed, const uint16_t *__restrict__ B, uint16_t *__restrict__ C, int M, int K,
    int N, int n_brows, const int32_t *__restrict__ order, XcdRuns runs) {
    using Cfg = BcsrCfg<BR, BC, BN, WM, WN, VEC>;
    constexpr int NT = Cfg::NT, KS = Cfg::KS, MT = Cfg::MT, NTL = Cfg::NTL;
    __shared__ __attribute__((aligned(16))) uint8_t lds[Cfg::LDS_BYTES];

    // Workgroups are handed to the 8 XCDs round-robin by flat id.  Each XCD gets a contiguous run of
    // the (N-tile major, block-row minor) tile order so that the workgroups sharing one XCD's L2 work
    // on the same column slab of B.  With an order, longest block-row first, the runs weigh the same: a compute unit takes
    // the next workgroup when one ends, so the last ones should be short.
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int u = runs.start[xcd] + local;
    if (u >= runs.start[xcd + 1]) return;
    const int nt = __builtin_amdgcn_readfirstlane(u / n_brows), pos = u - nt * n_brows;
    const int br = __builtin_amdgcn_readfirstlane(order ? order[pos] : pos);
    // Rows that are not 16-byte aligned: the last column tile moves left so that it ends at N, and its loads have no case of a
    // row's end.  (18944 x 3584 at 90 %, N = 4093, 128 / 64 / 32-row blocks 134 / 148 / 199 -> 113 / 125 / 173 us with plain loads
    // in every slice that does not reach past K; two slices ahead instead of one: 126 / 141 / 192.)  Where N does not fill one tile, chunks
    // of 8 columns that would pass N end there instead.
    const int n_own = nt * BN, n0 = !VEC && N >= BN && n_own > N - BN ? N - BN : n_own;
    const bool inner = N >= 8;
    auto chunk_col = [&](int col) __attribute__((always_inline)) { return inner && col > N - 8 ? N - 8 : col; };

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;

    const int blk0 = block_row_ptr[br], blk1 = block_row_ptr[br + 1];
    const int T = (blk1 - blk0) * Cfg::SPB;  // pipeline stages of this tile

    f32x16 acc[MT][NTL];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NTL; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    struct Stage {
        u32x4 a[Cfg::A_LD], b[Cfg::B_LD];
    };
    auto load_stage = [&](int t, Stage &f) __attribute__((always_inline)) {
        const int p = blk0 + t / Cfg::SPB, s = t % Cfg::SPB;
        const u32x4 *asrc = (const u32x4 *)(a_packed + (int64_t)p * (BR * BC) + (int64_t)s * (BR * KS));
#pragma unroll
        for (int i = 0; i < Cfg::A_LD; ++i) {
            int c = i * NT + tid;
            if (Cfg::A_CHUNKS % NT == 0 || c < Cfg::A_CHUNKS) f.a[i] = asrc[c];
        }
        const int krow0 = block_col_idx[p] * BC + s * KS;
        if (inner && krow0 + KS <= K) {
            const uint16_t *src = B + (int64_t)krow0 * N;
#pragma unroll
            for (int i = 0; i < Cfg::B_LD; ++i) {
                const int c = i * NT + tid;
                if (Cfg::B_CHUNKS % NT == 0 || c < Cfg::B_CHUNKS) {
                    const uint16_t *at = src + (int64_t)(c / Cfg::B_CPR) * N + chunk_col(n0 + c % Cfg::B_CPR * 8);
                    f.b[i] = VEC ? *(const u32x4 *)at : *(const u32x4_a2 *)at;
                }
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < Cfg::B_LD; ++i) {
            int c = i * NT + tid;
            if (Cfg::B_CHUNKS % NT == 0 || c < Cfg::B_CHUNKS) {
                int r = c / Cfg::B_CPR, cc = c % Cfg::B_CPR;
                int krow = krow0 + r, col = chunk_col(n0 + cc * 8);
                u32x4 v = {0u, 0u, 0u, 0u};
                if (krow < K && col < N) {  // rows past K belong to the zero padding of the last block column
                    const uint16_t *row = B + (int64_t)krow * N;
                    v = VEC ? *(const u32x4 *)(row + col) : load_tail8(row, col, N);
                }
                f.b[i] = v;
            }
        }
    };
    auto store_stage = [&](int buf, const Stage &f) __attribute__((always_inline)) {
        uint8_t *sa = lds + buf * Cfg::STAGE, *sb = sa + Cfg::A_STAGE;
#pragma unroll
        for (int i = 0; i < Cfg::A_LD; ++i) {
            int c = i * NT + tid;
            if (Cfg::A_CHUNKS % NT == 0 || c < Cfg::A_CHUNKS) *(u32x4 *)(sa + c * 16) = f.a[i];
        }
#pragma unroll
        for (int i = 0; i < Cfg::B_LD; ++i) {
            int c = i * NT + tid;
            if (Cfg::B_CHUNKS % NT == 0 || c < Cfg::B_CHUNKS) {
                int r = c / Cfg::B_CPR, cc = c % Cfg::B_CPR;
                *(u32x4 *)(sb + r * Cfg::PB + cc * 16) = f.b[i];
            }
        }
    };
    auto compute_stage = [&](int buf) {
        const uint8_t *sa = lds + buf * Cfg::STAGE, *sb = sa + Cfg::A_STAGE;
#pragma unroll
        for (int kk = 0; kk < Cfg::KK; ++kk) {
            bf16x8 af[MT], bfr[NTL];
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                int mtg = wm * MT + i;
                af[i] = *(const bf16x8 *)(sa + ((kk * (BR / 32) + mtg) * 64 + lane) * 16);
            }
            // transposing read: lane i of a 16-lane group addresses row i/4, 4 columns at 4*(i%4);
            // it receives the 4 rows of column (i) of the group's 16 columns
            const int krow = kk * 16 + 8 * (lane >> 5) + ((lane & 15) >> 2);
#pragma unroll
            for (int j = 0; j < NTL; ++j) {
                int col = wn * Cfg::TN + j * 32 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
                const uint8_t *p0 = sb + krow * Cfg::PB + col * 2;
                short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (short4v __attribute__((address_space(3))) *)(p0));
                short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (short4v __attribute__((address_space(3))) *)(p0 + 4 * Cfg::PB));
                short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                bfr[j] = __builtin_bit_cast(bf16x8, both);
            }
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NTL; ++j)
                    // operands swapped: D[n][m] = sum_k B[k][n] * A[m][k]
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
        }
    };

    if (T > 0) {
        Stage f;
        load_stage(0, f);
        store_stage(0, f);
        __syncthreads();
        for (int t = 0; t < T; ++t) {
            const int buf = t & 1;
            if (t + 1 < T) load_stage(t + 1, f);  // global loads fly while this stage is multiplied
            compute_stage(buf);
            if (t + 1 < T) store_stage(buf ^ 1, f);
            __syncthreads();
        }
    }

    // ---- epilogue: fp32 -> bf16, through LDS, 16-byte row stores --------------------------------
    uint8_t *sc = lds + wave * Cfg::C_WAVE;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NTL; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 v = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                bf16x4 hv = __builtin_convertvector(v, bf16x4);  // round to nearest even
                int mrow = i * 32 + (lane & 31);
                int ncol = j * 32 + 8 * q + 4 * (lane >> 5);
                *(bf16x4 *)(sc + mrow * Cfg::C_PITCH + ncol * 2) = hv;
            }
    __syncthreads();
    constexpr int CPR = Cfg::TN / 8;   // 16-byte units per staged row
    constexpr int RPI = 64 / CPR;      // rows per wave instruction
#pragma unroll
    for (int it = 0; it < Cfg::TM / RPI; ++it) {
        int row = it * RPI + lane / CPR, cc = lane % CPR;
        uint4 v = *(const uint4 *)(sc + row * Cfg::C_PITCH + cc * 16);
        int grow = br * BR + wm * Cfg::TM + row;
        const int own = n0 + wn * Cfg::TN + cc * 8, gcol = chunk_col(own);
        if (grow < M && own < N && own + 8 > n_own) {  // (a column of two tiles or chunks gets the same bits from both)
            uint16_t *dst = C + (int64_t)grow * N + gcol;
            if (VEC) {
                *(uint4 *)dst = v;
            } else if (gcol + 8 <= N) {
                *(u32x4_a2 *)dst = u32x4{v.x, v.y, v.z, v.w};
            } else {
                uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (gcol + e < N) dst[e] = (uint16_t)(w[e >> 1] >> (16 * (e & 1)));
            }
        }
    }
}

// ---- host side ------------------------------------------------------------------------------------

// Section IV-C: take the widest tile that divides N; when none does, the one that pads N the least.
static int choose_bn(int64_t N, const int *cand, int n) {
    int best = -1;
    for (int i = 0; i < n; ++i)
        if (N % cand[i] == 0 && cand[i] > best) best = cand[i];
    if (best > 0) return best;
    int64_t best_pad = -1;
    for (int i = 0; i < n; ++i) {
        int64_t pad = ceil_div(N, cand[i]) * cand[i];
        if (best_pad < 0 || pad < best_pad || (pad == best_pad && cand[i] > best)) {
            best_pad = pad;
            best = cand[i];
        }
    }
    return best;
}

// Section IV-C with both effects priced: a wider tile does more work per loaded A tile (cost per column falls
// with the width), a tile that does not divide N computes on padding.  Least padded width x cost; ties: wider.
static int choose_bn_weighted(int64_t N, const int *cand, const int *cost, int n) {
    int best = -1;
    int64_t best_total = -1;
    for (int i = 0; i < n; ++i) {
        const int64_t total = ceil_div(N, cand[i]) * cand[i] * cost[i];
        if (best < 0 || total < best_total || (total == best_total && cand[i] > best)) {
            best_total = total;
            best = cand[i];
        }
    }
    return best;
}

BcsrPlan bcsr_plan(const asp_handle *h, int64_t N, bool aligned) {
    BcsrPlan p;
    if (h->dtype == ASP_DT_F32) {  // (the fp32 kernel takes narrower tiles where a launch is small)
        static const int cand32[2] = {128, 256};
        p.vectorized = (aligned && N % 4 == 0) ? 1 : 0;
        p.bn = p.vectorized ? choose_bn(N, cand32, 2) : 128;
        p.n_tiles = (int32_t)ceil_div(N, p.bn);
        p.workgroups = h->n_brows * p.n_tiles;
        return p;
    }
    p.vectorized = (aligned && N % 8 == 0) ? 1 : 0;
    static const int cand[4] = {64, 128, 256, 512};
    // time per column of a tile of that width relative to a 512-wide one, in 1/64 (measured on the 128x128-block
    // projection workload at steady clocks: 0.529 / 0.376 / 0.290 / 0.251 ms for the same work)
    static const int cost[4] = {135, 96, 74, 64};
    const int env_bn = switches().bcsr_bn;  // benchmarking switch: caps the tile width
    if (!p.vectorized) {
        p.bn = 64;
    } else {
        // 512-wide tiles (one resident workgroup per compute unit) exist for 128x128 blocks and only pay
        // when every compute unit gets at least one tile
        int ncand = 3;
        const int64_t cus = h->n_cus > 0 ? h->n_cus : 256;
        // (smaller blocks: through the composite form with 128-row super-rows, when the handle has one)
        if (bcsr_wide_capable(h) && N < (1ll << 25)) {
            const int64_t rows = h->has_comp ? h->hc.n_nonempty : h->hb.n_nonempty > 0 ? h->hb.n_nonempty : h->n_brows;
            if (rows * ceil_div(N, 512) >= cus) ncand = 4;
        }
        if (env_bn == 64 || env_bn == 128 || env_bn == 256)
            while (ncand > 1 && cand[ncand - 1] > env_bn) --ncand;
        p.bn = choose_bn_weighted(N, cand, cost, ncand);
        // A launch with fewer tiles than compute units leaves part of the chip idle and every tile runs alone at
        // the latency of its K loop: take the next narrower width while that is so (the 28 block-rows of the case
        // study's down projection at N = 1024: 0.079 / 0.060 / 0.043 ms with 256- / 128- / 64-wide tiles).
        const int64_t rows_ne = h->hb.n_nonempty > 0 ? h->hb.n_nonempty : h->n_brows;
        while (p.bn > 64 && p.bn < 512 && rows_ne * ceil_div(N, p.bn) < cus) p.bn /= 2;
    }
    p.n_tiles = (int32_t)ceil_div(N, p.bn);
    p.workgroups = (p.bn == 512 && h->has_comp ? h->c_n_brows : h->n_brows) * p.n_tiles;
    return p;
}

// Runs of the XCDs over the register-staged kernel's tiles.  True: in the order longest block-row first, runs of equal weight;
// false: in the stored order, runs of as many tiles.
// Longest first where the tiles are more than the 4 or so that a compute unit holds at once (us, as stored / longest
// first: 4519 x 8812 at 90 %, 128-row, N = 4037 105 / 90; 1869 x 3209 at 50 %, 32-row, N = 4093 112 / 100; geometric lengths,
// 6593 x 6251 at 95 %, 64-row, N = 1437 53 / 45; with fewer tiles 8960 x 8011 at 75 %, 128-row, N = 535 75 / 80).
// Not where one XCD would get half of all tiles, next to nothing but empty block-rows to clear: the stored order then, an eighth
// of the tiles each (in the order of length the first eighth holds the longest ones).
bool register_staged_runs(const HostBcsr &b, int n_tiles, int64_t n_cus, int threads, XcdRuns &runs) {
    const int64_t nbr = (int64_t)b.block_row_ptr.size() - 1, total = nbr * n_tiles, even = ceil_div(total, 8);
    if (total > 4 * n_cus) {
        runs = cut_runs(b.length_prefix, nbr, n_tiles, 1, false);
        const int64_t longest = longest_run(runs);
        if (longest <= 4 * even && launch_fits(longest * 8, threads)) return true;
    }
    for (int x = 0; x <= 8; ++x) runs.start[x] = (int)std::min(total, x * even);
    return false;
}

// false: too many threads for a launch
template <int BR, int BN, int WM, int WN, bool VEC>
static bool launch(const asp_handle *h, const void *B, void *C, int64_t N, const BcsrPlan &p, hipStream_t stream) {
    if (!launch_fits(ceil_div(p.workgroups, 8) * 8, WM * WN * 64)) return false;
    XcdRuns runs;
    const int32_t *order = register_staged_runs(h->hb, p.n_tiles, h->n_cus, WM * WN * 64, runs) ? h->d_by_length : nullptr;
    const int64_t longest = longest_run(runs);
    dim3 grid((unsigned)(longest * 8)), block(WM * WN * 64);
    hipLaunchKernelGGL((bcsr_spmm_kernel<BR, BR, BN, WM, WN, VEC>), grid, block, 0, stream, h->d_row_ptr, h->d_col_idx,
                       (const uint16_t *)h->d_values, (const uint16_t *)B, (uint16_t *)C, (int)h->m, (int)h->k, (int)N,
                       (int)h->n_brows, order, runs);
    return true;
}

// Wide tiles where that leaves enough of them: A is read less often, but with few tiles the longest block-rows set the time.
// us, 64 / 128 / 256 wide, 128-row blocks: 18944 x 3584 at 90 %, N = 8001 338 / 257 / 199, 8000 x 2000 at 95 %, N = 6001 (1512
// tiles of 256) 42.6 / 40.0 / 37.3, 3940 x 1488 at 90 %, N = 5271 (651) - / 24.0 / 27.7, 5000 x 5000 at 90 %, N = 2001 (640 of 128) 32.4 /
// 34.0 / 43.0; 64-row: 359 / 272 / 232, 40.9 / 37.2 / 34.6 (3000), 3200 x 1920, geometric lengths, N = 6811 (1350) - / 52 / 58, 34.1 /
// 27.7 / 31.3; 32-row: 450 / 361 / 314, 50 / 46 / 40 (6000), 3057 x 2421, geometric lengths, N = 6099 (2304) - / 24.1 / 27.7, 41 / 34 / 33.
// And where N fills them: a column of a 128- or 256-wide tile costs about 0.72 and 0.6 of one of a 64-wide tile.  150 001 x 512 at
// 50 %, 64-row blocks, N = 70 32.5 / 22.1 / 32.8, 130 51 / 41 / 35, 257 83 / 67 / 74; 50 001 x 1024 at 80 %, 32-row, N = 513 51 / 47 / 49,
// 641 62 / 56 / 51; of 66 such products of 70 to 2050 columns the choice is the fastest or within 3 %, but for those whose number of
// 256-wide tiles is just short (128-row, N = 130, 1172 of them, 41 / 33).
int bcsr_unaligned_bn(const asp_handle *h, int64_t N) {
    const int64_t cost64 = 100 * 64 * ceil_div(N, 64), cost128 = 72 * 128 * ceil_div(N, 128), cost256 = 60 * 256 * ceil_div(N, 256);
    auto enough = [&](int bn, int64_t quarters) {  // tiles of that width, in quarters of the compute units
        return 4 * h->n_brows * ceil_div(N, bn) >= quarters * (int64_t)h->n_cus;
    };
    if (cost256 < cost128 && cost256 < cost64 && enough(256, h->b_row == 128 ? 20 : h->b_row == 64 ? 32 : 48)) return 256;
    return cost128 < cost64 && enough(128, h->b_row == 128 ? 11 : 16) ? 128 : 64;
}

asp_status_t bcsr_spmm_launch(const asp_handle *h, const void *B, void *C, int64_t N, hipStream_t stream) {
    const bool aligned = (((uintptr_t)B | (uintptr_t)C) & 15) == 0;
    const BcsrPlan p = bcsr_plan(h, N, aligned);
    if (p.workgroups * 8 >= (1ll << 31)) return fail(ASP_ERR_UNSUPPORTED, "too many output tiles");
    if (h->dtype == ASP_DT_F32) {
        if (!bcsr_f32_launch(h, B, C, N, stream)) return fail(ASP_ERR_UNSUPPORTED, "too many output tiles");
        hipError_t e32 = hipGetLastError();
        if (e32 != hipSuccess) return fail(ASP_ERR_HIP, std::string("BCSR fp32 kernel launch: ") + hipGetErrorString(e32));
        return ASP_OK;
    }
    const int key = h->b_row * 1000 + p.bn;
    const bool force_regstage = switches().bcsr_regstage;  // benchmarking switch: the synchronous-copy kernel
    if (!force_regstage && switches().bcsr_bn == 0 && bcsr_strip_launch(h, B, C, N, p, stream)) {
        // small launch: strips of block-rows
    } else if (p.vectorized && !force_regstage && N < (1ll << 25)) {
        if (!bcsr_wide_launch(h, B, C, N, p, stream) && !bcsr_dma_launch(h, B, C, N, p, stream))
            return fail(ASP_ERR_UNSUPPORTED, "no kernel for this block size / tile width");
    } else if (!p.vectorized) {  // 16-byte accesses at element alignment
        bool done = false;
        BcsrPlan w = p;
        // (narrower again where a single column tile of 2^29 rows would pass the threads of a launch)
        for (w.bn = bcsr_unaligned_bn(h, N); !done && w.bn >= 64; w.bn /= 2) {
            w.n_tiles = (int32_t)ceil_div(N, w.bn);
            w.workgroups = h->n_brows * w.n_tiles;
            switch (h->b_row * 1000 + w.bn) {
                case 128256: done = launch<128, 256, 2, 2, false>(h, B, C, N, w, stream); break;
                case 128128: done = launch<128, 128, 2, 2, false>(h, B, C, N, w, stream); break;
                case 128064: done = launch<128, 64, 2, 2, false>(h, B, C, N, w, stream); break;
                case 64256: done = launch<64, 256, 1, 4, false>(h, B, C, N, w, stream); break;
                case 64128: done = launch<64, 128, 2, 2, false>(h, B, C, N, w, stream); break;
                case 64064: done = launch<64, 64, 2, 2, false>(h, B, C, N, w, stream); break;
                case 32256: done = launch<32, 256, 1, 4, false>(h, B, C, N, w, stream); break;
                case 32128: done = launch<32, 128, 1, 4, false>(h, B, C, N, w, stream); break;
                case 32064: done = launch<32, 64, 1, 2, false>(h, B, C, N, w, stream); break;
            }
        }
        if (!done) return fail(ASP_ERR_UNSUPPORTED, "too many output tiles");
    } else {
        bool done = false;
        switch (key) {
            case 128256: done = launch<128, 256, 2, 2, true>(h, B, C, N, p, stream); break;
            case 128128: done = launch<128, 128, 2, 2, true>(h, B, C, N, p, stream); break;
            case 128064: done = launch<128, 64, 2, 2, true>(h, B, C, N, p, stream); break;
            case 64256: done = launch<64, 256, 1, 4, true>(h, B, C, N, p, stream); break;
            case 64128: done = launch<64, 128, 2, 2, true>(h, B, C, N, p, stream); break;
            case 64064: done = launch<64, 64, 2, 2, true>(h, B, C, N, p, stream); break;
            case 32256: done = launch<32, 256, 1, 4, true>(h, B, C, N, p, stream); break;
            case 32128: done = launch<32, 128, 1, 4, true>(h, B, C, N, p, stream); break;
            case 32064: done = launch<32, 64, 1, 2, true>(h, B, C, N, p, stream); break;
            default: return fail(ASP_ERR_UNSUPPORTED, "no kernel for this block size / tile width");
        }
        if (!done) return fail(ASP_ERR_UNSUPPORTED, "too many output tiles");
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(ASP_ERR_HIP, std::string("BCSR kernel launch: ") + hipGetErrorString(e));
    return ASP_OK;
}

}  // namespace asp

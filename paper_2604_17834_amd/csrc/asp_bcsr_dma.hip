// BCSR x dense SpMM, main gfx950 kernel: resident workgroups that stream K slices through an LDS ring
// filled by direct-to-LDS loads, without ever waiting for their own stores.
//
// Decomposition: an output tile is one (block-row, N-tile) pair of b_row x BN; its K loop walks the
// stored blocks of the block-row (paper, Section II-C) in slices of 32 k; each slice is multiplied with
// v_mfma_f32_32x32x16_bf16 (fp32 accumulation), operands swapped so that a lane ends with 4 adjacent
// output columns; the finished tile is rounded to bf16, transposed through LDS and stored as full
// 128-byte row segments.
//
// Asynchronous copy (the role TMA plays in the paper's Section III-B): global->LDS traffic never
// touches VGPRs.  Each wave issues global_load_lds_dwordx4 instructions, each dropping 64 lanes x 16
// bytes into one contiguous 1 KB LDS region while the lanes' global source addresses are free.
// Because the LDS side of such a load is lane-linear, the B slice cannot be padded per row; instead the
// source chunk of every lane is permuted so that row r's 64-byte units land XOR-swizzled by (r & 3):
// the four rows touched by one transposing read (ds_read_b64_tr_b16) then fall into disjoint banks.
// Rows of B past K (zero padding of A's last block column) and 16-byte chunks past N are redirected to
// the last valid row / chunk: they meet zeros of A or feed columns that are never stored.
//
// One continuous pipeline per workgroup.  A workgroup owns a fixed sequence of tiles and treats their
// slices as one stream: the ring (NS buffers) is refilled one slice per step, and the prefetch cursor
// runs on into the next tile while the current one is finished, so a tile's first loads overlap the
// previous tile's last multiplications, its epilogue and its stores.  Per step there is one fence-free
// barrier and one exact s_waitcnt: the wave counts every vector-memory operation it issues (loads of
// each slice, stores of each epilogue) and waits only until the operations issued after the slice it
// needs are the only ones outstanding.  Nothing ever waits for stores to C; with tiles of 1-10 blocks
// the store drain time of a tile is comparable to its multiply time, so waiting for it (a fenced
// barrier, or the end of a one-tile workgroup) left the matrix cores idle most of the time.
// The epilogue stages 32 x 64 pieces of the wave's tile in the one ring buffer that is free at a tile
// boundary, wave-privately, so it needs a single extra barrier per tile.
//
// Scheduling (Sections III-E/III-F of the paper discuss persistent kernels and dynamic tile scheduling
// on Hopper and reject them there for imbalance and atomic traffic).  Here the assignment is static and
// balanced by construction: block-rows are sorted by length once per handle; the tile order walks
// group_n adjacent N-tiles together, heaviest block-rows first; the order is cut into 8 runs of equal
// weight, one per XCD (workgroup id mod 8 -- workgroups are dealt to XCDs round-robin), so the B column
// slabs of a group stay in that XCD's private L2 and A blocks are fetched once per group; inside a run
// the XCD's workgroups take tiles round-robin, which deals sorted weights evenly.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>

#include "asp_bcsr_pipe.h"

namespace asp {

template <int BR, int BN, int WM, int WN, int NS, bool XT = false>
struct DmaCfg {
    static constexpr int KS = 32;
    static constexpr int NW = WM * WN;
    static constexpr int NT = NW * 64;
    static constexpr int TM = BR / WM, TN = BN / WN;
    static constexpr int MT = TM / 32, NTL = TN / 32;
    static constexpr int KK = KS / 16;
    static constexpr int SPB = BR / KS;             // slices per block (square blocks)
    static constexpr int A_STAGE = BR * KS * 2;     // bytes
    static constexpr int B_ROW = BN * 2;            // bytes per LDS row of B
    static constexpr int B_STAGE = KS * B_ROW;
    static constexpr int STAGE = A_STAGE + B_STAGE;
    static constexpr int A_R = A_STAGE / 1024, B_R = B_STAGE / 1024;  // 1 KB regions = wave-level loads
    static constexpr int A_LPW = A_R / NW, B_LPW = B_R / NW, LPW = A_LPW + B_LPW;
    static constexpr int CPRW = BN / 8;             // 16-byte chunks per B row
    // epilogue: a wave stages pieces of 32 rows x RW columns of the output matrix, privately, inside one ring buffer
    // (XT: of Y, whose rows are the tile's columns)
    static constexpr int EP_ROWS = XT ? TN : TM, EP_COLS = XT ? TM : TN;
    static constexpr int RW = (EP_COLS >= 64 && NW * 32 * (64 * 2 + 16) <= STAGE) ? 64 : 32;
    static constexpr int JR = RW / 32;              // MFMA tiles per piece
    static constexpr int C_PITCH = RW * 2 + 16;     // bytes
    static constexpr int C_WAVE = 32 * C_PITCH;
    static constexpr int CPR = RW / 8;              // 16-byte units per staged row
    static constexpr int RPI = 64 / CPR;            // rows per wave-level store
    static constexpr int NSTORE = (EP_ROWS / 32) * (EP_COLS / RW) * (32 / RPI);  // store instructions per wave and tile
    static constexpr int LDS_BYTES = NS * STAGE;
    static_assert(A_R % NW == 0 && B_R % NW == 0, "regions must split evenly over the waves");
    static_assert(TM % 32 == 0 && TN % 32 == 0, "wave tile must be made of 32x32 MFMA tiles");
    static_assert(NW * C_WAVE <= STAGE, "epilogue staging must fit into one ring buffer");
    static_assert(NS >= 3 && LDS_BYTES <= 163840, "ring");
    // swizzle of a row's 64-byte units: rows k..k+3 of a transposing read must not share banks
    __device__ static __forceinline__ int swz(int r) { return BN >= 128 ? (r & 3) : ((r >> 1) & 1); }
};

// rank_info[r] = {block-row, first stored block, number of stored blocks, block column of the first one} of the r-th heaviest block-row
//
// XT = true: Y[N x M] = X x A^T with K-contiguous X and Y, as in the kernel for 128x512 tiles (asp_bcsr_wide.hip), for
// launches that do not give every compute unit such a tile, and for small blocks without a composite form.  In the argument
// list B is X and C is Y; the tile's columns are tokens.  A slice of X is BN tokens x 64 bytes, laid out token-major in
// 1 KB regions of 16 tokens with the 16-byte chunks of a token XOR-swizzled by (token / 4) % 4, and read with plain 16-byte
// reads; the operands keep their order, so a lane ends with 4 adjacent outputs of one token.  Chunks past K are read
// from 16 zero bytes, so that nothing of the next token meets the zero padding of A.  K % 8 == 0 and M % 8 == 0.
//
// DYN = true (a benchmarking variant, ASP_BCSR_SCHEDULE=atomic: the dynamic tile scheduling that the paper's Sections
// III-E/III-F try on Hopper and reject): the resident workgroups of an XCD pull the tiles of its run from an atomic counter
// (sched[xcd], zeroed before the launch) instead of taking every stride-th one.  Thread 0 claims, the index travels
// through LDS under the barrier the tile boundary has anyway; the claim for the tile after the next one is made at each
// boundary, so its round trip is paid once per tile by wave 0.  Every workgroup leaves when its claim passes the end of
// the run.  Calls under this switch share the handle's counters and must be ordered on one stream.
// waits until at most j * LPW + EXTRA of the wave's vector-memory operations are outstanding (j <= J, wave-uniform;
// the counter has 6 bits), and for its LDS accesses and scalar loads
template <int LPW, int EXTRA, int J>
__device__ __forceinline__ void wait_slices(int j) {
    constexpr int n = J * LPW + EXTRA;
    if constexpr (J <= 0) {
        wait_vmcnt_and_lds<(n < 63 ? n : 63)>();
    } else {
        if (j >= J) wait_vmcnt_and_lds<(n < 63 ? n : 63)>();
        else wait_slices<LPW, EXTRA, J - 1>(j);
    }
}

static __device__ const uint4 xt_zero_chunk = {0u, 0u, 0u, 0u};

template <int BR, int BN, int WM, int WN, int NS, bool DYN = false, bool XT = false>
__global__ __launch_bounds__(WM *WN * 64, (BR / WM) * (BN / WN) > 8192 ? 1 : 2) void bcsr_spmm_dma_kernel(
    const int4 *__restrict__ rank_info, const int32_t *__restrict__ block_col_idx,
    const uint16_t *__restrict__ a_packed, const uint16_t *__restrict__ B, uint16_t *__restrict__ C, int M, int K,
    int N, int n_brows, int n_tiles, int group_n, XcdRuns runs, int *__restrict__ sched) {
    using Cfg = DmaCfg<BR, BN, WM, WN, NS, XT>;
    constexpr int NW = Cfg::NW, KS = Cfg::KS, MT = Cfg::MT, NTL = Cfg::NTL, LPW = Cfg::LPW;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[Cfg::LDS_BYTES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    // ---- this workgroup's tiles: every stride-th tile of its XCD's run ------------------------------
    // (the order of block-rows was built so that this deals every workgroup one weight-balanced list per
    // group of N-tiles)
    const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3, wg = blockIdx.x >> 3;
    const int run_begin = __builtin_amdgcn_readfirstlane(runs.start[xcd]);
    const int run_end = __builtin_amdgcn_readfirstlane(runs.start[xcd + 1]);
    auto tile_of_round = [&](int r) { return run_begin + r * stride + wg; };
    int round = 0;
    int *s_claim = nullptr;  // two LDS words, only in the dynamic variant
    if constexpr (DYN) {
        __shared__ int claim_words[2];
        s_claim = claim_words;
    }
    int idx_cur = tile_of_round(0), idx_n1 = tile_of_round(1);
    if constexpr (DYN) {
        if (tid == 0) {
            s_claim[0] = run_begin + atomicAdd(&sched[xcd], 1);
            s_claim[1] = run_begin + atomicAdd(&sched[xcd], 1);
        }
        __syncthreads();
        idx_cur = __builtin_amdgcn_readfirstlane(s_claim[0]);
        idx_n1 = __builtin_amdgcn_readfirstlane(s_claim[1]);
        __syncthreads();  // s_claim[0] is written again at the first tile boundary
    }
    if (idx_cur >= run_end) return;

    // ---- lane-invariant parts of the LDS read addresses ------------------------------------------
    const int a_off = lane * 16;
    // transposing read: lane i of a 16-lane group addresses row (i/4), 4 columns at 4*(i%4)
    const int krow_lane = 8 * (lane >> 5) + ((lane & 15) >> 2);          // + 16*kk (+4 for the upper half)
    const int sw = Cfg::swz(krow_lane) << 2;                              // same for krow_lane + 4 and + 16
    const int c_lane = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);         // chunk inside the 32-column tile
    const int sub = 8 * (lane & 1);                                       // byte inside the chunk
    int b_off[NTL];
#pragma unroll
    for (int j = 0; j < NTL; ++j) {
        const int c = (wn * Cfg::TN + j * 32) / 8 + c_lane;
        b_off[j] = krow_lane * Cfg::B_ROW + ((c ^ sw) * 16) + sub;
        if (XT) {  // token t, chunk (2 kk + lane / 32) of its 64 bytes: kk flips bit 5
            const int t = wn * Cfg::TN + j * 32 + (lane & 31);
            b_off[j] = (t >> 4) * 1024 + (t & 15) * 64 + (((lane >> 5) ^ ((t >> 2) & 3)) * 16);
        }
    }
    // B source: region jb = i*NW + wave of a slice holds the 16-byte slots [jb*64, jb*64+64); slot s is
    // row s / CPRW, position s % CPRW; the position is the swizzled chunk index.
    int b_row_in_slice[Cfg::B_LPW], b_chunk[Cfg::B_LPW];
#pragma unroll
    for (int i = 0; i < Cfg::B_LPW; ++i) {
        const int s = (i * NW + wave) * 64 + lane;
        const int r = s / Cfg::CPRW, cp = s % Cfg::CPRW;
        b_row_in_slice[i] = r;
        b_chunk[i] = cp ^ (Cfg::swz(r) << 2);
        if (XT) {  // a region is 16 tokens x 64 bytes
            b_row_in_slice[i] = (i * NW + wave) * 16 + (lane >> 2);
            b_chunk[i] = (lane & 3) ^ ((lane >> 4) & 3);
        }
    }
    const uint32_t a_voff = (uint32_t)(wave * 1024 + lane * 16);
    const uint32_t lds0 = lds_offset(lds);

    // ---- tile parameters ------------------------------------------------------------------------
    // (kept in named scalars: arrays indexed at run time would be placed in LDS or scratch by the
    // compiler, and everything read back from there counts as lane-varying)
    struct Tile {
        int br, n0, T;  // block-row, first column, number of K slices
        int blk0;       // first stored block of the block-row
        int bcol0;      // block column of that block (loaded early: no step waits for a dependent load)
    };
    auto decode = [&](int idx, Tile &t, uint32_t (&voff)[Cfg::B_LPW]) {
        const int per_group = group_n * n_brows;
        const int grp = idx / per_group, in_grp = idx - grp * per_group;
        const int left = n_tiles - grp * group_n;
        const int gw = left < group_n ? left : group_n;  // the last group may be narrower
        // heaviest block-row first in even groups, lightest first in odd ones: neighbours in the order,
        // which run at the same time, then have similar weights across group boundaries too
        const int pos = in_grp / gw, nt = grp * group_n + (in_grp - pos * gw);
        const int rank = (grp & 1) ? n_brows - 1 - pos : pos;
        const int4 ri = rank_info[rank];
        // the index is the same for the whole workgroup: tell the compiler, so that everything derived
        // from a tile's parameters stays in scalar registers
        t.br = __builtin_amdgcn_readfirstlane(ri.x);
        t.blk0 = __builtin_amdgcn_readfirstlane(ri.y);
        t.T = __builtin_amdgcn_readfirstlane(ri.z) * Cfg::SPB;
        t.bcol0 = t.T > 0 ? __builtin_amdgcn_readfirstlane(block_col_idx[t.blk0]) : 0;
        t.n0 = nt * BN;
#pragma unroll
        for (int i = 0; i < Cfg::B_LPW; ++i) {
            if (XT) {
                int tok = b_row_in_slice[i];
                const int last = N - 1 - t.n0;
                tok = tok < last ? tok : last;  // tokens past N only feed columns that are never stored
                voff[i] = (uint32_t)tok * (uint32_t)K * 2 + b_chunk[i] * 16;
                continue;
            }
            int col = t.n0 + 8 * b_chunk[i];
            col = col < N ? col : N - 8;  // chunks past N only feed columns that are never stored
            voff[i] = (uint32_t)(((int64_t)b_row_in_slice[i] * N + col) * 2);  // byte offset inside a slice of B
        }
    };

    // ---- the slice stream ---------------------------------------------------------------------------
    // cur_t is the tile being multiplied, nxt_t the one after it (if have_next).  The prefetch cursor is
    // the next slice to request; it carries its own copy of what it needs (pf_*), sits in the current tile
    // or, once that is fully requested, in the next one (pf_in_next), never further.
    // Buffers buf_c, buf_c+1, .. (mod NS) hold the `inflight` slices requested but not yet multiplied.
    // The counter of outstanding vector-memory operations retires in order: when the content of buf_c is needed, the
    // loads of the inflight - 1 slices behind it may be outstanding, and so may the NSTORE stores of the latest tile
    // while slices requested before them are still to be multiplied (`before_stores` of them).
    Tile cur_t, nxt_t;
    uint32_t nxt_voff[Cfg::B_LPW], pf_voff[Cfg::B_LPW];
    int have_next = 0;
    int pf_T = 0, pf_t = 0, pf_blk = 0, pf_s = 0, pf_in_next = 0;
    int64_t pf_tok = 0;                 // XT: first token of the cursor's tile
    int pf_bcol = 0, pf_bcol_next = 0;  // block column of the cursor's block and of the block after it
    int buf_c = 0, inflight = 0;
    int before_stores = 0;
    auto cursor_enter = [&](const Tile &t, const uint32_t (&voff)[Cfg::B_LPW]) {
        pf_T = t.T;
        pf_t = 0;
        pf_blk = t.blk0;
        pf_s = 0;
        pf_bcol_next = t.bcol0;
        pf_tok = t.n0;
#pragma unroll
        for (int i = 0; i < Cfg::B_LPW; ++i) pf_voff[i] = voff[i];
    };

    decode(idx_cur, cur_t, nxt_voff);
    cursor_enter(cur_t, nxt_voff);
    nxt_t = cur_t;
    if (idx_n1 < run_end) {
        have_next = 1;
        decode(idx_n1, nxt_t, nxt_voff);
    }

    // request the cursor's slice into ring buffer buf and move the cursor on
    auto issue_slice = [&](int buf) {
        const uint32_t stage = lds0 + buf * Cfg::STAGE;
        // the blocks of a block-row, and the slices of a block, are consecutive in a_packed
        const uint8_t *abase = (const uint8_t *)a_packed + ((int64_t)pf_blk * (BR * BR) + pf_s * (BR * KS)) * 2;
#pragma unroll
        for (int i = 0; i < Cfg::A_LPW; ++i)
            dma16_to_lds(abase + i * NW * 1024, a_voff, stage + (i * NW + wave) * 1024);
        if (pf_s == 0) {
            pf_bcol = pf_bcol_next;
            if (pf_t + Cfg::SPB < pf_T) pf_bcol_next = __builtin_amdgcn_readfirstlane(block_col_idx[pf_blk + 1]);
        }
        const int krow0 = pf_bcol * BR + pf_s * KS;
        const uint8_t *bbase = (const uint8_t *)(XT ? B + pf_tok * K + krow0 : B + (int64_t)krow0 * N);
        if (krow0 + KS <= K) {
#pragma unroll
            for (int i = 0; i < Cfg::B_LPW; ++i)
                dma16_to_lds(bbase, pf_voff[i], stage + Cfg::A_STAGE + (i * NW + wave) * 1024);
        } else if (XT) {  // the slice crosses K
#pragma unroll
            for (int i = 0; i < Cfg::B_LPW; ++i) {
                const bool in = krow0 + 8 * b_chunk[i] < K;
                dma16_to_lds(in ? (const void *)(bbase + pf_voff[i]) : (const void *)&xt_zero_chunk,
                             stage + Cfg::A_STAGE + (i * NW + wave) * 1024);
            }
        } else {
            // the slice crosses K: rows past K are read from row K-1, they meet the zero padding of A
#pragma unroll
            for (int i = 0; i < Cfg::B_LPW; ++i) {
                int krow = krow0 + b_row_in_slice[i];
                int back = krow < K ? 0 : krow - (K - 1);
                dma16_to_lds(bbase + pf_voff[i] - (int64_t)back * N * 2, stage + Cfg::A_STAGE + (i * NW + wave) * 1024);
            }
        }
        ++pf_t;
        if (++pf_s == Cfg::SPB) {
            pf_s = 0;
            ++pf_blk;
        }
    };
    // request the next slice of the stream, if there is one within reach; returns whether it did
    auto prefetch_one = [&]() -> bool {
        if (pf_t >= pf_T) {  // this tile is fully requested: step into the next one
            if (pf_in_next || !have_next || nxt_t.T == 0) return false;
            cursor_enter(nxt_t, nxt_voff);
            pf_in_next = 1;
        }
        int buf = buf_c + inflight;
        buf = buf >= NS ? buf - NS : buf;
        issue_slice(buf);
        ++inflight;
        return true;
    };
    // wait until the slice in buf_c has landed, and until this wave's LDS accesses and scalar loads are done
    auto wait_slice = [&]() {
        if (before_stores > 0) {
            --before_stores;
            wait_slices<LPW, Cfg::NSTORE, NS - 2>(inflight - 1);
        } else {
            wait_slices<LPW, 0, NS - 2>(inflight - 1);
        }
    };

    // MFMA operand fragments of one 16-wide k step of the slice in ring buffer buf
    struct Frags {
        bf16x8 a[MT], b[NTL];
    };
    auto load_frags = [&](int buf, int kk, Frags &f) {
        const uint8_t *sa = lds + buf * Cfg::STAGE, *sb = sa + Cfg::A_STAGE;
#pragma unroll
        for (int i = 0; i < MT; ++i) f.a[i] = *(const bf16x8 *)(sa + (kk * (BR / 32) + wm * MT + i) * 1024 + a_off);
#pragma unroll
        for (int j = 0; j < NTL; ++j) {
            if (XT) {
                f.b[j] = *(const bf16x8 *)(sb + (b_off[j] ^ (kk * 32)));
                continue;
            }
            const uint8_t *p0 = sb + kk * 16 * Cfg::B_ROW + b_off[j];
            short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3))) *)(p0));
            short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (short4v __attribute__((address_space(3))) *)(p0 + 4 * Cfg::B_ROW));
            short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            f.b[j] = __builtin_bit_cast(bf16x8, both);
        }
    };
    auto multiply = [&](f32x16 (&acc)[MT][NTL], const Frags &f) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NTL; ++j)
                // operands swapped: D[n][m] = sum_k B[k][n] * A[m][k]  (XT: D[m][n])
                acc[i][j] = XT ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[j], f.a[i], acc[i][j], 0, 0, 0);
    };
    static_assert(Cfg::KK == 2, "the step below is written for two k steps per slice");
    const bool k_aligned = K % BR == 0;  // then no slice reaches past row K of B

    for (;;) {
        const Tile tc = cur_t;
        // (re)fill the ring up to NS-1 slices: the buffer behind buf_c may still be read as the previous
        // tile's staging area until the next barrier
        while (inflight < NS - 1 && prefetch_one()) {
        }
        f32x16 acc[MT][NTL];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NTL; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

        for (int t = 0; t < tc.T; ++t) {
            // Steady state: the NS-1 slices t .. t+NS-2 are in flight or landed, no store is younger than any of them,
            // and the cursor is inside this tile at slice t+NS-1, which does not reach past K (only the last block of a
            // block-row can).  Then the wait is a constant and the request code is straight-line.  us, steady from the first slice
            // on and for any K, against from slice NS-1 on and K % BR == 0 only (rings of three): 5003 x 3331 at 80 %,
            // N = 2048, 128 / 64 / 32-row blocks 51 / 47.5 / 63 -> 41 / 36 / 46; 4096 x 4096, 64-row 36.3 -> 34.5.
            const bool steady = (k_aligned || pf_t < pf_T - Cfg::SPB) && before_stores == 0 && t + NS - 1 < tc.T &&
                                inflight == NS - 1 && !pf_in_next;
            if (steady) wait_vmcnt_and_lds<(NS - 2) * LPW>();
            else wait_slice();  // this wave's part of the slice in buf_c has landed
            barrier_no_fence();  // everybody's part has landed; the buffer behind buf_c is free
            Frags f0, f1;
            load_frags(buf_c, 0, f0);  // LDS reads first: their latency runs under the request code below
            if (steady) {
                const int buf = buf_c == 0 ? NS - 1 : buf_c - 1;
                const uint32_t stage = lds0 + buf * Cfg::STAGE;
                const uint8_t *abase = (const uint8_t *)a_packed + ((int64_t)pf_blk * (BR * BR) + pf_s * (BR * KS)) * 2;
#pragma unroll
                for (int i = 0; i < Cfg::A_LPW; ++i)
                    dma16_to_lds(abase + i * NW * 1024, a_voff, stage + (i * NW + wave) * 1024);
                if (pf_s == 0) {
                    pf_bcol = pf_bcol_next;
                    if (pf_t + Cfg::SPB < pf_T) pf_bcol_next = __builtin_amdgcn_readfirstlane(block_col_idx[pf_blk + 1]);
                }
                const int krow0 = pf_bcol * BR + pf_s * KS;
                const uint8_t *bbase = (const uint8_t *)(XT ? B + pf_tok * K + krow0 : B + (int64_t)krow0 * N);
#pragma unroll
                for (int i = 0; i < Cfg::B_LPW; ++i)
                    dma16_to_lds(bbase, pf_voff[i], stage + Cfg::A_STAGE + (i * NW + wave) * 1024);
                ++pf_t;
                if (++pf_s == Cfg::SPB) {
                    pf_s = 0;
                    ++pf_blk;
                }
            } else {
                while (inflight < NS && prefetch_one()) {
                }
                --inflight;
            }
            load_frags(buf_c, 1, f1);
            multiply(acc, f0);
            multiply(acc, f1);
            buf_c = buf_c + 1 == NS ? 0 : buf_c + 1;
        }

        // ---- tile boundary ------------------------------------------------------------------------
        // parameters of the tile after the next one: requested now, needed after the epilogue
        int idx_nn = tile_of_round(round + 2);
        Tile tnn = tc;
        uint32_t voff_nn[Cfg::B_LPW];
#pragma unroll
        for (int i = 0; i < Cfg::B_LPW; ++i) voff_nn[i] = 0;
        if (!DYN && idx_nn < run_end) decode(idx_nn, tnn, voff_nn);
        if constexpr (DYN) {
            if (tid == 0) s_claim[0] = run_begin + atomicAdd(&sched[xcd], 1);  // read by all after the barrier below
        }

        // the buffer behind buf_c holds nothing that is still needed once every wave got here
        wait_vmcnt_and_lds<63>();
        barrier_no_fence();
        if constexpr (DYN) {
            idx_nn = __builtin_amdgcn_readfirstlane(s_claim[0]);
            if (idx_nn < run_end) decode(idx_nn, tnn, voff_nn);
        }
        const bool interior = tc.br * BR + BR <= M && tc.n0 + BN <= N;
        int sbuf = buf_c == 0 ? NS - 1 : buf_c - 1;
        uint8_t *sc = lds + sbuf * Cfg::STAGE + wave * Cfg::C_WAVE;
        // first row and column of C (XT: of Y, rows are tokens) that this lane stores
        const int out_ld = XT ? M : N, out_rows = XT ? N : M, out_cols = XT ? M : N;
        const int row0 = tc.br * BR + wm * Cfg::TM, col0 = tc.n0 + wn * Cfg::TN;
        const int grow0 = (XT ? col0 : row0) + lane / Cfg::CPR;
        const int gcol0 = (XT ? row0 : col0) + (lane % Cfg::CPR) * 8;
        const uint8_t *scl = sc + (lane / Cfg::CPR) * Cfg::C_PITCH + (lane % Cfg::CPR) * 16;
#pragma unroll
        for (int i = 0; i < Cfg::EP_ROWS / 32; ++i)
#pragma unroll
            for (int jh = 0; jh < Cfg::EP_COLS / Cfg::RW; ++jh) {
                // fp32 -> bf16 (round to nearest even); lane holds row (lane & 31), 4 adjacent columns per q
#pragma unroll
                for (int jj = 0; jj < Cfg::JR; ++jj)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x16 &a = XT ? acc[jh * Cfg::JR + jj][i] : acc[i][jh * Cfg::JR + jj];
                        f32x4 v = {a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
                        bf16x4 hv = __builtin_convertvector(v, bf16x4);
                        *(bf16x4 *)(sc + (lane & 31) * Cfg::C_PITCH + (jj * 32 + 8 * q + 4 * (lane >> 5)) * 2) = hv;
                    }
                // LDS is in order within a wave: the reads below see the writes above
                uint16_t *cdst = C + (int64_t)(grow0 + i * 32) * out_ld + gcol0 + jh * Cfg::RW;
                if (interior) {
#pragma unroll
                    for (int it = 0; it < 32 / Cfg::RPI; ++it) {
                        uint4 v = *(const uint4 *)(scl + it * Cfg::RPI * Cfg::C_PITCH);
                        store_c16(cdst + (int64_t)it * Cfg::RPI * out_ld, v);
                    }
                } else {
#pragma unroll
                    for (int it = 0; it < 32 / Cfg::RPI; ++it) {
                        uint4 v = *(const uint4 *)(scl + it * Cfg::RPI * Cfg::C_PITCH);
                        if (grow0 + i * 32 + it * Cfg::RPI < out_rows && gcol0 + jh * Cfg::RW < out_cols)
                            store_c16(cdst + (int64_t)it * Cfg::RPI * out_ld, v);
                    }
                }
            }
        if (interior) {
            before_stores = inflight;  // exactly NSTORE stores were issued, none is waited for
        } else {
            // an edge tile issues a data-dependent number of stores: drain once so the count is exact again
            wait_vmcnt_and_lds<0>();
            before_stores = 0;
        }

        // ---- advance to the next tile ---------------------------------------------------------------
        if (!have_next) break;
        ++round;
        idx_cur = tile_of_round(round);
        cur_t = nxt_t;
        if (pf_in_next) pf_in_next = 0;          // the cursor's tile is now the current one
        else cursor_enter(nxt_t, nxt_voff);     // the cursor never left the finished tile: it follows
        if (idx_nn < run_end) {
            nxt_t = tnn;
#pragma unroll
            for (int i = 0; i < Cfg::B_LPW; ++i) nxt_voff[i] = voff_nn[i];
            have_next = 1;
        } else {
            have_next = 0;
        }
    }
}

// ---- host side ------------------------------------------------------------------------------------

// Cut the tile order into 8 runs of equal weight.  Tile weight = stored blocks of its block-row + 1
// (the 1 stands for the epilogue).  Groups of N-tiles repeat the same sorted list of block-rows, so a
// cut is found from the per-handle prefix sums over that list.
XcdRuns cut_runs(const std::vector<int64_t> &pre, int64_t nbr, int n_tiles, int group_n, bool turn) {
    const int64_t rows_weight = pre[nbr];
    const int64_t n_groups = ceil_div(n_tiles, group_n);
    const int64_t total_weight = rows_weight * n_tiles;
    XcdRuns r;
    r.start[0] = 0;
    for (int x = 1; x < 8; ++x) {
        const int64_t target = total_weight * x / 8;
        if (target >= total_weight) {  // (nothing to weigh)
            r.start[x] = (int)(nbr * n_tiles);
            continue;
        }
        const int64_t g = std::min(target / (group_n * rows_weight), n_groups - 1);  // whole groups before the cut
        const int64_t acc = g * group_n * rows_weight;
        const int64_t gw = std::min<int64_t>(group_n, n_tiles - g * group_n);
        // first position whose prefix (times the group width) reaches the remainder; odd groups walk
        // the block-rows lightest first (turn)
        const int64_t rem = target - acc;
        auto prefix = [&](int64_t j) { return turn && (g & 1) ? rows_weight - pre[nbr - j] : pre[j]; };
        int64_t lo = 0, hi = nbr;
        while (lo < hi) {
            int64_t mid = (lo + hi) / 2;
            if (prefix(mid) * gw < rem) lo = mid + 1; else hi = mid;
        }
        r.start[x] = (int)(g * group_n * nbr + lo * gw);
    }
    r.start[8] = (int)(nbr * n_tiles);
    for (int x = 1; x <= 8; ++x)
        if (r.start[x] < r.start[x - 1]) r.start[x] = r.start[x - 1];
    return r;
}

__global__ void bcsr_zero_sched_kernel(int *__restrict__ sched) {
    if (threadIdx.x < 8) sched[threadIdx.x] = 0;
}

static const std::vector<int64_t> &weight_prefix(const HostBcsr &b, int lists) {
    return lists == 64 ? b.weight_prefix_64 : lists == 32 ? b.weight_prefix_32 : b.sorted_weight_prefix;
}

// Workgroups of a ring launch, the same number on every XCD: one for every tile of the longest run where the chip holds them.
// Runs of equal weight differ in tiles, and with the mean number of workgroups one of them walked two (us, mean / longest:
// 3584 x 18944 at 90 %, 128-row, N = 3584 137 / 85, N = 3072 100 / 79; 3392 x 4864 at 50 %, N = 1464 75 / 54; 1664 x 3264 at
// 80 %, 32-row, K-contiguous, 1736 tokens 26.5 / 17.6).
static int64_t ring_workgroups(int64_t tiles, const XcdRuns &runs, int64_t resident) {
    const int64_t mean = std::max<int64_t>(8, std::min(tiles, resident) / 8 * 8);
    return std::min(std::max(mean, 8 * longest_run(runs)), std::max<int64_t>(8, resident / 8 * 8));
}

// as many lists as block-rows in a round
static int ring_lists(int64_t tiles, int64_t resident, int group_n) {
    const int64_t per_round = std::max<int64_t>(1, std::min(tiles, resident) / 8) / group_n;
    return per_round < 24 ? 16 : per_round < 48 ? 32 : 64;
}

// What the heaviest workgroup walks, in stored blocks and 1 for every tile, and the heaviest compute unit (every 32nd workgroup
// of its XCD), per workgroup that it holds.
RingLoad ring_heaviest(const HostBcsr &b, const RingWalk &walk, int n_tiles, int64_t n_cus, int per_cu) {
    const int64_t nbr = (int64_t)b.block_row_ptr.size() - 1, cus = std::max<int64_t>(1, n_cus / 8);
    const std::vector<int32_t> &info = walk.lists == 64 ? b.rank_info_64 : walk.lists == 32 ? b.rank_info_32 : b.rank_info;
    const XcdRuns runs = cut_runs(weight_prefix(b, walk.lists), nbr, n_tiles, walk.group_n);
    const int64_t wgs = ring_workgroups(nbr * n_tiles, runs, n_cus * per_cu) / 8;
    RingLoad most = {0, 0};
    std::vector<int64_t> load(wgs), unit(cus);
    for (int x = 0; x < 8; ++x) {
        std::fill(load.begin(), load.end(), 0);
        std::fill(unit.begin(), unit.end(), 0);
        int64_t w = 0;
        for_tiles(runs.start[x], runs.start[x + 1], nbr, n_tiles, walk.group_n, [&](int64_t rank) {
            load[w] += info[4 * rank + 2] + 1;
            if (++w == wgs) w = 0;
        });
        for (int64_t u = 0, v = 0; v < wgs; ++v, u = u + 1 < cus ? u + 1 : 0) unit[u] += load[v];
        most.workgroup = std::max(most.workgroup, *std::max_element(load.begin(), load.end()));
        most.unit = std::max(most.unit, (double)*std::max_element(unit.begin(), unit.end()) / per_cu);
    }
    return most;
}

// How many N-tiles are walked together (group_n), and in which of the orders (bcsr_build_schedule).
// Few N-tiles: an XCD reads the slab of B of one N-tile for many block-rows, whose requests meet in its 4 MB of L2; many: a
// block of A is fetched once for all of them.  Per tile that costs about BN / R and density x BR / group_n, with R the
// block-rows that an XCD walks at a time, so small blocks take few.  Us, groups of 1 / 2 / 4, 3584 x 18944 at 90 %: 32-row
// blocks N = 2048 64 / 87 / 110, N = 4096 129 / 183 / 229, K-contiguous 108 / 112 / 166, 259 / 267 / 345; 64-row N = 2048
// 53 / 60 / 66, K-contiguous 59 / 65 / 68; 128-row N = 2048 64 / 48 / 57, N = 4096 97 / 75 / 91, K-contiguous 62 / 48 / 58 and
// 125 / 89 / 79.
// The order: with as many lists as block-rows in a round the heaviest workgroup is even; 128-row blocks 16, whose rounds start
// in nearer block columns (3584 x 18944, N = 4096, groups of 2: 77 us, with 32 lists 89).
// That is the rule where there are many tiles.  With few rounds of them more depends on where the XCDs' runs end in the lists,
// so another group, in the order that is even for it, is taken where the estimate is 5 % less: the heaviest workgroup and
// compute unit, to powers that the measurements give (the rest of a launch goes on meanwhile), and a factor for the group that
// holds the slabs of B against the fetches of A.  (Us, rule / taken, at 90 %: 64-row, 10240 x 2560, N = 1536 27 / 21, K-contiguous
// 29 / 23; 2816 x 1536, N = 1472 11.4 / 9.3; 128-row, 6912 x 2688, N = 1104 17.5 / 14.6; 6144 x 4096 K-contiguous, 2048
// tokens 24 / 21.  Fitted to 649 launches, of which the rule is in the mean 1.07 times slower than the
// best of nine groups and orders, what is taken 1.04; 38 take more than 1.1 times as long with the rule as with groups of four
// in 16 lists, 9 with what is taken (3584 x 18944 K-contiguous, 2344 tokens 80 / 100).  All nine as candidates would give 1.02
// less and take three times as long to walk on the first call.)
RingWalk ring_walk(const HostBcsr &b, int64_t k, int b_row, int bn, bool xt, int n_tiles, int64_t n_cus, int per_cu) {
    const int64_t nbr = (int64_t)b.block_row_ptr.size() - 1, tiles = nbr * n_tiles;
    RingWalk rule;
    if (b_row == 32) rule.group_n = xt ? 2 : k * (8ll * bn) <= (9 << 19) ? 4 : 1;
    else if (b_row == 64) rule.group_n = 1;
    else rule.group_n = !xt && tiles <= n_cus * per_cu ? 2 : 4;
    rule.group_n = std::min(rule.group_n, n_tiles);
    rule.lists = b_row == 128 ? 16 : ring_lists(tiles, n_cus * per_cu, rule.group_n);
    if (n_tiles > 128 || tiles > 8192) return rule;
    // whole column tiles to every XCD, one at a time, of slabs that are twice its L2 (64-row, 3584 x 18944, N = 4096: 94 us, groups
    // of two in even lists 116)
    if (rule.group_n == 1 && n_tiles % 8 == 0 && k * (2ll * bn) > (8 << 20)) return rule;
    const double mean = (double)(b.block_col_idx.size() + nbr) * n_tiles / (double)(n_cus * per_cu);
    // of groups of one, two and four, at a slab of 8 MB for each N-tile and per doubling of it
    static const double factor[3][3] = {{0, 0.09, 0.35}, {0, 0, 0.05}, {0, -0.10, -0.14}};
    static const double doubling[3][3] = {{0, 0.03, 0.08}, {0, 0, 0.01}, {0, -0.01, -0.02}};
    const double slab = std::log2((double)k * bn * 2 / 8e6);
    auto estimate = [&](int group_n, double workgroup, double unit) {
        const int g = group_n >= 4 ? 2 : group_n >= 2 ? 1 : 0, size = b_row / 64;
        return 0.45 * std::log(workgroup) + 0.22 * std::log(unit) + factor[size][g] + slab * doubling[size][g];
    };
    auto cost = [&](const RingWalk &w) {
        const RingLoad most = ring_heaviest(b, w, n_tiles, n_cus, per_cu);
        return estimate(w.group_n, (double)most.workgroup, most.unit);
    };
    double best = cost(rule) - 0.05;
    RingWalk taken = rule;
    for (int group_n = 1; group_n <= 4 && group_n <= n_tiles; group_n *= 2) {
        const RingWalk w = {group_n, std::min(b_row == 128 ? 32 : 64, ring_lists(tiles, n_cus * per_cu, group_n))};
        if (w.group_n == rule.group_n && w.lists == rule.lists) continue;
        if (estimate(group_n, std::max(mean, (double)(b.max_blocks + 1)), mean) >= best) continue;  // nothing walks less
        const double c = cost(w);
        if (c < best) best = c, taken = w;
    }
    return taken;
}

// (a plan of the handle: it depends on nothing but the blocks and the tiles, so threads that meet here write the same)
static RingWalk kept_ring_walk(const asp_handle *h, int bn, bool xt, int n_tiles, int per_cu) {
    if (n_tiles > 128) return ring_walk(h->hb, h->k, h->b_row, bn, xt, n_tiles, h->n_cus, per_cu);
    std::atomic<uint8_t> &kept = h->ring_walks[xt][bn / 128][n_tiles];
    int v = kept.load(std::memory_order_relaxed);
    if (v == 0) {
        const RingWalk w = ring_walk(h->hb, h->k, h->b_row, bn, xt, n_tiles, h->n_cus, per_cu);
        v = w.group_n + w.lists;  // 1 .. 4 and 16, 32 or 64
        kept.store((uint8_t)v, std::memory_order_relaxed);
    }
    return RingWalk{v % 16, v / 16 * 16};
}

template <int BR, int BN, int WM, int WN, int NS, bool XT>
static void launch_dma(const asp_handle *h, const void *B, void *C, int64_t N, const BcsrPlan &p, hipStream_t stream) {
    const int env_group = switches().bcsr_group_n, env_wgs = switches().bcsr_wgs_per_cu;  // benchmarking switches
    // resident workgroups per CU: as many as LDS allows (the kernel is built for 2 waves per SIMD)
    const int fit = (int)(163840 / DmaCfg<BR, BN, WM, WN, NS, XT>::LDS_BYTES);
    const int per_cu = env_wgs > 0 ? env_wgs : std::max(1, std::min(fit, 8 / (WM * WN)));
    const int64_t resident = (int64_t)h->n_cus * per_cu;
    RingWalk walk;
    if (env_group > 0) {
        walk.group_n = std::min(env_group, p.n_tiles);
        walk.lists = BR == 128 ? 16 : ring_lists(p.workgroups, resident, walk.group_n);
    } else {
        walk = env_wgs > 0 ? ring_walk(h->hb, h->k, BR, BN, XT, p.n_tiles, h->n_cus, per_cu) : kept_ring_walk(h, BN, XT, p.n_tiles, per_cu);
    }
    const int group_n = walk.group_n;
    const int4 *rank_info = (const int4 *)(walk.lists == 64 ? h->d_rank_info_64 : walk.lists == 32 ? h->d_rank_info_32 : h->d_rank_info);
    const XcdRuns runs = cut_runs(weight_prefix(h->hb, walk.lists), h->n_brows, p.n_tiles, group_n);
    const int64_t workers = ring_workgroups(p.workgroups, runs, resident);
    dim3 grid((unsigned)workers), block(WM * WN * 64);
    // benchmarking switch: tiles pulled from per-XCD atomic counters (built for the 128 x 256 tiles of the ladder;
    // everything else keeps the static schedule)
    const bool env_atomic = switches().bcsr_atomic;
    if constexpr (BR == 128 && BN == 256 && !XT) {
        if (env_atomic && h->d_sched) {
            hipLaunchKernelGGL(bcsr_zero_sched_kernel, dim3(1), dim3(64), 0, stream, h->d_sched);
            hipLaunchKernelGGL((bcsr_spmm_dma_kernel<BR, BN, WM, WN, NS, true>), grid, block, 0, stream,
                               rank_info, h->d_col_idx, (const uint16_t *)h->d_values,
                               (const uint16_t *)B, (uint16_t *)C, (int)h->m, (int)h->k, (int)N, (int)h->n_brows,
                               p.n_tiles, group_n, runs, h->d_sched);
            return;
        }
    }
    hipLaunchKernelGGL((bcsr_spmm_dma_kernel<BR, BN, WM, WN, NS, false, XT>), grid, block, 0, stream, rank_info,
                       h->d_col_idx, (const uint16_t *)h->d_values, (const uint16_t *)B, (uint16_t *)C, (int)h->m,
                       (int)h->k, (int)N, (int)h->n_brows, p.n_tiles, group_n, runs, (int *)nullptr);
}

template <bool XT>
static bool launch_dma_tile(const asp_handle *h, const void *B, void *C, int64_t N, const BcsrPlan &p, hipStream_t stream) {
    // Buffers: as many as leave room for the workgroups that a compute unit can hold (two of four waves, four of two),
    // except 64 x 256, where a fourth one costs (3584 x 18944 at 90 %, N = 4096: 125.6 us with 3, 132 with 4).  Eight for
    // one workgroup a compute unit is no faster than these, and slower where there are two.
    switch (h->b_row * 1000 + p.bn) {
        case 128256: launch_dma<128, 256, 2, 2, 3, XT>(h, B, C, N, p, stream); return true;
        case 128128: launch_dma<128, 128, 2, 2, 5, XT>(h, B, C, N, p, stream); return true;
        case 128064: launch_dma<128, 64, 2, 2, 6, XT>(h, B, C, N, p, stream); return true;
        case 64256: launch_dma<64, 256, 1, 4, 3, XT>(h, B, C, N, p, stream); return true;
        case 64128: launch_dma<64, 128, 2, 2, 6, XT>(h, B, C, N, p, stream); return true;
        case 64064: launch_dma<64, 64, 1, 2, 5, XT>(h, B, C, N, p, stream); return true;
        case 32256:
            if constexpr (XT) return false;
            else launch_dma<32, 256, 1, 2, 3, XT>(h, B, C, N, p, stream);
            return true;
        case 32128: launch_dma<32, 128, 1, 2, 4, XT>(h, B, C, N, p, stream); return true;
        case 32064: launch_dma<32, 64, 1, 2, 6, XT>(h, B, C, N, p, stream); return true;
    }
    return false;
}

// needs N % 8 == 0, 8 <= N < 2^25 and 16-byte aligned B and C (the caller checked)
bool bcsr_dma_launch(const asp_handle *h, const void *B, void *C, int64_t N, const BcsrPlan &p, hipStream_t stream) {
    return launch_dma_tile<false>(h, B, C, N, p, stream);
}

// needs K % 8 == 0, M % 8 == 0, K < 2^22, N < 2^25 and 16-byte aligned X and Y (the caller checked)
bool bcsr_dma_xt_launch(const asp_handle *h, const void *X, void *Y, int64_t N, const BcsrPlan &p, hipStream_t stream) {
    return launch_dma_tile<true>(h, X, Y, N, p, stream);
}

}  // namespace asp

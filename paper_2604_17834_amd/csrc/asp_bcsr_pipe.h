// Device-side helpers shared by the BCSR kernels that fill an LDS ring with direct-to-LDS loads.
#pragma once

#include "asp_internal.h"

namespace asp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short short4v;
typedef __attribute__((ext_vector_type(8))) short short8v;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) void *lds_void_ptr;

// s_waitcnt vmcnt(N) lgkmcnt(0): at most N vector-memory operations (the newest ones) stay in flight,
// every LDS access and scalar load of this wave has completed
template <int N>
__device__ __forceinline__ void wait_vmcnt_and_lds() {
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
}

// Workgroup barrier without the memory fence of __syncthreads(): the fence would drain vmcnt to zero and
// with it the slices and stores that are meant to stay in flight.  Callers wait for what they need first.
__device__ __forceinline__ void barrier_no_fence() { __builtin_amdgcn_s_barrier(); }

// global_load_lds_dwordx4: LDS[lds_base + lane*16 .. +16) = 16 bytes at this lane's source address;
// lds_base is wave-uniform (it travels in M0).  Issued as inline assembly on purpose: for the builtin
// form the compiler cannot tell which LDS bytes the copy writes and drains vmcnt to zero before every
// later LDS read, which would serialise the ring.  Completion is tracked by hand.
// Form 1: per-lane 64-bit address.  Form 2: wave-uniform 64-bit base + per-lane 32-bit byte offset.
// The wave-uniform operands are passed through readfirstlane so that they sit in SGPRs even where the
// compiler's divergence analysis cannot prove that they are uniform.
__device__ __forceinline__ uint32_t uniform32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ const void *uniform_ptr(const void *p) {
    const uint64_t v = (uint64_t)(uintptr_t)p;
    const uint64_t lo = uniform32((uint32_t)v), hi = uniform32((uint32_t)(v >> 32));
    return (const void *)(uintptr_t)(lo | (hi << 32));
}
__device__ __forceinline__ void dma16_to_lds(const void *gptr, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(uniform32(lds_base))
                 : "memory", "m0");
}
__device__ __forceinline__ void dma16_to_lds(const void *sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(uniform_ptr(sbase)),
                 "s"(uniform32(lds_base))
                 : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_offset(const void *p) { return (uint32_t)(uintptr_t)(lds_void_ptr)p; }

// 16-byte store of finished output, marked non-temporal: C is written once and never read here, and
// plain stores were measured ~10 % slower end to end because the written lines displace B slabs in L2
// (a store-only kernel with this access pattern is faster with plain stores; the product is not).
__device__ __forceinline__ void store_c16(uint16_t *dst, uint4 v) {
    typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
    u32x4 w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, (u32x4 *)dst);
}

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));  // 16-byte accesses at element alignment

// Elements pos .. pos + 7 of a row of `end` bf16 elements, zeros from `end` on: the row's last 8 elements, moved down.
// (Loaded one by one they made the last column tile set the time of a launch: strips of 5003 x 3331, 80 %, 64 x 64 blocks,
// 1023 columns 58 us, 33 this way.)
__device__ __forceinline__ u32x4 load_tail8(const uint16_t *row, int pos, int end) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (pos >= end) return v;
    if (end < 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (pos + e < end) v[e >> 1] |= (uint32_t)row[pos + e] << (16 * (e & 1));
        return v;
    }
    const int first = pos + 8 <= end ? pos : end - 8, by = pos - first;
    v = *(const u32x4_a2 *)(row + first);
    if (by & 4) v = u32x4{v.z, v.w, 0u, 0u};
    if (by & 2) v = u32x4{v.y, v.z, v.w, 0u};
    if (by & 1) v = u32x4{v.x >> 16 | v.y << 16, v.y >> 16 | v.z << 16, v.z >> 16 | v.w << 16, v.w >> 16};
    return v;
}

// first tile of each XCD's run of the tile order, start[8] = number of tiles
struct XcdRuns {
    int start[9];
};
inline int64_t longest_run(const XcdRuns &r) {
    int64_t n = 0;
    for (int x = 0; x < 8; ++x) n = std::max<int64_t>(n, r.start[x + 1] - r.start[x]);
    return n;
}

// Cut the tile order (groups of group_n N-tiles, inside a group the n_rows heaviest block-rows, each repeated over the group's
// N-tiles, in the handle's order in even groups and backwards in odd ones, or always in order: turn = false) into 8 runs of
// equal weight; pre[] are the prefix sums of the block-rows' tile weights in that order.
XcdRuns cut_runs(const std::vector<int64_t> &pre, int64_t n_rows, int n_tiles, int group_n, bool turn = true);
// Calls tile(r) with the rank in the order of every tile first .. last - 1 of it.
template <class F>
inline void for_tiles(int64_t first, int64_t last, int64_t n_rows, int n_tiles, int group_n, F tile) {
    int64_t grp = first / (group_n * n_rows), in = first - grp * group_n * n_rows;
    int64_t gw = std::min<int64_t>(group_n, n_tiles - grp * group_n), pos = in / std::max<int64_t>(1, gw), j = in - pos * gw;
    for (int64_t i = first; i < last; ++i) {
        tile((grp & 1) ? n_rows - 1 - pos : pos);
        if (++j < gw) continue;
        j = 0;
        if (++pos < n_rows) continue;
        pos = 0;
        ++grp;
        gw = std::min<int64_t>(group_n, n_tiles - grp * group_n);
    }
}

struct RingWalk {
    int group_n, lists;
};
struct RingLoad {
    int64_t workgroup;
    double unit;
};
RingLoad ring_heaviest(const HostBcsr &b, const RingWalk &walk, int n_tiles, int64_t n_cus, int per_cu);
RingWalk ring_walk(const HostBcsr &b, int64_t k, int b_row, int bn, bool xt, int n_tiles, int64_t n_cus, int per_cu);
int64_t wide_heaviest(const HostBcsr &b, const BcsrShares &s, int n_tiles, int t);
int wide_shared_tiles(const HostBcsr &b, const BcsrShares &s, int64_t k, bool xt, int n_tiles, int64_t n_cus);
bool register_staged_runs(const HostBcsr &b, int n_tiles, int64_t n_cus, int threads, XcdRuns &runs);

}  // namespace asp

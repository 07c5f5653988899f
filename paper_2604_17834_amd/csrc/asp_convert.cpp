// Host-side format converters of the library: CSR -> BCSR and CSR -> WCSR (paper, Section II-C) and
// the host variant of the window sub-task list (Section III-C).  Values are bit-copied only.
//
// Work is spread over block-rows / windows with a shared atomic counter so that a few very long
// windows do not serialise the conversion.
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <functional>
#include <mutex>
#include <numeric>
#include <system_error>
#include <thread>

#include "asp_internal.h"

namespace asp {

namespace {

unsigned worker_count(int64_t items) {
    unsigned hw = std::thread::hardware_concurrency();
    if (hw == 0) hw = 1;
    hw = std::min(hw, 32u);
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(hw, items / 64 + 1));
}

// run fn(worker_index, first, last) over [0, n) in dynamically claimed chunks
// (by as many threads as `items` of the usual size are worth)
template <class F>
void parallel_chunks(int64_t n, int64_t chunk, F fn, int64_t items = 0) {
    unsigned nw = worker_count(std::max(n, items));
    std::atomic<int64_t> next{0};
    // An exception inside a worker (an allocation that fails) must not leave its thread: the first one is kept,
    // the other workers stop claiming chunks, and it is thrown again on the calling thread after all have joined.
    std::exception_ptr first_error;
    std::mutex error_mu;
    auto body = [&](unsigned wi) {
        try {
            for (;;) {
                int64_t b = next.fetch_add(chunk);
                if (b >= n) break;
                fn(wi, b, std::min(n, b + chunk));
            }
        } catch (...) {
            std::lock_guard<std::mutex> lock(error_mu);
            if (!first_error) first_error = std::current_exception();
            next.store(n);
        }
    };
    std::vector<std::thread> th;
    for (unsigned w = 1; w < nw; ++w) {
        try {
            th.emplace_back(body, w);
        } catch (const std::system_error &) {
            break;  // no further thread to be had: the ones that run (at least the caller) do all the chunks
        }
    }
    body(0);
    for (auto &t : th) t.join();
    if (first_error) std::rethrow_exception(first_error);
}

}  // namespace

std::string validate_csr(int64_t m, int64_t k, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx) {
    if (row_ptr[0] != 0) return "row_ptr[0] != 0";
    for (int64_t i = 0; i < m; ++i)
        if (row_ptr[i + 1] < row_ptr[i]) return "row_ptr decreases at row " + std::to_string(i);
    if (row_ptr[m] != nnz) return "row_ptr[m] != nnz";
    std::atomic<int64_t> bad_row{-1};
    parallel_chunks(m, 4096, [&](unsigned, int64_t b, int64_t e) {
        for (int64_t i = b; i < e; ++i) {
            int64_t prev = -1;
            for (int64_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p) {
                int64_t c = col_idx[p];
                if (c <= prev || c >= k) {
                    int64_t expect = -1;
                    bad_row.compare_exchange_strong(expect, i);
                    return;
                }
                prev = c;
            }
        }
    });
    if (bad_row.load() >= 0)
        return "row " + std::to_string(bad_row.load()) +
               ": column indices must be in [0,k) and strictly ascending (no duplicates)";
    return "";
}

// ------------------------------------------------------------------------------------------ BCSR
void csr_to_bcsr(int64_t m, int64_t k, const int32_t *row_ptr, const int32_t *col_idx, const void *values,
                 size_t esize, int32_t b_row, int32_t b_col, HostBcsr &out) {
    const int64_t nbr = ceil_div(m, b_row), nbc = ceil_div(k, b_col);
    out.block_row_ptr.assign(nbr + 1, 0);
    unsigned nw = worker_count(nbr);
    // stamp[w][J] == I + 1 marks "block column J already seen in block-row I" for worker w
    std::vector<std::vector<int64_t>> stamp(nw, std::vector<int64_t>(nbc, 0));

    // pass 1: number of touched block columns per block-row
    parallel_chunks(nbr, 16, [&](unsigned wi, int64_t b, int64_t e) {
        auto &st = stamp[wi];
        for (int64_t I = b; I < e; ++I) {
            int64_t r1 = std::min<int64_t>(m, (I + 1) * b_row);
            int32_t cnt = 0;
            for (int64_t p = row_ptr[I * b_row]; p < row_ptr[r1]; ++p) {
                int64_t J = col_idx[p] / b_col;
                if (st[J] != I + 1) {
                    st[J] = I + 1;
                    ++cnt;
                }
            }
            out.block_row_ptr[I + 1] = cnt;
        }
    });
    for (int64_t I = 0; I < nbr; ++I) out.block_row_ptr[I + 1] += out.block_row_ptr[I];
    const int64_t nb = out.block_row_ptr[nbr];
    const int64_t bsz = (int64_t)b_row * b_col;
    out.block_col_idx.assign(nb, 0);
    out.blocks.assign((size_t)nb * bsz * esize, 0);  // +0.0 everywhere

    // pass 2: ascending block columns, then scatter the entries
    std::vector<std::vector<int32_t>> slot(nw, std::vector<int32_t>(nbc, -1));
    for (auto &s : stamp) std::fill(s.begin(), s.end(), 0);
    parallel_chunks(nbr, 16, [&](unsigned wi, int64_t b, int64_t e) {
        auto &st = stamp[wi];
        auto &sl = slot[wi];
        for (int64_t I = b; I < e; ++I) {
            int64_t r0 = I * b_row, r1 = std::min<int64_t>(m, r0 + b_row);
            int32_t *cols = out.block_col_idx.data() + out.block_row_ptr[I];
            int32_t cnt = 0;
            for (int64_t p = row_ptr[r0]; p < row_ptr[r1]; ++p) {
                int32_t J = col_idx[p] / b_col;
                if (st[J] != I + 1) {
                    st[J] = I + 1;
                    cols[cnt++] = J;
                }
            }
            std::sort(cols, cols + cnt);
            for (int32_t t = 0; t < cnt; ++t) sl[cols[t]] = out.block_row_ptr[I] + t;
            for (int64_t i = r0; i < r1; ++i) {
                for (int64_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p) {
                    int32_t c = col_idx[p];
                    int32_t J = c / b_col;
                    size_t dst = ((size_t)sl[J] * bsz + (size_t)(i - r0) * b_col + (size_t)(c - J * b_col)) * esize;
                    std::memcpy(out.blocks.data() + dst, (const uint8_t *)values + (size_t)p * esize, esize);
                }
            }
        }
    });
}

// Exchanges entries between the heaviest list and another one while that makes the heavier of the two lighter: each time the
// pair of entries that makes it lightest.  With the lengths of every list in order the best difference between two lists
// takes one walk along both, not all pairs of their entries.
template <class Len>
static void exchange_entries(std::vector<std::vector<int32_t>> &lists, std::vector<int64_t> &load, Len len) {
    const int n = (int)lists.size();
    std::vector<std::vector<int32_t>> lens(n);
    for (int l = 0; l < n; ++l) {
        for (int32_t r : lists[l]) lens[l].push_back(len(r));
        std::sort(lens[l].begin(), lens[l].end());
    }
    auto replace = [](std::vector<int32_t> &v, int32_t from, int32_t by) {
        v.erase(std::lower_bound(v.begin(), v.end(), from));
        v.insert(std::lower_bound(v.begin(), v.end(), by), by);
    };
    for (int step = 0; step < 4 * n; ++step) {
        const int h = (int)(std::max_element(load.begin(), load.end()) - load.begin());
        // moving d blocks from h to l makes the heavier of the two min(d, load[h] - load[l] - d) lighter
        int64_t best = 0;
        int to = -1;
        for (int l = 0; l < n; ++l) {
            const int64_t apart = load[h] - load[l];
            if (l == h || apart <= 2 * best) continue;
            const std::vector<int32_t> &other = lens[l];
            size_t j = 0;
            for (int32_t mine : lens[h]) {
                while (j < other.size() && 2 * (int64_t)other[j] < 2 * (int64_t)mine - apart) ++j;  // the best partners: j - 1 and j
                for (size_t p = j > 0 ? j - 1 : 0; p < other.size() && p <= j; ++p) {
                    const int64_t d = mine - other[p], gain = std::min(d, apart - d);
                    if (gain > best) best = gain, to = l;
                }
            }
        }
        if (to < 0) break;
        const int64_t apart = load[h] - load[to];
        bool found = false;
        for (size_t i = 0; i < lists[h].size() && !found; ++i)
            for (size_t j = 0; j < lists[to].size() && !found; ++j) {
                const int32_t mine = len(lists[h][i]), other = len(lists[to][j]);
                const int64_t d = mine - other;
                if (std::min(d, apart - d) != best) continue;
                found = true;
                std::swap(lists[h][i], lists[to][j]);
                load[h] -= d, load[to] += d;
                replace(lens[h], mine, other);
                replace(lens[to], other, mine);
            }
    }
}

// Inside a list the order is free (the sum stays).  Entries go by the block column of their first block: the block-rows
// that run at the same time then start in the same few block columns, their first slabs of B are requested by several
// workgroups of the XCD at about the same time and cross the memory side of L2 once (7 % less time on 90 % Bernoulli
// masks than lists in order of weight).
static void sort_by_first_column(const HostBcsr &b, std::vector<std::vector<int32_t>> &lists) {
    for (auto &l : lists)
        std::stable_sort(l.begin(), l.end(), [&](int32_t x, int32_t y) {
            return b.block_col_idx[b.block_row_ptr[x]] < b.block_col_idx[b.block_row_ptr[y]];
        });
}

// The order of the main BCSR kernels: they deal its consecutive entries to the workgroups of an XCD round-robin, n_lists
// block-rows per round, so entry j belongs to list j % n_lists and a workgroup walks one list per group of N-tiles.  The
// non-empty block-rows (the first n_nonempty of `sorted`, heaviest first) are spread over the lists so that these have nearly
// the same sum of weights (stored blocks + 1 for the tile's epilogue); each list has an entry of every full round and perhaps
// one of the last, incomplete round.
template <class Len>
static void order_in_lists(const HostBcsr &b, const std::vector<int32_t> &sorted, int64_t n_nonempty, int n_lists, Len len,
                           std::vector<int32_t> &order) {
    std::vector<std::vector<int32_t>> lists(n_lists);
    std::vector<int64_t> load(n_lists, 0);
    for (int64_t r = 0; r < n_nonempty; ++r) {
        // among the lists with the fewest entries (the round being filled), the lightest one
        int best = -1;
        size_t fewest = lists[0].size();
        for (int l = 1; l < n_lists; ++l) fewest = std::min(fewest, lists[l].size());
        for (int l = 0; l < n_lists; ++l)
            if (lists[l].size() == fewest && (best < 0 || load[l] < load[best])) best = l;
        lists[best].push_back(sorted[r]);
        load[best] += len(sorted[r]) + 1;
    }
    // (Few entries to a list leave the rule above far off: 18944 x 3584 at 90 %, 32 lists, heaviest over mean 1.31 to 1.37
    // with 128-row blocks, 1.20 with 64, 1.15 with 32; after the exchanges 1.01 to 1.05.  Long lists are even as they are.)
    if (n_nonempty > n_lists && n_nonempty <= 64 * n_lists) exchange_entries(lists, load, len);
    // Lists with one entry more go first, so that the entries of the last, incomplete round are those of lists
    // 0, 1, ... and "entry j belongs to list j % n_lists" holds for every j.
    std::stable_sort(lists.begin(), lists.end(),
                     [](const std::vector<int32_t> &x, const std::vector<int32_t> &y) { return x.size() > y.size(); });
    sort_by_first_column(b, lists);
    order.reserve(sorted.size());
    for (size_t e = 0; order.size() < (size_t)n_nonempty; ++e)
        for (auto &l : lists)
            if (e < l.size()) order.push_back(l[e]);
}

// Scheduling data of the BCSR kernels: rank_info and the prefix sums of the tile weights in its order (and the same for
// groups of one N-tile), empty block-rows last.  LENGTH (the fp32 kernel, one workgroup per tile): longest block-row first
// (ties: lower block-row first), nothing else.  TILES: in 16 and 32 lists, all that 128x512 tiles take; ROWS_128: and longest
// first, for the register-staged kernel; ALL: and in 64 lists, which the ring kernel takes with smaller blocks.
void bcsr_build_schedule(HostBcsr &b, Orders orders) {
    const bool by_length = orders == Orders::LENGTH;
    const int64_t nbr = (int64_t)b.block_row_ptr.size() - 1;
    std::vector<int32_t> sorted(nbr);
    for (int64_t i = 0; i < nbr; ++i) sorted[i] = (int32_t)i;
    auto len = [&](int32_t r) { return b.block_row_ptr[r + 1] - b.block_row_ptr[r]; };
    std::stable_sort(sorted.begin(), sorted.end(), [&](int32_t x, int32_t y) { return len(x) > len(y); });
    int64_t n_nonempty = 0;
    while (n_nonempty < nbr && len(sorted[n_nonempty]) > 0) ++n_nonempty;
    b.n_nonempty = n_nonempty;

    auto fill = [&](int n_lists, std::vector<int32_t> &rank_info, std::vector<int64_t> &prefix) {
        std::vector<int32_t> order;
        if (n_lists > 0) order_in_lists(b, sorted, n_nonempty, n_lists, len, order);
        order.insert(order.end(), sorted.begin() + order.size(), sorted.end());
        rank_info.resize((size_t)nbr * 4);
        prefix.assign(nbr + 1, 0);
        for (int64_t r = 0; r < nbr; ++r) {
            const int32_t br = order[r];
            rank_info[4 * r + 0] = br;
            rank_info[4 * r + 1] = b.block_row_ptr[br];
            rank_info[4 * r + 2] = len(br);
            rank_info[4 * r + 3] = len(br) > 0 ? b.block_col_idx[b.block_row_ptr[br]] : 0;  // column of its first block
            prefix[r + 1] = prefix[r] + len(br) + 1;
        }
    };
    fill(by_length ? 0 : 16, b.rank_info, b.sorted_weight_prefix);
    if (by_length) return;
    fill(32, b.rank_info_32, b.weight_prefix_32);
    if (orders == Orders::TILES) return;
    b.by_length = sorted;
    b.length_prefix.assign(nbr + 1, 0);
    // What a tile costs beside its blocks, in blocks: 1, but a tile that is only cleared takes as long as 3 or 4 of them, which tells
    // where half of the block-rows are empty.  (Us, 1 / 3: 2048 block-rows of 32, lengths geometric, 3 column tiles of 128
    // 104 / 88, 5 139 / 126, 8 153 / 152; lengths alike 68 / 70, 102 / 103, 151 / 151; 30 % empty, 4 tiles 100 / 106.)
    const int64_t tile = 2 * n_nonempty <= nbr ? 3 : 1;
    for (int64_t r = 0; r < nbr; ++r) b.length_prefix[r + 1] = b.length_prefix[r] + len(b.by_length[r]) + tile;
    if (orders == Orders::ALL) fill(64, b.rank_info_64, b.weight_prefix_64);
}

// Lists for the N-tiles that are left when every XCD has had the same number of whole ones: t of them (1 to 23, no multiple of 8)
// are dealt to 256 workgroups, 256 / t to a tile, and a workgroup walks one list of its tile's block-rows.  Longest block-row first, each
// to the lightest of the lists with the fewest entries, then exchanges; without regard to the entries where that makes the
// heaviest list 5 % lighter (lists of one length keep the workgroups of an XCD in the same block columns).
void bcsr_build_shares(const HostBcsr &b, BcsrShares &out) {
    const int64_t n = b.n_nonempty;
    out = BcsrShares();
    const int64_t tile = 2;  // what a tile costs beside its blocks, in blocks
    if (n == 0 || n > BcsrShares::MAX_ROWS) return;
    auto len = [&](int32_t r) { return b.block_row_ptr[r + 1] - b.block_row_ptr[r]; };
    std::vector<int32_t> sorted(n);
    for (int64_t r = 0; r < n; ++r) sorted[r] = b.rank_info[4 * r];
    std::stable_sort(sorted.begin(), sorted.end(), [&](int32_t x, int32_t y) { return len(x) > len(y); });
    constexpr int SLOTS = BcsrShares::slot(BcsrShares::MAX_TILES) + 1;
    out.infos = (int64_t)b.rank_info_32.size() / 4 + SLOTS * n;
    out.lists = b.rank_info_32;
    out.load.assign(SLOTS * BcsrShares::WORKERS, 0);
    out.lists.resize((size_t)out.infos * 4 + SLOTS * BcsrShares::FIRST_PITCH);
    parallel_chunks(SLOTS, 1, [&](unsigned, int64_t lo, int64_t hi) {
        for (int64_t i = lo; i < hi; ++i) {
            const int n_lists = BcsrShares::WORKERS / (int)(i + i / 7 + 1);  // slot(t) = i
            std::vector<std::vector<int32_t>> lists;
            std::vector<int64_t> loads;
            int64_t longest = 0;
            for (int even = 1; even >= 0; --even) {
                std::vector<std::vector<int32_t>> cand(n_lists);
                std::vector<int64_t> load(n_lists, 0);
                for (int64_t r = 0; r < n; ++r) {
                    const size_t most = even ? (size_t)(r / n_lists) : (size_t)n;  // entries that a list may have already
                    int best = -1;
                    for (int l = 0; l < n_lists; ++l)
                        if (cand[l].size() <= most && (best < 0 || load[l] < load[best])) best = l;
                    cand[best].push_back(sorted[r]);
                    load[best] += len(sorted[r]) + tile;
                }
                if (n > n_lists) exchange_entries(cand, load, len);
                const int64_t w = *std::max_element(load.begin(), load.end());
                if (even || w * 100 < longest * 95) longest = w, lists.swap(cand), loads.swap(load);
            }
            sort_by_first_column(b, lists);
            int32_t *info = out.lists.data() + b.rank_info_32.size() + i * n * 4;
            int32_t *first = out.lists.data() + out.infos * 4 + i * BcsrShares::FIRST_PITCH;
            int32_t at = 0;
            for (int l = 0; l < n_lists; ++l) {
                first[l] = at;
                for (int32_t r : lists[l]) {
                    const int32_t v[4] = {r, b.block_row_ptr[r], len(r), b.block_col_idx[b.block_row_ptr[r]]};
                    std::copy(v, v + 4, info + 4 * at++);
                }
            }
            std::fill(first + n_lists, first + BcsrShares::FIRST_PITCH, at);
            std::copy(loads.begin(), loads.end(), out.load.begin() + i * BcsrShares::WORKERS);
        }
    }, n);
}

// Composite form of a bf16 BCSR matrix with 64x64 or 32x32 blocks, for the kernel written for 128x128 blocks
// (Section II-C's block product, regrouped): R = 128 / b block-rows make one 128-row super-row; the union of their
// block columns is cut into groups of R; a composite block holds, for each of its R columns j, the b-wide column
// strip [block(r_0, j); ...; block(r_{R-1}, j)] of the super-row's members (zeros where a block is not stored) as
// b / 32 consecutive 32-wide K slices.  slice_rows gives, per composite block, the first row of B that each of
// its four K slices multiplies (for a plain 128x128 block these would be 128 J + 0, 32, 64, 96).  Strips that pad
// the last group are zeros and repeat the rows of the last real strip.
//
// Members of a super-row need not be adjacent: every absent block of a strip is computed as zeros, so block-rows
// with similar block columns are put together (greedy: longest unassigned block-row first, then R - 1 times the
// unassigned block-row with the largest Jaccard index against the group's union of columns; on 50-90 %-sparse
// random masks this stores 12-24 % fewer composite blocks than grouping neighbours).  piece_rows
// gives, per super-row, the first row of C of each of its four 32-row pieces, -1 for a member that does not
// exist.  Block-rows without blocks form super-rows of their own at the end (their rows of C are cleared).
// Returns the work inflation: composite blocks x 128 x 128 over stored blocks x b x b.
double bcsr_build_composite(const HostBcsr &in, int64_t m, int64_t k, int32_t b, HostBcsr &out) {
    const int64_t nbr = (int64_t)in.block_row_ptr.size() - 1;
    const int32_t R = 128 / b, spv = b / 32;  // members of a super-row = strips per composite block; K slices per strip
    (void)m;
    auto len = [&](int64_t r) { return in.block_row_ptr[r + 1] - in.block_row_ptr[r]; };
    auto cols = [&](int64_t r) { return in.block_col_idx.data() + in.block_row_ptr[r]; };

    // ---- grouping ----------------------------------------------------------------------------------------
    int32_t nbc = 0;
    for (int32_t c : in.block_col_idx) nbc = std::max(nbc, c + 1);
    std::vector<int32_t> inv_ptr((size_t)nbc + 1, 0), inv(in.block_col_idx.size());
    for (int32_t c : in.block_col_idx) ++inv_ptr[c + 1];
    for (int32_t c = 0; c < nbc; ++c) inv_ptr[c + 1] += inv_ptr[c];
    {
        std::vector<int32_t> fill(inv_ptr.begin(), inv_ptr.end() - 1);
        for (int64_t r = 0; r < nbr; ++r)
            for (int32_t t = 0; t < len(r); ++t) inv[fill[cols(r)[t]]++] = (int32_t)r;
    }
    std::vector<int32_t> order;
    for (int64_t r = 0; r < nbr; ++r)
        if (len(r) > 0) order.push_back((int32_t)r);
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return len(x) > len(y); });
    std::vector<uint8_t> taken((size_t)nbr, 0), in_union((size_t)nbc, 0);
    std::vector<int32_t> shared((size_t)nbr, 0), touched, uni;
    std::vector<int32_t> members;  // R per super-row, -1 = none
    const int64_t budget = 1 << 18;  // shared-column counts examined per choice: bounds the work on dense matrices
    for (int32_t seed : order) {
        if (taken[seed]) continue;
        taken[seed] = 1;
        const size_t g0 = members.size();
        members.push_back(seed);
        uni.assign(cols(seed), cols(seed) + len(seed));
        for (int32_t c : uni) in_union[c] = 1;
        while (members.size() - g0 < (size_t)R) {
            touched.clear();
            int64_t spent = 0;
            for (int32_t c : uni) {
                for (int32_t q = inv_ptr[c]; q < inv_ptr[c + 1] && spent < budget; ++q, ++spent) {
                    const int32_t r = inv[q];
                    if (taken[r]) continue;
                    if (shared[r]++ == 0) touched.push_back(r);
                }
                if (spent >= budget) break;
            }
            // best Jaccard index with the group's union: shared / (union + own - shared), compared as fractions
            int32_t best = -1;
            int64_t best_num = 0, best_den = 1;
            const int64_t usize = (int64_t)uni.size();
            for (int32_t r : touched) {
                const int64_t num = shared[r], den = usize + len(r) - shared[r];
                const int64_t lhs = num * best_den, rhs = best_num * den;
                if (best < 0 || lhs > rhs || (lhs == rhs && r < best)) best = r, best_num = num, best_den = den;
                shared[r] = 0;
            }
            if (best < 0) break;  // nobody shares a column: the group stays short
            taken[best] = 1;
            members.push_back(best);
            for (int32_t t = 0; t < len(best); ++t) {
                const int32_t c = cols(best)[t];
                if (!in_union[c]) in_union[c] = 1, uni.push_back(c);
            }
        }
        for (int32_t c : uni) in_union[c] = 0;
        // members in ascending block-row order (rows of C of a tile ascend), padded with -1
        std::sort(members.begin() + g0, members.end());
        while (members.size() - g0 < (size_t)R) members.push_back(-1);
    }
    {   // block-rows without blocks
        size_t g0 = members.size();
        for (int64_t r = 0; r < nbr; ++r)
            if (len(r) == 0) {
                members.push_back((int32_t)r);
                if (members.size() - g0 == (size_t)R) g0 = members.size();
            }
        while ((members.size() - g0) % R != 0) members.push_back(-1);
    }
    const int64_t nsr = (int64_t)members.size() / R;

    // ---- composite blocks --------------------------------------------------------------------------------
    out = HostBcsr();
    out.block_row_ptr.assign(nsr + 1, 0);
    out.piece_rows.assign((size_t)nsr * 4, -1);
    std::vector<std::vector<int32_t>> unis((size_t)nsr);
    parallel_chunks(nsr, 16, [&](unsigned, int64_t lo, int64_t hi) {
        for (int64_t sr = lo; sr < hi; ++sr) {
            auto &u = unis[sr];
            for (int32_t t = 0; t < R; ++t) {
                const int32_t br = members[sr * R + t];
                if (br < 0) continue;
                u.insert(u.end(), cols(br), cols(br) + len(br));
                for (int32_t i = 0; i < spv; ++i) out.piece_rows[4 * sr + t * spv + i] = br * b + 32 * i;
            }
            std::sort(u.begin(), u.end());
            u.erase(std::unique(u.begin(), u.end()), u.end());
            out.block_row_ptr[sr + 1] = (int32_t)ceil_div((int64_t)u.size(), R);
        }
    });
    for (int64_t sr = 0; sr < nsr; ++sr) out.block_row_ptr[sr + 1] += out.block_row_ptr[sr];
    const int64_t nc = out.block_row_ptr[nsr];
    out.block_col_idx.assign(nc, 0);
    out.slice_rows.assign((size_t)nc * 4, 0);
    out.blocks.assign((size_t)nc * 128 * 128 * 2, 0);
    const uint16_t *src = (const uint16_t *)in.blocks.data();
    uint16_t *dst = (uint16_t *)out.blocks.data();
    parallel_chunks(nsr, 4, [&](unsigned, int64_t lo, int64_t hi) {
        for (int64_t sr = lo; sr < hi; ++sr) {
            const auto &u = unis[sr];
            for (int64_t c = out.block_row_ptr[sr]; c < out.block_row_ptr[sr + 1]; ++c) {
                const int64_t first = (c - out.block_row_ptr[sr]) * R;
                for (int32_t v = 0; v < R; ++v) {
                    const bool real = first + v < (int64_t)u.size();
                    const int32_t j = u[real ? first + v : u.size() - 1];
                    // a slice must not reach past K: in the last, partly filled block column it starts early enough
                    // to end at K, and its values move right by the same amount (the columns it then overlaps with
                    // an earlier slice stay zero here)
                    int32_t shift[4] = {0, 0, 0, 0};
                    for (int32_t t = 0; t < spv; ++t) {
                        const int64_t k0 = (int64_t)j * b + 32 * t;
                        const int64_t r0 = std::min<int64_t>(k0, k - 32);
                        shift[t] = (int32_t)(k0 - r0);
                        out.slice_rows[4 * c + v * spv + t] = (int32_t)r0;
                    }
                    if (!real) continue;
                    for (int32_t t = 0; t < R; ++t) {
                        const int32_t br = members[sr * R + t];
                        if (br < 0) continue;
                        const int32_t *cb = cols(br), *ce = cb + len(br);
                        const int32_t *hit = std::lower_bound(cb, ce, j);
                        if (hit == ce || *hit != j) continue;
                        const uint16_t *sb = src + (int64_t)(hit - in.block_col_idx.data()) * b * b;
                        for (int32_t r = 0; r < b; ++r)
                            for (int32_t sl = 0; sl < spv; ++sl) {
                                if (shift[sl] >= 32) continue;  // the slice lies past K altogether: zeros
                                std::memcpy(dst + c * 128 * 128 + ((int64_t)t * b + r) * 128 + v * b + 32 * sl + shift[sl],
                                            sb + (int64_t)r * b + 32 * sl, (size_t)(32 - shift[sl]) * 2);
                            }
                    }
                }
                out.block_col_idx[c] = out.slice_rows[4 * c] / 128;  // the schedule orders block-rows by this
            }
        }
    });
    bcsr_build_schedule(out, Orders::TILES);
    bcsr_pack_fragments_bf16(out, 128, 128, out.packed);
    out.blocks = std::vector<uint8_t>();  // only the packed form is used
    const double stored = (double)in.block_col_idx.size() * b * b;
    return stored > 0 ? (double)nc * 128 * 128 / stored : 0.0;
}

// Kernel-internal order of a bf16 block: for each 16-wide k slice, for each group of 32 rows, the 64
// lanes of a wavefront hold 8 consecutive k each (lane l: row l % 32, k offset 8 * (l / 32)), which
// is the A/B operand layout of v_mfma_f32_32x32x16_bf16.  A pure permutation of the canonical block.
void bcsr_pack_fragments_bf16(const HostBcsr &in, int32_t b_row, int32_t b_col, std::vector<uint8_t> &packed) {
    const int64_t nb = (int64_t)in.block_col_idx.size();
    const int64_t bsz = (int64_t)b_row * b_col;
    packed.resize(in.blocks.size());
    const uint16_t *src = (const uint16_t *)in.blocks.data();
    uint16_t *dst = (uint16_t *)packed.data();
    const int32_t mtiles = b_row / 32, kslices = b_col / 16;
    parallel_chunks(nb, 4, [&](unsigned, int64_t b, int64_t e) {
        for (int64_t q = b; q < e; ++q) {
            const uint16_t *s = src + q * bsz;
            uint16_t *d = dst + q * bsz;
            for (int32_t ks = 0; ks < kslices; ++ks)
                for (int32_t mt = 0; mt < mtiles; ++mt)
                    for (int32_t lane = 0; lane < 64; ++lane) {
                        int32_t row = mt * 32 + lane % 32, col = ks * 16 + 8 * (lane / 32);
                        std::memcpy(d, s + (int64_t)row * b_col + col, 16);
                        d += 8;
                    }
        }
    });
}

// Kernel-internal order of an fp32 block: for each 16-wide k slice, each group of 32 rows and each group of
// 8 k, lane l of a wavefront holds the 4 values A[l % 32][2t + l / 32], t = 0..3: the A operands of four
// consecutive v_mfma_f32_32x32x2_f32 (lane l feeds row l % 32, k index l / 32).  A pure permutation.
void bcsr_pack_fragments_f32(const HostBcsr &in, int32_t b_row, int32_t b_col, std::vector<uint8_t> &packed) {
    const int64_t nb = (int64_t)in.block_col_idx.size();
    const int64_t bsz = (int64_t)b_row * b_col;
    packed.resize(in.blocks.size());
    const uint32_t *src = (const uint32_t *)in.blocks.data();
    uint32_t *dst = (uint32_t *)packed.data();
    const int32_t mtiles = b_row / 32, kslices = b_col / 16;
    parallel_chunks(nb, 4, [&](unsigned, int64_t b, int64_t e) {
        for (int64_t q = b; q < e; ++q) {
            const uint32_t *s = src + q * bsz;
            uint32_t *d = dst + q * bsz;
            for (int32_t ks = 0; ks < kslices; ++ks)
                for (int32_t mt = 0; mt < mtiles; ++mt)
                    for (int32_t kg = 0; kg < 2; ++kg)
                        for (int32_t lane = 0; lane < 64; ++lane)
                            for (int32_t t = 0; t < 4; ++t) {
                                int32_t row = mt * 32 + lane % 32, col = ks * 16 + kg * 8 + 2 * t + lane / 32;
                                *d++ = s[(int64_t)row * b_col + col];
                            }
        }
    });
}

// ------------------------------------------------------------------------------------------ WCSR
namespace {

// Columns of one window, ascending with duplicates between rows removed: sort the window's CSR entries (they
// are one contiguous range of col_idx) by column.  A k-way merge of the sorted rows costs rows x distinct
// columns and was 30x slower for 64-row windows with ~1000 columns.
// key = column << 32 | entry index inside the window (the window's entries are fewer than 2^31).
struct WindowSorter {
    std::vector<uint64_t> key;
    std::vector<uint8_t> row_of;  // row inside the window of each entry

    // distinct columns only
    int64_t count(const int32_t *row_ptr, const int32_t *col_idx, int64_t r0, int64_t r1) {
        const int64_t p0 = row_ptr[r0], n = row_ptr[r1] - p0;
        if (r1 - r0 == 1) return n;  // a row's columns are distinct already
        key.resize((size_t)n);
        for (int64_t e = 0; e < n; ++e) key[e] = (uint32_t)col_idx[p0 + e];
        std::sort(key.begin(), key.end());
        return (int64_t)(std::unique(key.begin(), key.end()) - key.begin());
    }

    // emit(t, col) once per distinct column in ascending order with its rank t; hit(t, row_in_window, p) once
    // per CSR entry p that sits in that column
    template <class Emit, class Hit>
    void place(const int32_t *row_ptr, const int32_t *col_idx, int64_t r0, int64_t r1, Emit emit, Hit hit) {
        const int64_t p0 = row_ptr[r0], n = row_ptr[r1] - p0;
        key.resize((size_t)n);
        row_of.resize((size_t)n);
        for (int64_t r = r0; r < r1; ++r)
            for (int64_t p = row_ptr[r]; p < row_ptr[r + 1]; ++p) {
                key[p - p0] = ((uint64_t)(uint32_t)col_idx[p] << 32) | (uint64_t)(p - p0);
                row_of[p - p0] = (uint8_t)(r - r0);
            }
        std::sort(key.begin(), key.end());
        int64_t t = -1;
        int32_t prev = -1;
        for (int64_t i = 0; i < n; ++i) {
            const int32_t col = (int32_t)(key[i] >> 32);
            const int64_t e = (int64_t)(key[i] & 0xFFFFFFFFu);
            if (col != prev) {
                emit(++t, col);
                prev = col;
            }
            hit(t, (int)row_of[e], p0 + e);
        }
    }
};

}  // namespace

bool csr_to_wcsr(int64_t m, int64_t k, const int32_t *row_ptr, const int32_t *col_idx, const void *values,
                 size_t esize, int32_t b_row, int32_t b_col, HostWcsr &out) {
    (void)k;
    const int64_t nw = ceil_div(m, b_row);
    out.window_row_ptr.assign(nw + 1, 0);
    parallel_chunks(nw, 64, [&](unsigned, int64_t b, int64_t e) {
        WindowSorter ws;
        for (int64_t w = b; w < e; ++w) {
            int64_t r0 = w * b_row, r1 = std::min<int64_t>(m, r0 + b_row);
            int64_t u = ws.count(row_ptr, col_idx, r0, r1);
            out.window_row_ptr[w + 1] = (int32_t)(ceil_div(u, b_col) * b_col);
        }
    });
    int64_t total = 0;  // packed positions are 32-bit: padding can push them past what the entries needed
    for (int64_t w = 0; w < nw; ++w) total += out.window_row_ptr[w + 1];
    if (total > INT32_MAX) return false;
    for (int64_t w = 0; w < nw; ++w) out.window_row_ptr[w + 1] += out.window_row_ptr[w];
    const int64_t padded = out.window_row_ptr[nw];
    out.window_col_idx.assign(padded, -1);
    out.values.reset((size_t)padded * b_row * esize);
    const int64_t tile = (int64_t)b_row * b_col;
    parallel_chunks(nw, 64, [&](unsigned, int64_t b, int64_t e) {
        WindowSorter ws;
        for (int64_t w = b; w < e; ++w) {
            int64_t r0 = w * b_row, r1 = std::min<int64_t>(m, r0 + b_row);
            const int64_t p0 = out.window_row_ptr[w];
            ws.place(
                row_ptr, col_idx, r0, r1, [&](int64_t t, int32_t col) { out.window_col_idx[p0 + t] = col; },
                [&](int64_t t, int r, int64_t p) {
                    int64_t pc = p0 + t;
                    size_t dst = (size_t)((pc / b_col) * tile + (int64_t)r * b_col + pc % b_col) * esize;
                    std::memcpy(out.values.data() + dst, (const uint8_t *)values + (size_t)p * esize, esize);
                });
        }
    });
    return true;
}

void wcsr_tasks_host(const std::vector<int32_t> &wrp, int32_t task_cols, std::vector<int32_t> &tasks) {
    tasks.clear();
    for (size_t w = 0; w + 1 < wrp.size(); ++w) {
        const int32_t lo = wrp[w], hi = wrp[w + 1];
        const int32_t split = (hi - lo > task_cols) ? 1 : 0;
        for (int64_t c = lo; c < hi; c += task_cols) {  // 64-bit: position + task_cols may pass 2^31
            tasks.push_back((int32_t)w);
            tasks.push_back((int32_t)c);
            tasks.push_back((int32_t)std::min<int64_t>(hi, c + task_cols));
            tasks.push_back(split);
        }
    }
}

namespace {

// Reorders tasks (four ints each, four tasks to a workgroup) so that each of the 8 XCDs, which take workgroups
// round-robin, gets one contiguous range of the given order with an eighth of the weight: tasks that are neighbours
// in the order then meet in one L2.  Shorter ranges are filled up with empty tasks.  Lists too short for that stay (false).
bool deal_to_xcds(std::vector<int32_t> &tasks, const std::vector<int64_t> &weight) {
    const size_t n = weight.size();
    if (n < 256) return false;  // less than a workgroup per compute unit and XCD to tell apart
    int64_t total = 0;
    for (int64_t w : weight) total += w;
    size_t cut[9] = {0};
    int64_t sum = 0;
    int x = 1;
    for (size_t t = 0; t < n; ++t) {
        while (x < 8 && sum >= total * x / 8) cut[x++] = t;
        sum += weight[t];
    }
    while (x < 9) cut[x++] = n;
    size_t most = 0;
    for (x = 0; x < 8; ++x) most = std::max(most, cut[x + 1] - cut[x]);
    most = (most + 3) / 4 * 4;
    std::vector<int32_t> dealt(most * 8 * 4, 0);
    for (x = 0; x < 8; ++x)
        for (size_t t = cut[x]; t < cut[x + 1]; ++t) {
            const size_t i = t - cut[x], to = (i / 4 * 8 + x) * 4 + i % 4;
            std::copy(tasks.begin() + 4 * t, tasks.begin() + 4 * t + 4, dealt.begin() + 4 * to);
        }
    tasks.swap(dealt);
    return true;
}

}  // namespace

namespace {

// Collects tasks of consecutive whole rows, up to 63 of them and `target` entries each (a longer row is its own task).
struct RowRuns {
    const std::vector<int32_t> &row_ptr;
    int64_t target;
    std::vector<int32_t> tasks;
    std::vector<int64_t> weight;
    int64_t first = -1, last = -1;  // open task: rows [first, last)

    RowRuns(const std::vector<int32_t> &rp, int64_t t) : row_ptr(rp), target(t) {}
    void close() {
        if (first < 0) return;
        tasks.insert(tasks.end(), {(int32_t)first, (int32_t)(last - first), row_ptr[first], row_ptr[last]});
        weight.push_back(row_ptr[last] - row_ptr[first] + 2 * (last - first));
        first = -1;
    }
    void add(int64_t r, int64_t len) {
        if (first >= 0 && (last - first >= 63 || row_ptr[last] - row_ptr[first] + len > target)) close();
        if (first < 0) first = r;
        last = r + 1;
    }
};

// Enough tasks for four rounds of the chip's 8192 waves, 32 to 256 entries each.
int64_t run_target(int64_t entries) { return std::max<int64_t>(32, std::min<int64_t>(256, entries / 32768)); }

}  // namespace

void wcsr_build_rows(int64_t m, const int32_t *row_ptr, const int32_t *col_idx, size_t esize, int32_t b_row,
                     int32_t task_cols, const HostWcsr &in, HostRows &out) {
    const auto &wrp = in.window_row_ptr;
    const int64_t nw = (int64_t)wrp.size() - 1;
    // Bytes per packed column and per entry at 128 columns of B: the gathered row in both, the tile column and index
    // against column and value.  (Two entries in one packed column read the row of B once instead of twice.)
    const int64_t row_b = 128 * (int64_t)esize, tile_b = b_row * (int64_t)esize + 4, entry_b = 4 + (int64_t)esize;
    auto by_rows = [&](int64_t w) {
        const int64_t nnz = row_ptr[std::min<int64_t>(m, (w + 1) * b_row)] - row_ptr[w * b_row];
        int64_t padded = wrp[w + 1] - wrp[w], real = padded;
        while (real > 0 && in.window_col_idx[wrp[w] + real - 1] < 0) --real;
        // (the kernels' lists hold scratch rows as ints)
        if (in.ws_slot[w] >= 0 && (in.ws_slot[w] + ceil_div(padded, task_cols)) * b_row > (1ll << 31)) return false;
        return nnz * (row_b + entry_b) <= real * row_b + padded * tile_b;
    };
    out = HostRows();
    out.row_ptr.assign(m + 1, 0);
    int64_t entries = 0;
    std::vector<uint8_t> sparse((size_t)nw);
    for (int64_t w = 0; w < nw; ++w) {
        sparse[w] = by_rows(w);
        const int64_t r0 = w * b_row, r1 = std::min<int64_t>(m, r0 + b_row);
        if (sparse[w]) {
            if (out.runs.empty() || out.runs.back().second != row_ptr[r0]) out.runs.push_back({row_ptr[r0], row_ptr[r0]});
            out.runs.back().second = row_ptr[r1];
        }
        for (int64_t r = r0; r < r1; ++r) {
            if (sparse[w]) entries += row_ptr[r + 1] - row_ptr[r];
            out.row_ptr[r + 1] = (int32_t)entries;
        }
    }
    out.n_entries = entries;

    // Nearly dense rows: chunks that cover the same columns should run together, so that a row of B is fetched into an
    // XCD's L2 once for all of them.  An XCD holds up to 1024 waves; with R such rows cut every W columns they span
    // W * 1024 / R columns at a time.  Short spans hit L2 more often, long chunks pay their start less often: the best
    // time is at spans of 16 MB of B (64 rows of 200 000 entries over 2 000 000 columns, N = 64: 0.264 / 0.236 / 0.296 ms
    // at 4 / 8 / 16 MB there, where a row of B has 256 bytes, with one wave to a chunk's columns; 0.343 ms
    // with chunks of task_cols = 512; the present kernel takes 0.207 ms at 8 MB and finds 80 % of its lines in L2).  The span is counted at 128 columns of B.  Taken for the R longest rows for
    // which a chunk keeps 32 entries, when at least two of their entries meet in a column on average.
    const int64_t FIT = (16 << 20) / (128 * (int64_t)esize), MIN_CHUNK = 32;
    int32_t k_used = 1;
    std::vector<int64_t> longest;
    for (int64_t w = 0; w < nw; ++w)
        if (sparse[w])
            for (int64_t r = w * b_row; r < std::min<int64_t>(m, (w + 1) * b_row); ++r)
                if (row_ptr[r + 1] - row_ptr[r] > task_cols) {
                    longest.push_back(row_ptr[r + 1] - row_ptr[r]);
                    k_used = std::max(k_used, col_idx[row_ptr[r + 1] - 1] + 1);
                }
    std::sort(longest.begin(), longest.end(), std::greater<int64_t>());
    int64_t dense_len = INT64_MAX, dense_width = 0, sum = 0;  // rows of at least dense_len entries: cut every dense_width columns
    for (size_t i = 0; i < longest.size(); ++i) {
        sum += longest[i];
        const int64_t W = FIT * (int64_t)(i + 1) / 1024;
        if (longest[i] * W >= MIN_CHUNK * (int64_t)k_used && sum >= 2 * (int64_t)k_used) dense_len = longest[i], dense_width = W;
    }

    out.dense_len = dense_len;
    int64_t in_long_rows = 0;
    for (int64_t len : longest) in_long_rows += len;
    RowRuns runs(out.row_ptr, run_target(entries - in_long_rows));
    std::vector<int32_t> chunks;
    std::vector<std::pair<int32_t, int64_t>> chunk_key;  // (first column, index)
    for (int64_t w = 0; w < nw; ++w) {
        if (!sparse[w]) {
            runs.close();
            continue;
        }
        const int64_t r0 = w * b_row, r1 = std::min<int64_t>(m, r0 + b_row);
        int64_t slot = in.ws_slot[w] >= 0 ? (int64_t)in.ws_slot[w] * b_row : -1;
        for (int64_t r = r0; r < r1; ++r) {
            const int64_t len = row_ptr[r + 1] - row_ptr[r];
            if (len > task_cols) {  // (then the window is split and owns at least this many rows of scratch)
                runs.close();
                int64_t step = task_cols;
                if (len >= dense_len) {  // (no more chunks than the row's share of its window's scratch rows)
                    const int64_t rows_left = (int64_t)ceil_div(wrp[w + 1] - wrp[w], task_cols) * b_row;
                    // whole batches of the kernel: 64 entries at the widths where it matters most
                    step = std::max<int64_t>(1, (len * dense_width / k_used + 32) / 64) * 64;
                    step = std::max(step, ceil_div(2 * (row_ptr[r1] - row_ptr[r0]), rows_left));
                    step = std::min<int64_t>(task_cols, step);
                }
                const int64_t parts = ceil_div(len, step);
                out.split.insert(out.split.end(), {(int32_t)r, (int32_t)slot, (int32_t)parts, 0});
                for (int64_t j = 0; j < parts; ++j) {
                    const int64_t lo = j * step, hi = std::min<int64_t>(len, lo + step);
                    chunk_key.push_back({col_idx[row_ptr[r] + lo], (int64_t)chunk_key.size()});
                    chunks.insert(chunks.end(), {(int32_t)r, (int32_t)slot, (int32_t)(out.row_ptr[r] + lo),
                                                 (int32_t)(out.row_ptr[r] + hi)});
                    ++slot;
                }
                continue;
            }
            runs.add(r, len);
        }
    }
    runs.close();
    std::sort(chunk_key.begin(), chunk_key.end());
    std::vector<int64_t> chunk_weight;
    for (auto &c : chunk_key) {
        const int32_t *t = chunks.data() + 4 * c.second;
        out.chunks.insert(out.chunks.end(), t, t + 4);
        chunk_weight.push_back(t[3] - t[2]);
    }
    deal_to_xcds(out.chunks, chunk_weight);
    deal_to_xcds(runs.tasks, runs.weight);
    out.tasks.swap(runs.tasks);

    // the windows that stay with the tile kernels
    std::vector<int64_t> tile_weight;
    for (int64_t w = 0; w < nw; ++w) {
        if (sparse[w]) continue;
        const int32_t lo = wrp[w], hi = wrp[w + 1], split = hi - lo > task_cols;
        if (split) out.tile_split.push_back((int32_t)w);
        for (int64_t c = lo; c < hi; c += task_cols) {
            const int64_t e = std::min<int64_t>(hi, c + task_cols);
            out.tile_tasks.insert(out.tile_tasks.end(), {(int32_t)w, (int32_t)c, (int32_t)e, split});
            tile_weight.push_back(e - c + 16);
        }
    }
    // Neighbouring windows of a band share rows of B.  Lists that the chip holds at once: one range for each XCD (60 000 rows,
    // band of 27, N = 256, height 16: bf16 19.3 against 16.8 us, fp32 34.9 / 34.6; 20 000 rows, band of 9, fp32 9.5 / 8.5).  Longer ones
    // round-robin: they sweep the band anyway, and ranges are up to 3 % slower (1 000 000 rows, band of 13 and 24 long rows).
    if (tile_weight.size() <= 4096) out.tiles_dealt = deal_to_xcds(out.tile_tasks, tile_weight);
}

// Which rows walk in groups (asp_wcsr_groups.hip), and how.
//
// The columns are cut into 8 ranges of equal work.  A row leaves one or several pieces in each range that it has entries in,
// and the pieces of a range are dealt to that range's tasks by themselves, the longest to the task with the least so far: a
// task holds as many entries as its neighbours whatever columns the rows store, all of them or those of a community.  A piece
// is a partial sum that is written and read once more, so rows take part from 8 entries a range on, the longest as many as 256
// tasks a range hold: with more, an XCD's waves would walk the columns a second time (rows that cannot go by whole rows
// because they are longer than task_cols do so all the same).  Rows with more than half of a task's share in a range leave
// several pieces there, entry by entry, and so that a sum has at most 160 terms and no more than task_cols: fp32 sums in one piece a
// range were twice as far from the 64-bit ones as chunks of task_cols = 512.
// Not done for a few nearly dense rows (the chunks of asp_wcsr_rows.hip find their rows of B in L2 already: 2 000 000
// rows with 64 of 200 000 entries, N = 64 216 us in chunks and 219 here), where the rows share few columns (two entries a column
// on average), for less than 64 entries a task (16 915 rows with 118 000 entries, N = 200 36 us by rows, 39 here), where scratch memory, whose
// size is that of the tiles' partial sums, does not hold the sums of all pieces, where a range would pass 2^24 columns, where one
// range has a quarter more to walk than the mean, and where short tasks would make short pieces (524 288 rows of Zipf lengths, fp32, N
// = 128, task_cols = 16 / 32 / 64 / 128: 692 / 568 / 538 / 555 us by rows, 732 / 608 / 488 / 460 here; 200 003 rows, bf16, 253 / 149 /
// 112 / 108 and 219 / 154 / 116 / 110).
void wcsr_build_groups(int64_t m, const int32_t *row_ptr, const int32_t *col_idx, const void *values, size_t esize,
                       int32_t b_row, int32_t task_cols, const HostWcsr &in, const HostRows &rows, HostGroups &out) {
    constexpr int64_t S = HostGroups::RANGES, MIN_PIECE = 8, GROUPS = 256, MIN_ROWS = 128, MIN_TASK = 64, MAX_TERMS = 128, NEAR_ENTRIES = 4500000, MIN_TASK_COLS = 48;
    const int64_t R = HostGroups::rows(esize);
    out = HostGroups();
    if (task_cols < MIN_TASK_COLS) return;
    const auto &wrp = in.window_row_ptr;
    const int64_t nw = (int64_t)wrp.size() - 1;
    auto walked = [&](int64_t r) { return rows.row_ptr[r + 1] > rows.row_ptr[r]; };
    auto length = [&](int64_t r) { return (int64_t)row_ptr[r + 1] - row_ptr[r]; };
    std::vector<int32_t> longest;  // rows, longest first
    for (int64_t r = 0; r < m; ++r)
        if (walked(r) && length(r) >= S * MIN_PIECE) longest.push_back((int32_t)r);
    if ((int64_t)longest.size() < MIN_ROWS) return;
    std::sort(longest.begin(), longest.end(), [&](int32_t a, int32_t b) {
        return length(a) != length(b) ? length(a) > length(b) : a < b;
    });
    const int64_t shortest = length(longest.back());
    int64_t n = std::min<int64_t>(longest.size(), GROUPS * R);
    while (n < (int64_t)longest.size() && length(longest[n]) > task_cols) ++n;
    longest.resize((size_t)n);

    int64_t total = 0;
    int32_t k_used = 1;
    for (int32_t r : longest) total += length(r), k_used = std::max(k_used, col_idx[row_ptr[r + 1] - 1] + 1);
    if (total < 2 * (int64_t)k_used || total < MIN_TASK * GROUPS * S) return;

    // ranges of columns with as many entries each, to 1 / 65536 of the columns
    int shift = 0;
    while ((k_used >> shift) >= 65536) ++shift;
    std::vector<int64_t> count(65537, 0);
    int64_t counted = 0;
    for (int32_t r : longest)  // (every eighth entry tells; from another one in every row, or the first columns would count for more)
        for (int64_t p = (int64_t)row_ptr[r] + r % 8; p < row_ptr[r + 1]; p += 8, ++counted) ++count[col_idx[p] >> shift];
    std::vector<int32_t> start((size_t)S + 1, k_used);
    start[0] = 0;
    int64_t sum = 0, s = 1;
    for (int64_t b = 0; b < 65537 && s < S; ++b) {
        while (s < S && sum >= counted * s / S) start[s++] = (int32_t)std::min<int64_t>(b << shift, k_used);
        sum += count[b];
    }
    for (s = 0; s < S; ++s) out.span = std::max<int64_t>(out.span, start[s + 1] - start[s]);
    if (out.span > (1 << 24)) return;

    // where each row crosses from one range to the next, and how many pieces it leaves in each
    std::vector<int32_t> cuts((size_t)(n * (S + 1)));
    parallel_chunks(n, 256, [&](unsigned, int64_t b, int64_t e) {
        for (int64_t i = b; i < e; ++i) {
            const int32_t *lo = col_idx + row_ptr[longest[i]], *hi = col_idx + row_ptr[longest[i] + 1], *it = lo;
            for (int64_t j = 0; j <= S; ++j) {
                it = j == S ? hi : std::lower_bound(it, hi, start[j]);
                cuts[i * (S + 1) + j] = (int32_t)(it - lo);
            }
        }
    });
    const int64_t share = std::max(MIN_PIECE, total / (2 * GROUPS * S));
    const int64_t cut_at = std::min<int64_t>({MAX_TERMS, share, task_cols}), most = std::min<int64_t>(cut_at * 5 / 4, task_cols);
    auto in_range = [&](int64_t i, int64_t j) { return (int64_t)cuts[i * (S + 1) + j + 1] - cuts[i * (S + 1) + j]; };
    auto pieces = [&](int64_t i, int64_t j) {
        const int64_t c = in_range(i, j);
        return c <= most ? (int64_t)(c > 0) : ceil_div(c, cut_at);
    };
    int64_t n_pieces[S] = {0};
    for (int64_t i = 0; i < n; ++i)
        for (int64_t j = 0; j < S; ++j) n_pieces[j] += pieces(i, j);
    std::vector<int64_t> kept;  // the rows that take part, as places in `longest`
    for (int64_t i = n - 1; i >= 0; --i) {
        bool full = false;
        for (int64_t j = 0; j < S; ++j) full |= n_pieces[j] > GROUPS * R && in_range(i, j) > 0;
        if (full && length(longest[i]) <= task_cols) {
            total -= length(longest[i]);
            for (int64_t j = 0; j < S; ++j) n_pieces[j] -= pieces(i, j);
        } else {
            kept.push_back(i);
        }
    }
    std::reverse(kept.begin(), kept.end());
    const int64_t widest = *std::max_element(n_pieces, n_pieces + S);
    const int64_t G = std::min(std::max(GROUPS, ceil_div(widest, R)), widest);
    if (G * S > (1 << 24)) return;  // (one launch takes fewer than 2^32 threads)

    // scratch rows: one for every piece, those of a row one after the other, in the windows whose own split rows are all here
    std::vector<uint8_t> grouped((size_t)m, 0);
    for (int64_t i : kept) grouped[longest[i]] = 1;
    std::vector<std::pair<int64_t, int64_t>> room;
    for (int64_t w = 0; w < nw; ++w) {
        if (in.ws_slot[w] < 0) continue;
        const int64_t r0 = w * b_row, r1 = std::min<int64_t>(m, r0 + b_row);
        bool is_free = rows.row_ptr[r1] > rows.row_ptr[r0];
        for (int64_t r = r0; r < r1 && is_free; ++r) is_free = length(r) <= task_cols || grouped[r];
        if (!is_free) continue;
        const int64_t lo = (int64_t)in.ws_slot[w] * b_row, hi = lo + ceil_div(wrp[w + 1] - wrp[w], task_cols) * b_row;
        if (!room.empty() && room.back().second == lo) room.back().second = hi;
        else room.push_back({lo, hi});
    }
    struct Piece {
        int32_t row, part, parts, size;  // row: its place in `longest`; entries c with c % parts == part of the row's range
        int32_t slot;
    };
    std::vector<Piece> in_ranges[S];
    size_t at = 0;
    for (int64_t i : kept) {
        int64_t need = 0;
        for (int64_t j = 0; j < S; ++j) need += pieces(i, j);
        while (at < room.size() && room[at].second - room[at].first < need) ++at;
        if (at == room.size()) return;
        out.split.insert(out.split.end(), {longest[i], (int32_t)room[at].first, (int32_t)need, 0});
        for (int64_t j = 0; j < S; ++j) {
            const int64_t c = in_range(i, j), np = pieces(i, j);
            for (int64_t p = 0; p < np; ++p)
                in_ranges[j].push_back({(int32_t)i, (int32_t)p, (int32_t)np, (int32_t)ceil_div(c - p, np), (int32_t)room[at].first++});
        }
    }

    // range j of group g is task j G + g: pieces to tasks, the longest first to the task with the fewest entries so far
    std::vector<std::vector<Piece>> task((size_t)(S * G));
    std::vector<int64_t> n_entries((size_t)(S * G), 0);
    parallel_chunks(S, 1, [&](unsigned, int64_t b, int64_t e) {
        for (int64_t j = b; j < e; ++j) {
            auto &all = in_ranges[j];
            std::stable_sort(all.begin(), all.end(), [](const Piece &x, const Piece &y) { return x.size > y.size; });
            std::vector<std::pair<int64_t, int64_t>> heap;  // (entries, group), least first
            for (int64_t g = 0; g < G; ++g) heap.push_back({0, g});
            const std::greater<std::pair<int64_t, int64_t>> more;
            for (const Piece &p : all) {
                std::pop_heap(heap.begin(), heap.end(), more);
                auto &least = heap.back();
                task[j * G + least.second].push_back(p);
                n_entries[j * G + least.second] = least.first += p.size;
                if ((int64_t)task[j * G + least.second].size() == R) heap.pop_back();
                else std::push_heap(heap.begin(), heap.end(), more);
            }
        }
    }, total);
    if (*std::max_element(n_entries.begin(), n_entries.end()) * (4 * S * G) > 5 * total + 64 * S * G) {
        out = HostGroups();
        return;
    }

    std::vector<int64_t> first((size_t)(S * G) + 1, 0);
    for (int64_t t = 0; t < S * G; ++t) first[t + 1] = first[t] + ceil_div(n_entries[t], 16) * 16;
    if (first[S * G] / 16 > INT32_MAX) {
        out = HostGroups();
        return;
    }
    out.entries.reset((size_t)first[S * G] * 8);
    uint64_t *const entries = (uint64_t *)out.entries.data();
    out.tasks.resize((size_t)(S * G) * 4);
    out.slots.assign((size_t)(S * G * R), -1);
    parallel_chunks(S * G, 8, [&](unsigned, int64_t b, int64_t e) {
        for (int64_t t = b; t < e; ++t) {
            const int64_t j = t / G;
            uint64_t *const dst = entries + first[t], *const end = entries + first[t + 1], *to = dst;
            for (size_t i = 0; i < task[t].size(); ++i) {
                const Piece &p = task[t][i];
                out.slots[t * R + i] = p.slot;
                const int64_t row = row_ptr[longest[p.row]], c1 = cuts[p.row * (S + 1) + j + 1];
                for (int64_t c = cuts[p.row * (S + 1) + j] + p.part; c < c1; c += p.parts) {
                    const int64_t q = row + c;
                    uint32_t v = esize == 2 ? (uint32_t)((const uint16_t *)values)[q] << 16 : ((const uint32_t *)values)[q];
                    *to++ = ((uint64_t)((uint32_t)(col_idx[q] - start[j]) << 8 | (uint32_t)i) << 32) | v;
                }
            }
            std::sort(dst, to);
            const uint64_t fill = to > dst ? (to[-1] >> 40 << 40) | (uint64_t)R << 32 : 0;
            for (; to < end; ++to) *to = fill;
            for (to = dst; to < end; ++to) *to = *to >> 32 | *to << 32;  // the key is the first word
            const int32_t td[4] = {(int32_t)(first[t] / 16), (int32_t)((end - dst) / 16), start[j], 0};
            std::copy(td, td + 4, out.tasks.begin() + 4 * t);
        }
    });

    // the rest: chunks of other rows stay where they are dealt to, runs of whole rows without the grouped ones
    bool any = false;
    out.chunks = rows.chunks;
    for (size_t c = 0; c < out.chunks.size(); c += 4) {
        if (out.chunks[c + 2] < out.chunks[c + 3] && !grouped[out.chunks[c]]) any = true;
        else std::fill(out.chunks.begin() + c, out.chunks.begin() + c + 4, 0);
    }
    if (!any) out.chunks.clear();
    int64_t left = rows.n_entries - total;
    for (size_t i = 0; i < rows.split.size(); i += 4)
        if (!grouped[rows.split[i]]) {
            out.split.insert(out.split.end(), rows.split.begin() + i, rows.split.begin() + i + 4);
            left -= length(rows.split[i]);
        }
    // rows of many pieces first, which are added by more threads (wcsr_rows_sum_launch)
    std::vector<int32_t> by_count[2];
    for (size_t i = 0; i < out.split.size(); i += 4) {
        auto &to = by_count[out.split[i + 2] > HostGroups::MANY_PIECES ? 0 : 1];
        to.insert(to.end(), out.split.begin() + i, out.split.begin() + i + 4);
    }
    out.n_many = (int64_t)by_count[0].size() / 4;
    out.split = std::move(by_count[0]);
    out.split.insert(out.split.end(), by_count[1].begin(), by_count[1].end());
    // How many columns the long rows store where the walk by rows is at one time: the different ones in the rows of 2^17
    // consecutive entries, the mean of 16 places, where a quarter of those entries or more store a column again.  Asked where there
    // are many entries: with fewer, chunks of 512 are the last that the walk by rows ends with, and groups are the better ones on
    // any columns (204 512 rows, 4.0 million entries within 30 000 of the diagonal, fp32, N = 192 414 us by rows, 310 in groups;
    // 358 770 rows, 4.6 million within 3000, N = 100 265 / 290).
    if (rows.n_entries > NEAR_ENTRIES) {
        constexpr int64_t PLACES = 16, SPAN = 1 << 17;
        int64_t stored[PLACES], different[PLACES];
        parallel_chunks(PLACES, 1, [&](unsigned, int64_t b, int64_t e) {
            for (int64_t q = b; q < e; ++q) {
                const int64_t e0 = (rows.n_entries - SPAN) * q / (PLACES - 1);
                std::vector<int32_t> cols;
                for (int64_t r = std::upper_bound(rows.row_ptr.begin(), rows.row_ptr.end(), e0) - rows.row_ptr.begin() - 1;
                     r < m && rows.row_ptr[r] < e0 + SPAN; ++r)
                    if (walked(r) && length(r) >= shortest) cols.insert(cols.end(), col_idx + row_ptr[r], col_idx + row_ptr[r + 1]);
                std::sort(cols.begin(), cols.end());
                stored[q] = (int64_t)cols.size();
                different[q] = std::unique(cols.begin(), cols.end()) - cols.begin();
            }
        }, rows.n_entries);
        const int64_t all = std::accumulate(stored, stored + PLACES, (int64_t)0), diff = std::accumulate(different, different + PLACES, (int64_t)0);
        if (4 * diff < 3 * all) out.near_cols = std::max<int64_t>(1, diff / PLACES);
    }
    RowRuns runs(rows.row_ptr, run_target(left));
    for (int64_t w = 0; w < nw; ++w) {
        const int64_t r0 = w * b_row, r1 = std::min<int64_t>(m, r0 + b_row);
        if (rows.row_ptr[r1] == rows.row_ptr[r0] && row_ptr[r1] > row_ptr[r0]) {  // by tiles
            runs.close();
            continue;
        }
        for (int64_t r = r0; r < r1; ++r)
            if (grouped[r] || length(r) > task_cols) runs.close();
            else runs.add(r, length(r));
    }
    runs.close();
    deal_to_xcds(runs.tasks, runs.weight);
    out.row_tasks.swap(runs.tasks);
    out.n_groups = G;
}

// Nearly dense rows that walk their entries over columns of B in LDS (asp_wcsr_dense.hip): those whose chunks would be cut at the
// same columns, in equal numbers to a pass over B, 64 at most, when a column holds 4.5 entries of every pass in the mean (2 000 000 rows, band of
// 27, N = 64, long rows with a tenth of the columns, chunks / so: 32 of them 412 / 420 us, 48 452 / 424, 64 488 / 427), and each row has
// scratch rows for 64 ranges of columns.  (So a row has 18 entries in a block of 256 columns in the mean, and the table of their first entries
// takes a 36th of the entries' bytes at most.)  All of them or none: 36 rows left of 100 lose more as chunks, whose rows of B are met less
// often then, than the others gain (600 000 rows, N = 64 139 by chunks, 171).  The rest keeps its lists.
void wcsr_build_dense(int64_t m, const int32_t *row_ptr, const int32_t *col_idx, int32_t b_row, int32_t task_cols, const HostWcsr &in,
                      const HostRows &rows, HostDense &out) {
    constexpr int64_t MIN_RANGES = 64;
    out = HostDense();
    auto length = [&](int32_t r) { return (int64_t)row_ptr[r + 1] - row_ptr[r]; };
    int32_t k_used = 1;
    std::vector<int32_t> candidates;  // (rows are in order: those of a window are together)
    for (size_t i = 0; i < rows.split.size(); i += 4)
        if (length(rows.split[i]) >= rows.dense_len) {
            candidates.push_back(rows.split[i]);
            k_used = std::max(k_used, col_idx[row_ptr[rows.split[i] + 1] - 1] + 1);
        }
    if (candidates.empty()) return;
    const size_t per_pass = ceil_div(candidates.size(), ceil_div(candidates.size(), HostDense::ROWS));
    int64_t entries = 0, meet = INT64_MAX;
    std::vector<uint8_t> dense((size_t)m, 0);
    for (size_t c = 0; c < candidates.size(); c += per_pass) {
        const size_t end = std::min(candidates.size(), c + per_pass);
        int64_t sum = 0;
        for (size_t i = c; i < end; ++i) sum += length(candidates[i]), dense[candidates[i]] = 1;
        meet = std::min(meet, 10 * sum / k_used);
        entries += sum;
    }
    if (meet < 45) return;
    int64_t fewest = HostDense::RANGES;
    for (size_t i = 0; i < rows.split.size();) {
        const int64_t w = rows.split[i] / b_row;
        int64_t in_window = 0;
        bool all = true;
        size_t end = i;
        for (; end < rows.split.size() && rows.split[end] / b_row == w; end += 4) {
            if (dense[rows.split[end]]) ++in_window;
            else all = false;
        }
        // a row's scratch rows: an even share of its window's, or what its chunks had beside rows that stay with theirs
        const int64_t share = in_window > 0 ? ceil_div(in.window_row_ptr[w + 1] - in.window_row_ptr[w], task_cols) * b_row / in_window : 0;
        int64_t slot = (int64_t)in.ws_slot[w] * b_row;
        for (; i < end; i += 4) {
            if (!dense[rows.split[i]]) continue;
            fewest = std::min<int64_t>(fewest, all ? share : rows.split[i + 2]);
            out.rows.insert(out.rows.end(), {rows.split[i], (int32_t)(all ? slot : rows.split[i + 1]), 0, 0});
            slot += share;
        }
    }
    const int64_t n = (int64_t)out.rows.size() / 4, blocks = ceil_div(k_used, HostDense::COLS);
    if (n > 65535 * HostDense::ROWS || std::min(fewest, blocks) < MIN_RANGES) return;
    out.per_pass = (int64_t)per_pass;
    out.meet_tenths = meet;
    out.blocks = blocks;
    out.ranges = std::min(fewest, blocks);
    out.ptr.resize((size_t)((blocks + 1) * n));
    parallel_chunks(n, 1, [&](unsigned, int64_t b, int64_t e) {
        for (int64_t i = b; i < e; ++i) {
            const int32_t r = out.rows[4 * i];
            const int32_t *const lo = col_idx + row_ptr[r], *const hi = col_idx + row_ptr[r + 1], *it = lo;
            for (int64_t j = 0; j <= blocks; ++j) {
                it = j == blocks ? hi : std::lower_bound(it, hi, (int32_t)(j * HostDense::COLS));
                out.ptr[i * (blocks + 1) + j] = (int32_t)(rows.row_ptr[r] + (it - lo));
            }
        }
    }, entries);
    for (int64_t i = 0; i < n; ++i)
        out.split.insert(out.split.end(), {out.rows[4 * i], out.rows[4 * i + 1], (int32_t)out.ranges, 0});
    for (size_t i = 0; i < rows.split.size(); i += 4)
        if (!dense[rows.split[i]]) out.split.insert(out.split.end(), rows.split.begin() + i, rows.split.begin() + i + 4);
    out.tasks = rows.tasks;
    out.chunks = rows.chunks;
    bool any = false;
    for (size_t c = 0; c < out.chunks.size(); c += 4) {
        if (out.chunks[c + 2] < out.chunks[c + 3] && !dense[out.chunks[c]]) any = true;
        else std::fill(out.chunks.begin() + c, out.chunks.begin() + c + 4, 0);
    }
    if (!any) out.chunks.clear();
}

// Chunks and single rows that a workgroup takes instead of a wave: those with more entries than half of what each of the chip's 8192
// waves would have, and more than 64.  They run on the XCD that the lists have them on.
// us, by waves / so: 19 732 rows of Zipf lengths, degree 17, fp32, N = 64 29.1 / 15.4; 57 008, degree 24, N = 19 53 / 40;
// 182 898, degree 11, bf16, N = 32 68 / 56; 51 331, degree 9, fp32, N = 221 86 / 71; with more entries less (2^20 rows, N = 31 473 /
// 466).  From as many entries on as such a wave would have, rather than half: up to 1.1 / 1.3 times as long; from a quarter on: the same.
// The chunks of nearly dense rows are not among them: they are many, and meet in L2 as they are dealt.  Where a wave walks an entry at a
// time it can pay to share those of more than 100 entries too (wcsr_share_chunks): `wide` holds the lists for that.
void wcsr_build_teams(int64_t n_entries, const HostRows &rows, std::vector<int32_t> &chunks, std::vector<int32_t> &tasks,
                      std::vector<int32_t> &teams, HostWide &wide) {
    const int64_t least = std::max<int64_t>(65, n_entries / (2 * 8192));
    auto length = [&](int32_t r) { return (int64_t)rows.row_ptr[r + 1] - rows.row_ptr[r]; };
    std::vector<int32_t> of_xcd[8];  // four to a workgroup, which the XCDs take round-robin
    // takes tasks out of a list
    auto take = [&](std::vector<int32_t> &list, bool whole, auto fits) {
        bool left = false;
        for (size_t i = 0; i < list.size(); i += 4) {
            if (whole ? list[i + 1] == 0 : list[i + 2] >= list[i + 3]) continue;  // fills up
            if (!fits(&list[i])) {
                left = true;
                continue;
            }
            auto &to = of_xcd[i / 16 % 8];
            to.insert(to.end(), {list[i], whole ? -1 : list[i + 1], list[i + 2], list[i + 3]});
            std::fill(list.begin() + i, list.begin() + i + 4, 0);
        }
        if (!left) list.clear();
    };
    // a list of them, `per` to a workgroup
    auto deal = [&](std::vector<int32_t> &out, size_t per) {
        size_t most = 0;
        for (auto &v : of_xcd) most = std::max(most, ceil_div(v.size() / 4, per) * per);
        out.assign(most * 8 * 4, 0);
        for (size_t x = 0; x < 8; ++x) {
            for (size_t i = 0; i < of_xcd[x].size() / 4; ++i)
                std::copy(of_xcd[x].begin() + 4 * i, of_xcd[x].begin() + 4 * i + 4, out.begin() + 4 * ((i / per * 8 + x) * per + i % per));
            of_xcd[x].clear();
        }
    };
    take(chunks, false, [&](const int32_t *c) { return c[3] - c[2] >= least && length(c[0]) < rows.dense_len; });
    take(tasks, true, [&](const int32_t *c) { return c[3] - c[2] >= least && c[1] == 1; });
    deal(teams, 1);

    wide = HostWide();
    std::vector<uint8_t> shared;  // rows
    for (size_t i = 0; i < rows.split.size(); i += 4)
        if (const int32_t r = rows.split[i]; length(r) >= rows.dense_len && length(r) > std::max<int64_t>(least, 100) * rows.split[i + 2]) {
            shared.resize(rows.row_ptr.size());
            shared[r] = 1;
        }
    if (shared.empty()) return;
    wide.chunks = chunks;
    take(wide.chunks, false, [&](const int32_t *c) {
        if (!shared[c[0]]) return false;
        ++wide.count;
        wide.len += c[3] - c[2];
        return true;
    });
    deal(wide.teams, 1);
    if (wide.count > 0) wide.len /= wide.count;
    take(wide.chunks, false, [](const int32_t *) { return true; });
    deal(wide.chunks, 4);
}

void wcsr_zero_windows(const std::vector<int32_t> &wrp, int32_t task_cols, std::vector<int32_t> &zw) {
    zw.clear();
    for (size_t w = 0; w + 1 < wrp.size(); ++w) {
        int32_t n = wrp[w + 1] - wrp[w];
        if (n == 0 || n > task_cols) zw.push_back((int32_t)w);
    }
}

}  // namespace asp

// Prints the work lists that the converters make of a synthetic matrix, for tests/test_wcsr_lists.py and test_bcsr_order.py.
//   order L..        BCSR block-rows of L blocks each: the orders of the tile kernels in 16, 32 and 64 lists
//   shares L..       the lists for shared N-tiles, and what they weigh
//   wide N K X C L.. a launch of N 128x512 tiles to a block-row, K columns (X = 1: K-contiguous), C compute units: how many are
//                    shared, the runs of the pairs, and what the heaviest workgroup walks with 0, 1, ... shared ones
//   ring N K B W X P L..  a launch of the ring kernel: N column tiles W wide, blocks of B, P workgroups to a compute unit: the group
//                    and order taken, and for each what the heaviest workgroup walks and the starts of the XCDs' runs
//   staged T C L..   the register-staged kernel's launch of T column tiles on C compute units: 1 (longest block-row first) or 0
//                    (as stored), the starts of the XCDs' runs, the order longest first
//   groups M K W T E L..  M rows of K columns with L.. entries in turn (in W adjacent columns, other ones for every row; 0: in
//                    all), tasks of T columns, values of E bytes: the products of the rows' values (1, 2, 3) with (column % 13 + 1),
//                    by the lists of groups, chunks and runs: "row r difference times" ("tile r times" for rows that go tile by
//                    tile); and how many groups there are, the entries of their largest task and of all, the most terms of a
//                    sum in a task, the scratch rows there are and that they use, the columns that near rows meet in, and how many
//                    rows have their scratch rows added by many threads, the fewest of one and the most of another; and how many of
//                    how many split rows a product with 128 columns adds so
//   dense M K H T L..  M rows of K columns with L.. entries in turn, spread over all, in windows of H rows, tasks of T columns: the
//                    ranges and blocks of columns, the nearly dense rows, the size of the table of their first entries and the rows to a
//                    pass over B; the fewest entries of a pass; and, by their lists, "row r difference times" as above
//   teams M K H T L..  the same rows by waves and workgroups: how many workgroups, those for chunks of nearly dense rows, and how many
//                    these are, of how many entries; the least entries of the others, how many of them nearly dense rows have, and of
//                    what waves walk what is as long; chunks that change their XCD; and "row r difference times difference times" without and with the chunks shared
//   share D N C L    whether workgroups share C chunks of L entries for N columns, D: fp32 (0) or bf16 (1)
//   apply K R C T N..  whether R nearly dense rows over K columns, of whose chunks C can be shared, T tenths of an entry a column, go through
//                    LDS for N.. columns of B, 50 to a pass
//   launches W T     the walk by rows of W waves and T workgroups before them: first and end wave and workgroups of each launch
//   f32 B R U L N..  R block-rows of height B in fp32, U blocks, the longest row L, on 256 compute units: whether one wave takes a tile
//   unaligned B R N..  R block-rows of height B on 256 compute units: the tile width for N.. columns in rows that are not aligned
//   columns H T N..  T tasks of windows of height H in fp32: the columns of a lane for N.. columns
//   xt B R U L N     a BCSR handle of R block-rows, U blocks of B x B, the longest row L: the row tiles of the staged strips that N
//                    tokens on 256 compute units take in asp_spmm_xt, 0: none
//   slots S          two windows of 16 rows with 20 scattered entries each, tasks of 8 columns, scratch slots from S on
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "asp_bcsr_pipe.h"

static void print(const char *name, const std::vector<int32_t> &v, size_t width) {
    for (size_t i = 0; i < v.size(); i += width) {
        std::printf("%s", name);
        for (size_t j = 0; j < width; ++j) std::printf(" %d", v[i + j]);
        std::printf("\n");
    }
}

static int slots(int32_t first) {
    const int64_t m = 32, per_row = 20, k = m * per_row;
    std::vector<int32_t> rp(m + 1), ci(k);
    for (int64_t r = 0; r <= m; ++r) rp[r] = (int32_t)(r * per_row);
    for (int64_t r = 0; r < m; ++r)
        for (int64_t j = 0; j < per_row; ++j) ci[r * per_row + j] = (int32_t)(j * m + r);
    std::vector<float> values(k, 1.f);
    asp::HostWcsr w;
    if (!asp::csr_to_wcsr(m, k, rp.data(), ci.data(), values.data(), 4, 16, 8, w)) return 1;
    w.ws_slot = {first, first + 40};
    asp::HostRows rows;
    asp::wcsr_build_rows(m, rp.data(), ci.data(), 4, 16, 8, w, rows);
    print("split", rows.split, 4);
    print("chunk", rows.chunks, 4);
    print("tile", rows.tile_tasks, 4);
    print("tile_split", rows.tile_split, 1);
    return 0;
}

static void schedule(const std::vector<int32_t> &lengths, asp::HostBcsr &b) {
    b.block_row_ptr.assign(1, 0);
    for (int32_t n : lengths) {
        for (int32_t j = 0; j < n; ++j) b.block_col_idx.push_back(j);
        b.block_row_ptr.push_back((int32_t)b.block_col_idx.size());
    }
    asp::bcsr_build_schedule(b, asp::Orders::ALL);
}

static int shares(const std::vector<int32_t> &lengths) {
    asp::HostBcsr b;
    schedule(lengths, b);
    asp::BcsrShares s;
    asp::bcsr_build_shares(b, s);
    std::printf("infos %lld\n", (long long)s.infos);
    if (s.lists.empty()) return 0;
    const size_t whole = lengths.size() * 4, n = (size_t)b.n_nonempty * 4;
    print("whole", std::vector<int32_t>(s.lists.begin(), s.lists.begin() + whole), 4);
    for (int t = 1; t <= asp::BcsrShares::MAX_TILES; ++t) {
        if (t % 8 == 0) continue;
        const int slot = asp::BcsrShares::slot(t);
        char name[16];
        std::snprintf(name, sizeof name, "t%d", t);
        const auto info = s.lists.begin() + whole + slot * n;
        print(name, std::vector<int32_t>(info, info + n), 4);
        std::snprintf(name, sizeof name, "first%d", t);
        const auto first = s.lists.begin() + s.infos * 4 + slot * asp::BcsrShares::FIRST_PITCH;
        print(name, std::vector<int32_t>(first, first + asp::BcsrShares::FIRST_PITCH), 1);
        std::snprintf(name, sizeof name, "load%d", t);
        const auto load = s.load.begin() + slot * asp::BcsrShares::WORKERS;
        print(name, std::vector<int32_t>(load, load + asp::BcsrShares::WORKERS), 1);
    }
    return 0;
}

static int order(const std::vector<int32_t> &lengths) {
    asp::HostBcsr b;
    schedule(lengths, b);
    print("16", b.rank_info, 4);
    print("32", b.rank_info_32, 4);
    print("64", b.rank_info_64, 4);
    const std::vector<int64_t> *prefix[3] = {&b.sorted_weight_prefix, &b.weight_prefix_32, &b.weight_prefix_64};
    for (int i = 0; i < 3; ++i)
        for (int64_t v : *prefix[i]) std::printf("prefix%d %lld\n", 16 << i, (long long)v);
    return 0;
}

static int wide(int n_tiles, int64_t k, bool xt, int64_t n_cus, const std::vector<int32_t> &lengths) {
    asp::HostBcsr b;
    schedule(lengths, b);
    asp::BcsrShares s;
    asp::bcsr_build_shares(b, s);
    std::printf("shared %d\n", asp::wide_shared_tiles(b, s, k, xt, n_tiles, n_cus));
    const asp::XcdRuns runs = asp::cut_runs(b.sorted_weight_prefix, b.n_nonempty, n_tiles, 2);
    for (int x = 0; x <= 8; ++x) std::printf("start %d\n", runs.start[x]);
    std::printf("heaviest 0 %lld\n", (long long)asp::wide_heaviest(b, s, n_tiles, 0));
    for (int t = n_tiles % 8; t > 0 && t <= std::min(n_tiles, asp::BcsrShares::MAX_TILES); t += 8)
        std::printf("heaviest %d %lld\n", t, (long long)asp::wide_heaviest(b, s, n_tiles, t));
    return 0;
}

static int ring(int n_tiles, int64_t k, int b_row, int bn, bool xt, int per_cu, const std::vector<int32_t> &lengths) {
    asp::HostBcsr b;
    schedule(lengths, b);
    const asp::RingWalk taken = asp::ring_walk(b, k, b_row, bn, xt, n_tiles, 256, per_cu);
    std::printf("taken %d %d\n", taken.group_n, taken.lists);
    for (int group = 1; group <= 4; group *= 2)
        for (int lists = 16; lists <= 64; lists *= 2) {
            const int group_n = std::min(group, n_tiles);
            const auto &prefix = lists == 64 ? b.weight_prefix_64 : lists == 32 ? b.weight_prefix_32 : b.sorted_weight_prefix;
            const asp::XcdRuns runs = asp::cut_runs(prefix, lengths.size(), n_tiles, group_n);
            const asp::RingLoad most = asp::ring_heaviest(b, asp::RingWalk{group_n, lists}, n_tiles, 256, per_cu);
            std::printf("walk %d %d %lld", group_n, lists, (long long)most.workgroup);
            for (int x = 0; x <= 8; ++x) std::printf(" %d", runs.start[x]);
            std::printf("\n");
        }
    return 0;
}

static int staged(int n_tiles, int64_t n_cus, const std::vector<int32_t> &lengths) {
    asp::HostBcsr b;
    schedule(lengths, b);
    asp::XcdRuns runs;
    std::printf("sorted %d\n", (int)asp::register_staged_runs(b, n_tiles, n_cus, 256, runs));
    for (int x = 0; x <= 8; ++x) std::printf("start %d\n", runs.start[x]);
    print("order", b.by_length, 1);
    return 0;
}

static int groups(int64_t m, int64_t k, int64_t w, int32_t task_cols, size_t esize, const std::vector<int32_t> &lengths) {
    std::vector<int32_t> rp(1, 0), ci;
    const int64_t cols = w > 0 ? w : k;
    for (int64_t r = 0; r < m; ++r) {
        const int64_t n = lengths[r % lengths.size()], c0 = r * 7919 % (k / cols) * cols;
        for (int64_t j = 0; j < n; ++j) ci.push_back((int32_t)(c0 + j * cols / n + (r * 7919 + j) % std::max<int64_t>(1, cols / n)));
        rp.push_back((int32_t)ci.size());
    }
    std::vector<uint8_t> values(ci.size() * esize);
    for (size_t e = 0; e < ci.size(); ++e) {
        const float v = (float)(1 + e % 3);
        uint32_t bits;
        std::memcpy(&bits, &v, 4);
        if (esize == 4) std::memcpy(&values[e * 4], &bits, 4);
        else values[2 * e] = (uint8_t)(bits >> 16), values[2 * e + 1] = (uint8_t)(bits >> 24);
    }
    asp::HostWcsr hw;
    if (!asp::csr_to_wcsr(m, k, rp.data(), ci.data(), values.data(), esize, 16, 8, hw)) return 1;
    int64_t slots = 0;
    for (size_t i = 0; i + 1 < hw.window_row_ptr.size(); ++i) {
        const int64_t n = hw.window_row_ptr[i + 1] - hw.window_row_ptr[i];
        hw.ws_slot.push_back(n > task_cols ? (int32_t)slots : -1);
        if (n > task_cols) slots += asp::ceil_div(n, task_cols);
    }
    asp::HostRows rows;
    asp::wcsr_build_rows(m, rp.data(), ci.data(), esize, 16, task_cols, hw, rows);
    asp::HostGroups g;
    asp::wcsr_build_groups(m, rp.data(), ci.data(), values.data(), esize, 16, task_cols, hw, rows, g);
    auto b = [](int64_t col) { return (double)(col % 13 + 1); };
    std::vector<int64_t> at;  // where the entries walked row by row are
    for (auto &r : rows.runs)
        for (int64_t p = r.first; p < r.second; ++p) at.push_back(p);
    auto walk = [&](int64_t e0, int64_t e1) {
        double sum = 0;
        for (int64_t e = e0; e < e1; ++e) sum += (1 + at[e] % 3) * b(ci[at[e]]);
        return sum;
    };
    std::vector<double> ws(slots * 16, 0), c(m, 0);
    std::vector<int> ws_times(slots * 16, 0), times(m, 0);
    const int64_t R = asp::HostGroups::rows(esize), S = asp::HostGroups::RANGES;
    int64_t largest = 0, all = 0, terms = 0, used = 0;
    const uint64_t *entries = (const uint64_t *)g.entries.data();
    if (g.n_groups == 0) return std::printf("groups 0\n"), 0;
    for (int64_t t = 0; t < S * g.n_groups; ++t) {
        const int32_t *td = &g.tasks[4 * t];
        double sum[64] = {0};
        int64_t n[64] = {0}, in_task = 0;
        if (td[0] < 0 || 128 * ((int64_t)td[0] + td[1]) > (int64_t)g.entries.size()) return std::printf("task %lld\n", (long long)t), 1;
        for (int64_t e = 16 * (int64_t)td[0]; e < 16 * ((int64_t)td[0] + td[1]); ++e) {
            const uint32_t key = (uint32_t)entries[e], bits = (uint32_t)(entries[e] >> 32);
            float v;
            std::memcpy(&v, &bits, 4);
            if (td[2] + (int64_t)(key >> 8) >= k || (key & 255) > R) return std::printf("entry %lld of task %lld\n", (long long)e, (long long)t), 1;
            if ((int64_t)(key & 255) < R) sum[key & 255] += v * b(td[2] + (key >> 8)), terms = std::max(terms, ++n[key & 255]), ++in_task;
        }
        largest = std::max(largest, in_task), all += in_task;
        for (int64_t r = 0; r < R; ++r) {
            const int32_t slot = g.slots[t * R + r];
            if (slot >= 0) ws.at(slot) = sum[r], ++ws_times[slot], ++used;
        }
    }
    for (size_t i = 0; i < g.chunks.size(); i += 4)
        if (g.chunks[i + 2] < g.chunks[i + 3]) ws.at(g.chunks[i + 1]) = walk(g.chunks[i + 2], g.chunks[i + 3]), ++ws_times[g.chunks[i + 1]], ++used;
    for (size_t i = 0; i < g.row_tasks.size(); i += 4)
        for (int64_t r = g.row_tasks[i]; r < g.row_tasks[i] + g.row_tasks[i + 1]; ++r)
            c.at(r) = walk(rows.row_ptr[r], rows.row_ptr[r + 1]), ++times[r];
    for (size_t i = 0; i < g.split.size(); i += 4) {
        for (int64_t j = g.split[i + 1]; j < g.split[i + 1] + g.split[i + 2]; ++j) {
            c.at(g.split[i]) += ws.at(j);
            if (ws_times[j] != 1) return std::printf("scratch row %lld written %d times\n", (long long)j, ws_times[j]), 1;
        }
        ++times[g.split[i]];
    }
    int64_t fewest = INT32_MAX, most = 0;
    for (size_t i = 0; i < g.split.size(); i += 4)
        if ((int64_t)i < 4 * g.n_many) fewest = std::min<int64_t>(fewest, g.split[i + 2]);
        else most = std::max<int64_t>(most, g.split[i + 2]);
    std::printf("groups %lld\nlargest %lld %lld\nterms %lld\nscratch %lld %lld\nnear %lld\nmany %lld %lld %lld\n", (long long)g.n_groups, (long long)largest, (long long)all, (long long)terms,
                (long long)slots * 16, (long long)used, (long long)g.near_cols, (long long)g.n_many, (long long)fewest, (long long)most);
    asp_handle h;
    h.dtype = esize == 2 ? ASP_DT_BF16 : ASP_DT_F32, h.m = m, h.k = k, h.n_groups = g.n_groups, h.group_span = g.span, h.group_many = g.n_many;
    h.n_split_rows = (int64_t)rows.split.size() / 4, h.scratch_rows = asp::split_scratch_rows(rows.split);
    h.n_g_split_rows = (int64_t)g.split.size() / 4, h.g_scratch_rows = asp::split_scratch_rows(g.split);
    std::printf("sums %lld %lld\n", (long long)asp::wcsr_rows_sum_many(&h, 128), (long long)h.n_g_split_rows);
    for (int64_t r = 0; r < m; ++r) {
        double want = 0;
        for (int64_t e = rp[r]; e < rp[r + 1]; ++e) want += (1 + e % 3) * b(ci[e]);
        if (rows.row_ptr[r + 1] - rows.row_ptr[r] != rp[r + 1] - rp[r]) {
            std::printf("tile %lld %d\n", (long long)r, times[r]);
            continue;
        }
        std::printf("row %lld %lld %d\n", (long long)r, (long long)(c[r] - want), times[r]);
    }
    return 0;
}

// Rows of L.. entries in turn over all k columns, in fp32 (1, 2, 3), and what is made of them.
struct Spread {
    std::vector<int32_t> rp{0}, ci;
    std::vector<float> values;
    asp::HostWcsr hw;
    asp::HostRows rows;
    std::vector<int64_t> at;  // where the entries walked row by row are
    int64_t slots = 0;

    bool make(int64_t m, int64_t k, int32_t height, int32_t task_cols, const std::vector<int32_t> &lengths) {
        for (int64_t r = 0; r < m; ++r) {
            const int64_t n = lengths[r % lengths.size()];
            for (int64_t j = 0; j < n; ++j) ci.push_back((int32_t)(j * k / n + (r * 7919 + j) % std::max<int64_t>(1, k / n)));
            rp.push_back((int32_t)ci.size());
        }
        for (size_t e = 0; e < ci.size(); ++e) values.push_back((float)(1 + e % 3));
        if (!asp::csr_to_wcsr(m, k, rp.data(), ci.data(), values.data(), 4, height, 8, hw)) return false;
        for (size_t i = 0; i + 1 < hw.window_row_ptr.size(); ++i) {
            const int64_t n = hw.window_row_ptr[i + 1] - hw.window_row_ptr[i];
            hw.ws_slot.push_back(n > task_cols ? (int32_t)slots : -1);
            if (n > task_cols) slots += asp::ceil_div(n, task_cols);
        }
        asp::wcsr_build_rows(m, rp.data(), ci.data(), 4, height, task_cols, hw, rows);
        for (auto &r : rows.runs)
            for (int64_t p = r.first; p < r.second; ++p) at.push_back(p);
        return true;
    }
    double walk(int64_t e0, int64_t e1) const {
        double sum = 0;
        for (int64_t e = e0; e < e1; ++e) sum += (1 + at[e] % 3) * (double)(ci[at[e]] % 13 + 1);
        return sum;
    }
};

static int dense(int64_t m, int64_t k, int32_t height, int32_t task_cols, const std::vector<int32_t> &lengths) {
    Spread a;
    if (!a.make(m, k, height, task_cols, lengths)) return 1;
    asp::HostDense d;
    asp::wcsr_build_dense(m, a.rp.data(), a.ci.data(), height, task_cols, a.hw, a.rows, d);
    const int64_t n = d.ranges > 0 ? (int64_t)d.rows.size() / 4 : 0;
    std::printf("dense %lld %lld %lld %lld %lld\n", (long long)d.ranges, (long long)d.blocks, (long long)n, (long long)d.ptr.size(),
                (long long)d.per_pass);
    if (n == 0) return 0;
    std::vector<double> ws(a.slots * height, 0), c(m, 0);
    std::vector<int> ws_times(a.slots * height, 0), times(m, 0);
    int64_t fewest = INT64_MAX, entries = 0;
    for (int64_t i = 0; i < n; ++i) {
        const int32_t *ptr = &d.ptr[i * (d.blocks + 1)], row = d.rows[4 * i];
        if (i % d.per_pass == 0 && i > 0) fewest = std::min(fewest, entries), entries = 0;
        entries += ptr[d.blocks] - ptr[0];
        if (ptr[0] != a.rows.row_ptr[row] || ptr[d.blocks] != a.rows.row_ptr[row + 1]) return std::printf("ends of row %d\n", row), 1;
        for (int64_t x = 0; x < d.ranges; ++x) {
            const int64_t slot = d.rows[4 * i + 1] + x;
            for (int64_t b = d.blocks * x / d.ranges; b < d.blocks * (x + 1) / d.ranges; ++b) {
                for (int64_t e = ptr[b]; e < ptr[b + 1]; ++e)
                    if (a.ci[a.at[e]] / asp::HostDense::COLS != b) return std::printf("entry %lld in block %lld\n", (long long)e, (long long)b), 1;
                ws.at(slot) += a.walk(ptr[b], ptr[b + 1]);
            }
            ++ws_times[slot];
        }
    }
    std::printf("fewest %lld\n", (long long)std::min(fewest, entries));
    for (size_t i = 0; i < d.chunks.size(); i += 4)
        if (d.chunks[i + 2] < d.chunks[i + 3]) ws.at(d.chunks[i + 1]) = a.walk(d.chunks[i + 2], d.chunks[i + 3]), ++ws_times[d.chunks[i + 1]];
    for (size_t i = 0; i < d.tasks.size(); i += 4)
        for (int64_t r = d.tasks[i]; r < d.tasks[i] + d.tasks[i + 1]; ++r) c.at(r) = a.walk(a.rows.row_ptr[r], a.rows.row_ptr[r + 1]), ++times[r];
    for (size_t i = 0; i < d.split.size(); i += 4) {
        for (int64_t j = d.split[i + 1]; j < d.split[i + 1] + d.split[i + 2]; ++j) {
            c.at(d.split[i]) += ws.at(j);
            if (ws_times[j] != 1) return std::printf("scratch row %lld written %d times\n", (long long)j, ws_times[j]), 1;
        }
        ++times[d.split[i]];
    }
    for (int64_t r = 0; r < m; ++r) {
        if (a.rows.row_ptr[r + 1] == a.rows.row_ptr[r] && a.rp[r + 1] > a.rp[r]) continue;  // by tiles
        double want = 0;
        for (int64_t e = a.rp[r]; e < a.rp[r + 1]; ++e) want += (1 + e % 3) * (double)(a.ci[e] % 13 + 1);
        std::printf("row %lld %lld %d\n", (long long)r, (long long)(c[r] - want), times[r]);
    }
    return 0;
}

static int teams(int64_t m, int64_t k, int32_t height, int32_t task_cols, const std::vector<int32_t> &lengths) {
    Spread a;
    if (!a.make(m, k, height, task_cols, lengths)) return 1;
    auto dense_row = [&](int64_t r) { return a.rows.row_ptr[r + 1] - a.rows.row_ptr[r] >= a.rows.dense_len; };
    std::vector<int32_t> chunks = a.rows.chunks, tasks = a.rows.tasks, list;
    asp::HostWide wide;
    asp::wcsr_build_teams(a.rows.n_entries, a.rows, chunks, tasks, list, wide);
    const auto &shared = wide.teams;
    auto on_xcd = [&](const int32_t *c, size_t xcd) {
        size_t t = 0;
        while (t < chunks.size() && !std::equal(c, c + 4, chunks.begin() + t)) t += 4;
        return t < chunks.size() && t / 16 % 8 == xcd;
    };
    std::printf("teams %zu %zu %lld %lld\n", list.size() / 4, shared.size() / 4, (long long)wide.count, (long long)wide.len);
    int64_t least = INT64_MAX, of_dense = 0, as_long = 0, moved = 0;
    for (size_t i = 0; i < list.size(); i += 4)
        if (list[i + 2] < list[i + 3]) least = std::min<int64_t>(least, list[i + 3] - list[i + 2]), of_dense += dense_row(list[i]);
    const int64_t line = std::max<int64_t>(65, a.rows.n_entries / 16384);
    for (size_t i = 0; i < chunks.size(); i += 4) as_long += chunks[i + 3] - chunks[i + 2] >= line && !dense_row(chunks[i]);
    for (size_t i = 0; i < tasks.size(); i += 4) as_long += tasks[i + 1] == 1 && tasks[i + 3] - tasks[i + 2] >= line;
    for (size_t i = 0; i < shared.size(); i += 4) moved += shared[i + 2] < shared[i + 3] && !on_xcd(&shared[i], i / 4 % 8);
    for (size_t i = 0; i < wide.chunks.size(); i += 4) moved += wide.chunks[i + 2] < wide.chunks[i + 3] && !on_xcd(&wide.chunks[i], i / 16 % 8);
    std::printf("least %lld %lld %lld\nmoved %lld\n", (long long)least, (long long)of_dense, (long long)as_long, (long long)moved);
    std::vector<double> c[2];
    std::vector<int> times[2];
    for (int mode = 0; mode < 2; ++mode) {
        std::vector<double> ws(a.slots * height, 0);
        std::vector<int> ws_times(a.slots * height, 0);
        c[mode].assign(m, 0), times[mode].assign(m, 0);
        auto all = [&](const std::vector<int32_t> &of) {
            for (size_t i = 0; i < of.size(); i += 4) {
                if (of[i + 2] >= of[i + 3]) continue;
                if (of[i + 1] < 0) c[mode].at(of[i]) = a.walk(of[i + 2], of[i + 3]), ++times[mode][of[i]];
                else ws.at(of[i + 1]) = a.walk(of[i + 2], of[i + 3]), ++ws_times[of[i + 1]];
            }
        };
        all(list);
        if (mode == 1 && wide.count > 0) all(shared), all(wide.chunks);
        else all(chunks);
        for (size_t i = 0; i < tasks.size(); i += 4)
            for (int64_t r = tasks[i]; r < tasks[i] + tasks[i + 1]; ++r) c[mode].at(r) = a.walk(a.rows.row_ptr[r], a.rows.row_ptr[r + 1]), ++times[mode][r];
        for (size_t i = 0; i < a.rows.split.size(); i += 4) {
            for (int64_t j = a.rows.split[i + 1]; j < a.rows.split[i + 1] + a.rows.split[i + 2]; ++j) {
                c[mode].at(a.rows.split[i]) += ws.at(j);
                if (ws_times[j] != 1) return std::printf("scratch row %lld written %d times\n", (long long)j, ws_times[j]), 1;
            }
            ++times[mode][a.rows.split[i]];
        }
    }
    for (int64_t r = 0; r < m; ++r) {
        if (a.rows.row_ptr[r + 1] == a.rows.row_ptr[r] && a.rp[r + 1] > a.rp[r]) continue;  // by tiles
        double want = 0;
        for (int64_t e = a.rp[r]; e < a.rp[r + 1]; ++e) want += (1 + e % 3) * (double)(a.ci[e] % 13 + 1);
        std::printf("row %lld %lld %d %lld %d\n", (long long)r, (long long)(c[0][r] - want), times[0][r], (long long)(c[1][r] - want), times[1][r]);
    }
    return 0;
}

static int xt(char **argv) {
    asp_handle h;
    h.b_row = std::atoi(argv[0]), h.n_brows = std::atoll(argv[1]), h.n_units = std::atoll(argv[2]), h.hb.max_blocks = std::atoll(argv[3]);
    h.n_cus = 256;
    std::printf("staged %d\n", asp::bcsr_xt_staged_strips(&h, std::atoll(argv[4])));
    return 0;
}

static int launches(int64_t waves, int64_t n_teams) {
    for (int64_t first = 0, end; first < waves || n_teams > 0; first = end, n_teams = 0) {
        end = asp::rows_launch_end(waves, first, n_teams);
        std::printf("launch %lld %lld %lld\n", (long long)first, (long long)end, (long long)(n_teams + asp::ceil_div(end - first, 4)));
        if (end <= first && waves > 0) return 1;
    }
    return 0;
}

int main(int argc, char **argv) {
    if (argc == 7 && std::strcmp(argv[1], "xt") == 0) return xt(argv + 2);
    if (argc == 3 && std::strcmp(argv[1], "slots") == 0) return slots((int32_t)std::atoll(argv[2]));
    if (argc == 4 && std::strcmp(argv[1], "launches") == 0) return launches(std::atoll(argv[2]), std::atoll(argv[3]));
    auto is = [&](const char *what, int first) { return argc > first && std::strcmp(argv[1], what) == 0; };
    auto lengths = [&](int first) {
        std::vector<int32_t> v;
        for (int i = first; i < argc; ++i) v.push_back(std::atoi(argv[i]));
        return v;
    };
    if (is("order", 2)) return order(lengths(2));
    if (is("shares", 2)) return shares(lengths(2));
    if (is("groups", 7))
        return groups(std::atoll(argv[2]), std::atoll(argv[3]), std::atoll(argv[4]), std::atoi(argv[5]), std::atoll(argv[6]), lengths(7));
    if (is("f32", 6)) {
        asp_handle h;
        h.b_row = std::atoi(argv[2]), h.n_brows = std::atoll(argv[3]), h.n_units = std::atoll(argv[4]), h.hb.max_blocks = std::atoll(argv[5]);
        h.n_cus = 256;
        for (int32_t n : lengths(6)) std::printf("one %d\n", (int)asp::bcsr_f32_one_wave(&h, n));
        return 0;
    }
    if (is("unaligned", 4)) {
        asp_handle h;
        h.b_row = std::atoi(argv[2]), h.n_brows = std::atoll(argv[3]), h.n_cus = 256;
        for (int32_t n : lengths(4)) std::printf("bn %d\n", asp::bcsr_unaligned_bn(&h, n));
        return 0;
    }
    if (is("columns", 4)) {
        asp_handle h;
        h.b_row = std::atoi(argv[2]), h.n_tile_tasks = std::atoll(argv[3]);
        for (int32_t n : lengths(4)) std::printf("columns %d\n", asp::wcsr_lane_columns(&h, n));
        return 0;
    }
    if (argc == 6 && std::strcmp(argv[1], "share") == 0) {
        asp_handle h;
        h.dtype = std::atoi(argv[2]) ? ASP_DT_BF16 : ASP_DT_F32;
        std::printf("share %d\n", (int)asp::wcsr_share_chunks(&h, std::atoll(argv[3]), std::atoll(argv[4]), std::atoll(argv[5])));
        return 0;
    }
    if (is("teams", 6))
        return teams(std::atoll(argv[2]), std::atoll(argv[3]), std::atoi(argv[4]), std::atoi(argv[5]), lengths(6));
    if (is("apply", 6)) {
        asp_handle h;
        h.k = std::atoll(argv[2]), h.n_dense = std::atoll(argv[3]), h.dense_per_pass = 50, h.dtype = ASP_DT_F32;
        h.wide.count = std::atoll(argv[4]), h.wide.len = 192, h.dense_meet_tenths = std::atoll(argv[5]);
        for (int32_t n : lengths(6)) std::printf("apply %d\n", (int)asp::wcsr_dense_apply(&h, n));
        return 0;
    }
    if (is("dense", 6))
        return dense(std::atoll(argv[2]), std::atoll(argv[3]), std::atoi(argv[4]), std::atoi(argv[5]), lengths(6));
    if (is("staged", 4)) return staged(std::atoi(argv[2]), std::atoll(argv[3]), lengths(4));
    if (is("ring", 8))
        return ring(std::atoi(argv[2]), std::atoll(argv[3]), std::atoi(argv[4]), std::atoi(argv[5]), std::atoi(argv[6]) != 0,
                    std::atoi(argv[7]), lengths(8));
    if (is("wide", 6)) return wide(std::atoi(argv[2]), std::atoll(argv[3]), std::atoi(argv[4]) != 0, std::atoll(argv[5]), lengths(6));
    return 2;
}

// Host-side layout of the jagged window tiles: which rows form tiles, each
// tile's lanes in order of row length, its window's sectors, and its slices'
// headers.  Pure C++ (no HIP calls); the positions and values are then
// filled on the device from the CSR arrays.  The same for the sweep tiles of
// scattered orderings (sweep.hip).
#include <algorithm>
#include <atomic>
#include <cstring>
#include <thread>

#include "internal.h"
#include "shares.h"

namespace spmvlib {

bool build_jag_plan(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *row_ptr, const int32_t *col_idx,
                    int long_len, JagPlan &J) {
    J = JagPlan{};
    const auto len_of = [row_ptr](int32_t r) { return row_ptr[r + 1] - row_ptr[r]; };
    // runs of rows of at most kJagMaxLen entries, in tiles of 256 rows
    std::vector<int32_t> first, rows;
    int64_t long_entries = 0;
    for (int32_t r = 0; r < n_rows;) {
        if (len_of(r) > kJagMaxLen) {
            if (len_of(r) > long_len) long_entries += len_of(r);
            ++r;
            continue;
        }
        int32_t r1 = r + 1;
        while (r1 < n_rows && r1 - r < kJagRows && len_of(r1) <= kJagMaxLen) ++r1;
        first.push_back(r);
        rows.push_back(r1 - r);
        r = r1;
    }
    const int32_t n_cand = (int32_t)first.size();
    // tiles cut short by longer rows leave lanes idle
    if (n_cand == 0 || (int64_t)n_cand * (kJagRows / 2) > n_rows) return false;
    const int nth = std::max(1, std::min({32, (int)std::thread::hardware_concurrency(), n_cand / 64}));
    std::vector<std::vector<int32_t>> lists(nth);
    std::vector<int64_t> off((size_t)n_cand, 0);
    std::vector<int32_t> count((size_t)n_cand, -1);  // sectors; -1: the window does not fit
    std::atomic<int64_t> left_out{0};  // entries of tiles whose window does not fit
    run_shares(nth, [&](int t) {
        // a tile's sectors: at most kJagMaxSectors + 1 in a table of 1,024
        // (a mark per sector of x would take n_cols / 2 bytes per thread)
        constexpr uint32_t kSlots = 1024;
        static_assert(2 * kJagMaxSectors <= kSlots, "half full at most, one more for the sector that is too many");
        std::vector<int32_t> table(kSlots), u;
        std::vector<int32_t> &out = lists[t];
        // contiguous shares: the tiles' lists follow each other in order
        const int32_t c0 = (int32_t)((int64_t)n_cand * t / nth), c1 = (int32_t)((int64_t)n_cand * (t + 1) / nth);
        for (int32_t i = c0; i < c1; ++i) {
            u.clear();
            std::fill(table.begin(), table.end(), -1);
            const int32_t s = row_ptr[first[i]], e = row_ptr[first[i] + rows[i]];
            for (int32_t k = s; k < e && (int)u.size() <= kJagMaxSectors; ++k) {
                const int32_t sc = col_idx[k] / kJagSector;
                uint32_t at = (uint32_t)sc * 2654435769u >> 22;
                while (table[at] != sc && table[at] >= 0) at = (at + 1) % kSlots;
                if (table[at] != sc) {
                    table[at] = sc;
                    u.push_back(sc);
                }
            }
            if ((int)u.size() > kJagMaxSectors) {
                // more than the rule below allows: the rest need not be looked at
                if (8 * (left_out += e - s) > nnz - long_entries) return;
                continue;
            }
            std::sort(u.begin(), u.end());
            off[i] = (int64_t)out.size();
            count[i] = (int32_t)u.size();
            out.insert(out.end(), u.begin(), u.end());
        }
    });
    if (8 * left_out > nnz - long_entries) return false;
    // Worth it when nearly all of the entries that row tiles would work lie
    // in the tiles and the staged words do not outnumber them (a scattered
    // ordering touches a sector of 8 words per entry, and gathering x
    // directly reads less).
    int64_t entries = 0, words = 0;
    int32_t most = 0;
    for (int32_t i = 0; i < n_cand; ++i) {
        if (count[i] < 0) continue;
        entries += row_ptr[first[i] + rows[i]] - row_ptr[first[i]];
        words += (int64_t)count[i] * kJagSector;
        most = std::max(most, count[i]);
        ++J.n_tiles;
    }
    if (J.n_tiles == 0 || 8 * entries < 7 * (nnz - long_entries) || words > entries) return false;
    J.stride = std::max((most + 15) / 16 * 16, 16);
    J.width = most * kJagSector;
    constexpr int kSlices = kJagRows / kJagSlice;
    const size_t nt = (size_t)J.n_tiles;
    if (nt * J.stride > (size_t)INT32_MAX) return false;
    J.hdr.assign(nt * kSlices * kJagHdr, 0);
    J.slot.resize(nt * kJagRows);
    J.sect.assign(nt * J.stride, 0);
    int64_t vb = 0, pb = 0;
    int32_t t = 0, longest = 0;
    std::vector<int32_t> tile_of((size_t)n_cand, -1);
    for (int32_t i = 0; i < n_cand; ++i)
        if (count[i] >= 0) tile_of[i] = t++;
    // lanes in order of row length (longest first), counts of the slices' runs
    run_shares(nth, [&](int sh) {
        const int32_t c0 = (int32_t)((int64_t)n_cand * sh / nth), c1 = (int32_t)((int64_t)n_cand * (sh + 1) / nth);
        for (int32_t i = c0; i < c1; ++i) {
            if (tile_of[i] < 0) continue;
            const size_t tile = (size_t)tile_of[i];
            std::memcpy(&J.sect[tile * J.stride], lists[sh].data() + off[i], sizeof(int32_t) * (size_t)count[i]);
            uint16_t *slot = &J.slot[tile * kJagRows];
            int at[kJagMaxLen + 1] = {};
            for (int32_t r = 0; r < kJagRows; ++r) ++at[r < rows[i] ? len_of(first[i] + r) : 0];
            for (int l = kJagMaxLen, sum = 0; l >= 0; --l) {
                const int n = at[l];
                at[l] = sum;
                sum += n;
            }
            for (int32_t r = 0; r < kJagRows; ++r) {
                const int l = r < rows[i] ? len_of(first[i] + r) : 0;
                slot[at[l]++] = (uint16_t)(l << 8 | r);
            }
            for (int sl = 0; sl < kSlices; ++sl) {
                int32_t *h = &J.hdr[(tile * kSlices + sl) * kJagHdr];
                h[2] = count[i];
                h[3] = first[i];
                h[4] = rows[i];
                // a sector reaching past x's last word needs word-wise staging
                h[5] = count[i] > 0 && ((int64_t)J.sect[tile * J.stride + count[i] - 1] + 1) * kJagSector > n_cols;
                uint8_t *c = reinterpret_cast<uint8_t *>(h + 8);
                for (int l = 0; l < kJagSlice; ++l)
                    for (int j = 0; j < slot[sl * kJagSlice + l] >> 8; ++j) ++c[j];
            }
        }
    });
    for (size_t sl = 0; sl < nt * kSlices; ++sl) {
        int32_t *h = &J.hdr[sl * kJagHdr];
        const uint8_t *c = reinterpret_cast<const uint8_t *>(h + 8);
        h[0] = (int32_t)vb;
        h[1] = (int32_t)pb;
        for (int j = 0; j < kJagMaxLen; ++j) {
            vb += c[j];
            if (j % 8 == 0 || j % 8 == 2 || j % 8 == 5) pb += c[j];
            if (c[j]) longest = std::max(longest, j + 1);
        }
    }
    J.n_entries = vb;
    J.n_words = pb;
    J.groups = (longest + 3) / 4;
    // the rows left to row tiles (long rows are segments of their own)
    int32_t r = 0;
    for (int32_t i = 0; i <= n_cand; ++i) {
        if (i < n_cand && count[i] < 0) continue;
        const int32_t stop = i < n_cand ? first[i] : n_rows;
        if (stop > r) J.rest.emplace_back(r, stop);
        if (i < n_cand) r = first[i] + rows[i];
    }
    return true;
}

double lines_per_entry(int32_t n_rows, const int32_t *row_ptr, const int32_t *col_idx, int long_len, int rows,
                       int blocks) {
    int64_t lines = 0, entries = 0;
    std::vector<int32_t> u;
    const int32_t all = (int32_t)(((int64_t)n_rows + rows - 1) / rows), step = std::max(1, all / blocks);
    for (int32_t b = 0; b < all; b += step) {
        u.clear();
        for (int32_t r = b * rows; r < n_rows && r - b * rows < rows; ++r)
            if (row_ptr[r + 1] - row_ptr[r] <= long_len)
                for (int32_t k = row_ptr[r]; k < row_ptr[r + 1]; ++k) u.push_back(col_idx[k] / 16);
        entries += (int64_t)u.size();
        std::sort(u.begin(), u.end());
        lines += std::unique(u.begin(), u.end()) - u.begin();
    }
    return entries ? (double)lines / (double)entries : 0.0;
}

bool build_sweep_plan(int32_t n_rows, int32_t n_cols, const int32_t *row_ptr, const int32_t *col_idx, int long_len,
                      int n_cus, SweepPlan &S) {
    S = SweepPlan{};
    if (lines_per_entry(n_rows, row_ptr, col_idx, long_len, 256, 32) < 0.75) return false;
    const auto len_of = [row_ptr](int32_t r) { return row_ptr[r + 1] - row_ptr[r]; };
    // entries of the runs of rows between long rows: a tile ends with its run
    std::vector<int64_t> run;
    int64_t entries = 0;
    for (int32_t r = 0, last = -2; r < n_rows; ++r) {
        if (len_of(r) > long_len) continue;
        if (r != last + 1) run.push_back(0);
        run.back() += len_of(r);
        entries += len_of(r);
        last = r;
    }
    if (entries < kSweepMinNnz) return false;
    // Tiles of at least `target` entries, as many as whole rounds of one
    // workgroup per CU hold: the smallest such target for each number of
    // rounds, and of those the quickest.  A workgroup takes as long as for its
    // entries and some 3,600 more (2M-row kNN mesh, tiles of 20,480 / 16,384 /
    // 8,192 / 4,096 entries: 117 / 122 / 143 / 175 us).
    const auto cost = [n_cus](int64_t rounds, int64_t target) { return rounds * n_cus * (target + 3600); };
    const int64_t least = (entries + (int64_t)n_cus * kSweepTarget - 1) / ((int64_t)n_cus * kSweepTarget);
    constexpr int kMoreRounds = 3;
    if ((int64_t)run.size() > (least + kMoreRounds) * n_cus) return false;
    int32_t target = 0;
    int64_t best = INT64_MAX;
    for (int64_t rounds = least; rounds <= least + kMoreRounds; ++rounds) {
        int32_t lo = 1, hi = kSweepTarget + 1;  // the first that fits lies in [lo, hi]; hi: none
        while (lo < hi) {
            const int32_t mid = (lo + hi) / 2;
            int64_t tiles = 0;
            for (const int64_t e : run) tiles += std::max<int64_t>((e + mid - 1) / mid, 1);
            if (tiles <= rounds * n_cus) hi = mid;
            else lo = mid + 1;
        }
        if (lo <= kSweepTarget && cost(rounds, lo) < best) {
            target = lo;
            best = cost(rounds, lo);
        }
    }
    if (!target) return false;
    int64_t chains = 0;  // the tiles' longest rows
    for (int32_t r = 0; r < n_rows;) {
        if (len_of(r) > long_len) {
            ++r;
            continue;
        }
        const int32_t s = row_ptr[r];
        int32_t r1 = r, longest = 0;
        while (r1 < n_rows && len_of(r1) <= long_len && (row_ptr[r1] - s < target || len_of(r1) == 0) &&
               row_ptr[r1 + 1] - s <= kSweepTile)
            longest = std::max(longest, len_of(r1++));
        chains += longest;
        S.bound.push_back(r);
        S.bound.push_back(r1);
        S.width = std::max(S.width, row_ptr[r1] - s);
        r = r1;
    }
    const int32_t nt = (int32_t)(S.bound.size() / 2);
    // Row tiles take as long as 1.5 to 1.9 times the entries in the same unit, a
    // tile's longest row (one lane's chain) up to 4 per entry: where many long
    // rows leave small tiles, or many tiles hold such a row, row tiles are the
    // quicker (kNN mesh, row / sweep tiles: 2M rows with 64 / 512 rows of 2,100
    // entries for long rows 190 / 127 and 199 / 208 us; 2M rows, 2,000 rows of 1,000
    // entries 222 / 189; 804K rows, 200 rows of 2,000 entries 73 / 78).
    const int64_t rounds = (nt + n_cus - 1) / n_cus;
    if (2 * (cost(rounds, target) + 4 * chains) > 3 * entries) return false;
    S.n = (size_t)row_ptr[n_rows];
    S.place.reset(new uint16_t[S.n]);  // the long rows' parts stay unset and unread
    // order of column, to 1/2048 of the columns' range (a stable counting
    // sort per tile)
    int shift = 0;
    while (((int64_t)n_cols >> shift) > 2047) ++shift;
    const int nth = std::max(1, std::min({32, (int)std::thread::hardware_concurrency(), nt / 8}));
    run_shares(nth, [&](int t) {
        int32_t at[2049];
        for (int32_t i = (int32_t)((int64_t)nt * t / nth); i < (int32_t)((int64_t)nt * (t + 1) / nth); ++i) {
            const int32_t s = row_ptr[S.bound[2 * i]], e = row_ptr[S.bound[2 * i + 1]];
            std::memset(at, 0, sizeof at);
            for (int32_t k = s; k < e; ++k) ++at[(col_idx[k] >> shift) + 1];
            for (int b = 0; b < 2048; ++b) at[b + 1] += at[b];
            for (int32_t k = s; k < e; ++k) S.place[(size_t)s + at[col_idx[k] >> shift]++] = (uint16_t)(k - s);
        }
    });
    return true;
}

}  // namespace spmvlib

// Sliced rows of large levels (sell_rows), run by tests/test_sliced_layout_cpu.py
// (CPU only): what the tiles store against a brute-force look at the rows, and
// which levels are stored that way:
//  * even rows: the tiles cover the rows in order, whole aggregates, at most
//    256 rows; inside a tile the rows are sorted by length, ties in row order;
//    every row's entries start at its position in the tile, and an entry's
//    position names its column in the tile's dictionary (sorted, no longer than
//    2048);
//  * the same with scattered rows, whose tiles are cut for their dictionaries;
//  * never more than 1.4 times the entries: uneven rows and badly scattered
//    ones are not stored this way at all;
//  * the lines of the rule: longest rows of 128 and 129, four times the mean.
// Exit status 0 when every check holds; the first failures are printed.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "common.hpp"

using namespace pamg;

static int failures = 0;
#define CHECK(cond, ...)                          \
    do {                                          \
        if (!(cond)) {                            \
            if (++failures <= 10) {               \
                std::printf(__VA_ARGS__);         \
                std::printf("\n");                \
            }                                     \
        }                                         \
    } while (0)

struct Case {
    int32_t n = 0, nc = 0;
    std::vector<int32_t> rp, ci, aggptr;
};

// n rows of `base` columns around the diagonal; in row i, extra(i) more, either
// anywhere (scattered) or next to those.
template <class F>
static Case make(std::mt19937& rng, int32_t n, int base, bool scattered, int agg, F extra) {
    Case c;
    c.n = n;
    c.rp.assign(n + 1, 0);
    std::vector<int32_t> row;
    for (int32_t i = 0; i < n; ++i) {
        row.clear();
        const int m = base + (scattered ? 0 : extra(i));
        const int32_t first = std::max(0, std::min(i - m / 2, n - m));
        for (int k = 0; k < m; ++k) row.push_back(first + k);
        if (scattered)
            for (int k = extra(i); k > 0; --k) row.push_back((int32_t)(rng() % (unsigned)n));
        std::sort(row.begin(), row.end());
        row.erase(std::unique(row.begin(), row.end()), row.end());
        c.ci.insert(c.ci.end(), row.begin(), row.end());
        c.rp[i + 1] = (int32_t)c.ci.size();
    }
    if (agg > 0) {
        c.aggptr.push_back(0);
        while (c.aggptr.back() < n)
            c.aggptr.push_back(std::min<int32_t>(n, c.aggptr.back() + 1 + (int32_t)(rng() % (unsigned)agg)));
        c.nc = (int32_t)c.aggptr.size() - 1;
    }
    return c;
}

// The largest and smallest number of rows in a tile of S, everything checked.
static void check_tiles(const char* name, const Case& c, const SellRows& S, int* most, int* least) {
    const int64_t nt = (int64_t)S.tiles.size() / 8;
    CHECK(nt > 0, "%s: not stored in sliced rows", name);
    if (nt == 0) return;
    CHECK(5 * S.entries <= 7 * (int64_t)c.ci.size(), "%s: %lld stored for %zu entries", name,
          (long long)S.entries, c.ci.size());
    int32_t row = 0, coarse = 0;
    int64_t at = 0, dict = 0;
    *most = 0;
    *least = 1 << 30;
    for (int64_t t = 0; t < nt; ++t) {
        const int32_t* d = &S.tiles[8 * t];
        CHECK(d[0] == row && d[1] > d[0] && d[1] - d[0] <= 256, "%s tile %lld: rows %d..%d", name, (long long)t, d[0], d[1]);
        CHECK(d[2] == at && d[3] == dict && d[4] <= kSellDict && d[4] <= S.max_len, "%s tile %lld: base %d dictionary %d + %d",
              name, (long long)t, d[2], d[3], d[4]);
        if (c.nc) {
            CHECK(d[5] == coarse && c.aggptr[d[5]] == d[0] && c.aggptr[d[6]] == d[1], "%s tile %lld: aggregates", name,
                  (long long)t);
            coarse = d[6];
        }
        row = d[1];
        *most = std::max(*most, d[1] - d[0]);
        *least = std::min(*least, d[1] - d[0]);
        CHECK(std::is_sorted(S.col.begin() + d[3], S.col.begin() + d[3] + d[4]), "%s tile %lld: dictionary order", name,
              (long long)t);
        int32_t longest = 0, last = 1 << 30, lastrow = -1;
        for (int32_t q = 0; q < d[1] - d[0]; ++q) {
            const int32_t i = d[0] + (int32_t)(S.slot[d[0] + q] & 0xffff), len = (int32_t)(S.slot[d[0] + q] >> 16);
            CHECK(i < d[1] && len == c.rp[i + 1] - c.rp[i] && S.rowpos[i] == d[2] + q, "%s row %d: slot", name, i);
            CHECK(len < last || (len == last && i > lastrow), "%s row %d: order", name, i);
            last = len;
            lastrow = i;
            longest = std::max(longest, len);
            for (int32_t k = 0; k < len; ++k) {
                const int32_t e = c.rp[i] + k;
                CHECK(S.local[e] < d[4] && S.col[d[3] + S.local[e]] == c.ci[e], "%s row %d entry %d", name, i, k);
            }
        }
        at += (int64_t)kSlice * longest;
        dict += d[4];
    }
    CHECK(row == c.n && at == S.entries && dict == (int64_t)S.col.size(), "%s: covered", name);
}

int main() {
    std::mt19937 rng(20260501);
    const int32_t n = 1050011;
    int most = 0, least = 0;
    const auto slices = [](const Case& c) {
        int32_t longest = 0;
        for (int32_t i = 0; i < c.n; ++i) longest = std::max(longest, c.rp[i + 1] - c.rp[i]);
        return sell_applies(c.n, (int64_t)c.ci.size(), longest) ? sell_rows(c.rp, c.ci, c.aggptr, c.n, c.nc) : SellRows();
    };
    {
        const Case c = make(rng, n, 7, false, 2, [&](int32_t i) { return (i / 1000) % 9 == 0 ? 1 : 0; });
        check_tiles("even rows", c, slices(c), &most, &least);
        CHECK(most > 200 && least > 150, "even rows: tiles of %d to %d rows", least, most);
    }
    {
        const Case c = make(rng, n, 7, false, 0, [&](int32_t i) { return i % 5 == 0 ? 1 : 0; });
        check_tiles("no aggregates", c, slices(c), &most, &least);
    }
    {
        // one row in 25 with 10 and one in 100 with 20 columns anywhere: 228 rows
        // have 2,500 and 4,800 distinct columns, halved once and twice
        const Case c = make(rng, n, 7, true, 16, [&](int32_t i) {
            const int32_t s = (i / 2000) % 100;
            return s < 3 ? 10 : s == 50 ? 20 : 0;
        });
        check_tiles("scattered rows", c, slices(c), &most, &least);
        CHECK(most > 200 && least < 80, "scattered rows: tiles of %d to %d rows", least, most);
    }
    {
        const Case c = make(rng, n, 7, false, 2, [&](int32_t i) { return i % 256 == 0 ? 93 : 0; });
        CHECK(slices(c).tiles.empty(), "one row of 100 in 256: sliced");
    }
    {
        const Case c = make(rng, n, 7, false, 2, [&](int32_t i) { return i % 64 == 0 ? 22 : 0; });
        CHECK(slices(c).tiles.empty(), "one row of 29 in 64: sliced");
    }
    {
        const Case c = make(rng, n, 7, true, 2, [&](int32_t i) { return 20; });
        CHECK(slices(c).tiles.empty(), "scattered columns everywhere: sliced");
    }
    const int64_t big = 4 * kSellMinRows;
    CHECK(sell_applies(big, 128 * big, 128) && !sell_applies(big, 128 * big, 129), "rows of 128 and 129");
    CHECK(sell_applies(big, 7 * big, 28) && !sell_applies(big, 7 * big, 29), "rows of four times the mean");
    CHECK(sell_applies(kSellMinRows, 7ll * kSellMinRows, 7) && !sell_applies(kSellMinRows - 1, 7ll * kSellMinRows, 7),
          "least rows");
    std::printf("%d failures\n", failures);
    return failures == 0 ? 0 : 1;
}

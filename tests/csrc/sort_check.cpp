// sort_longest_first against std::stable_sort: every size around the digit sort's limit, lengths of one digit to three.
#include <algorithm>
#include <cstdio>
#include <random>

#include "prep.h"

int main()
{
    using Item = std::pair<int64_t, int32_t>;
    std::mt19937_64 rng(1);
    const int64_t most[] = {1, 2, 2047, 2048, 2049, int64_t(1) << 22, (int64_t(1) << 31) - 1};
    int checked = 0;
    for (size_t n : {0, 1, 2, 255, 256, 257, 1000, 5000})
        for (int64_t m : most)
            for (int kind = 0; kind < 4; ++kind) {
                std::vector<Item> v(n);
                for (size_t i = 0; i < n; ++i) {
                    const int64_t x = kind == 0 ? (int64_t)(rng() % (uint64_t)(m + 1)) : kind == 1 ? (int64_t)i % (m + 1)
                                      : kind == 2 ? m - (int64_t)i % (m + 1) : (rng() & 1 ? m : 0);
                    v[i] = {x, (int32_t)i};
                }
                auto want = v;
                std::stable_sort(want.begin(), want.end(), [](const Item& a, const Item& b) { return a.first > b.first; });
                gpe::sort_longest_first(&v);
                if (v != want) {
                    std::printf("n %zu, lengths to %lld, kind %d differ\n", n, (long long)m, kind);
                    return 1;
                }
                ++checked;
            }
    std::printf("%d orders\n", checked);
    return 0;
}

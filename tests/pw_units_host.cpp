// Walks the work units of the grouped widening step on the host (the index
// arithmetic the kernels use, csrc/pw_units.hpp) for arbitrary offsets: the
// records fit the workspace's array, no unit leaves [0, T), and every group in
// range is covered once and alone.
#include "pw_units.hpp"

#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

using namespace voila;

static long g_unlisted = 0;

static int check(const std::vector<int32_t>& seg, int T, int rows) {
    const int M = (int)seg.size() - 1;
    std::vector<int> lo(M), n(M);
    std::vector<long> first(M);
    long total = 0;
    for (int m = 0; m < M; ++m) {
        pw_rows(seg.data(), m, T, lo[m], n[m]);
        first[m] = total;
        total += pw_unit_count(n[m], rows);
    }
    const int listed = pw_listed(total, T, M);
    std::vector<PwUnit> units;
    if (listed >= 0) {
        std::vector<PwUnit> records(pw_unit_capacity(T, M), PwUnit{-1, 0, 0});
        for (int m = 0; m < M; ++m)
            for (int q = 0; q < pw_unit_count(n[m], rows); ++q) {
                const long at = (int)first[m] + q;
                if (at < 0 || at >= (long)records.size()) return 1;
                records[at] = pw_unit(m, lo[m], n[m], q, rows);
            }
        units.assign(records.begin(), records.begin() + listed);
    } else {
        ++g_unlisted;
        for (long u = 0; u < pw_unlisted_units(M, rows); ++u)
            units.push_back(pw_unlisted_unit(seg.data(), T, u, rows));
    }
    std::vector<long> rows_of(M, 0), next(M, -1);
    for (const PwUnit& u : units) {
        if (u.group < 0 || u.group >= M) return 2;
        const int k = u.end - u.first < rows ? u.end - u.first : rows;
        if (k < 0) return 7;
        if (k == 0) continue;
        if (u.first < lo[u.group] || (long)u.first + k > (long)lo[u.group] + n[u.group]) return 3;
        if (u.first < 0 || (long)u.first + k > T) return 4;
        if (next[u.group] >= 0 && u.first != next[u.group]) return 5;
        next[u.group] = (long)u.first + k;
        rows_of[u.group] += k;
    }
    for (int m = 0; m < M; ++m)
        if (rows_of[m] != n[m]) return 6;
    return 0;
}

int main() {
    std::mt19937 rng(12345);
    auto uni = [&](int a, int b) { return (int)std::uniform_int_distribution<long>(a, b)(rng); };
    long cases = 0;
    for (int rows : {32, 64}) {
        // offsets that fall and rise again: every other group spans everything
        for (int T : {1, 31, 32, 33, 64, 1000, 8191, 8192})
            for (int M : {1, 2, 3, 4, 41, 64, 301}) {
                std::vector<int32_t> seg(M + 1);
                for (int m = 0; m <= M; ++m) seg[m] = m % 2 ? T : 0;
                if (int r = check(seg, T, rows)) return printf("alternating T %d M %d rows %d: %d\n", T, M, rows, r), 1;
                ++cases;
            }
        // arbitrary values, in and out of range, and well-formed ones with one entry spoiled
        for (int it = 0; it < 4000; ++it) {
            const int T = uni(0, 1) ? uni(0, 200) : uni(0, 20000), M = uni(1, 40), kind = uni(0, 3);
            std::vector<int32_t> seg(M + 1);
            for (auto& v : seg) v = kind == 1 ? uni(-5, T + 5) : uni(0, T);
            if (kind == 2)
                for (auto& v : seg)
                    if (uni(0, 3) == 0) v = uni(0, 1) ? INT32_MAX - uni(0, 40) : INT32_MIN + uni(0, 40);
            if (kind == 3) {
                std::sort(seg.begin(), seg.end());
                seg[0] = 0;
                seg[M] = T;
                if (uni(0, 1)) seg[uni(0, M)] = uni(-1, T + 1);
            }
            if (int r = check(seg, T, rows)) return printf("case %d T %d M %d kind %d rows %d: %d\n", it, T, M, kind, rows, r), 1;
            ++cases;
        }
    }
    if (g_unlisted == 0) return printf("no case without a list\n"), 1;
    printf("%ld offset arrays, %ld of them not listed\n", cases, g_unlisted);
    return 0;
}

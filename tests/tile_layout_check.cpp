// Host check of the row tiles of the batched products (formats.cpp): every
// row is in one tile, decoding the tiles' blocks the way the kernels do gives
// the matrix back with each row's entries in its own order, and no tile of
// more than one row has more columns than the limit.
#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <numeric>
#include <random>
#include <set>

#include "../paper_1204_2586_amd/csrc/host/setup.hpp"

using namespace auxp;

static void fail(const char *what, int n, int tile, int cap)
{
    std::printf("FAIL %s (n %d, tile %d, cap %d)\n", what, n, tile, cap);
    std::exit(1);
}

static void check(int n, int most, int reach, int tile, int cap, unsigned seed)
{
    std::mt19937 g(seed);
    Csr a;
    a.n = a.m = n;
    a.ptr.push_back(0);
    for (int i = 0; i < n; i++) {
        std::set<int> row{i};                            // as in A_h, the diagonal is always there
        for (int k = (int)(g() % (unsigned)most); k > 0; k--) row.insert((i + (int)(g() % (unsigned)reach)) % n);
        for (int c : row) {
            a.col.push_back(c);
            a.val.push_back(1.0 + (double)(g() % 1000));
        }
        a.ptr.push_back((int)a.col.size());
    }
    std::vector<int> order(n), iperm(n);
    std::iota(order.begin(), order.end(), 0);
    iperm = order;
    for (int i = 0; i + 1 < n; i += 2) std::swap(order[i], order[i + 1]);
    std::shuffle(iperm.begin(), iperm.end(), g);
    std::vector<int> row_of(n);
    for (int i = 0; i < n; i++) row_of[iperm[i]] = i;
    Tiles t;
    build_tiles(a, order, iperm, tile, cap, t);
    std::vector<char> have(n, 0);
    int most_cols = 0;
    for (int k = 0; k < t.ntiles; k++) {
        const int nc = t.col_off[k + 1] - t.col_off[k];
        most_cols = std::max(most_cols, nc);
        int rows = 0;
        for (int i = 0; i < tile; i++) {
            const int r = t.rows[(size_t)k * tile + i];
            if (r < 0) continue;
            rows++;
            if (have[r]++) fail("row twice", n, tile, cap);
            const int q = row_of[r], gr = k * (tile / 8) + i / 8;
            int e = a.ptr[q];
            for (int j = 0; j < 8 * (t.grp_off[gr + 1] - t.grp_off[gr]); j++) {
                const size_t at = 64 * (size_t)(t.grp_off[gr] + j / 8) + 8 * (i % 8) + j % 8;
                if (t.lidx[at] >= nc) fail("position", n, tile, cap);
                if (e < a.ptr[q + 1]) {
                    if (t.val[at] != a.val[e] || t.ucols[t.col_off[k] + t.lidx[at]] != iperm[a.col[e]])
                        fail("entry", n, tile, cap);
                    e++;
                } else if (t.val[at] != 0.0) {
                    fail("padding", n, tile, cap);
                }
            }
            if (e != a.ptr[q + 1]) fail("row too short", n, tile, cap);
        }
        if (rows == 0) fail("empty tile", n, tile, cap);
        if (rows > 1 && nc > cap) fail("columns", n, tile, cap);
    }
    if (std::count(have.begin(), have.end(), 1) != n) fail("rows", n, tile, cap);
    if (most_cols != t.max_cols) fail("max_cols", n, tile, cap);
    if ((size_t)t.grp_off.back() * 64 != t.val.size()) fail("size", n, tile, cap);
}

int main()
{
    unsigned seed = 1;
    for (int tile : {64, 128})
        for (int n : {1, 7, 8, 9, 63, 64, 65, 127, 128, 129, 1000})
            for (int most : {1, 7, 8, 9, 40})
                for (int cap : {8, 64, 504}) check(n, most, std::min(n, 100), tile, cap, seed++);
    check(200000, 20, 150, 64, 312, seed);               // several shares of the curve
    std::printf("OK\n");
    return 0;
}

// Host check of the padding of the device layouts (formats.cpp): every stored
// entry that a kernel multiplies for a row, padding included, points at a
// column of that row.  One 16-bit range per slot, two, 32-bit columns, rows of
// very different lengths in one slice; row tiles.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <random>
#include <set>

#include "../paper_1204_2586_amd/csrc/host/setup.hpp"

using namespace auxp;

static void fail(const char *what, int n, int row)
{
    std::printf("FAIL %s (n %d, row %d)\n", what, n, row);
    std::exit(1);
}

// rows of 1 to `most` entries, the diagonal among them: near it, or for every
// other entry `jump` rows further on
static Csr matrix(int n, int most, int reach, int jump, unsigned seed)
{
    std::mt19937 g(seed);
    Csr a;
    a.n = a.m = n;
    for (int i = 0; i < n; i++) {
        std::set<int> row{i};
        for (int k = (int)(g() % (unsigned)most); k > 0; k--)
            row.insert((int)(((int64_t)i + g() % (unsigned)reach + (k % 2 ? jump : 0)) % n));
        for (int c : row) {
            a.col.push_back(c);
            a.val.push_back(1.0 + (double)(g() % 1000));
        }
        a.ptr.push_back((int)a.col.size());
    }
    return a;
}

static void check_sell(const Csr &a, int window, bool index16, bool permute)
{
    Sell s;
    build_sell(a, 64, window, index16, s, permute);
    for (int r = 0; r < a.n; r++) {
        const int sl = r / 64, l = r % 64, i = s.perm[r];
        const std::set<int> own(a.col.begin() + a.ptr[i], a.col.begin() + a.ptr[i + 1]);
        for (int j = 0; j < (int)((s.slice_off[sl + 1] - s.slice_off[sl]) / 64); j++) {
            const size_t at = sell_pos((size_t)s.slice_off[sl], j, l), slot = (size_t)s.slice_off[sl] / 64 + j;
            const int c = s.wide_off[sl] >= 0 ? s.wide[(size_t)s.wide_off[sl] + (at - (size_t)s.slice_off[sl])]
                                              : s.base[2 * slot + (s.off[at] >> 15)] + (s.off[at] & 0x7fff);
            if (!own.count(permute ? s.perm[c] : c)) fail("sliced ELL", a.n, i);
        }
    }
}

static void check_tiles(const Csr &a, int tile, int cap)
{
    std::vector<int> order(a.n), iperm(a.n), row_of(a.n);
    std::iota(order.begin(), order.end(), 0);
    iperm = order;
    std::shuffle(iperm.begin(), iperm.end(), std::mt19937(3));
    for (int i = 0; i < a.n; i++) row_of[iperm[i]] = i;
    Tiles t;
    build_tiles(a, order, iperm, tile, cap, t);
    for (int k = 0; k < t.ntiles * tile; k++) {
        if (t.rows[k] < 0) continue;
        const int i = row_of[t.rows[k]], g = k / 8;
        const std::set<int> own(a.col.begin() + a.ptr[i], a.col.begin() + a.ptr[i + 1]);
        for (int j = 0; j < 8 * (t.grp_off[g + 1] - t.grp_off[g]); j++) {
            const size_t at = 64 * (size_t)(t.grp_off[g] + j / 8) + 8 * (k % 8) + j % 8;
            if (!own.count(row_of[t.ucols[t.col_off[k / tile] + t.lidx[at]]])) fail("tiles", a.n, i);
        }
    }
}

int main()
{
    for (int n : {1, 63, 65, 512, 1000})
        for (int most : {1, 2, 3, 4, 5, 9, 30}) {
            const Csr a = matrix(n, most, std::min(n, 50), 0, (unsigned)(n + most));
            for (int window : {1 << 30, 64}) {
                for (bool permute : {true, false}) {
                    check_sell(a, window, true, permute);
                    check_sell(a, window, false, permute);
                }
            }
            for (int tile : {32, 64, 128}) check_tiles(a, tile, 40);
        }
    // two ranges; columns anywhere, so 32-bit where the rows are of one length and where they are not
    check_sell(matrix(150000, 6, 300, 75000, 1), 4096, true, true);
    check_sell(matrix(150000, 6, 300, 75000, 1), 100, true, false);
    check_sell(matrix(200000, 6, 200000, 0, 2), 1 << 30, true, true);
    check_sell(matrix(200000, 3, 200000, 0, 3), 64, true, true);
    std::printf("OK\n");
    return 0;
}

// Host check of the sliced-ELL layout of the P^k operator (formats.cpp):
// decoding every stored entry the way the kernels do gives the matrix back,
// for the three column forms (one 16-bit range per slot, two, 32-bit).
#include <cstdio>
#include <cstdlib>
#include <map>
#include <random>

#include "../paper_1204_2586_amd/csrc/host/setup.hpp"

using namespace auxp;

static void fail(const char *what)
{
    std::printf("FAIL %s\n", what);
    std::exit(1);
}

static Csr random_csr(int n, int m, int most, int reach, unsigned seed)
{
    std::mt19937 g(seed);
    Csr a;
    a.n = n;
    a.m = m;
    a.ptr.push_back(0);
    for (int i = 0; i < n; i++) {
        std::map<int, double> row;
        const int len = (int)(g() % (unsigned)(most + 1));
        for (int k = 0; k < len; k++) {
            // near the diagonal, near a second place, or anywhere
            const int c = reach == 0 ? (int)(g() % (unsigned)m)
                                     : (i + (int)(g() % (unsigned)reach) + (k % 2 ? m / 2 : 0)) % m;
            row[c] = 1.0 + (double)(g() % 1000);
        }
        for (auto &cv : row) {
            a.col.push_back(cv.first);
            a.val.push_back(cv.second);
        }
        a.ptr.push_back((int)a.col.size());
    }
    return a;
}

static void check(const Csr &a, int window, bool index16, bool permute, int want_short, int want_narrow)
{
    Sell s;
    build_sell(a, 64, window, index16, s, permute);
    if (s.nslices != (a.n + 63) / 64) fail("slices");
    int narrow = 0, shorts = 0;
    std::vector<int> pos;
    if (permute) pos = sell_positions(a, s);
    std::vector<char> used(s.val.size(), 0);
    for (int sl = 0; sl < s.nslices; sl++) {
        if (s.slice_off[sl] % 256) fail("slice offset");
        if ((s.slice_off[sl + 1] - s.slice_off[sl]) / 64 != (s.width[sl] + 3) / 4 * 4) fail("width");
        shorts += s.wide_off[sl] < 0;
        for (int l = 0; l < 64 && sl * 64 + l < a.n; l++) {
            const int i = s.perm[sl * 64 + l];
            std::map<int, double> row;
            int last = -1;
            for (int j = 0; j < (s.slice_off[sl + 1] - s.slice_off[sl]) / 64; j++) {
                const size_t at = sell_pos((size_t)s.slice_off[sl], j, l);
                const int slot = s.slice_off[sl] / 64 + j;
                int c;
                if (s.wide_off[sl] >= 0) c = s.wide[s.wide_off[sl] + (at - s.slice_off[sl])];
                else c = s.base[2 * slot + (s.off[at] >> 15)] + (s.off[at] & 0x7fff);
                if (c < 0 || c >= std::max(a.m, 1)) fail("column out of range");
                if (s.val[at] != 0.0) {
                    row[permute ? s.perm[c] : c] += s.val[at];
                    if (c <= last) fail("entries not in increasing column");
                    last = c;
                    used[at] = 1;
                }
            }
            std::map<int, double> want;
            for (int e = a.ptr[i]; e < a.ptr[i + 1]; e++) {
                want[a.col[e]] = a.val[e];
                if (permute && (s.val[pos[e]] != a.val[e] || !used[pos[e]])) fail("position");
            }
            if (row != want) fail("row");
        }
    }
    for (size_t e = 0; e < used.size(); e++)
        if (!used[e] && s.val[e] != 0.0) fail("padding");
    if (shorts != (index16 ? s.short_slices : 0)) fail("count of 16-bit slices");
    narrow = s.narrow_slices;
    const int all = s.nslices;
    auto ok = [&](int want, int have) { return want < 0 || (want == 0 ? have == 0 : want == 1 ? have > 0 && have < all : have == all); };
    if (!ok(want_short, s.short_slices) || !ok(want_narrow, narrow)) {
        std::printf("%d slices, %d short, %d narrow\n", all, s.short_slices, narrow);
        fail("column forms");
    }
}

int main()
{
    // want: 0 none, 1 some, 2 all, -1 not checked
    for (int n : {0, 1, 63, 64, 65, 200})
        for (int most : {0, 1, 3, 4, 5, 17})
            for (int window : {1 << 30, 64, 100}) {
                const Csr a = random_csr(n, std::max(n, 1), most, 0, (unsigned)(n + most));
                check(a, window, true, true, 2, 2);
                check(a, window, false, true, n ? 0 : -1, n ? 0 : -1);
                check(a, window, true, false, 2, 2);
            }
    // one reach near the diagonal and one half way round: two ranges
    check(random_csr(200000, 200000, 6, 300, 1), 4096, true, true, 1, 1);
    // columns anywhere: 32-bit, but for the empty rows at the end of each window
    check(random_csr(200000, 200000, 6, 0, 2), 4096, true, true, 1, 1);
    // wide rectangular rows, columns not renumbered
    check(random_csr(300, 150000, 9, 200, 3), 64, true, false, -1, -1);
    std::printf("OK\n");
    return 0;
}

// Host check of the patches of the matrix-free operator (formats.cpp): summing
// one number per tet and node the way the kernels do (slots of a patch, its
// complete dofs, the partial sums of the shared ones) gives every dof's sum
// over its tets, and every index stays inside what it points into.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <random>

#include "../paper_1204_2586_amd/csrc/host/setup.hpp"

using namespace auxp;

static void check(int n, int nt, int nloc, int reach, int tp, unsigned seed)
{
    auto fail = [&](const char *what) {
        std::printf("FAIL %s (n %d, nt %d, nloc %d, tp %d)\n", what, n, nt, nloc, tp);
        std::exit(1);
    };
    std::mt19937 g(seed);
    std::vector<int> emap((size_t)nt * nloc), order(nt);
    std::iota(order.begin(), order.end(), 0);
    for (int i = 0; i + 1 < nt; i += 2) std::swap(order[i], order[i + 1]);
    std::vector<double> want(n, 0.0);
    for (int t = 0; t < nt; t++)
        for (int a = 0; a < nloc; a++) {
            // distinct dofs near the tet's place, some eliminated
            int d = n ? (int)((int64_t)t * n / nt + (int64_t)a * reach + (int)(g() % (unsigned)reach)) % n : -1;
            if (g() % 8 == 0) d = -1;
            for (int b = 0; b < a; b++)
                if (emap[(size_t)t * nloc + b] == d) d = -1;
            emap[(size_t)t * nloc + a] = d;
            if (d >= 0) want[d] += 64 * t + a;
        }
    Patches h;
    build_patches(n, nt, nloc, emap, order, tp, h);
    const int nb = (nloc + 3) / 4;
    if (h.word.size() != (size_t)h.npatch * tp / 16 * nb * 64 || h.tet.size() != (size_t)h.npatch * tp) fail("sizes");
    std::vector<double> have(n, 0.0), part(h.sh_ptr.back(), -1.0);
    std::vector<char> done(n, 0), tets(nt, 0);
    int most = 0;
    for (int p = 0; p < h.npatch; p++) {
        const int *m = &h.meta[4 * (size_t)p];
        most = std::max(most, m[1]);
        std::vector<double> ys((size_t)tp * nloc, -1.0);
        int in_patch = 0;
        for (int t = 0; t < tp; t++) {
            const int tet = h.tet[(size_t)p * tp + t];
            in_patch += tet >= 0;
            if (tet >= 0 && tets[tet]++) fail("tet twice");
            for (int a = 0; a < 4 * nb; a++) {
                const uint32_t w = h.word[(((size_t)p * tp + t) / 16 * nb + a / 4) * 64 + 16 * (a % 4) + t % 16];
                const int at = w & 0xffff, slot = w >> 16, d = tet >= 0 && a < nloc ? emap[(size_t)tet * nloc + a] : -1;
                if (d < 0) {
                    if (at != m[1] || slot != 0xffff) fail("missing node");
                    continue;
                }
                if (at >= m[1] || h.dof[m[0] + at] != d) fail("place of a dof");
                if (slot >= tp * nloc || ys[slot] != -1.0) fail("slot");
                if (slot < (int)(h.range[m[0] + at] & 0xffff) || slot >= (int)(h.range[m[0] + at] >> 16)) fail("slot range");
                ys[slot] = 64 * tet + a;
            }
        }
        if (in_patch == 0) fail("empty patch");
        for (int i = 0; i < m[1]; i++) {
            double s = 0.0;
            for (uint32_t q = h.range[m[0] + i] & 0xffff; q < h.range[m[0] + i] >> 16; q++) s += ys.at(q);
            if (i < m[2]) {
                if (done[h.dof[m[0] + i]]++) fail("dof twice");
                have[h.dof[m[0] + i]] = s;
            } else {
                double &v = part.at(h.pos.at(m[3] + i - m[2]));
                if (v != -1.0) fail("partial sum twice");
                v = s;
            }
        }
    }
    for (size_t k = 0; k < h.sh_dof.size(); k++) {
        if (done[h.sh_dof[k]]++) fail("shared dof twice");
        for (int q = h.sh_ptr[k]; q < h.sh_ptr[k + 1]; q++) have[h.sh_dof[k]] += part.at(q);
    }
    if (have != want) fail("sums");
    if (most != h.max_dofs || std::count(tets.begin(), tets.end(), 1) != nt) fail("counts");
}

int main()
{
    unsigned seed = 1;
    for (int nloc : {10, 20, 35})
        for (int tp : {16, 64, 128})
            for (int nt : {1, 5, 15, 16, 17, 127, 128, 129, 700})
                for (int n : {0, 1, 300}) check(n, nt, nloc, 4, tp, seed++);
    check(60000, 40000, 20, 6, 128, seed);
    std::printf("OK\n");
    return 0;
}

// Device storage formats built on the host (once per setup).
//
// Sliced ELLPACK for the P^k operator.  Rows keep the dof order (which is
// lexicographic in the vertex multisets, so neighbours along one mesh axis
// are adjacent in memory) except that within each window of `window`
// consecutive rows longer rows come first (stable): the rows of a slice then
// have nearly equal lengths.  Consecutive groups of `slice` rows form slices,
// padded to the slice's longest row with zero values; four consecutive
// entries of a row are adjacent, so one load of a lane brings four values (16
// or 32 bytes) or four columns.  A row's entries are sorted by internal
// column: entry j of the slice's rows then mostly points into one or two
// short ranges, and its columns are stored as 16-bit words, a range selector
// and a 15-bit offset from one of the slot's two bases.  On the cube meshes
// one range is enough for 52 % (P2, 48^3), 66 % (P3, 25^3) and 95 % (P4, 14^3)
// of the slices, two for 98.7 % (P2, 64^3) to 100 %; the others keep 32-bit
// columns.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <numeric>
#include <stdexcept>

#include "parallel.hpp"
#include "setup.hpp"

namespace auxp {

namespace {

// rows of [w0, w1) by decreasing length, stable (a counting sort)
template <typename Len>
void sort_window(int w0, int w1, Len len, std::vector<int> &perm)
{
    int top = 0;
    for (int i = w0; i < w1; i++) top = std::max(top, len(i));
    std::vector<int> at((size_t)top + 2, 0);
    for (int i = w0; i < w1; i++) at[top - len(i) + 1]++;
    for (int l = 0; l <= top; l++) at[l + 1] += at[l];
    for (int i = w0; i < w1; i++) perm[w0 + at[top - len(i)]++] = i;
}

// the entries of original row i in the layout's order: column in the layout,
// and in the low half the entry
void row_entries(const Csr &A, int i, const int *iperm, std::vector<uint64_t> &out)
{
    const int n = A.ptr[i + 1] - A.ptr[i];
    out.resize(n);
    for (int q = 0; q < n; q++) {
        const int e = A.ptr[i] + q;
        out[q] = (uint64_t)(uint32_t)(iperm ? iperm[A.col[e]] : A.col[e]) << 32 | (uint32_t)e;
    }
    if (iperm) std::sort(out.begin(), out.end());
}

// contiguous shares of [0, n) over the worker threads
template <typename F>
void for_shares(int n, size_t work, F f)
{
    const int nt = std::max(1, std::min(setup_threads(work), n));
    run_tasks(nt, [&](int t) { f((int)((int64_t)n * t / nt), (int)((int64_t)n * (t + 1) / nt)); });
}

}  // namespace

std::vector<int64_t> sell_offsets(const std::vector<int> &width, int slice)
{
    std::vector<int64_t> off(width.size() + 1, 0);
    int64_t entries = 0;
    for (size_t s = 0; s < width.size(); s++) {
        entries += (int64_t)width[s] * slice;
        off[s + 1] = off[s] + (int64_t)((width[s] + kSellGroup - 1) / kSellGroup) * kSellGroup * slice;
    }
    if (entries > 0x7fffffff) throw std::invalid_argument("operator too large for 32-bit ELL offsets");
    return off;
}

void build_sell(const Csr &A, int slice, int window, bool index16, Sell &out, bool permute_cols)
{
    if (slice != 64) throw std::invalid_argument("build_sell: slices of 64 rows");
    const int n = A.n;
    out = Sell();
    out.n = n;
    out.slice = slice;
    out.perm.resize(n);
    auto len = [&](int i) { return A.ptr[i + 1] - A.ptr[i]; };
    const int nwin = n ? (int)(((int64_t)n + window - 1) / window) : 0;
    for_shares(nwin, (size_t)n, [&](int a, int b) {
        for (int w = a; w < b; w++)
            sort_window((int)((int64_t)w * window), (int)std::min<int64_t>(n, (int64_t)(w + 1) * window), len, out.perm);
    });
    out.iperm.assign(n, 0);
    for (int i = 0; i < n; i++) out.iperm[out.perm[i]] = i;
    const int ns = out.nslices = (n + slice - 1) / slice;
    out.width.assign(ns, 0);
    for (int s = 0; s < ns; s++)
        for (int r = s * slice; r < std::min(n, (s + 1) * slice); r++) out.width[s] = std::max(out.width[s], len(out.perm[r]));
    out.slice_off = sell_offsets(out.width, slice);
    const size_t total = (size_t)out.slice_off.back();
    std::vector<int> col(total);
    out.val.resize(total);
    out.base.resize(total / slice * 2);
    out.off.resize(index16 ? total : 0);
    std::vector<char> kind(ns, 2);             // 0: one range per slot, 1: two, 2: 32-bit columns
    const int *ip = permute_cols ? out.iperm.data() : nullptr;
    for_shares(ns, A.col.size() / 8, [&](int sa, int sb) {
        std::vector<uint64_t> row;
        for (int s = sa; s < sb; s++) {
            const size_t e0 = (size_t)out.slice_off[s], e1 = (size_t)out.slice_off[s + 1];
            const int r0 = s * slice, r1 = std::min(n, r0 + slice);
            std::fill(col.begin() + e0, col.begin() + e1, -1);
            std::fill(out.val.begin() + e0, out.val.begin() + e1, 0.0);
            for (int r = r0; r < r1; r++) {
                row_entries(A, out.perm[r], ip, row);
                for (int j = 0; j < (int)row.size(); j++) {
                    const size_t at = sell_pos(e0, j, r - r0);
                    col[at] = (int)(row[j] >> 32);
                    out.val[at] = A.val[(uint32_t)row[j]];
                }
            }
            // Padding entries (value 0) repeat the last column of their own
            // row, so that an Inf or NaN in a vector meets only the rows that
            // have it.  (A row without entries takes its slot's first column.)
            const int slots = (int)((e1 - e0) / slice);
            for (int r = r0; r < r1; r++) {
                const int last = len(out.perm[r]) - 1;
                for (int j = last + 1; last >= 0 && j < slots; j++)
                    col[sell_pos(e0, j, r - r0)] = col[sell_pos(e0, last, r - r0)];
            }
            // the two ranges of every slot
            char k = 0;
            for (int j = 0; j < slots; j++) {
                int64_t lo = INT32_MAX, hi = -1, second = INT32_MAX;
                for (int l = 0; l < slice; l++) {
                    const int c = col[sell_pos(e0, j, l)];
                    if (c >= 0) {
                        lo = std::min<int64_t>(lo, c);
                        hi = std::max<int64_t>(hi, c);
                    }
                }
                if (hi < 0) lo = hi = 0;
                if (hi - lo >= 65536) {
                    for (int l = 0; l < slice; l++) {
                        const int c = col[sell_pos(e0, j, l)];
                        if (c >= lo + 32768) second = std::min<int64_t>(second, c);
                    }
                    k = std::max(k, (char)(hi - second < 32768 ? 1 : 2));
                } else {
                    second = lo + 32768;
                }
                const size_t t = e0 / slice + j;
                out.base[2 * t] = (int)lo;
                out.base[2 * t + 1] = (int)std::min<int64_t>(second, INT32_MAX);
                for (int l = 0; l < slice; l++) {
                    const size_t at = sell_pos(e0, j, l);
                    if (col[at] < 0) col[at] = (int)lo;
                    if (index16)
                        out.off[at] = (uint16_t)(col[at] < second ? (col[at] - lo) & 0x7fff
                                                                  : 0x8000 | ((col[at] - second) & 0x7fff));
                }
            }
            if (index16) kind[s] = k;
        }
    });
    out.wide_off.assign(ns, -1);
    int64_t wide = 0;
    for (int s = 0; s < ns; s++) {
        out.narrow_slices += kind[s] == 0;
        out.short_slices += kind[s] < 2;
        if (kind[s] == 2) {
            out.wide_off[s] = wide;
            wide += out.slice_off[s + 1] - out.slice_off[s];
        }
    }
    out.wide.resize((size_t)wide);
    for (int s = 0; s < ns; s++)
        if (kind[s] == 2)
            std::copy(col.begin() + out.slice_off[s], col.begin() + out.slice_off[s + 1],
                      out.wide.begin() + out.wide_off[s]);
}

std::vector<int> sell_positions(const Csr &A, const Sell &s)
{
    if (s.slice_off.back() > (int64_t)UINT32_MAX) throw std::invalid_argument("sell_positions: too many entries");
    std::vector<int> pos(A.col.size());
    for_shares(s.n, A.col.size() / 8, [&](int a, int b) {
        std::vector<uint64_t> row;
        for (int r = a; r < b; r++) {
            row_entries(A, s.perm[r], s.iperm.data(), row);
            for (int j = 0; j < (int)row.size(); j++)
                pos[(uint32_t)row[j]] = (int)(uint32_t)sell_pos((size_t)s.slice_off[r / s.slice], j, r % s.slice);
        }
    });
    return pos;
}

void build_tiles(const Csr &A, const std::vector<int> &order, const std::vector<int> &iperm, int tile, int cap,
                 Tiles &out)
{
    if (tile % 8) throw std::invalid_argument("build_tiles: tiles of a multiple of eight rows");
    const int n = A.n, groups = tile / 8;
    out = Tiles();
    out.n = n;
    out.tile = tile;
    auto len = [&](int i) { return A.ptr[i + 1] - A.ptr[i]; };
    // the tiles' first places on the curve: shares of it in parallel, each cut greedily
    // (at most 64, each with a mark per column)
    const int share = std::max(65536, (n + 63) / 64), shares = (int)(((int64_t)n + share - 1) / share);
    std::vector<std::vector<int>> cut(shares);
    run_tasks(std::max(shares, 1), [&](int sh) {
        if (sh >= shares) return;
        std::vector<int> seen(n, -1);
        const int end = (int)std::min<int64_t>(n, (int64_t)(sh + 1) * share);
        int rows = 0, count = 0, id = -1;
        for (int r = sh * share; r < end; r++) {
            const int i = order[r];
            int more = 0;
            for (int e = A.ptr[i]; e < A.ptr[i + 1]; e++) more += id < 0 || seen[A.col[e]] != id;
            if (id < 0 || rows == tile || count + more > cap) {
                id = r;
                cut[sh].push_back(r);
                rows = count = 0;
            }
            for (int e = A.ptr[i]; e < A.ptr[i + 1]; e++)
                if (seen[A.col[e]] != id) {
                    seen[A.col[e]] = id;
                    count++;
                }
            rows++;
        }
    });
    std::vector<int> first;
    for (const std::vector<int> &c : cut) first.insert(first.end(), c.begin(), c.end());
    out.ntiles = (int)first.size();
    first.push_back(n);
    out.rows.assign((size_t)out.ntiles * tile, -1);
    out.grp_off.assign((size_t)out.ntiles * groups + 1, 0);
    out.col_off.assign((size_t)out.ntiles + 1, 0);
    // the rows of each tile (of A, by decreasing length), its distinct columns and block counts
    std::vector<int> arow((size_t)out.ntiles * tile, -1);
    std::vector<std::vector<int>> cols(out.ntiles);
    for_shares(out.ntiles, A.col.size() / 4, [&](int ta, int tb) {
        for (int t = ta; t < tb; t++) {
            int *r = &arow[(size_t)t * tile];
            const int cnt = first[t + 1] - first[t];
            std::copy(order.begin() + first[t], order.begin() + first[t + 1], r);
            std::stable_sort(r, r + cnt, [&](int a, int b) { return len(a) > len(b); });
            std::vector<int> &c = cols[t];
            for (int i = 0; i < cnt; i++) {
                out.rows[(size_t)t * tile + i] = iperm[r[i]];
                for (int e = A.ptr[r[i]]; e < A.ptr[r[i] + 1]; e++) c.push_back(iperm[A.col[e]]);
            }
            std::sort(c.begin(), c.end());
            c.erase(std::unique(c.begin(), c.end()), c.end());
            for (int g = 0; g < groups; g++)
                out.grp_off[(size_t)t * groups + g + 1] = 8 * g < cnt ? (len(r[8 * g]) + 7) / 8 : 0;
        }
    });
    int64_t blocks = 0, ncols = 0;
    for (size_t g = 1; g < out.grp_off.size(); g++) {
        blocks += out.grp_off[g];
        if (blocks > 0x7fffffff) throw std::invalid_argument("build_tiles: operator too large");
        out.grp_off[g] = (int)blocks;
    }
    for (int t = 0; t < out.ntiles; t++) {
        if (cols[t].size() > 65535) throw std::invalid_argument("build_tiles: tile too wide for 16-bit positions");
        ncols += (int64_t)cols[t].size();
        out.max_cols = std::max(out.max_cols, (int)cols[t].size());
        out.col_off[t + 1] = (int)ncols;
    }
    out.ucols.resize((size_t)ncols);
    out.lidx.resize((size_t)blocks * 64);
    out.val.resize((size_t)blocks * 64);
    for_shares(out.ntiles, A.col.size() / 4, [&](int ta, int tb) {
        for (int t = ta; t < tb; t++) {
            const std::vector<int> &c = cols[t];
            std::copy(c.begin(), c.end(), out.ucols.begin() + out.col_off[t]);
            const size_t e0 = (size_t)out.grp_off[(size_t)t * groups] * 64, e1 = (size_t)out.grp_off[(size_t)(t + 1) * groups] * 64;
            std::fill(out.lidx.begin() + e0, out.lidx.begin() + e1, 0);
            std::fill(out.val.begin() + e0, out.val.begin() + e1, 0.0);
            for (int i = 0; i < tile; i++) {
                const int r = arow[(size_t)t * tile + i];
                if (r < 0) continue;
                const size_t b0 = (size_t)out.grp_off[(size_t)t * groups + i / 8] * 64 + 8 * (i % 8);
                // padding entries repeat the row's last column
                const int g = t * groups + i / 8, padded = 8 * (out.grp_off[(size_t)g + 1] - out.grp_off[g]);
                uint16_t p = 0;
                for (int e = A.ptr[r], j = 0; j < padded; e++, j++) {
                    const size_t at = b0 + 64 * (size_t)(j / 8) + j % 8;
                    if (e < A.ptr[r + 1]) {
                        p = (uint16_t)(std::lower_bound(c.begin(), c.end(), iperm[A.col[e]]) - c.begin());
                        out.val[at] = A.val[e];
                    }
                    out.lidx[at] = p;
                }
            }
        }
    });
}

Csr permute_symmetric(const Csr &A, const std::vector<int> &perm, const std::vector<int> &iperm)
{
    Csr B;
    B.n = A.n;
    B.m = A.m;
    B.ptr.assign((size_t)A.n + 1, 0);
    std::vector<std::pair<int, double>> row;
    for (int r = 0; r < A.n; r++) {
        const int i = perm[r];
        row.clear();
        for (int e = A.ptr[i]; e < A.ptr[i + 1]; e++) row.push_back({iperm[A.col[e]], A.val[e]});
        std::sort(row.begin(), row.end());
        for (auto &cv : row) {
            B.col.push_back(cv.first);
            B.val.push_back(cv.second);
        }
        B.ptr[r + 1] = (int)B.col.size();
    }
    return B;
}

Csr permute_rows(const Csr &A, const std::vector<int> &perm)
{
    Csr B;
    B.n = A.n;
    B.m = A.m;
    B.ptr.assign((size_t)A.n + 1, 0);
    for (int r = 0; r < A.n; r++) {
        int i = perm[r];
        B.col.insert(B.col.end(), A.col.begin() + A.ptr[i], A.col.begin() + A.ptr[i + 1]);
        B.val.insert(B.val.end(), A.val.begin() + A.ptr[i], A.val.begin() + A.ptr[i + 1]);
        B.ptr[r + 1] = (int)B.col.size();
    }
    return B;
}

void build_patches(int n, int nt, int nloc, const std::vector<int> &emap, const std::vector<int> &order, int tp,
                   Patches &out)
{
    if (tp % 16 || (int64_t)tp * nloc >= 65535) throw std::invalid_argument("build_patches: places per patch");
    const int nb = (nloc + 3) / 4;
    out = Patches();
    out.tp = tp;
    const int np = out.npatch = (nt + tp - 1) / tp;
    std::vector<int> first(np + 1);
    for (int p = 0; p <= np; p++) first[p] = (int)std::min<int64_t>(nt, (int64_t)p * tp);
    out.tet.assign((size_t)np * tp, -1);
    std::vector<std::vector<int>> dofs(np);
    std::vector<int> patches_of((size_t)n + 1, 0);
    for_shares(np, (size_t)nt * 8, [&](int pa, int pb) {
        for (int p = pa; p < pb; p++) {
            std::copy(order.begin() + first[p], order.begin() + first[p + 1], out.tet.begin() + (size_t)p * tp);
            std::vector<int> &d = dofs[p];
            for (int r = first[p]; r < first[p + 1]; r++)
                for (int a = 0; a < nloc; a++)
                    if (const int i = emap[(size_t)order[r] * nloc + a]; i >= 0) d.push_back(i);
            std::sort(d.begin(), d.end());
            d.erase(std::unique(d.begin(), d.end()), d.end());
        }
    });
    for (const std::vector<int> &d : dofs)
        for (int i : d) patches_of[i]++;
    // the shared dofs' partial sums
    std::vector<int> next(n, -1);
    out.sh_ptr.push_back(0);
    for (int i = 0; i < n; i++)
        if (patches_of[i] > 1) {
            next[i] = out.sh_ptr.back();
            out.sh_dof.push_back(i);
            if (next[i] > 0x7fffffff - patches_of[i]) throw std::invalid_argument("build_patches: too many shared dofs");
            out.sh_ptr.push_back(next[i] + patches_of[i]);
        }
    out.meta.resize((size_t)4 * np);
    int64_t nd = 0;
    for (int p = 0; p < np; p++) {
        std::vector<int> &d = dofs[p];
        std::stable_partition(d.begin(), d.end(), [&](int i) { return patches_of[i] == 1; });
        int in = 0;
        while (in < (int)d.size() && patches_of[d[in]] == 1) in++;
        const int m[4] = {(int)nd, (int)d.size(), in, (int)out.pos.size()};
        std::copy(m, m + 4, out.meta.begin() + 4 * (size_t)p);
        for (size_t i = in; i < d.size(); i++) out.pos.push_back(next[d[i]]++);
        nd += (int64_t)d.size();
        if (nd > 0x7fffffff) throw std::invalid_argument("build_patches: too many patch dofs");
        out.max_dofs = std::max(out.max_dofs, (int)d.size());
    }
    out.dof.resize((size_t)nd);
    out.range.resize((size_t)nd);
    out.word.resize((size_t)np * tp / 16 * nb * 64);
    for_shares(np, (size_t)nt * 16, [&](int pa, int pb) {
        std::vector<int> fill;
        for (int p = pa; p < pb; p++) {
            const std::vector<int> &d = dofs[p];
            const int *m = &out.meta[4 * (size_t)p], cnt = m[1];
            std::copy(d.begin(), d.end(), out.dof.begin() + m[0]);
            auto local = [&](int i) {
                const auto b = patches_of[i] == 1 ? d.begin() : d.begin() + m[2];
                return (int)(std::lower_bound(b, patches_of[i] == 1 ? d.begin() + m[2] : d.end(), i) - d.begin());
            };
            fill.assign((size_t)cnt + 1, 0);
            for (int r = first[p]; r < first[p + 1]; r++)
                for (int a = 0; a < nloc; a++)
                    if (const int i = emap[(size_t)order[r] * nloc + a]; i >= 0) fill[local(i) + 1]++;
            for (int i = 0; i < cnt; i++) fill[i + 1] += fill[i];
            for (int i = 0; i < cnt; i++) out.range[(size_t)m[0] + i] = (uint32_t)fill[i] | (uint32_t)fill[i + 1] << 16;
            for (int t = 0; t < tp; t++)
                for (int a = 0; a < 4 * nb; a++) {
                    const int r = first[p] + t;
                    const int i = r < first[p + 1] && a < nloc ? emap[(size_t)order[r] * nloc + a] : -1;
                    uint32_t w = 0xffff0000u | (uint32_t)cnt;
                    if (i >= 0) {
                        const int l = local(i);
                        w = (uint32_t)l | (uint32_t)fill[l]++ << 16;
                    }
                    const size_t tile = ((size_t)p * tp + t) / 16;
                    out.word[(tile * nb + a / 4) * 64 + 16 * (a % 4) + t % 16] = w;
                }
        }
    });
}

std::vector<int> morton_order(const std::vector<double> &xyz, int n)
{
    double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300};
    for (int i = 0; i < n; i++)
        for (int c = 0; c < 3; c++) {
            lo[c] = std::min(lo[c], xyz[3 * (size_t)i + c]);
            hi[c] = std::max(hi[c], xyz[3 * (size_t)i + c]);
        }
    // spread the 21 low bits of v to every third bit
    auto spread = [](uint64_t v) {
        v &= 0x1fffff;
        v = (v | v << 32) & 0x1f00000000ffffULL;
        v = (v | v << 16) & 0x1f0000ff0000ffULL;
        v = (v | v << 8) & 0x100f00f00f00f00fULL;
        v = (v | v << 4) & 0x10c30c30c30c30c3ULL;
        v = (v | v << 2) & 0x1249249249249249ULL;
        return v;
    };
    std::vector<std::pair<uint64_t, int>> code((size_t)n);
    for (int i = 0; i < n; i++) {
        uint64_t m = 0;
        for (int c = 0; c < 3; c++) {
            const double span = hi[c] - lo[c];
            const double t = span > 0 ? (xyz[3 * (size_t)i + c] - lo[c]) / span : 0.0;
            const uint64_t q = (uint64_t)std::min(2097151.0, std::max(0.0, std::floor(t * 2097151.0 + 0.5)));
            m |= spread(q) << c;
        }
        code[i] = {m, i};
    }
    std::sort(code.begin(), code.end());
    std::vector<int> ord((size_t)n);
    for (int r = 0; r < n; r++) ord[r] = code[r].second;
    return ord;
}

Csr renumber_cols(const Csr &A, const std::vector<int> &map, int split)
{
    Csr B;
    B.n = A.n;
    B.m = A.m;
    B.ptr.assign((size_t)A.n + 1, 0);
    std::vector<std::pair<int, double>> row;
    for (int r = 0; r < A.n; r++) {
        row.clear();
        for (int e = A.ptr[r]; e < A.ptr[r + 1]; e++) {
            const int j = A.col[e];
            row.push_back({j < split ? map[j] : split + map[j - split], A.val[e]});
        }
        std::sort(row.begin(), row.end());
        for (auto &cv : row) {
            B.col.push_back(cv.first);
            B.val.push_back(cv.second);
        }
        B.ptr[r + 1] = (int)B.col.size();
    }
    return B;
}

void build_ell(const Csr &A, int lanes, Ell &out)
{
    if (lanes < 1 || lanes > 64 || (64 % lanes) != 0) throw std::invalid_argument("build_ell: lanes must divide 64");
    const int rows = 64 / lanes;
    out = Ell();
    out.n = A.n;
    out.lanes = lanes;
    out.nslices = (A.n + rows - 1) / rows;
    out.slice_off.assign((size_t)out.nslices + 1, 0);
    for (int s = 0; s < out.nslices; s++) {
        int width = 0;
        for (int q = 0; q < rows && s * rows + q < A.n; q++) {
            const int i = s * rows + q;
            width = std::max(width, (A.ptr[i + 1] - A.ptr[i] + lanes - 1) / lanes);
        }
        out.slice_off[s + 1] = out.slice_off[s] + 64 * width;
    }
    out.col.assign((size_t)out.slice_off[out.nslices], 0);
    out.val.assign((size_t)out.slice_off[out.nslices], 0.0);
    for (int s = 0; s < out.nslices; s++)
        for (int q = 0; q < rows && s * rows + q < A.n; q++) {
            const int i = s * rows + q;
            for (int e = A.ptr[i], k = 0; e < A.ptr[i + 1]; e++, k++) {
                const size_t at = (size_t)out.slice_off[s] + (size_t)(k / lanes) * 64 + q * lanes + k % lanes;
                out.col[at] = A.col[e];
                out.val[at] = A.val[e];
            }
        }
}

}  // namespace auxp

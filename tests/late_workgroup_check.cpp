// Kernels whose first workgroup may set the stop flag that they also test, run
// on the host as a late workgroup sees them: the flag is set after one of its
// wavefronts has read it and before the others have.  The wavefronts have to
// meet at every barrier, and the iterate must stay as it is: the sum that
// stops the solve is negative, but not without the share of one wavefront.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include <hip/hip_runtime.h>

#include "../paper_1204_2586_amd/csrc/hip/kernels.hip"
#include "../paper_1204_2586_amd/csrc/hip/stokes.hip"

using namespace auxp;

static int failures = 0;

static void expect(bool ok, const char *kernel, int early, int set, const char *what)
{
    if (ok) return;
    std::printf("FAIL %s, wavefront %d early, flag %d: %s\n", kernel, early, set, what);
    failures++;
}

int main()
{
    const int n = 700, grid = 3, block = 1, maxit = 50;
    std::vector<double> x(n, 1.0), r(n, 2.0), z(n, 0.5), p(n, 0.25), p2(n, 0.25), q(n, 0.125), d(n, 1.0);
    std::vector<double> parts(3 * kMaxBlocks, 0.0), out(3 * kMaxBlocks, 0.0), hist(3 * (maxit + 2), 1.0), scal(8, 0.0);
    // tridiagonal, as CSR and as one group of four slots per slice
    std::vector<int> ptr{0}, col;
    std::vector<double> val;
    const int ns = (n + 63) / 64;
    std::vector<int4> meta(ns);
    std::vector<int> wide((size_t)ns * 256, 0);
    std::vector<double> sval((size_t)ns * 256, 0.0);
    for (int s = 0; s < ns; s++) meta[s] = make_int4(s, 1, s, 3);
    for (int i = 0; i < n; i++) {
        int j = 0;
        for (int c = std::max(i - 1, 0); c <= std::min(i + 1, n - 1); c++, j++) {
            col.push_back(c);
            val.push_back(c == i ? 2.0 : -1.0);
            wide[(size_t)(i / 64) * 256 + 4 * (i % 64) + j] = c;
            sval[(size_t)(i / 64) * 256 + 4 * (i % 64) + j] = c == i ? 2.0 : -1.0;
        }
        ptr.push_back((int)col.size());
    }
    int iter = 3, done = 0;
    CgState st{&iter, &done, hist.data(), hist.data() + maxit + 2, hist.data() + 2 * (maxit + 2), scal.data(), maxit};
    DevSellView A{n, ns, 1, meta.data(), nullptr, nullptr, wide.data(), sval.data()};

    for (int early = 0; early < 4; early++)
        for (int set = 0; set < 2; set++) {
            auto run = [&](const char *name, bool bad, const std::function<void()> &kernel) {
                // the first wavefront reads partials 0 .. 63
                for (int i = 0; i < 256; i++)
                    parts[i] = parts[kMaxBlocks + i] = bad && i / 64 == (early ? 0 : 3) ? -1000.0 : 1.0;
                done = 0;
                iter = 3;
                const std::vector<double> x0 = x;
                const bool met = host_hip::run(256, block, grid, early, [&] { done = set ? 3 : 0; }, kernel);
                expect(met, name, early, set, "the wavefronts part at a barrier");
                if (bad) expect(x == x0, name, early, set, "the iterate changes after the stop");
                else if (!set) expect(x != x0, name, early, set, "the iterate stays");
            };
            for (int bad = 0; bad < 2; bad++) {
                if (bad || !set) {
                    run("k_cg_update_prep", bad, [&] {
                        k_cg_update_prep<double, true>(n, x.data(), r.data(), p.data(), q.data(), st, out.data(), d.data(),
                                                       z.data(), nullptr, parts.data(), 256);
                    });
                    run("k_mass_update", bad, [&] {
                        k_mass_update(n, x.data(), r.data(), p.data(), q.data(), d.data(), z.data(), parts.data(), 256, 3,
                                      out.data(), st);
                    });
                }
            }
            // (these write no iterate)
            auto meet = [&](const char *name, const std::function<void()> &kernel) { run(name, true, kernel); };
            meet("k_cg_product", [&] {
                k_cg_product<1>(A, z.data(), p.data(), p2.data(), q.data(), parts.data(), 256, out.data(), st);
            });
            meet("k_cg_product, two wavefronts per slice", [&] {
                k_cg_product<2>(A, z.data(), p.data(), p2.data(), q.data(), parts.data(), 256, out.data(), st);
            });
            meet("k_mass_product", [&] {
                k_mass_product<4, true>(n, ptr.data(), col.data(), val.data(), z.data(), p.data(), p2.data(), q.data(),
                                        parts.data(), 256, 3, 1e-12, out.data(), st);
            });
            meet("k_mass_direction", [&] { k_mass_direction(n, z.data(), p.data(), parts.data(), 256, 3, 1e-12, st); });
            const RrFinish fin{parts.data(), 256, st};
            meet("k_sell_sweep", [&] {
                k_sell_sweep<double, double, double, double, false, true, 2>(A, d.data(), r.data(), z.data(), q.data(),
                                                                             nullptr, nullptr, &done, nullptr, fin);
            });
            meet("k_sell_sweep, four wavefronts per slice", [&] {
                k_sell_sweep<double, double, double, double, false, true, 4>(A, d.data(), r.data(), z.data(), q.data(),
                                                                             nullptr, nullptr, &done, nullptr, fin);
            });
        }
    if (failures == 0) std::printf("OK\n");
    return failures != 0;
}

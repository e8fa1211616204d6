// Host check of div6_quad (paper_2102_12416_amd/csrc/jc_div6.h), the division
// of the resident sweeps, against the host's IEEE division s / 6: every
// combination of edge values in the four places, and random values of every
// exponent beside ordinary ones, each in each place.  Built host-only by
// tests/test_div6_quad_cpu.py.  Any NaN matches any NaN.  Prints "checked <n>
// mismatches <m>"; exits 0 only when m == 0.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "jc_div6.h"

static double from64(uint64_t u)
{
    double x;
    std::memcpy(&x, &u, 8);
    return x;
}

static bool same(double a, double b)
{
    return (std::isnan(a) && std::isnan(b)) || std::memcmp(&a, &b, 8) == 0;
}

__attribute__((noinline)) static double ieee(double s) { return s / 6.0; }

static uint64_t n_checked = 0, n_bad = 0;

static void check(const double s[4])
{
    double v[4];
    jc::div6_quad(s[0], s[1], s[2], s[3], v[0], v[1], v[2], v[3]);
    ++n_checked;
    for (int k = 0; k < 4; ++k)
        if (!same(v[k], ieee(s[k])) && n_bad++ < 20)
            std::fprintf(stderr, "place %d of %a %a %a %a: got %a want %a\n", k, s[0], s[1], s[2], s[3], v[k], ieee(s[k]));
}

int main()
{
    const double edge[] = {0.0, -0.0, 0x1p-1074, -0x1p-1074, 3.5e-320, 0x1p-1022, -0x1.8p-1000, 0x1p-1000, 1.0, -6.0,
                           1.0 / 3.0, 1e300, 1.7e308, -1.7e308, INFINITY, -INFINITY, NAN};
    const int n = sizeof(edge) / sizeof(edge[0]);
    for (int a = 0; a < n; ++a)
        for (int b = 0; b < n; ++b)
            for (int c = 0; c < n; ++c)
                for (int d = 0; d < n; ++d) {
                    const double s[4] = {edge[a], edge[b], edge[c], edge[d]};
                    check(s);
                }
    uint64_t st = 0x12416;
    auto next = [&] {
        uint64_t z = (st += 0x9e3779b97f4a7c15ull);
        z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
        z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
        return z ^ (z >> 31);
    };
    for (uint64_t e = 0; e < 2048; ++e)
        for (int k = 0; k < 4000; ++k) {
            const uint64_t r = next();
            const double x = from64((r & 0x800fffffffffffffull) | (e << 52));
            double s[4] = {1.5, -2.25, 3e-9, 7e11};
            s[k & 3] = x;
            check(s);
            const double t[4] = {x, from64(next()), from64(next()), from64(next())};
            check(t);
        }
    std::printf("checked %llu mismatches %llu\n", (unsigned long long)n_checked, (unsigned long long)n_bad);
    return n_bad != 0;
}

// Host-side check of row_class_sum (dev.hpp), the first and last stage of the
// one-block solver's reductions: over rows of random numbers of mixed size, the
// four lanes of a class hold the same bits, and the sum is theirs to rounding.
// Built and run on the CPU by test_reductions_host.py; it launches nothing on a GPU.
#include <cmath>
#include <cstdio>
#include <random>

#include "dev.hpp"

using namespace lqs;

struct Row {
    double a[16];
    Row operator+(const Row &o) const
    {
        Row r;
        for (int i = 0; i < 16; ++i) r.a[i] = a[i] + o.a[i];
        return r;
    }
};
struct HostRows {
    template <int N> static Row by(const Row &v)
    {
        Row r;
        for (int i = 0; i < 16; ++i) r.a[i] = v.a[(i + 16 - N) & 15];
        return r;
    }
};

int main()
{
    std::mt19937_64 gen(5);
    std::normal_distribution<double> normal;
    long bad = 0;
    for (int trial = 0; trial < 20000; ++trial) {
        Row v;
        for (double &x : v.a) x = normal(gen) * std::exp2((double)(gen() % 8));
        const Row s = row_class_sum(v, HostRows());
        for (int c = 0; c < 4; ++c) {
            long double want = 0, mag = 0;
            for (int i = c; i < 16; i += 4) {
                want += v.a[i];
                mag += std::fabs(v.a[i]);
            }
            for (int i = c; i < 16; i += 4) bad += s.a[i] != s.a[c] || std::fabs(s.a[i] - want) > 4e-16 * mag;
        }
    }
    std::printf("bad %ld\n", bad);
    return bad != 0;
}

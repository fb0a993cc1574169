// Runs the library's pairwise sum on vectors whose exact sum is known: one 1 and
// N - 1 values of 2^-53, half an ulp of 1.  Added one after another they all vanish
// (an error of N - 1 halves); pairwise at most ceil(log2 N) roundings of at most
// half an ulp of a sum below 1.1 happen on the way of any value.
#include <cstdio>
#include <vector>

#include "sums.hpp"

template <int N>
int check(int step)
{
    int bad = 0;
    int levels = 0;
    while ((1 << levels) < N) ++levels;
    const double h = 0x1p-53;
    for (int at = 0; at < N; ++at) {   // the place of the 1
        std::vector<double> v((size_t)N * step, 1e300);
        for (int i = 0; i < N; ++i) v[(size_t)i * step] = i == at ? 1.0 : h;
        const double off = (syk::pairwise_sum<N>(v.data(), step) - 1.0) / h - (N - 1);
        if (!(off <= levels && off >= -levels)) {
            std::printf("N=%d step=%d 1 at %d: off by %g halves of an ulp, bound %d\n", N, step, at, off, levels);
            ++bad;
        }
    }
    double serial = 1.0;
    for (int i = 1; i < N; ++i) serial += h;
    if (N >= 8 && (N - 1) - (serial - 1.0) / h <= levels) {   // the values do tell the two orders apart
        std::printf("N=%d: a serial sum would pass\n", N);
        ++bad;
    }
    return bad;
}

template <int N>
int check_all()
{
    int bad = check<N>(1) + check<N>(3);
    if constexpr (N > 1) bad += check_all<N - 1>();
    return bad;
}

int main()
{
    const int bad = check_all<17>();
    std::printf("%s\n", bad ? "BAD" : "pairwise sums ok");
    return bad != 0;
}

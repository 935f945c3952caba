// Host-only checks of the rules in fft_tile.h by which a kernel picks the form of a
// direct stage, over every radix, length and width that a tile takes. Exit status 0
// when all hold.
#include <cstdio>

#include "fft_tile.h"

using namespace ips;

static int g_fail = 0;

static void expect(bool ok, const char *what, int R, int NR, int lgs)
{
    if (ok) return;
    if (++g_fail < 20) std::printf("FAILED: %s (R = %d, positions %d, 2^%d sequences)\n", what, R, NR, lgs);
}

// rounds of a thread over the items of ST x QT outputs
template <int NT>
static int rounds(int R, int NR, int lgs, int ST, int QT)
{
    return ((NR << lgs) / ST * ((R + QT - 1) / QT) + NT - 1) / NT;
}

template <bool F64, int MAXE, int NT>
static void check(int maxn)
{
    constexpr int Q2 = F64 ? 2 : 4;
    for (int R = 7; R < maxn; ++R) {
        bool prime = true;
        for (int q = 2; q * q <= R; ++q) prime = prime && R % q != 0;
        if (!prime) continue;
        for (int NR = 2; NR * R <= maxn; NR += 2)
            for (int lgs = 0; (NR * R) << lgs <= MAXE * NT && lgs <= 4; ++lgs) {
                const bool sh = direct_shared<F64, NT>(R, NR, lgs);
                const int ST = lgs > 0 ? 2 : 1, QT = lgs > 0 ? Q2 : 2 * Q2;
                const int r1 = rounds<NT>(R, NR, lgs, 1, 1), rs = rounds<NT>(R, NR, lgs, ST, QT);
                expect(r1 <= direct_items<MAXE, 1, 1>(), "held items, one output at a time", R, NR, lgs);
                expect(rs <= (lgs > 0 ? direct_items<MAXE, 2, Q2>() : direct_items<MAXE, 1, 2 * Q2>()),
                       "held items, shared", R, NR, lgs);
                // tiles without an output per thread never share, and a thread that
                // shares reads less than one that does not
                expect(r1 > 1 || !sh, "a tile of fewer outputs than threads shares", R, NR, lgs);
                expect(sh == (rs * (ST + QT) <= 2 * r1), "LDS reads of the shared form", R, NR, lgs);
            }
    }
}

int main()
{
    check<true, 4, 256>(2048);
    check<true, 8, 256>(2048);
    check<true, 16, 256>(2048);
    check<false, 4, 256>(2048);
    check<false, 8, 256>(2048);
    check<false, 16, 256>(2048);
    check<true, 4, 1024>(4096);
    check<true, 8, 1024>(8192);
    check<false, 4, 1024>(4096);
    check<false, 8, 1024>(8192);
    if (g_fail) return 1;
    std::printf("tile rules hold\n");
    return 0;
}

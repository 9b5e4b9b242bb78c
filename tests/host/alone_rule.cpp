// The rule that gives a phase workgroup four lanes per site (alone_on_cu in tables.h): by its LDS, or
// by the number of blocks of a colour against the CUs of the device or partition at hand.
#include <cstdio>

#include "../../paper_1210_7398_amd/csrc/tables.h"

int main() {
    const size_t all = 160 * 1024;
    sapq_geom G;  // 8^3 x 16 in 4^4 blocks: 16 blocks of a colour
    for (int m = 0; m < 4; ++m) { G.L[m] = m == 3 ? 16 : 8; G.block[m] = 4; }
    struct { int np; size_t lds; int n_cu; bool want; } cases[] = {
        {1, 24672, 256, true}, {1, 24672, 16, true}, {1, 24672, 15, false},  // by the number of blocks
        {2, 24672, 256, false},                                              // a split block never so
        {1, all / 2 + 96, 1, true}, {2, all / 2 + 96, 1, true}, {1, all / 2, 1, false}};
    int fails = 0;
    for (auto &c : cases) fails += sapq::alone_on_cu(&G, c.np, c.lds, all, c.n_cu) != c.want;
    printf(fails ? "%d failures\n" : "the rule holds\n", fails);
    return fails;
}

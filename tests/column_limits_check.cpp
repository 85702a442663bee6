// Host check of the column search's limits: every column of every root that it
// takes unit by unit is fixed under its own number, alone, second or third, and
// none reads as "no column".
#include <cstdio>

#include "bc_device.h"

using namespace bcdev;

int main()
{
    unsigned roots = 0, bad = 0;
    for (uint32_t du = 1; du <= 64 * kColRootPlanes + 64; ++du) {
        if (!col_root_fits(du, 1)) continue;
        ++roots;
        const uint32_t c = du - 1;   // the first unit's column
        bad += (du + 63) / 64 > kColRootPlanes;
        bad += c == kColNone || col_pack(c, kColNone, kColNone) == col_pack(kColNone, kColNone, kColNone);
        bad += col_fixed(col_pack(c, kColNone, kColNone), 0) != c;
        bad += col_fixed(col_pack(0, c, kColNone), 1) != c || col_fixed(col_pack(0, c, kColNone), 2) != kColNone;
        bad += col_fixed(col_pack(1, 0, c), 2) != c || col_fixed(col_pack(1, 0, c), 0) != 1;
    }
    printf("roots %u bad %u\n", roots, bad);
    return bad != 0 || roots < 1000;
}

// Host check of the several-sweeps shapes (linked from libj3d.so): the
// workgroups that the planner counts on per compute unit fit its 160 KB of
// LDS, with equal and with unequal blocks.  Exit status 0 when every case holds.
#include <cstdio>

#include "j3d_internal.hpp"

using namespace j3d;

int main()
{
    long bad = 0, n_cases = 0;
    for (int s = 0; s < mshape_count(); ++s) {
        const MShapeInfo mi = mshape_info(s);
        for (int g = 0; g < 2; ++g) {
            ++n_cases;
            if (mi.per_cu[g] >= 1 && (long)mi.per_cu[g] * mi.lds[g] <= 160 * 1024) continue;
            std::printf("shape %d general %d: %d workgroups of %d bytes\n", s, g, mi.per_cu[g], mi.lds[g]);
            ++bad;
        }
    }
    std::printf("%ld cases, %ld bad\n", n_cases, bad);
    return bad ? 1 : 0;
}

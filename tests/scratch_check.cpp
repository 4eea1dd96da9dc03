// Host check of the one-shot solve's tables (scratch_layout and scratch_tiles):
// the several-sweeps plan is bounded by what blocks and maps leave, so that the
// one chosen fits.  Exit status 0 when every case holds.
#include <cstdio>

#include "j3d_host.hpp"

using namespace j3d;

int main()
{
    long bad = 0, n_cases = 0;
    for (size_t nblocks : {1, 8, 512, 4096, 13000, 16383})
        for (size_t nmaps : {6, 1200, 49160, 200000}) {
            ++n_cases;
            const uint64_t most = scratch_tiles(nblocks, nmaps);
            const bool room = scratch_layout(nblocks, 0, nmaps).total <= kScratchBytes;
            if (room ? scratch_layout(nblocks, most, nmaps).total <= kScratchBytes &&
                           scratch_layout(nblocks, most + 8, nmaps).total > kScratchBytes
                     : most == 0)
                continue;
            std::printf("%zu blocks, %zu map entries: %llu tiles\n", nblocks, nmaps, (unsigned long long)most);
            ++bad;
        }
    // very wide, shallow grids: the plan taken fits, or none is
    for (int64_t ny = 15000; ny <= 16250; ny += 250) {
        ++n_cases;
        j3d_problem p{};
        p.n[0] = 16384;
        p.n[1] = ny;
        p.n[2] = 4;
        for (int a = 0; a < 3; ++a) p.nblk[a] = 1;
        Plan plan;
        const size_t nmaps = 2 * (size_t)(p.n[0] + p.n[1] + p.n[2]);
        MultiPlan m;
        if (make_plan(1, &p, false, &plan) == J3D_OK)
            make_multi(plan, nullptr, 256, scratch_tiles(1, nmaps), &m);
        if (m.shape < 0 || scratch_layout(1, m.tiles.size(), nmaps).total <= kScratchBytes) continue;
        std::printf("16384 x %ld x 4: shape %d, %zu tiles\n", (long)ny, m.shape, m.tiles.size());
        ++bad;
    }
    std::printf("%ld cases, %ld bad\n", n_cases, bad);
    return bad ? 1 : 0;
}

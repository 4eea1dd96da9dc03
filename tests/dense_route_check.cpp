// Host check of how the copies between a dense grid and its blocks run
// (dense_shape, linked from libj3d.so): by blocks where these are large and
// alike, cell by cell where they are small, narrow or very uneven.  Exit
// status 0 when every case holds.
#include <cstdio>
#include <vector>

#include "j3d_host.hpp"

using namespace j3d;

static long bad = 0, n_cases = 0;

static void check(const std::vector<int64_t> &x, const std::vector<int64_t> &y, const std::vector<int64_t> &z,
                  bool one, bool pairs, const char *what)
{
    ++n_cases;
    const std::vector<int64_t> *ext[3] = {&x, &y, &z};
    Decomp d;
    for (int a = 0; a < 3; ++a) {
        d.ext[a] = *ext[a];
        d.nb[a] = (int32_t)d.ext[a].size();
        d.n[a] = 0;
        for (int64_t e : d.ext[a]) {
            d.org[a].push_back(d.n[a]);
            d.n[a] += e;
        }
    }
    const DenseShape s = dense_shape(d);
    if (s.by_block[0] == one && s.by_block[1] == pairs) return;
    std::printf("%s: by blocks %d, in pairs %d\n", what, s.by_block[0], s.by_block[1]);
    ++bad;
}

static std::vector<int64_t> same(int count, int64_t e) { return std::vector<int64_t>((size_t)count, e); }
static std::vector<int64_t> skew(int64_t big, int count, int64_t small)
{
    std::vector<int64_t> v = same(count + 1, small);
    v[0] = big;
    return v;
}

int main()
{
    auto cube = [](std::vector<int64_t> v, bool one, bool pairs, const char *what) { check(v, v, v, one, pairs, what); };
    // measured at least 1.5 times as fast by blocks
    cube(same(1, 1), true, true, "one cell");
    cube(same(1, 401), true, true, "one block");
    cube(same(8, 64), true, true, "512^3 as 64^3 blocks");
    cube(same(32, 16), true, true, "512^3 as 16^3 blocks");
    cube(skew(400, 1, 112), true, true, "512^3 as 400 and 112");
    check(same(1, 512), same(1, 512), same(512, 1), true, true, "512^3 in planes");
    // measured at least 1.3 times as fast by cells
    cube(same(64, 1), false, false, "64^3 in single cells");
    cube(same(64, 4), false, false, "256^3 as 4^3 blocks");
    cube(same(64, 8), false, false, "512^3 as 8^3 blocks");
    cube(skew(505, 7, 1), false, false, "512^3, seven single cells an axis");
    cube(skew(121, 7, 1), false, false, "128^3, seven single cells an axis");
    cube(skew(400, 7, 16), false, false, "512^3 as 400 and seven times 16");
    cube(skew(416, 3, 32), false, false, "512^3 as 416 and three times 32");
    check(same(1, 512), same(512, 1), same(512, 1), false, false, "512^3 in rows");
    check(same(512, 1), same(1, 512), same(1, 512), false, false, "512^3 in x slices");
    // the grids of the GPU test
    check({64, 1, 5}, {45, 1, 4}, {1, 30, 9}, false, false, "uneven, by cells");
    check({150, 1, 1}, same(2, 64), {250, 1, 1, 1, 1}, false, false, "more cells than one transfer, by cells");
    check({128, 24}, same(2, 128), {70, 80}, true, true, "more cells than one transfer, by blocks");
    std::printf("%ld cases, %ld bad\n", n_cases, bad);
    return bad ? 1 : 0;
}

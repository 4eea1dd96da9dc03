// Host check of the multi-sweep tiles (cut_axis and make_multi, linked from
// libj3d.so).  Every shape's axis cuts cover the axis, start on the asked
// grid and fit the lanes with their halo; the planner's tiles of even and
// uneven decompositions cover every cell once, fit their shape, and with
// unequal blocks lie in one block row along z and read at most kMultiSegs.
// Exit status 0 when every case holds.
#include <cstdio>
#include <random>
#include <vector>

#include "j3d_host.hpp"

using namespace j3d;

static long bad = 0, n_cases = 0;

static void expect(bool ok, const char *what, long a, long b, long c)
{
    if (ok) return;
    if (bad < 20) std::printf("%s: %ld %ld %ld\n", what, a, b, c);
    ++bad;
}

static void check_plan(const int64_t n[3], const int32_t nb[3], const std::vector<int64_t> ext[3])
{
    ++n_cases;
    j3d_problem p{};
    for (int a = 0; a < 3; ++a) {
        p.n[a] = n[a];
        p.nblk[a] = nb[a];
        p.split[a] = ext[a].data();
    }
    Plan plan;
    expect(make_plan(1, &p, true, &plan) == J3D_OK, "plan", n[0], n[1], n[2]);
    MultiPlan m;
    make_multi(plan, nullptr, 256, plan.mtiles_cap, &m);
    if (m.shape < 0) {  // only where unequal blocks are too shallow
        int64_t low = n[2];
        for (int64_t e : ext[2]) low = e < low ? e : low;
        expect(low < 5, "no shape", n[0], n[1], n[2]);
        return;
    }
    const MShapeInfo mi = mshape_info(m.shape);
    expect(m.tiles.size() <= plan.mtiles_cap && m.prefix.back() == (int32_t)m.tiles.size(), "table", n[0], n[1], n[2]);
    std::vector<unsigned char> seen((size_t)(n[0] * n[1] * n[2]), 0);
    auto row = [&](int64_t z) {
        int32_t b = 0;
        while (b + 1 < nb[2] && plan.probs[0].d.org[2][b + 1] <= z) ++b;
        return b;
    };
    for (const Tile &t : m.tiles) {
        const bool in = t.x0 >= 0 && t.y0 >= 0 && t.z0 >= 0 && t.nxv > 0 && t.nyv > 0 && t.nzv > 0 &&
                        t.x0 + t.nxv <= n[0] && t.y0 + t.nyv <= n[1] && t.z0 + t.nzv <= n[2];
        expect(in, "tile outside the grid", t.x0, t.y0, t.z0);
        if (!in) continue;
        const int T = mi.t;
        expect(t.nxv + std::min(T, t.x0 + 1) + std::min<int64_t>(T, n[0] - t.x0 - t.nxv + 1) <= 64, "lanes", t.x0,
               t.nxv, n[0]);
        expect(t.nyv + std::min(T, t.y0 + 1) + std::min<int64_t>(T, n[1] - t.y0 - t.nyv + 1) <= mi.rows, "rows", t.y0,
               t.nyv, n[1]);
        if (m.general && plan.blocks.size() > 1) {
            const int32_t lo = row(std::max(0, t.z0 - T)), hi = row(std::min<int64_t>(n[2] - 1, t.z0 + t.nzv - 1 + T));
            expect(row(t.z0) == row(t.z0 + t.nzv - 1), "tile across block rows", t.z0, t.nzv, n[2]);
            expect(hi - lo < kMultiSegs, "block rows read", lo, hi, n[2]);
        }
        for (int64_t z = t.z0; z < t.z0 + t.nzv; ++z)
            for (int64_t y = t.y0; y < t.y0 + t.nyv; ++y)
                for (int64_t x = t.x0; x < t.x0 + t.nxv; ++x) ++seen[(size_t)((z * n[1] + y) * n[0] + x)];
    }
    long miss = 0;
    for (unsigned char c : seen) miss += c != 1;
    expect(miss == 0, "cells not covered once", n[0], n[1], n[2]);
}

int main()
{
    std::vector<Piece> px;
    for (int s = 0; s < mshape_count(); ++s) {
        const MShapeInfo mi = mshape_info(s);
        for (int cap : {64, mi.rows})
            for (int align : {1, 8})
                for (int32_t n = 1; n <= 700; ++n) {
                    if (align > 1 && (n % align || cap != 64)) continue;
                    ++n_cases;
                    cut_axis(n, cap, mi.t, align, &px);
                    int32_t at = 0;
                    for (const Piece &q : px) {
                        expect(q.at == at && q.len > 0 && q.at % align == 0, "piece", n, q.at, q.len);
                        expect(q.len + std::min(mi.t, q.at + 1) + std::min(mi.t, n - q.at - q.len + 1) <= cap, "fits",
                               n, q.at, q.len);
                        at += q.len;
                    }
                    expect(at == n, "axis covered", n, at, cap);
                }
    }
    std::mt19937_64 rng(3);
    for (int rep = 0; rep < 250; ++rep) {
        int64_t n[3];
        int32_t nb[3];
        std::vector<int64_t> ext[3];
        const bool even = rep % 3 == 0;
        for (int a = 0; a < 3; ++a) {
            nb[a] = 1 + (int32_t)(rng() % 4);
            const int64_t e = 1 + (int64_t)(rng() % (rep % 5 == 0 ? 9 : 45));
            n[a] = 0;
            for (int32_t i = 0; i < nb[a]; ++i) {
                ext[a].push_back(even ? e : 1 + (int64_t)(rng() % (rep % 5 == 0 ? 9 : 45)));
                n[a] += ext[a].back();
            }
        }
        check_plan(n, nb, ext);
    }
    std::printf("%ld cases, %ld bad\n", n_cases, bad);
    return bad ? 1 : 0;
}

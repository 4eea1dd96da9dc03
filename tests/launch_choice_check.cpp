// Host check of when several sweeps go into one launch (MultiPlan::pays and
// pays_all, linked from libj3d.so): never for a single sweep, not where the
// tiles' lanes or planes are mostly ring or blocks too far apart, always for
// long runs of ordinary grids.  Exit status 0 when every case holds.
#include <cstdio>
#include <vector>

#include "j3d_host.hpp"

using namespace j3d;

static long bad = 0, n_cases = 0;
typedef std::vector<int64_t> Ext;

static Ext same(int count, int64_t e) { return Ext((size_t)count, e); }

static void expect(bool ok, const char *grid, const char *what, long k)
{
    ++n_cases;
    if (ok) return;
    std::printf("%s: %s at %ld\n", grid, what, k);
    ++bad;
}

static void check(const char *name, const Ext &x, const Ext &y, const Ext &z, bool pays)
{
    const Ext *ext[3] = {&x, &y, &z};
    j3d_problem p{};
    for (int a = 0; a < 3; ++a) {
        p.nblk[a] = (int32_t)ext[a]->size();
        p.split[a] = ext[a]->data();
        for (int64_t e : *ext[a]) p.n[a] += e;
    }
    Plan plan;
    expect(make_plan(1, &p, true, &plan) == J3D_OK, name, "plan", 0);
    MultiPlan m;
    make_multi(plan, nullptr, 256, plan.mtiles_cap, &m);
    expect(!m.pays(1), name, "one sweep", 1);
    expect(m.pays(50) == pays, name, "fifty sweeps", 50);
    if (pays)
        for (long k : {4, 8, 12, 100}) expect(m.pays(k), name, "many sweeps", k);
    else
        for (long k : {2, 3, 4, 8, 100}) expect(!m.pays(k), name, "thin grid", k);
}

// One count of a grid in block rows a few planes deep.
static void check_rows(const char *name, const Ext &z, long k, bool pays)
{
    const Ext x{100, 156}, y{128, 128};
    const Ext *ext[3] = {&x, &y, &z};
    j3d_problem p{};
    for (int a = 0; a < 3; ++a) {
        p.nblk[a] = (int32_t)ext[a]->size();
        p.split[a] = ext[a]->data();
        for (int64_t e : *ext[a]) p.n[a] += e;
    }
    Plan plan;
    expect(make_plan(1, &p, true, &plan) == J3D_OK, name, "plan", 0);
    MultiPlan m;
    make_multi(plan, nullptr, 256, plan.mtiles_cap, &m);
    expect(m.pays(k) == pays, name, "sweeps", k);
}

static void check_batch(int64_t iters, bool pays)
{
    j3d_problem p[3] = {};
    const int64_t edge[3] = {64, 100, 37};
    for (int i = 0; i < 3; ++i)
        for (int a = 0; a < 3; ++a) {
            p[i].n[a] = edge[(i + a) % 3];
            p[i].nblk[a] = 1;
        }
    Plan plan;
    expect(make_plan(3, p, true, &plan) == J3D_OK, "batch", "plan", 0);
    for (int i = 0; i < 3; ++i) plan.probs[i].iters = iters - i > 0 ? iters - i : 0;
    std::vector<int32_t> order{0, 1, 2};
    MultiPlan m;
    make_multi(plan, &order, 256, plan.mtiles_cap, &m);
    expect(m.shape >= 0 && m.pays_all() == pays, "batch", "sweeps", iters);
}

// Blocks whose fields lie further apart than a 32-bit offset reaches.
static void check_reach(int64_t nx, int32_t bx, int64_t edge, bool ok, const char *name)
{
    j3d_problem p{};
    p.n[0] = nx;
    p.n[1] = p.n[2] = edge;
    p.nblk[0] = bx;
    p.nblk[1] = p.nblk[2] = 1;
    Plan plan;
    expect(make_plan(1, &p, true, &plan) == J3D_OK, name, "plan", 0);
    MultiPlan m;
    make_multi(plan, nullptr, 256, plan.mtiles_cap, &m);
    expect((m.shape >= 0) == ok, name, "shape", m.shape);
    expect(ok || !m.pays(50), name, "fifty sweeps", 50);
}

int main()
{
    check_reach(1600, 2, 800, false, "two blocks of 800^3, 8.2 GB");
    check_reach(1024, 2, 512, true, "two blocks of 512^3, 2.2 GB");
    check_reach(1600, 1, 800, true, "one block of 8.2 GB");
    // measured 1.4 to 3 times as fast several to a launch (50 sweeps)
    check("33x35x31", {33}, {35}, {31}, true);
    check("64^3", {64}, {64}, {64}, true);
    check("157x211x183", {157}, {211}, {183}, true);
    check("256^3 as 4^3", same(4, 64), same(4, 64), same(4, 64), true);
    check("512^3 as 8^3", same(8, 64), same(8, 64), same(8, 64), true);
    check("512^3", {512}, {512}, {512}, true);
    check("160^3 uneven", {40, 60, 60}, {50, 55, 55}, {45, 60, 55}, true);
    check("1 x 1 x 65536", {1}, {1}, {65536}, true);
    check("16 x 16 x 4096", {16}, {16}, {4096}, true);
    check("2048 x 2048 x 4", {2048}, {2048}, {4}, true);
    // measured 2 and 2.4 times as slow
    check("1 x 1024 x 1024", {1}, {1024}, {1024}, false);
    check("1 x 65536 x 1", {1}, {65536}, {1}, false);
    // 341 against 306 us, 155 against 146; 2585 against 3420
    Ext four = same(62, 4), five = same(50, 5);
    four.push_back(3);
    four.push_back(5);
    five.push_back(6);
    check_rows("256^3 in rows of 4 planes", four, 4, false);
    check_rows("256^3 in rows of 5 planes", five, 2, false);
    check_rows("256^3 in rows of 5 planes", five, 50, true);
    check_batch(0, false);
    check_batch(1, false);
    check_batch(100, true);
    std::printf("%ld cases, %ld bad\n", n_cases, bad);
    return bad ? 1 : 0;
}

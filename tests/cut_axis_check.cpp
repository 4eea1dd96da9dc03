// Host check of the axis cuts (cut_axis, linked from libj3d.so): as few pieces
// as fit the lanes or rows, every piece within its limit, and sizes up to the
// largest axis the library accepts.  Exit status 0 when every case holds.
#include <climits>
#include <cstdio>
#include <vector>

#include "j3d_host.hpp"

using namespace j3d;

static long bad = 0, n_cases = 0;

static void expect(bool ok, const char *what, long n, long cap, long t)
{
    if (ok) return;
    if (bad < 20) std::printf("%s: n %ld cap %ld t %ld\n", what, n, cap, t);
    ++bad;
}

// Fewest pieces whatever their lengths: greedy, each as long as fits.
static int32_t fewest(int32_t n, int cap, int t)
{
    int32_t at = 0, m = 0;
    while (at < n) {
        const int lo = std::min(t, at + 1);
        int32_t len = n - at;
        if (len + lo + 1 > cap) {  // not the last piece: a ring above, down to one cell at the axis' end
            len = std::min(n - at - 1, cap - lo - 1);
            while (len + lo + std::min(t, n - at - len + 1) > cap) --len;
        }
        at += len;
        ++m;
    }
    return m;
}

int main()
{
    std::vector<Piece> px;
    for (int s = 0; s < mshape_count(); ++s) {
        const MShapeInfo mi = mshape_info(s);
        for (int cap : {64, mi.rows}) {
            for (int32_t n = 1; n <= 1200; ++n) {
                ++n_cases;
                cut_axis(n, cap, mi.t, 1, &px);
                expect((int32_t)px.size() == fewest(n, cap, mi.t), "more pieces than needed", n, cap, mi.t);
                expect((int32_t)px.size() == cut_axis_count(n, cap, mi.t, 1), "count", n, cap, mi.t);
                int32_t at = 0;
                for (const Piece &q : px) {
                    expect(q.at == at && q.len >= 1 &&
                               q.len + std::min(mi.t, q.at + 1) + std::min(mi.t, n - q.at - q.len + 1) <= cap,
                           "piece", n, cap, mi.t);
                    // lanes along x take the boundary column from their own end of the axis only
                    expect(cap != 64 || px.size() == 1 || q.len >= mi.t, "thinner than the ring", n, cap, mi.t);
                    at += q.len;
                }
                expect(at == n, "axis covered", n, cap, mi.t);
            }
            if (cap == 64)  // starts on multiples of 8: as few pieces, none thinner than the ring
                for (int32_t n = 8; n <= 4096; n += 8) {
                    ++n_cases;
                    cut_axis(n, cap, mi.t, 8, &px);
                    const int inner = (cap - 2 * mi.t) / 8 * 8, end = (cap - mi.t - 1) / 8 * 8;
                    expect(px.size() == 1 ? n <= cap - 2
                                          : n <= 2 * end + inner * ((int64_t)px.size() - 2) &&
                                                (px.size() == 2 || n > 2 * end + inner * ((int64_t)px.size() - 3)),
                           "more pieces than needed (align 8)", n, cap, mi.t);
                    int32_t at = 0;
                    for (const Piece &q : px) {
                        const bool edge = q.at == 0 || q.at + q.len == n;
                        expect(q.at == at && q.at % 8 == 0 && q.len >= std::min(8, n) &&
                                   (px.size() == 1 || q.len <= (edge ? end : inner)),
                               "piece (align 8)", n, q.at, q.len);
                        at += q.len;
                    }
                    expect(at == n, "axis covered (align 8)", n, at, mi.t);
                }
            for (int32_t n : {INT_MAX, INT_MAX - 1, INT_MAX - mi.t, INT_MAX - 7}) {
                ++n_cases;
                const int inner = cap - 2 * mi.t;
                const int64_t m = cut_axis_count(n, cap, mi.t, 1);
                expect(m == ((int64_t)n - 2 * (mi.t - 1) + inner - 1) / inner, "largest axes", n, cap, mi.t);
            }
        }
    }
    // the size of a long thin grid: a query that does no device work
    j3d_problem p{};
    p.n[0] = INT_MAX;
    p.n[1] = p.n[2] = 1;
    p.auto_parts = 4096;
    uint64_t bytes = 0;
    ++n_cases;
    expect(j3d_arena_bytes(&p, &bytes) == J3D_OK && bytes > 16ull * INT_MAX, "arena of the largest axis", INT_MAX, 0, 0);
    std::printf("%ld cases, %ld bad\n", n_cases, bad);
    return bad ? 1 : 0;
}

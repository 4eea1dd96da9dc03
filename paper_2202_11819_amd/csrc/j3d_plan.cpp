// j3d_plan.cpp -- host-only planning and the host-only C-ABI queries.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>

#include "j3d_host.hpp"

namespace j3d {

namespace {
thread_local std::string g_last_error;
}

j3d_status set_error(j3d_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return st;
}

void clear_error() { g_last_error.clear(); }

const char *last_error_text() { return g_last_error.c_str(); }

uint64_t stream_start(uint64_t seed, uint64_t pid)
{
    // SplitMix64 (Steele, Lea, Flood 2014): state advances by the golden gamma,
    // the output is the mixed state.  Output number m from state s mixes
    // s + m*gamma.
    uint64_t z = seed + (pid + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

j3d_status auto_split(const int64_t n[3], int32_t parts, int32_t nb[3])
{
    if (parts < 1) return set_error(J3D_EINVAL, "auto split: parts must be >= 1 (got %d)", parts);
    if (parts > (1 << 22)) return set_error(J3D_EINVAL, "auto split: %d blocks, more than 2^22", parts);
    bool found = false;
    unsigned __int128 best = 0;
    int32_t bc[3] = {0, 0, 0};
    for (int32_t a = 1; a <= parts && a <= n[0]; ++a) {
        if (parts % a) continue;
        for (int32_t b = 1; b <= parts / a; ++b) {
            if ((parts / a) % b) continue;
            const int32_t c = parts / a / b;
            if (a > n[0] || b > n[1] || c > n[2]) continue;
            // total area of the cuts between blocks (the communication volume)
            const unsigned __int128 cost =
                (unsigned __int128)(a - 1) * (uint64_t)(n[1] * n[2]) +
                (unsigned __int128)(b - 1) * (uint64_t)(n[0] * n[2]) +
                (unsigned __int128)(c - 1) * (uint64_t)(n[0] * n[1]);
            const bool better = !found || cost < best ||
                                (cost == best && (c > bc[2] || (c == bc[2] && b > bc[1])));
            if (better) {
                found = true;
                best = cost;
                bc[0] = a;
                bc[1] = b;
                bc[2] = c;
            }
        }
    }
    if (!found)
        return set_error(J3D_EINVAL, "auto split: no factorisation of %d blocks fits %lldx%lldx%lld",
                         parts, (long long)n[0], (long long)n[1], (long long)n[2]);
    nb[0] = bc[0];
    nb[1] = bc[1];
    nb[2] = bc[2];
    return J3D_OK;
}

j3d_status resolve_decomp(const j3d_problem *p, Decomp *d)
{
    if (!p) return set_error(J3D_EINVAL, "problem is NULL");
    for (int a = 0; a < 3; ++a) {
        if (p->n[a] < 1 || p->n[a] > INT32_MAX)
            return set_error(J3D_EINVAL, "n[%d] = %lld out of range [1, 2^31-1]", a, (long long)p->n[a]);
        d->n[a] = p->n[a];
    }
    for (int f = 0; f < 6; ++f)
        if (!std::isfinite(p->bc[f])) return set_error(J3D_EINVAL, "bc[%d] is not finite", f);
    const bool all_zero = p->nblk[0] == 0 && p->nblk[1] == 0 && p->nblk[2] == 0;
    if (all_zero) {
        if (p->split[0] || p->split[1] || p->split[2])
            return set_error(J3D_EINVAL, "explicit splits need explicit block counts");
        const int32_t parts = p->auto_parts == 0 ? 1 : p->auto_parts;
        j3d_status st = auto_split(d->n, parts, d->nb);
        if (st != J3D_OK) return st;
        for (int a = 0; a < 3; ++a) {
            d->ext[a].assign(d->nb[a], d->n[a] / d->nb[a]);
            for (int64_t i = 0; i < d->n[a] % d->nb[a]; ++i) d->ext[a][i] += 1;
        }
    } else {
        for (int a = 0; a < 3; ++a) {
            const int32_t nb = p->nblk[a];
            if (nb < 1 || nb > d->n[a])
                return set_error(J3D_EINVAL, "nblk[%d] = %d out of range [1, n[%d]]", a, nb, a);
            d->nb[a] = nb;
            if (p->split[a]) {
                int64_t sum = 0;
                d->ext[a].resize(nb);
                for (int32_t i = 0; i < nb; ++i) {
                    const int64_t e = p->split[a][i];
                    if (e < 1) return set_error(J3D_EINVAL, "split[%d][%d] = %lld < 1", a, i, (long long)e);
                    d->ext[a][i] = e;
                    sum += e;
                }
                if (sum != d->n[a])
                    return set_error(J3D_EINVAL, "split[%d] sums to %lld, not n[%d] = %lld", a,
                                     (long long)sum, a, (long long)d->n[a]);
            } else {
                if (d->n[a] % nb)
                    return set_error(J3D_EINVAL, "even split needs n[%d] %% nblk[%d] == 0 (%lld %% %d)",
                                     a, a, (long long)d->n[a], nb);
                d->ext[a].assign(nb, d->n[a] / nb);
            }
        }
    }
    for (int a = 0; a < 3; ++a) {
        d->org[a].resize(d->nb[a]);
        int64_t o = 0;
        for (int32_t i = 0; i < d->nb[a]; ++i) {
            d->org[a][i] = o;
            o += d->ext[a][i];
        }
    }
    const int64_t nblocks = (int64_t)d->nb[0] * d->nb[1] * d->nb[2];
    if (nblocks > (1 << 22)) return set_error(J3D_EINVAL, "%lld blocks: more than 2^22", (long long)nblocks);
    for (int32_t bz = 0; bz < d->nb[2]; ++bz)
        for (int32_t by = 0; by < d->nb[1]; ++by)
            for (int32_t bx = 0; bx < d->nb[0]; ++bx) {
                const int64_t ex = d->ext[0][bx], ey = d->ext[1][by], ez = d->ext[2][bz];
                if (block_field_cells(ex, ey, ez) > INT32_MAX || ey * ez > INT32_MAX / 2 ||
                    ex * ez > INT32_MAX || ex * ey > INT32_MAX)
                    return set_error(J3D_EINVAL, "block %lldx%lldx%lld exceeds 2^31 cells with halos",
                                     (long long)ex, (long long)ey, (long long)ez);
                // the sweep addresses one plane (with its ghost rows) by 32-bit byte offsets
                if (plane_stride(row_pitch(ex), ey) * 8 > INT32_MAX)
                    return set_error(J3D_EINVAL, "block %lldx%lldx%lld: an x-y plane exceeds 2^28 cells",
                                     (long long)ex, (long long)ey, (long long)ez);
            }
    return J3D_OK;
}

namespace {

struct Bump {
    uint64_t off = 0;
    uint64_t take(uint64_t bytes, uint64_t align = 256)
    {
        off = align_up(off, align);
        const uint64_t at = off;
        off += bytes;
        return at;
    }
};

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

int max_ez(const Plan &plan, int32_t b0, int32_t b1)
{
    int m = 1;
    for (int32_t b = b0; b < b1; ++b) m = plan.blocks[b].ext[2] > m ? plan.blocks[b].ext[2] : m;
    return m;
}

}  // namespace

DenseShape dense_shape(const Decomp &d)
{
    DenseShape s{1, 1, {d.nb[0], d.nb[1], d.nb[2]}, true, {true, true}};
    int64_t most[3] = {1, 1, 1};
    for (int a = 0; a < 3; ++a)
        for (int64_t e : d.ext[a]) most[a] = std::max(most[a], e);
    for (int64_t e : d.ext[0]) s.even_rows = s.even_rows && e % 2 == 0;
    s.max_plane = (int32_t)(most[0] * most[1]);
    s.max_depth = (int32_t)most[2];
    const double blocks = (double)d.nb[0] * d.nb[1] * d.nb[2];
    if (blocks == 1) return s;
    // Measured on MI355X over 40 decompositions, from 64^3 in single cells to
    // 640^3 uneven: a run by blocks takes 3.2 ns (5.2 ns in pairs) however full
    // it is, its dense rows' share of partly written cache lines on top; a
    // workgroup that finds no run 0.27 ns; by cells 5.4 ns per 1000.
    double rows = 0;
    for (int32_t b = 0; b < d.nb[0]; ++b) {
        const bool lines = d.n[0] % 16 == 0 && d.org[0][b] % 16 == 0 && d.ext[0][b] % 16 == 0;
        rows += (double)d.ext[0][b] + (lines ? 0 : 24);
    }
    rows /= (double)d.n[0];
    const double by_cells = 5.4e-3 * (double)d.n[0] * (double)d.n[1] * (double)d.n[2];
    for (int pairs = 0; pairs < 2; ++pairs) {
        const int per = kDenseRun << pairs;
        const bool flat = dense_flat(s.max_plane, per);
        double runs = 0;
        for (int64_t ey : d.ext[1])
            for (int64_t ex : d.ext[0]) {
                if (!flat) runs += (double)ceil_div(ex * ey, per) * (double)d.n[2];
                for (int32_t b = 0; flat && b < d.nb[2]; ++b) runs += (double)ceil_div(ex * ey * d.ext[2][b], per);
            }
        const double depth = s.max_depth;
        const double grid = blocks * (flat ? std::ceil(s.max_plane * depth / per)
                                           : std::ceil((double)s.max_plane / per) * depth);
        s.by_block[pairs] = runs * (pairs ? 5.2 : 3.2) * rows + (grid - runs) * 0.27 < by_cells;
    }
    return s;
}

int find_variant(int tile_x, int tile_y, int threads)
{
    for (int v = 0; v < variant_count(); ++v) {
        const VariantInfo vi = variant_info(v);
        if (vi.tile_x == tile_x && vi.tile_y == tile_y && vi.threads == threads) return v;
    }
    return -1;
}

int find_flat_variant(int threads, int cells, int prefetch)
{
    for (int v = 0; v < variant_count(); ++v) {
        const VariantInfo vi = variant_info(v);
        if (vi.tile_x == 0 && vi.tile_y == cells && vi.threads == threads && vi.prefetch == prefetch) return v;
    }
    return -1;
}

uint64_t count_tiles(const Plan &plan, int variant, int zchunk)
{
    const VariantInfo vi = variant_info(variant);
    const int zc = zchunk > 0 ? zchunk : max_ez(plan, 0, (int32_t)plan.blocks.size());
    uint64_t n = 0, of = 0;
    const int32_t *last = nullptr;  // a block's neighbours in the table mostly have its extents
    for (const BlockDesc &B : plan.blocks) {
        if (!last || B.ext[0] != last[0] || B.ext[1] != last[1] || B.ext[2] != last[2]) {
            int64_t ntx, nty;
            tiles_xy(vi, B.ext[0], B.ext[1], &ntx, &nty);
            of = (uint64_t)(ntx * nty * ceil_div(B.ext[2], zc));
            last = B.ext;
        }
        n += of;
    }
    return n;
}

// The end pieces have the ring on one side only and one boundary cell on the
// other, so they can hold t - 1 cells more than the inner ones.
int32_t cut_axis_count(int32_t n, int cap, int t, int align)
{
    if (n <= cap - 2) return 1;
    const int32_t inner = (cap - 2 * t) / align * align, end = (cap - t - 1) / align * align;
    return (int32_t)(2 + std::max<int64_t>(0, ((int64_t)n - 2 * end + inner - 1) / inner));
}

void cut_axis(int32_t n, int cap, int t, int align, std::vector<Piece> *out)
{
    const int32_t m = cut_axis_count(n, cap, t, align);
    out->assign(1, Piece{0, n});
    if (m == 1) return;
    // Where all m pieces fit so, end pieces t - 1 cells shorter than the inner
    // ones: boundary tiles take longer (512^3, 10 x 10 tiles: 13.78 ms per 100
    // sweeps against 13.95 with end pieces the longer ones).
    auto shorter_ends = [&](int32_t i) {
        const int64_t at = i * ((int64_t)n + 2 * (t - 1)) / m - (t - 1);
        return (int32_t)((at + align / 2) / align * align);
    };
    // Else end pieces t - 1 cells longer, which always fits; with starts on
    // multiples of `align`, pieces of an even multiple (a whole number of cache
    // lines for align 8) or one more: a start inside a line splits it between tiles.
    const int32_t units = n / align, inner = (cap - 2 * t) / align;
    const int32_t even = std::min(inner / 2 * 2, ((units + m - 1) / m + 1) / 2 * 2);
    const int32_t extra = units - even * m;  // pieces one unit longer: pairs first, an odd one last
    const int32_t first = extra <= 0 ? 0 : inner > even ? extra / 2 * 2 : extra - 1;
    auto longer_ends = [&](int32_t i) {
        if (align == 1) return (int32_t)(i * ((int64_t)n - 2 * (t - 1)) / m + (t - 1));
        return (even * i + std::min(i, first)) * align;
    };
    auto cut = [&](auto start) {
        out->clear();
        for (int32_t i = 0, at = 0; i < m; ++i) {
            const int32_t next = i + 1 < m ? start(i + 1) : n, len = next - at;
            if (len < 1 || len + std::min(t, at + 1) + std::min(t, n - next + 1) > cap) return false;
            out->push_back({at, len});
            at = next;
        }
        return true;
    };
    if (!cut(shorter_ends)) cut(longer_ends);
}

namespace {

constexpr int kMinMultiZ = 4;

int x_align(const ProbPlan &pp)
{
    if (pp.nblocks == 1) return pp.d.n[0] % 8 ? 1 : 8;
    for (int64_t e : pp.d.ext[0])
        if (e % 8) return 1;
    return 8;
}

uint64_t multi_tiles_bound(const Plan &plan)
{
    uint64_t best = 0;
    for (int s = 0; s < mshape_count(); ++s) {
        const MShapeInfo mi = mshape_info(s);
        uint64_t n = 0;
        for (const ProbPlan &pp : plan.probs) {
            n += (uint64_t)cut_axis_count((int32_t)pp.d.n[0], 64, mi.t, x_align(pp)) *
                 cut_axis_count((int32_t)pp.d.n[1], mi.rows, mi.t, 1) * ceil_div(pp.d.n[2], kMinMultiZ);
        }
        best = std::max(best, n);
    }
    return best;
}

// Plane steps of a tile: its planes and the ramp on both sides, in rounds of two.
int64_t multi_steps(const MShapeInfo &mi, int64_t planes)
{
    return (planes + 2 * mi.t + 1) / 2 * 2;
}

// Estimated microseconds per sweep of a launch of `tiles` tiles of `steps`
// plane steps each.  Fitted to MI355X timings of every shape on 13 grids from
// 33x35x31 to 1024^3:
//   - a plane step issues about 13 instructions per cell, stage and wave
//     (7 FP64, 4 DPP, 2 for the boundary) and 15 more, and waits about 0.3 us
//     for LDS, barrier and dependent chains; the fit gives an instruction 1.8
//     ns per SIMD, where FP64 and DPP ones alone measured 2.0;
//   - a tile starts with about 3 us of table lookups and first loads, with
//     unequal blocks 0.9 us more for each of a thread's rows (256^3 in block
//     rows of 5 planes: 200 us a launch by 64-row tiles, 158 without);
//   - memory moves 17 bytes per cell and launch at 5.3 TB/s, at 3.2 TB/s where
//     tiles end inside cache lines and the grid is past the last-level cache;
//   - the two overlap only in part: the third root of the sum of cubes.
// Constants refitted to 5200 timings of 47 grids, with four other shapes,
// measured 0.996 of the speed over 22 solves, batches and pools: not kept.
// The planner asks for some 250 of them while a solver is created, so where the
// larger part alone is above `worse` no root is taken (any value above it does).
double multi_cost(const MShapeInfo &mi, bool general, int cus, double tiles, double steps, double cells, bool ragged,
                  double worse = HUGE_VAL)
{
    auto up = [](double v) {
        const double k = (double)(int64_t)v;
        return k < v ? k + 1 : k;
    };
    const double c = std::min<double>(mi.per_cu[general], up(tiles / cus));  // workgroups sharing a compute unit
    const int cpt = mi.rows * 64 / mi.threads;                              // cells per thread
    const double valu = mi.threads / 256 * (cpt * mi.t * 13.0 + 15) * 0.0018;
    const double step = c * valu + 0.3;
    const double start = general ? 3.0 + 0.9 * cpt : 3.0;
    const double compute = up(tiles / (cus * c)) * (steps * step + start);
    const double hbm = cells * 17.0 / (ragged && cells > 1.6e7 ? 3.2e6 : 5.3e6);
    const double least = (std::max(compute, hbm) + 3.0) / mi.t;
    if (least > worse) return least;
    return (std::cbrt(compute * compute * compute + hbm * hbm * hbm) + 3.0) / mi.t;
}

// What a launch of the one-sweep kernel takes, from the blocks added so far.
// Fitted to MI355X timings of 21 grids from 8^3 to 640^3, thin, uneven and
// decomposed ones among them, within 20%: a compute unit takes a tile at a
// time, 2.5 us and, for each plane it reads, 0.13 us and 0.31 us per 1024 cells
// of the shape; memory moves the cells and the rings and planes around them at
// 5.9 TB/s; third root of the sum of cubes.
struct SingleCost {
    VariantInfo vi;
    int zchunk;  // 0: whole blocks
    int64_t ex = 0, ey = 0, ez = 0;
    double n = 0, steps = 0, moved = 0;  // of a block of these extents
    double tiles = 0, all_steps = 0, cells = 0;

    SingleCost(const j3d_tune &t) : vi(variant_info(t.variant)), zchunk(t.zchunk) {}

    void add(const BlockDesc &B)
    {
        if (B.ext[0] != ex || B.ext[1] != ey || B.ext[2] != ez) {
            ex = B.ext[0];
            ey = B.ext[1];
            ez = B.ext[2];
            int64_t ntx, nty;
            tiles_xy(vi, ex, ey, &ntx, &nty);
            const int64_t ntz = zchunk > 0 ? ceil_div(ez, zchunk) : 1;
            n = (double)(ntx * nty * ntz);
            steps = (double)(ntx * nty) * (double)(ez + 2 * ntz);
            moved = (double)(ex * ey) * (double)(2 * ez + 2 * ntz) + 2.0 * (double)(nty * ex + ntx * ey) * (double)ez;
        }
        tiles += n;
        all_steps += steps;
        cells += moved;
    }
    double us(int cus) const
    {
        if (tiles == 0) return 0;
        const double step = 0.13 + 0.31 * (vi.tile_x ? vi.tile_x * vi.tile_y : vi.tile_y) / 1024;
        const double compute = std::ceil(tiles / cus) * (all_steps / tiles * step + 2.5), hbm = cells * 8 / 5.9e6;
        return std::cbrt(compute * compute * compute + hbm * hbm * hbm) + 0.5;
    }
};

// Byte span of a tile's blocks from its first block's field: the lane offsets
// are 32-bit.
bool multi_span_ok(const Plan &plan, const ProbPlan &pp, const std::vector<Piece> &px, const std::vector<Piece> &py,
                   int t)
{
    const Decomp &d = pp.d;
    if (pp.nblocks == 1) return true;
    const BlockDesc &first = plan.blocks[pp.block_begin], &last = plan.blocks[pp.block_begin + pp.nblocks - 1];
    if ((last.off[0] - first.off[0] + block_field_cells(last.ext[0], last.ext[1], last.ext[2])) * 8 <= 0xFFFFF000ll)
        return true;  // all of the problem's fields within reach
    auto owner = [](const std::vector<int64_t> &org, int64_t c) {
        return (int32_t)(std::upper_bound(org.begin(), org.end(), c) - org.begin()) - 1;
    };
    for (const Piece &y : py)
        for (const Piece &x : px) {
            const int32_t ax = owner(d.org[0], std::max(0, x.at - t)), ay = owner(d.org[1], std::max(0, y.at - t));
            const int32_t ex = owner(d.org[0], std::min<int64_t>(d.n[0] - 1, x.at + x.len - 1 + t));
            const int32_t ey = owner(d.org[1], std::min<int64_t>(d.n[1] - 1, y.at + y.len - 1 + t));
            for (int32_t bz = 0; bz < d.nb[2]; ++bz) {
                const BlockDesc &A = plan.blocks[pp.block_begin + ax + d.nb[0] * (ay + d.nb[1] * bz)];
                const BlockDesc &B = plan.blocks[pp.block_begin + ex + d.nb[0] * (ey + d.nb[1] * bz)];
                const int64_t end = B.off[0] - A.off[0] + block_field_cells(B.ext[0], B.ext[1], B.ext[2]);
                if (end * 8 > 0xFFFFF000ll) return false;
            }
        }
    return true;
}

}  // namespace

void fill_prob(const Plan &plan, int32_t i, int64_t maps_base, ProbDesc *pd)
{
    std::memset(pd, 0, sizeof *pd);
    const ProbPlan &pp = plan.probs[i];
    pd->res_slot = i;
    pd->limit = pp.iters;
    pd->flags = PF_RES_LAST;
    for (int a = 0; a < 3; ++a) {
        pd->nb[a] = pp.d.nb[a];
        pd->n[a] = (int32_t)pp.d.n[a];
    }
    pd->maps_off = (int64_t)pp.maps_off - maps_base;
}

namespace {

// z pieces of a problem: near-equal, at most zc planes.  With unequal blocks
// (general) each lies in one block row, and the rows are at least t deep, so a
// tile reads its own row and its two neighbours at most.  Calls
// cut(start, planes, pieces) for each uncut stretch, whose piece i starts at
// i * planes / pieces; false if a row is too shallow.
template <class F>
bool cut_z(const ProbPlan &pp, bool general, int t, int zc, F cut)
{
    const bool rows = general && pp.nblocks > 1;
    for (int32_t b = 0; b < (rows ? pp.d.nb[2] : 1); ++b) {
        const int64_t at = rows ? pp.d.org[2][b] : 0, len = rows ? pp.d.ext[2][b] : pp.d.n[2];
        if (rows && len < t) return false;
        cut(at, len, ceil_div(len, zc));
    }
    return true;
}

}  // namespace

void make_multi(const Plan &plan, const std::vector<int32_t> *order, int cus, uint64_t cap, MultiPlan *m,
                const j3d_tune *one, int only)
{
    *m = MultiPlan{};
    m->prefix.assign(1, 0);
    const int32_t count = (int32_t)(order ? order->size() : plan.probs.size());
    auto prob = [&](int32_t k) -> const ProbPlan & { return plan.probs[order ? (*order)[k] : k]; };
    int64_t depth = 1;
    bool ragged = false;
    for (int32_t k = 0; k < count; ++k) {
        const ProbPlan &pp = prob(k);
        const BlockDesc &A = plan.blocks[pp.block_begin];
        for (int32_t b = pp.block_begin; b < pp.block_begin + pp.nblocks; ++b)
            for (int a = 0; a < 3; ++a) m->general = m->general || plan.blocks[b].ext[a] != A.ext[a];
        depth = std::max(depth, pp.d.n[2]);
        ragged = ragged || x_align(pp) == 1;
    }
    // The z stretches to cut, those of equal depth together: a pool round of 256
    // requests is planned while the GPU waits (250 us by requests, 60 by depths).
    // The problems of a group run together for as many sweeps as they have more
    // than the next group (a batch, longest first; else all in one).
    struct Stretch {
        int32_t group, len, k;
    };
    std::vector<Stretch> zs;
    std::vector<double> group_sweeps, group_cells;
    double cells = 0;
    for (int32_t k = 0; k < count; ++k) {
        const ProbPlan &pp = prob(k);
        cut_z(pp, m->general, 0, 1, [&](int64_t, int64_t len, int64_t) {
            zs.push_back({(int32_t)group_cells.size(), (int32_t)len, k});
        });
        cells += (double)pp.d.n[0] * pp.d.n[1] * pp.d.n[2];
        if (k + 1 < count && pp.iters == prob(k + 1).iters) continue;
        group_sweeps.push_back(k + 1 < count ? (double)(pp.iters - prob(k + 1).iters)
                                             : std::max(1.0, (double)pp.iters));
        group_cells.push_back(cells);
    }
    std::sort(zs.begin(), zs.end(), [](const Stretch &a, const Stretch &b) {
        return a.group != b.group ? a.group < b.group : a.len != b.len ? a.len < b.len : a.k < b.k;
    });
    struct Column {
        int32_t group, len;
        double xy;  // tiles of an x-y plane
    };
    std::vector<Column> columns;
    std::vector<Piece> px, py;
    std::vector<int64_t> xy(count);
    int best_shape = -1, best_zc = 0;
    double best = 0;
    for (int s = 0; s < mshape_count(); ++s) {
        const MShapeInfo mi = mshape_info(s);
        bool ok = only < 0 || s == only;
        for (int32_t k = 0; k < count && ok; ++k) {
            const ProbPlan &pp = prob(k);
            xy[k] = (int64_t)cut_axis_count((int32_t)pp.d.n[0], 64, mi.t, x_align(pp)) *
                    cut_axis_count((int32_t)pp.d.n[1], mi.rows, mi.t, 1);
            if (pp.nblocks > 1) {
                cut_axis((int32_t)pp.d.n[0], 64, mi.t, x_align(pp), &px);
                cut_axis((int32_t)pp.d.n[1], mi.rows, mi.t, 1, &py);
                ok = multi_span_ok(plan, pp, px, py, mi.t) &&
                     cut_z(pp, m->general, mi.t, 1, [](int64_t, int64_t, int64_t) {});
            }
        }
        if (!ok) continue;
        columns.clear();
        for (const Stretch &z : zs)
            if (!columns.empty() && columns.back().group == z.group && columns.back().len == z.len)
                columns.back().xy += (double)xy[z.k];
            else
                columns.push_back({z.group, z.len, (double)xy[z.k]});
        int32_t last_zc = 0;
        for (int64_t nc = 1; nc <= ceil_div(depth, kMinMultiZ); nc += 1 + (count > 1 ? nc / 8 : nc / 16)) {
            const int32_t zc = (int32_t)ceil_div(depth, nc);
            if (zc == last_zc) continue;
            last_zc = zc;
            double tiles = 0, steps = 0, cost = 0;
            for (size_t i = 0; i < columns.size(); ++i) {
                const Column &c = columns[i];
                const int32_t n = (c.len - 1) / zc + 1, low = c.len / n, more = c.len - low * n;
                // n pieces: `more` of them a plane deeper than the others
                tiles += c.xy * n;
                steps += c.xy * (double)(more * multi_steps(mi, low + 1) + (n - more) * multi_steps(mi, low));
                if ((i + 1 == columns.size() || columns[i + 1].group != c.group) && group_sweeps[c.group] > 0)
                    cost += group_sweeps[c.group] *
                            multi_cost(mi, m->general, cus, tiles, steps / tiles, group_cells[c.group], ragged,
                                       best_shape < 0 ? HUGE_VAL : best / group_sweeps[c.group]);
            }
            if (tiles > (double)cap) break;
            if (best_shape < 0 || cost < best) {
                best = cost;
                best_shape = s;
                best_zc = zc;
            }
        }
    }
    if (best_shape < 0) return;
    const MShapeInfo mi = mshape_info(best_shape);
    j3d_tune t1;
    if (one)
        t1 = *one;
    else
        default_tune(plan, cus, &t1);
    SingleCost single(t1);
    MShapeInfo mi2 = mi;
    mi2.t = kShortSweeps;
    double steps = 0, steps2 = 0;
    cells = 0;
    for (int32_t k = 0; k < count; ++k) {
        const ProbPlan &pp = prob(k);
        cut_axis((int32_t)pp.d.n[0], 64, mi.t, x_align(pp), &px);
        cut_axis((int32_t)pp.d.n[1], mi.rows, mi.t, 1, &py);
        cut_z(pp, m->general, mi.t, best_zc, [&](int64_t at, int64_t len, int64_t n) {
            for (int64_t i = 0; i < n; ++i) {
                const int32_t z0 = (int32_t)(at + i * len / n), nzv = (int32_t)(at + (i + 1) * len / n) - z0;
                const int below = mi.t - std::min(mi.t, z0 + 1);  // no ramp below the boundary plane
                steps += (double)(px.size() * py.size() * (multi_steps(mi, nzv) - below / 2 * 2));
                steps2 += (double)(px.size() * py.size() * multi_steps(mi2, nzv));
                for (const Piece &y : py)
                    for (const Piece &x : px) {
                        Tile t{};
                        t.block = pp.block_begin;
                        t.x0 = x.at;
                        t.nxv = x.len;
                        t.y0 = y.at;
                        t.nyv = y.len;
                        t.z0 = z0;
                        t.nzv = nzv;
                        m->tiles.push_back(t);
                    }
            }
        });
        m->prefix.push_back((int32_t)m->tiles.size());
        cells += (double)pp.d.n[0] * pp.d.n[1] * pp.d.n[2];
        for (int32_t b = pp.block_begin; b < pp.block_begin + pp.nblocks; ++b) single.add(plan.blocks[b]);
        // what problem k has more than the next one, in launches and in sweeps
        const int64_t more = k + 1 < count ? prob(k + 1).iters : 0;
        const int64_t launches = ceil_div(pp.iters, mi.t) - ceil_div(more, mi.t);
        const double tiles = (double)m->tiles.size();
        if (k + 1 == count || pp.iters > more) {
            m->launch_us = mi.t * multi_cost(mi, m->general, cus, tiles, steps / tiles, cells, ragged);
            // two stages hide less of a plane's latency: measured 3 to 25% above the fit
            m->short_us = 1.15 * mi2.t * multi_cost(mi2, m->general, cus, tiles, steps2 / tiles, cells, ragged);
            m->sweep_us = single.us(cus);
            m->all_us += (double)launches * m->launch_us;
            m->all_single_us += (double)(pp.iters - more) * m->sweep_us;
        }
    }
    tile_work(m->tiles, &m->work);
    m->shape = best_shape;
    m->t = mi.t;
}

j3d_status make_plan(int32_t count, const j3d_problem *probs, bool with_sr, Plan *plan)
{
    if (count < 1 || !probs) return set_error(J3D_EINVAL, "need at least one problem");
    plan->blocks.clear();
    plan->probs.assign(count, ProbPlan{});
    plan->with_sr = with_sr;
    plan->max_face = 0;
    plan->max_cells = 0;
    for (int32_t i = 0; i < count; ++i) {
        ProbPlan &pp = plan->probs[i];
        j3d_status st = resolve_decomp(&probs[i], &pp.d);
        if (st != J3D_OK) return st;
        pp.dense = dense_shape(pp.d);
        for (int f = 0; f < 6; ++f) pp.bc[f] = probs[i].bc[f];
        pp.s0 = stream_start(probs[i].seed, probs[i].pid);
        pp.block_begin = (int32_t)plan->blocks.size();
        const Decomp &d = pp.d;
        pp.nblocks = d.nb[0] * d.nb[1] * d.nb[2];
        if ((int64_t)plan->blocks.size() + pp.nblocks > (1 << 22))
            return set_error(J3D_EINVAL, "more than 2^22 blocks in total");
        auto index = [&](int32_t bx, int32_t by, int32_t bz) {
            return pp.block_begin + bx + d.nb[0] * (by + d.nb[1] * bz);
        };
        for (int32_t bz = 0; bz < d.nb[2]; ++bz)
            for (int32_t by = 0; by < d.nb[1]; ++by)
                for (int32_t bx = 0; bx < d.nb[0]; ++bx) {
                    BlockDesc B;
                    std::memset(&B, 0, sizeof B);
                    B.ext[0] = (int32_t)d.ext[0][bx];
                    B.ext[1] = (int32_t)d.ext[1][by];
                    B.ext[2] = (int32_t)d.ext[2][bz];
                    B.org[0] = (int32_t)d.org[0][bx];
                    B.org[1] = (int32_t)d.org[1][by];
                    B.org[2] = (int32_t)d.org[2][bz];
                    B.pitch = (int32_t)row_pitch(B.ext[0]);
                    B.prob = i;
                    B.nbr[0] = bx > 0 ? index(bx - 1, by, bz) : -1;
                    B.nbr[1] = bx + 1 < d.nb[0] ? index(bx + 1, by, bz) : -1;
                    B.nbr[2] = by > 0 ? index(bx, by - 1, bz) : -1;
                    B.nbr[3] = by + 1 < d.nb[1] ? index(bx, by + 1, bz) : -1;
                    B.nbr[4] = bz > 0 ? index(bx, by, bz - 1) : -1;
                    B.nbr[5] = bz + 1 < d.nb[2] ? index(bx, by, bz + 1) : -1;
                    const int64_t ex = B.ext[0], ey = B.ext[1], ez = B.ext[2];
                    B.face_total = 2 * (ey * ez + ex * ez + ex * ey);
                    const int64_t mf = std::max(ey * ez, std::max(ex * ez, ex * ey));
                    plan->max_face = (int32_t)std::max<int64_t>(plan->max_face, mf);
                    plan->max_cells = (int32_t)std::max<int64_t>(plan->max_cells, block_field_cells(ex, ey, ez));
                    plan->blocks.push_back(B);
                }
    }

    Bump bump;
    const uint64_t nb = plan->blocks.size();
    plan->off_blocks = bump.take(nb * sizeof(BlockDesc));
    plan->off_probs = bump.take((uint64_t)count * sizeof(ProbDesc));
    uint64_t cap = 0;
    for (int v = 0; v < variant_count(); ++v) cap = std::max(cap, count_tiles(*plan, v, kMinZchunk));
    plan->tiles_cap = cap;
    plan->off_tiles = bump.take(cap * sizeof(Tile));
    plan->mtiles_cap = multi_tiles_bound(*plan);
    plan->off_mtiles = bump.take(plan->mtiles_cap * sizeof(Tile));
    for (ProbPlan &pp : plan->probs)
        pp.maps_off = bump.take((uint64_t)(pp.d.n[0] + pp.d.n[1] + pp.d.n[2]) * 2 * sizeof(int32_t));
    plan->off_res = bump.take((uint64_t)(count + 1) * sizeof(uint64_t));
    plan->off_queue = bump.take(16 * sizeof(uint32_t));
    for (int q = 0; q < 2; ++q)
        for (ProbPlan &pp : plan->probs) {
            pp.f_off[q] = align_up(bump.off, 4096);
            uint64_t cells = 0;
            for (int32_t b = pp.block_begin; b < pp.block_begin + pp.nblocks; ++b) {
                BlockDesc &B = plan->blocks[b];
                const uint64_t c = (uint64_t)block_field_cells(B.ext[0], B.ext[1], B.ext[2]);
                B.off[q] = (int64_t)(bump.take(c * sizeof(double), 4096) / sizeof(double));
                cells += c;
            }
            pp.field_cells = cells;
        }
    for (int q = 0; q < 2; ++q)
        for (BlockDesc &B : plan->blocks)
            B.xoff[q] = (int64_t)(bump.take(2 * (uint64_t)B.ext[1] * B.ext[2] * sizeof(double)) /
                                  sizeof(double));
    if (with_sr)
        for (BlockDesc &B : plan->blocks)
            B.sr_off = (int64_t)(bump.take(2 * (uint64_t)B.face_total * sizeof(double)) / sizeof(double));
    link_halo_sources(plan->blocks.data(), plan->blocks.size());
    uint64_t bounce = 0;
    for (const ProbPlan &pp : plan->probs) {
        const int64_t n0 = pp.d.n[0], n1 = pp.d.n[1], n2 = pp.d.n[2];
        uint64_t need = (uint64_t)std::max(n0 * n1, std::max(n1 * n2, n0 * n2));
        need = std::max<uint64_t>(need, std::min<uint64_t>((uint64_t)(n0 * n1 * n2), 1ull << 22));
        bounce = std::max(bounce, need);
    }
    plan->bounce_doubles = bounce;
    plan->off_bounce = bump.take(bounce * sizeof(double), 4096);
    plan->total = align_up(bump.off, 4096);
    return J3D_OK;
}

void make_tiles(const Plan &plan, int32_t b0, int32_t b1, int variant, int zchunk,
                std::vector<Tile> *tiles, std::vector<int32_t> *block_first)
{
    const VariantInfo vi = variant_info(variant);
    const int zc = zchunk > 0 ? zchunk : max_ez(plan, 0, (int32_t)plan.blocks.size());
    if (block_first) block_first->clear();
    for (int32_t b = b0; b < b1; ++b) {
        const BlockDesc &B = plan.blocks[b];
        if (block_first) block_first->push_back((int32_t)tiles->size());
        int64_t ntx, nty;
        tiles_xy(vi, B.ext[0], B.ext[1], &ntx, &nty);
        const int ex = B.ext[0], ey = B.ext[1], ez = B.ext[2];
        const int ntz = (int)ceil_div(ez, zc);
        // z is cut into ntz near-equal pieces, so no tile is a thin remainder
        for (int tz = 0; tz < ntz; ++tz)
            for (int ty = 0; ty < (int)nty; ++ty)
                for (int tx = 0; tx < (int)ntx; ++tx) {
                    Tile t{};
                    t.block = b;
                    t.tx = tx;
                    t.ty = ty;
                    t.tz = tz;
                    if (vi.tile_x == 0) {  // flattened: x pieces on 16-column boundaries, y near-equal
                        const FlatShape f = flat_shape(ex, ey, vi.threads, vi.tile_y);
                        t.x0 = flat_x0(ex, f.tnx, tx);
                        t.nxv = flat_x0(ex, f.tnx, tx + 1) - t.x0;
                    } else {  // fixed: TX-wide columns, y near-equal
                        t.x0 = tx * vi.tile_x;
                        t.nxv = std::min(vi.tile_x, ex - t.x0);
                    }
                    t.y0 = (int32_t)((int64_t)ty * ey / nty);
                    t.nyv = (int32_t)((int64_t)(ty + 1) * ey / nty) - t.y0;
                    t.z0 = (int32_t)((int64_t)tz * ez / ntz);
                    t.nzv = (int32_t)((int64_t)(tz + 1) * ez / ntz) - t.z0;
                    tiles->push_back(t);
                }
    }
    if (block_first) block_first->push_back((int32_t)tiles->size());
}

void tile_work(const std::vector<Tile> &tiles, std::vector<uint64_t> *prefix)
{
    // A tile's time is set by the planes it streams, whatever share of its
    // lanes hold a cell (measured: weighting by cells balanced the batched
    // workload worse than equal counts), plus a fixed cost of about one plane
    // for its first memory latency.
    constexpr uint64_t kTileFixed = 1;  // planes
    prefix->assign(tiles.size() + 1, 0);
    uint64_t acc = 0;
    for (size_t i = 0; i < tiles.size(); ++i) {
        acc += (uint64_t)(tiles[i].nzv + 2) + kTileFixed;
        (*prefix)[i + 1] = acc;
    }
}

void default_tune(const Plan &plan, int cus, j3d_tune *t)
{
    // Shapes measured fastest on MI355X (one workgroup per tile; the
    // persistent schedule never won for a single problem):
    //   <= 64 wide:         flattened tiles of 512 threads, 2 cells each (64 x 16
    //                       on 64-wide blocks), through 64 planes;
    //   widths not a multiple of 16 (rows ending inside a cache line), or
    //   129..192 wide:      flattened tiles of 512 threads, 4 cells each, which
    //                       write whole lines at row ends, z-chunks of 32;
    //   <= 128:             128 x 16 tiles of 512 threads, z-chunks of 32;
    //   wider:              128 x 32 tiles of 1024 threads, z-chunks of 64.
    int exm = 1;
    bool ragged = false;
    for (const BlockDesc &B : plan.blocks) {
        exm = std::max(exm, B.ext[0]);
        ragged = ragged || B.ext[0] % 16 != 0;
    }
    int v, zc;
    if (exm <= 64) {
        v = find_flat_variant(512, 1024, 3);
        zc = 64;
    } else if (ragged || (exm > 128 && exm <= 192)) {
        v = find_flat_variant(512, 2048, 1);
        zc = 32;
    } else if (exm <= 128) {
        v = find_variant(128, 16, 512);
        zc = 32;
    } else {
        v = find_variant(128, 32, 1024);
        zc = 64;
    }
    if (v < 0) v = 0;  // a shape missing from the table: any variant is correct, only slower
    t->variant = v;
    t->blocks_per_cu = 0;
    // a shallower chunk if the launch would otherwise have too few workgroups
    // to fill the chip
    const int ezm = max_ez(plan, 0, (int32_t)plan.blocks.size());
    while (zc > 16 && count_tiles(plan, v, zc) < (uint64_t)(2 * (cus > 0 ? cus : 256))) zc = (zc + 1) / 2;
    t->zchunk = zc >= ezm ? 0 : zc;
}

j3d_status check_tune(const Plan &plan, const j3d_tune *t, int *zchunk_eff)
{
    if (t->variant < 0 || t->variant >= variant_count())
        return set_error(J3D_EINVAL, "tune variant %d out of range [0, %d)", t->variant, variant_count());
    if (t->zchunk < 0) return set_error(J3D_EINVAL, "tune zchunk %d < 0", t->zchunk);
    if (t->blocks_per_cu < 0 || t->blocks_per_cu > 32)
        return set_error(J3D_EINVAL, "tune blocks_per_cu %d out of range [0, 32]", t->blocks_per_cu);
    const uint64_t n = count_tiles(plan, t->variant, t->zchunk);
    if (n > plan.tiles_cap || n > INT32_MAX)
        return set_error(J3D_EINVAL, "tune gives %llu tiles, more than the table holds (%llu)",
                         (unsigned long long)n, (unsigned long long)plan.tiles_cap);
    *zchunk_eff = t->zchunk > 0 ? t->zchunk : max_ez(plan, 0, (int32_t)plan.blocks.size());
    return J3D_OK;
}

}  // namespace j3d

using namespace j3d;

extern "C" {

const char *j3d_last_error(void) { return last_error_text(); }

const char *j3d_version(void) { return "j3d 0.1 (gfx950)"; }

j3d_status j3d_auto_split(const int64_t n[3], int32_t parts, int32_t nblk_out[3])
{
    if (!n || !nblk_out) return set_error(J3D_EINVAL, "NULL argument");
    for (int a = 0; a < 3; ++a)
        if (n[a] < 1) return set_error(J3D_EINVAL, "n[%d] < 1", a);
    int32_t nb[3];
    j3d_status st = auto_split(n, parts, nb);
    if (st != J3D_OK) return st;
    for (int a = 0; a < 3; ++a) nblk_out[a] = nb[a];
    return J3D_OK;
}

j3d_status j3d_block_extents(const j3d_problem *p, int32_t nblk_out[3], int64_t *extents_out,
                             int64_t cap)
{
    if (!nblk_out) return set_error(J3D_EINVAL, "nblk_out is NULL");
    Decomp d;
    j3d_status st = resolve_decomp(p, &d);
    if (st != J3D_OK) return st;
    const int64_t need = (int64_t)d.nb[0] + d.nb[1] + d.nb[2];
    if (extents_out && cap < need)
        return set_error(J3D_EINVAL, "extents_out holds %lld values, %lld needed", (long long)cap,
                         (long long)need);
    for (int a = 0; a < 3; ++a) nblk_out[a] = d.nb[a];
    if (extents_out) {
        int64_t k = 0;
        for (int a = 0; a < 3; ++a)
            for (int64_t e : d.ext[a]) extents_out[k++] = e;
    }
    return J3D_OK;
}

j3d_status j3d_arena_bytes(const j3d_problem *p, uint64_t *bytes)
{
    if (!bytes) return set_error(J3D_EINVAL, "bytes is NULL");
    Plan plan;
    j3d_status st = make_plan(1, p, true, &plan);
    if (st != J3D_OK) return st;
    *bytes = plan.total;
    return J3D_OK;
}

j3d_status j3d_field_bytes(const j3d_problem *p, uint64_t *bytes)
{
    if (!bytes) return set_error(J3D_EINVAL, "bytes is NULL");
    Plan plan;
    j3d_status st = make_plan(1, p, true, &plan);
    if (st != J3D_OK) return st;
    uint64_t b = 0;
    for (const BlockDesc &B : plan.blocks)
        b += 2 * sizeof(double) *
             ((uint64_t)block_field_cells(B.ext[0], B.ext[1], B.ext[2]) + 2ull * B.ext[1] * B.ext[2]);
    *bytes = b;
    return J3D_OK;
}

j3d_status j3d_variant_info(int32_t variant, int32_t *tile_x, int32_t *tile_y, int32_t *threads)
{
    if (variant < 0 || variant >= variant_count())
        return set_error(J3D_EINVAL, "variant %d out of range [0, %d)", variant, variant_count());
    const VariantInfo vi = variant_info(variant);
    if (tile_x) *tile_x = vi.tile_x;
    if (tile_y) *tile_y = vi.tile_y;
    if (threads) *threads = vi.threads;
    return J3D_OK;
}

j3d_status j3d_batch_arena_bytes(int32_t count, const j3d_problem *probs, uint64_t *bytes)
{
    if (!bytes) return set_error(J3D_EINVAL, "bytes is NULL");
    Plan plan;
    j3d_status st = make_plan(count, probs, true, &plan);
    if (st != J3D_OK) return st;
    *bytes = plan.total;
    return J3D_OK;
}

}  // extern "C"

// j3d_multisweep.hip -- several Jacobi sweeps per launch (temporal blocking),
// on undivided and on decomposed grids, alone or many problems at once.
//
// One sweep per launch reads and writes 16 bytes per cell update and is bound
// by HBM (512^3: 386 us a sweep).  Here a workgroup owns an x-y tile of the
// *grid* (whatever blocks it lies in), marches along z and carries T sweeps at
// once: stage s computes plane k-1-s of iterate t+s+1 while plane k of iterate
// t arrives, so T sweeps cost one read and one write of the grid.  Tiles
// overlap by T cells on each side and recompute that ring.
//
//   - Lanes run along x (a wave is 64 columns of the tile), a thread holds RY
//     rows, NW waves are stacked along y.  Per stage a thread keeps planes q-1
//     and q of its cells in registers; x neighbours come from the neighbouring
//     lanes (DPP moves), y neighbours from its own registers and, at the
//     strip's two ends, from the neighbouring waves through LDS; the plane
//     above arrives from the stage before.  So the LDS carries 2 rows in RY
//     instead of every cell, and one barrier per plane serves all T stages.
//   - What bounds it: vector issue and memory, overlapping in part.  Seven FP64
//     operations and four DPP moves per update and lane, times the ring's share
//     of lanes (64 x 64 lanes hold 56 x 56 cells at T = 4), are 168 k vector
//     instructions per SIMD for 4 sweeps of 512^3: 0.34 ms at the 2.0 ns that an
//     FP64 or DPP instruction was measured to take.  The launch moves 2.42 GB,
//     0.39 ms at the streaming copy's 6.15 TB/s, and takes 0.54 ms.
//   - Measured and rejected: the x neighbours through the LDS crossbar
//     (ds_bpermute for one side: 16.2 against 14.2 ms per 100 sweeps of 512^3,
//     for both 21), two more planes of prefetch (the same), non-temporal
//     loads (10% slower: the ring cells of a tile are its neighbours' cells
//     and are found in L2).
//
// 512^3 as 8^3 blocks of 64^3: 134 us a sweep (1000 GLUP/s) against 384 us one
// sweep per launch; 64^3: 3.6 against 11.4 us; 33x35x31: 3.3 against 11.4 us
// (a sweep's share of 50, with the call).
//
// Each value is the 7-term sum of the same operands in the same order as in a
// single sweep (centre, x-, x+, y-, y+, z-, z+, each addition rounded, then
// one multiplication by fl(1/7); built with -ffp-contract=off), so the result
// has the bits of separate sweeps.  Cells of the Dirichlet layer keep their
// value through the stages; what lies beyond it is never an operand of a
// stored cell.  A launch of fewer sweeps than it has stages lets the first ones
// pass their input on; one or two sweeps run in a form of two stages.  Halos
// between blocks are read as the neighbours' interior cells, so nothing is
// packed, exchanged or handed over.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "j3d_internal.hpp"

namespace j3d {
namespace {

constexpr double kW = 1.0 / 7.0;  // fl(1/7)
constexpr uint32_t kOut = 0xFFFFFF00u;       // a lane offset outside every resource
constexpr uint32_t kMaxSpan = 0xFFFFF000u;   // largest resource

typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(4))) BlockDesc KBlock;
typedef const __attribute__((address_space(4))) ProbDesc KProb;
typedef const __attribute__((address_space(4))) int32_t kint32;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void *p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}

__device__ __forceinline__ double bload(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}

template <int AUX>
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, uint32_t off, double v)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, v), r, (int)off, 0, AUX);
}

// The value of the lane below (x-) / above (x+); 0 past the wave's ends.
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v)
{
    const i32x2 i = __builtin_bit_cast(i32x2, v);
    i32x2 o;
    o.x = __builtin_amdgcn_mov_dpp(i.x, CTRL, 0xf, 0xf, true);
    o.y = __builtin_amdgcn_mov_dpp(i.y, CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, o);
}
__device__ __forceinline__ double from_below(double v) { return lane_shift<0x138>(v); }  // wave_shr:1
__device__ __forceinline__ double from_above(double v) { return lane_shift<0x130>(v); }  // wave_shl:1

// Holds a value's computation where it stands: the compiler otherwise sinks
// the middle rows' sums past the step's rare branches and keeps their DPP
// operands instead (64 x 64 tiles: 310 registers instead of 230).
__device__ __forceinline__ void keep_here(double &v) { asm volatile("" : "+v"(v)); }

// v[r] = b[r] in the lanes of m[r]: one move under the execution mask instead of
// two selects.  Every lane of a wave is active here, so the mask goes back to
// all ones.  Also keeps the values' computation in its place (see the step).
template <int N>
__device__ __forceinline__ void keep_lanes(double *v, const double *b, const uint64_t *m)
{
    if constexpr (N >= 4) {
        asm volatile("s_mov_b64 exec, %8\n\tv_mov_b64_e32 %0, %4\n\ts_mov_b64 exec, %9\n\tv_mov_b64_e32 %1, %5\n\t"
                     "s_mov_b64 exec, %10\n\tv_mov_b64_e32 %2, %6\n\ts_mov_b64 exec, %11\n\tv_mov_b64_e32 %3, %7\n\t"
                     "s_mov_b64 exec, -1"
                     : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3])
                     : "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "s"(m[0]), "s"(m[1]), "s"(m[2]), "s"(m[3]));
        keep_lanes<N - 4>(v + 4, b + 4, m + 4);
    } else if constexpr (N >= 2) {
        asm volatile("s_mov_b64 exec, %4\n\tv_mov_b64_e32 %0, %2\n\ts_mov_b64 exec, %5\n\tv_mov_b64_e32 %1, %3\n\t"
                     "s_mov_b64 exec, -1"
                     : "+v"(v[0]), "+v"(v[1])
                     : "v"(b[0]), "v"(b[1]), "s"(m[0]), "s"(m[1]));
        keep_lanes<N - 2>(v + 2, b + 2, m + 2);
    } else if constexpr (N == 1) {
        asm volatile("s_mov_b64 exec, %2\n\tv_mov_b64_e32 %0, %1\n\ts_mov_b64 exec, -1"
                     : "+v"(v[0])
                     : "v"(b[0]), "s"(m[0]));
    }
}

__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int NW_, int RY_, int T_>
struct MShape {
    static constexpr int NW = NW_, RY = RY_, T = T_, NT = NW * 64;
    // Shared memory of a workgroup, in elements: edge rows (both halves of the
    // double buffer), x boundary values, the residual's wave maxima; and for
    // blocks of unequal extents the lane offsets and x sources per block row.
    static constexpr int kEdge = 2 * T * NW * 128, kX = NW * 64, kRed = NW;
    static constexpr int kTab = kMultiSegs * NT * RY, kXTab = kMultiSegs * NT;
    static constexpr int lds(bool general)
    {
        return (kEdge + kX + kRed) * 8 + (general ? kTab * 4 + kXTab * 8 : 0);
    }
};

// One tile's place in its problem, uniform over the workgroup.
struct MGeo {
    double *base;
    const char *end;     // end of the arena
    KBlock *blocks;      // the problem's first block
    kint32 *mx, *my, *mz;
    int nx, ny, nz, nb0, nb1, nb2;
    int x0, y0, z0, nxv, nyv, nzv;
    int hl, ht;          // halo columns / rows below the tile held by the workgroup
    int p, ns;
    bool res;
};

// Streams one tile.  GEN: blocks of unequal extents (plane strides differ from
// lane to lane).  EDGE: some column or row of the tile's lanes lies on the
// boundary layer; XE: a column does, so its values come from the x-halo
// arrays.  Returns the last sweep's largest change where it is asked for.
template <class S, bool GEN, bool EDGE, bool XE>
__device__ __forceinline__ double multi_tile(const MGeo &g, double *E, double *LX, uint32_t *tab, int64_t *xtab)
{
    constexpr int NW = S::NW, RY = S::RY, T = S::T;
    // Equal blocks: stores stream (non-temporal).  Unequal ones: tiles end inside
    // cache lines, which L2 joins with the neighbour tile's half (640^3 uneven:
    // 22.5 against 22.9 ms per 50 sweeps at T = 4, 17.2 against 17.8 at T = 5).
    constexpr int kStore = GEN ? 0 : 2;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool multi = g.nb0 * g.nb1 * g.nb2 > 1;

    const int gx = g.x0 - g.hl + lane;
    const int row0 = g.y0 - g.ht + w * RY;  // this wave's first row
    const bool inx = gx >= 0 && gx < g.nx;
    const bool isx = gx == -1 || gx == g.nx;  // a column of the x boundary layer

    // lowest block of the tile's extended rectangle: the offsets' origin
    int bxa = 0, bya = 0;
    int bx = 0, lx = gx;
    if (multi) {
        bxa = g.mx[2 * max(g.x0 - g.hl, 0)];
        bya = g.my[2 * max(g.y0 - g.ht, 0)];
        const int c = min(max(gx, 0), g.nx - 1);
        bx = ((const int32_t *)g.mx)[2 * c];
        lx = ((const int32_t *)g.mx)[2 * c + 1];
    }
    const int p = g.p;
    auto blk = [&](int bz) __attribute__((always_inline)) -> KBlock * {
        return g.blocks + bxa + g.nb0 * (bya + g.nb1 * bz);
    };
    const int pitchA = blk(0)->pitch, eyA = blk(0)->ext[1];
    const int64_t psA = plane_stride(pitchA, eyA);
    const int64_t delta = blk(0)->off[p ^ 1] - blk(0)->off[p];
    // Bytes a plane's resource spans: the plane itself, or with several blocks
    // what is left of the arena (behind the last plane of the block row, for
    // equal blocks: the same for all its planes), as far as 32-bit offsets go.
    auto reach = [&](const char *at) __attribute__((always_inline)) -> uint32_t {
        const uint64_t left = (uint64_t)(g.end - at);
        return left < kMaxSpan ? (uint32_t)left : kMaxSpan;
    };
    auto row_span = [&](const char *field, int ez) __attribute__((always_inline)) -> uint32_t {
        return multi ? reach(field + (ez + 1) * psA * 8) : (uint32_t)(psA * 8);
    };

    // per-lane byte offsets of this wave's rows from plane lz of block (bxa, bya, bz)
    uint32_t vin[RY], vout[GEN ? RY : 1], dst[GEN ? RY : 1] = {};
    auto offsets = [&](int bz, uint32_t *v) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            const int gy = row0 + r;
            const bool ok = inx && gy >= -1 && gy <= g.ny;
            uint32_t o;
            if (!multi) {
                o = (uint32_t)(gy + 1) * (uint32_t)pitchA * 8u + (uint32_t)gx * 8u;
            } else {
                const int cy = min(max(gy, 0), g.ny - 1);
                const int by = g.my[2 * cy];
                int ly = g.my[2 * cy + 1];
                ly += gy < 0 ? -1 : (gy >= g.ny ? 1 : 0);
                const int i = bx + g.nb0 * (by + g.nb1 * bz);
                const BlockDesc *B = (const BlockDesc *)g.blocks + i;
                const int64_t ps = plane_stride(B->pitch, B->ext[1]);
                int64_t d = B->off[p] - blk(bz)->off[p] + (int64_t)(ly + 1) * B->pitch + lx;
                if (GEN) {
                    d += ps - psA;
                    dst[r] = ok ? (uint32_t)((ps - psA) * 8) : 0u;
                }
                o = (uint32_t)(d * 8);
            }
            v[r] = ok ? o : kOut;
        }
    };
    // a lane (row) outside the tile's cells stores nothing: kOut or-ed into its offset
    const uint32_t vlane = lane >= g.hl && lane < g.hl + g.nxv ? 0u : kOut;
    auto srow = [&](int r) __attribute__((always_inline)) -> uint32_t {
        const int cy = w * RY + r - g.ht;
        return cy >= 0 && cy < g.nyv ? 0u : kOut;
    };
    // lanes whose cell keeps its value: boundary layer and beyond
    const uint64_t fx = EDGE ? __builtin_amdgcn_ballot_w64(!inx) : 0ull;
    auto fixrow = [&](int r) __attribute__((always_inline)) -> uint64_t {
        return row0 + r < 0 || row0 + r >= g.ny ? ~0ull : fx;
    };

    const int k0 = max(g.z0 - T, -1), k1 = g.z0 + g.nzv - 1 + T;
    const int zlast = min(k1, g.nz);  // last plane read
    // input cursor: plane zl is plane lzl of block row bzl
    int zl = k0, bzl = 0, lzl = k0, ezl = g.nz;
    if (multi) {
        const int c = max(k0, 0);
        bzl = g.mz[2 * c];
        lzl = k0 < 0 ? -1 : g.mz[2 * c + 1];
        ezl = blk(bzl)->ext[2];
    }
    const char *lp = (const char *)(g.base + blk(bzl)->off[p]);
    uint32_t span_in = row_span(lp, ezl);
    lp += (int64_t)(lzl + 1) * psA * 8;
    int bzo = 0, lzo = g.z0, ezo = g.nz;
    if (multi) {
        bzo = g.mz[2 * g.z0];
        lzo = g.mz[2 * g.z0 + 1];
        ezo = blk(bzo)->ext[2];
    }
    char *op = (char *)(g.base + blk(bzo)->off[p] + delta);
    uint32_t span_out = row_span(op, ezo);
    op += (int64_t)(lzo + 1) * psA * 8;
    if (!GEN) {
        offsets(bzl, vin);
    } else {
        // offsets of the block rows this tile reads (at most kMultiSegs), kept in LDS:
        // vector loads inside the plane loop would shorten every wait for a plane
        uint32_t v[RY];
        const int last = multi ? g.mz[2 * min(k1, g.nz - 1)] : 0;
        for (int b = bzl; b <= last; ++b) {
            offsets(b, v);
#pragma unroll
            for (int r = 0; r < RY; ++r) tab[((b - bzl) * RY + r) * S::NT + threadIdx.x] = v[r];
        }
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            vin[r] = tab[r * S::NT + threadIdx.x];
            vin[r] += dst[r] * (uint32_t)lzl;  // dst is 0 in lanes outside
            const uint32_t o = tab[((bzo - bzl) * RY + r) * S::NT + threadIdx.x];
            vout[r] = (vlane | srow(r)) ? kOut : o + dst[r] * (uint32_t)lzo;
        }
    }
    const int bz0 = bzl;

    // x boundary values: lane i < RY loads row i's x- value, lane 32 + i its x+
    // value (other lanes read a valid cell), handed to the rows through LDS
    const double *xb = g.base + blk(0)->off[p];
    uint32_t xey = 0;
    auto xsource = [&](int bz) __attribute__((always_inline)) {
        const int gy = row0 + (lane & 31), side = lane >> 5;
        if ((lane & 31) >= RY || gy < 0 || gy >= g.ny || (side ? g.x0 + g.nxv < g.nx : g.x0 > 0)) return;
        int i = 0, ly = gy;
        if (multi) {
            const int by = ((const int32_t *)g.my)[2 * gy];
            ly = ((const int32_t *)g.my)[2 * gy + 1];
            i = (side ? g.nb0 - 1 : 0) + g.nb0 * (by + g.nb1 * bz);
        }
        const BlockDesc *B = (const BlockDesc *)g.blocks + i;
        xb = g.base + B->xoff[p] + (side ? (int64_t)B->ext[1] * B->ext[2] : 0) + ly;
        xey = (uint32_t)B->ext[1];
    };
    if (XE) {
        if (GEN) {
            const int last = multi ? g.mz[2 * min(k1, g.nz - 1)] : 0;
            for (int b = last; b >= bzl; --b) {
                xsource(b);
                xtab[(b - bzl) * S::NT + threadIdx.x] = xb - g.base;
            }
        } else {
            xsource(bzl);
        }
    }
    const uint64_t xm = __builtin_amdgcn_ballot_w64(isx);

    double St[T][2][RY];       // stage s: planes q-1 and q of iterate t+s, alternating
    double L[2][RY], X[2] = {};  // planes on their way in, and their x boundary values
#pragma unroll
    for (int r = 0; r < RY; ++r)
#pragma unroll
        for (int s = 0; s < T; ++s) St[s][0][r] = St[s][1][r] = 0.0;

    auto load = [&](double (&d)[RY], double &x) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rz = plane_rsrc(lp, zl <= zlast ? (GEN && multi ? reach(lp) : span_in) : 0u);
#pragma unroll
        for (int r = 0; r < RY; ++r) d[r] = bload(rz, vin[r]);
        if (XE) x = xb[(uint64_t)xey * (uint32_t)min(max(lzl, 0), ezl - 1)];
    };
    auto advance_in = [&]() __attribute__((always_inline)) {
        ++zl;
        ++lzl;
        lp += psA * 8;
        if (GEN) {
#pragma unroll
            for (int r = 0; r < RY; ++r) vin[r] += dst[r];
        }
        if (lzl == ezl && zl <= zlast && zl < g.nz) {
            ++bzl;
            lzl = 0;
            ezl = blk(bzl)->ext[2];
            lp = (const char *)(g.base + blk(bzl)->off[p]);
            span_in = row_span(lp, ezl);
            lp += psA * 8;
            if (GEN) {
#pragma unroll
                for (int r = 0; r < RY; ++r) vin[r] = tab[((bzl - bz0) * RY + r) * S::NT + threadIdx.x];
            }
            if (XE) {
                if (GEN)
                    xb = g.base + xtab[(bzl - bz0) * S::NT + threadIdx.x];
                else  // equal blocks: every lane's array moves by the same distance
                    xb += blk(bzl)->xoff[p] - blk(bzl - 1)->xoff[p];
            }
        }
    };
    // The stores of the two steps before the first, dropped: the waits for a
    // plane then count the same memory operations on the way into the loops as
    // inside them, and never wait for a younger plane.
    auto no_stores = [&]() __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t none = plane_rsrc(op, 0u);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            bstore<kStore>(none, kOut, 0.0);
            asm volatile("" ::: "memory");  // or equal stores are merged
        }
    };
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        load(L[i], X[i]);
        advance_in();
        no_stores();
    }

    double rmax = 0.0;
    uint32_t zbits = 0;  // bit 31-s: plane k-1-s lies on a z face
    // stages of a shorter launch that pass their input on, from bit 31 down
    const uint32_t idle = (uint32_t)(0xffffffff00000000ull >> (T - g.ns));
    uint64_t xms[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) xms[r] = xm;
    auto step = [&](auto zm, const int k, const int j) __attribute__((always_inline)) {
        constexpr bool ZM = decltype(zm)::value;  // some stage may be on a z face (or idle)
        double *Ew = E + j * (T * NW * 128);
        const double *Er = E + (j ^ 1) * (T * NW * 128);
        double up[T], dn[T];
        auto read_edges = [&](int s) __attribute__((always_inline)) {
            up[s] = Er[(s * NW + max(w - 1, 0)) * 128 + 64 + lane];
            dn[s] = Er[(s * NW + min(w + 1, NW - 1)) * 128 + lane];
        };
        read_edges(0);
        if (T > 1) read_edges(1);
        auto edges = [&](int s, double first, double last) __attribute__((always_inline)) {
            Ew[(s * NW + w) * 128 + lane] = first;
            Ew[(s * NW + w) * 128 + 64 + lane] = last;
        };
        auto part = [&](int s, int r) __attribute__((always_inline)) {
            const double(&B)[RY] = St[s][j ^ 1];
            double t = B[r];
            t += from_below(B[r]);
            t += from_above(B[r]);
            t += r > 0 ? B[r > 0 ? r - 1 : 0] : up[s];
            t += r < RY - 1 ? B[r < RY - 1 ? r + 1 : r] : dn[s];
            t += St[s][j][r];
            return t;
        };
        if (ZM) zbits = zbits >> 1 | ((uint32_t)((k - 1) | (g.nz - k)) & 0x80000000u);
        const uint32_t still = (uint32_t)__builtin_amdgcn_readfirstlane((int)(zbits | idle));
        double pa[RY], W[RY];
#pragma unroll
        for (int r = 0; r < RY; ++r) pa[r] = part(0, r);
#pragma unroll
        for (int s = 0; s < T; ++s) {
            double pn[RY], v[RY];
            if (s + 2 < T) read_edges(s + 2);
            if (s + 1 < T) {
#pragma unroll
                for (int r = 0; r < RY; ++r) pn[r] = part(s + 1, r);
            }
            if (s == 0) {
                if (XE) {
                    double xv[RY];
                    LX[w * 64 + lane] = X[j];
#pragma unroll
                    for (int r = 0; r < RY; ++r) xv[r] = LX[w * 64 + (gx < 0 ? 0 : 32) + r];
                    keep_lanes<RY>(L[j], xv, xms);
                }
#pragma unroll
                for (int r = 0; r < RY; ++r) St[0][j][r] = L[j][r];
                edges(0, L[j][0], L[j][RY - 1]);
            }
            const int q = k - 1 - s;  // the plane this stage computes
#pragma unroll
            for (int r = 0; r < RY; ++r) v[r] = (pa[r] + St[s][j][r]) * kW;
            if (EDGE || ZM) {
                const uint64_t zf = ZM && (still << s & 0x80000000u) ? ~0ull : 0ull;
                uint64_t m[RY];
#pragma unroll
                for (int r = 0; r < RY; ++r) m[r] = zf | (EDGE ? fixrow(r) : 0ull);
                keep_lanes<RY>(v, St[s][j ^ 1], m);
            } else {
#pragma unroll
                for (int r = 0; r < RY; ++r) keep_here(v[r]);
            }
            if (s == T - 1 && g.res && q >= g.z0 && q < g.z0 + g.nzv) {
#pragma unroll
                for (int r = 0; r < RY; ++r) {
                    const double d = (vlane | srow(r)) == 0u ? fabs(v[r] - St[s][j ^ 1][r]) : 0.0;
                    rmax = d > rmax ? d : rmax;
                }
            }
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                if (s < T - 1)
                    St[s < T - 1 ? s + 1 : s][j][r] = v[r];
                else
                    W[r] = v[r];
                pa[r] = pn[r];
            }
            if (s == 0) load(L[j], X[j]);
            if (s < T - 1) edges(s + 1, v[0], v[RY - 1]);
        }
        advance_in();
        const int q = k - T;
        const bool st = q >= g.z0 && q < g.z0 + g.nzv;
        const __amdgpu_buffer_rsrc_t ro = plane_rsrc(op, st ? (GEN && multi ? reach(op) : span_out) : 0u);
#pragma unroll
        for (int r = 0; r < RY; ++r) bstore<kStore>(ro, GEN ? vout[GEN ? r : 0] : vin[r] | vlane | srow(r), W[r]);
        if (st) {
            ++lzo;
            op += psA * 8;
            if (GEN) {
#pragma unroll
                for (int r = 0; r < RY; ++r) vout[GEN ? r : 0] += vout[GEN ? r : 0] != kOut ? dst[GEN ? r : 0] : 0u;
            }
            if (!GEN && lzo == ezo && q + 1 < g.nz) {  // GEN: a tile's cells lie in one block row
                ++bzo;
                lzo = 0;
                ezo = blk(bzo)->ext[2];
                op = (char *)(g.base + blk(bzo)->off[p] + delta);
                span_out = row_span(op, ezo);
                op += psA * 8;
            }
        }
        lds_barrier();
    };

    // Two steps a round: the planes' registers alternate.  The arriving plane is
    // moved into place (2% more instructions) so that two steps suffice: with
    // its registers rotating as well a round was four, and fetching that code
    // cost a small launch up to 9 us (157x211x183: 1370 against 1311 us for 30
    // launches; 64^3: 467 against 415 us for 25; 512^3: 15.1 against 14.5 ms).
    int k = k0;
    auto round = [&](auto zm) __attribute__((always_inline)) {
        step(zm, k, 0);
        step(zm, k + 1, 1);
        k += 2;
    };
    if (!EDGE && g.ns == T) {
        while (k < T && k <= k1) round(std::true_type{});
        const int kf = min(k1, g.nz - 1);
        while (k <= kf) round(std::false_type{});
        zbits = 0;  // the planes computed so far lie inside
    }
    while (k <= k1) round(std::true_type{});
    return rmax;
}

template <class S, bool GEN>
__global__ __launch_bounds__(S::NT)  void multisweep_kernel(MultiArgs a)
{
    constexpr int NW = S::NW, T = S::T;
    __shared__ double E[S::kEdge];
    __shared__ double LX[S::kX];
    __shared__ double red[S::kRed];
    __shared__ uint32_t tab[GEN ? S::kTab : 1];
    __shared__ int64_t xtab[GEN ? S::kXTab : 1];
    const int xcd = blockIdx.x % kXcdCount, jj = blockIdx.x / kXcdCount;
    typedef const __attribute__((address_space(4))) char kchar;
    const kint32 *xc = (const kint32 *)((kchar *)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(MultiArgs, xcut));
    const int t = xc[xcd] + jj;
    if (t >= xc[xcd + 1]) return;
    typedef const __attribute__((address_space(4))) Tile KTile;
    KTile *tl = (KTile *)(a.tiles + a.tile_begin + t);
    const int first = tl->block;
    KProb *P = (KProb *)(a.probs + ((KBlock *)(a.blocks + first))->prob);
    MGeo g;
    if (a.flags & MS_MULTI) {
        const int64_t done = a.step * T;
        if (done >= P->limit) return;
        g.p = (int)((P->base + a.step) & 1);
        g.ns = (int)(P->limit - done < T ? P->limit - done : T);
        g.res = (P->flags & PF_RES_LAST) && done + g.ns == P->limit;
    } else {
        g.p = a.parity;
        g.ns = a.nsweeps;
        g.res = (a.flags & MS_RES) != 0;
    }
    g.base = a.base;
    g.end = a.end;
    g.blocks = (KBlock *)(a.blocks + first);
    g.nx = P->n[0];
    g.ny = P->n[1];
    g.nz = P->n[2];
    g.nb0 = P->nb[0];
    g.nb1 = P->nb[1];
    g.nb2 = P->nb[2];
    g.mx = (kint32 *)(a.maps + P->maps_off);
    g.my = g.mx + 2 * g.nx;
    g.mz = g.my + 2 * g.ny;
    g.x0 = tl->x0;
    g.y0 = tl->y0;
    g.z0 = tl->z0;
    g.nxv = tl->nxv;
    g.nyv = tl->nyv;
    g.nzv = tl->nzv;
    g.hl = min(T, g.x0 + 1);
    g.ht = min(T, g.y0 + 1);
    double rmax = 0.0;
    // every stage computes cells strictly inside the grid along x and y
    const bool xe = g.x0 < T || g.x0 + g.nxv + T > g.nx, ye = g.y0 < T || g.y0 + g.nyv + T > g.ny;
    if (xe)
        rmax = multi_tile<S, GEN, true, true>(g, E, LX, tab, xtab);
    else if (ye)
        rmax = multi_tile<S, GEN, true, false>(g, E, LX, tab, xtab);
    else
        rmax = multi_tile<S, GEN, false, false>(g, E, LX, tab, xtab);
    if (g.res) {
        double m = rmax;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double q = __shfl_xor(m, o);
            m = q > m ? q : m;
        }
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
        __syncthreads();
        if (threadIdx.x == 0) {
            double v = 0.0;
            for (int i = 0; i < NW; ++i) v = red[i] > v ? red[i] : v;
            __hip_atomic_fetch_max(a.res + P->res_slot, (unsigned long long)__double_as_longlong(v),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Shapes: waves, rows per thread, sweeps, workgroups that fit a compute unit
// with equal and with unequal blocks (by registers, and by the 160 KB of LDS:
// the general kernels' tables leave room for one).  The planner
// picks by estimated time (multi_cost); each is the fastest somewhere:
// 64 x 64 lanes and T = 4 on large equal blocks, 64 x 48 and T = 5 where
// memory is slow (ragged widths), fewer rows where the grid is too small to
// give every compute unit a tile, T = 3 where the ring of small problems eats
// the gain of a fourth sweep (a batch of 32..256-wide grids).
#define J3D_MSHAPES(M) \
    M(8, 8, 4, 1, 1)   \
    M(8, 6, 4, 1, 1)   \
    M(8, 6, 5, 1, 1)   \
    M(8, 4, 4, 1, 1)   \
    M(8, 4, 3, 2, 1)   \
    M(8, 3, 4, 2, 1)   \
    M(8, 2, 4, 2, 1)

// A launch of one or two sweeps runs the same tiles by the two-stage form of
// its shape: fewer stages and a ramp of two planes instead of T.
struct MEntry {
    MShapeInfo info;
    void (*fn[2])(MultiArgs);   // T sweeps: equal, unequal blocks
    void (*fn2[2])(MultiArgs);  // up to two
};
#define M(NW, RY, T, PC, PG)                                                                                        \
    {{NW * RY, T, NW * 64, {PC, PG}, {MShape<NW, RY, T>::lds(false), MShape<NW, RY, T>::lds(true)}},               \
     {multisweep_kernel<MShape<NW, RY, T>, false>, multisweep_kernel<MShape<NW, RY, T>, true>},                    \
     {multisweep_kernel<MShape<NW, RY, 2>, false>, multisweep_kernel<MShape<NW, RY, 2>, true>}},
const MEntry kM[] = {J3D_MSHAPES(M)};
#undef M
}  // namespace

int mshape_count() { return (int)(sizeof kM / sizeof kM[0]); }
MShapeInfo mshape_info(int i) { return kM[i].info; }

int launch_multisweep(int shape, bool general, const MultiArgs &a, int grid, void *stream)
{
    if (shape < 0 || shape >= mshape_count() || grid < 1) return (int)hipErrorInvalidValue;
    MultiArgs b = a;
    if (b.xcut[kXcdCount] == 0) {
        if (grid != b.tile_count) return (int)hipErrorInvalidValue;
        const int q = b.tile_count / kXcdCount, r = b.tile_count % kXcdCount;
        for (int x = 0; x <= kXcdCount; ++x) b.xcut[x] = x * q + (x < r ? x : r);
    }
    const MEntry &e = kM[shape];
    hipLaunchKernelGGL((a.nsweeps <= kShortSweeps ? e.fn2 : e.fn)[general], dim3(grid), dim3(e.info.threads), 0,
                       (hipStream_t)stream, b);
    return (int)hipGetLastError();
}

}  // namespace j3d

// rows.hip -- formation of the rows of the pCT linear system on gfx950.
//
// Each proton history gives one equation: the chord lengths of its most
// likely path (MLP) through the voxels, times the voxel RSPs, sum to its
// WEPL (arXiv 1803.01112, Section I).  One lane forms one row:
//   1. the MLP vertices at depths j*step along the beam axis, from the
//      Fermi-Eyges / Highland scattering moments of the entry->vertex and
//      vertex->exit slabs and the 2x2 Gaussian conditioning of the lateral
//      (t, dt/du) and vertical (v, dv/du) states on the entry and exit
//      measurements, all in float64;
//   2. a Siddon parametric walk of every polyline segment (crossings of the
//      integer grid planes merged in order, voxel of a piece taken at its
//      midpoint), merging consecutive pieces in the same voxel.
// Decisions that pick voxel indices are taken in float64; chords are
// rounded to float32 (or float16) only when written.  This file must be
// compiled with -ffp-contract=off so that no multiply-add is fused.
#include <algorithm>
#include <type_traits>

#include "tvs_internal.hpp"

namespace tvs {
namespace {

constexpr double kE0 = 13.6;     // MeV, Highland constant
constexpr double kX0 = 360.8;    // mm, radiation length of water
constexpr int kThreads = 256;
constexpr int64_t kFewLines = 40000;   // hull lines that are bound by latency
// Row kernels: at least 3 wavefronts per SIMD (two vertices evaluated side by
// side fit only two: 14.0 against 11.5 ms for 4M rows of 200x200x16); the
// tile-list kernel's kRoom instance holds 2, leaving room for DROP waves.
constexpr int kRowWaves = 3;
// List entries staged per lane before they are written (LDS: 8 bytes each,
// 32 KB per 256-lane workgroup with float32 chords); slot k of lane l at
// k * kStageRow + l, so that a lane's slots fall into different banks.
constexpr int kStage = 16;
constexpr int kStageRow = kThreads + 1;

__device__ inline double ipow(double base, int e)
{
    double r = 1.0;
    for (int i = 0; i < e; i++) r *= base;
    return r;
}

// n! for n <= 9 (every use has a compile-time n after unrolling)
__device__ inline double fact(int n)
{
    constexpr double f[10] = {1.0, 1.0, 2.0, 6.0, 24.0, 120.0, 720.0, 5040.0, 40320.0, 362880.0};
    return f[n];
}

// a / b, correctly rounded (the IEEE quotient bit for bit), from y = 1/b
// rounded to nearest: a * y corrected twice by its residual a - b q (exact
// in an FMA).  After the first correction the estimate lies within one ulp
// of a / b; from there one correction with a correctly rounded reciprocal
// gives the correctly rounded quotient (Markstein's theorem; it needs no
// underflow or overflow on the way, which holds for every quotient it is
// used for here).  Five float64 operations against the eleven, one of them a
// quarter-rate reciprocal, of a general division.
__device__ inline double div_rn(double a, double b, double y)
{
    double q = a * y;
    double r = fma(-q, b, a);
    q = fma(r, y, q);
    r = fma(-q, b, a);
    return fma(r, y, q);
}

// a / n for a small integer n known at compile time (after unrolling).
__device__ inline double div_int(double a, int n)
{
    if ((n & (n - 1)) == 0) return a / (double)n;     // power of two: exact multiply
    return div_rn(a, (double)n, 1.0 / (double)n);
}

// Reciprocal of b rounded to nearest: the hardware's estimate, two Newton
// steps, then one correction by the exact residual (Markstein's theorem).  It
// and the two functions below leave out the scaling and special cases of the
// general operations; their operands are finite and far from underflow.
__device__ inline double recip_rn(double b)
{
    double y = __builtin_amdgcn_rcp(b);
    y = fma(fma(-b, y, 1.0), y, y);
    y = fma(fma(-b, y, 1.0), y, y);
    return fma(fma(-b, y, 1.0), y, y);
}

// a / b rounded to nearest: the quotient by an almost correct reciprocal,
// corrected once by its exact residual.
__device__ inline double quot_rn(double a, double b)
{
    double y = __builtin_amdgcn_rcp(b);
    y = fma(fma(-b, y, 1.0), y, y);
    y = fma(fma(-b, y, 1.0), y, y);
    const double q = a * y;
    return fma(fma(-b, q, a), y, q);
}

// sqrt(x) rounded to nearest, x > 0: one step of Goldschmidt's iteration from the
// hardware's 1 / sqrt(x) for g -> sqrt(x) and h -> 1 / (2 sqrt(x)), then two
// corrections of g by its exact residual.
__device__ inline double sqrt_rn(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    return fma(fma(-g, g, x), h, g);
}

// Natural logarithm of a positive, finite, normal x: x = m 2^e with m in
// [sqrt(1/2), sqrt(2)), ln m = 2 atanh(s) = 2 (s + s^3/3 + ... + s^21/21),
// s = (m - 1) / (m + 1), |s| <= 0.1716 (first omitted term below 2e-19).
// A fixed sequence of float64 operations (no library logarithm, whose last
// bit differs between math libraries), so the Highland factor, and with it
// every vertex, is the same double wherever the rows are formed.
__device__ inline double series_log(double x)
{
    int e = 0;
    double m = frexp(x, &e);
    if (m < 0.70710678118654752440) {
        m = m * 2.0;
        e = e - 1;
    }
    const double s = quot_rn(m - 1.0, m + 1.0);
    const double z = s * s;
    double p = 1.0 / 21.0;
    p = p * z + 1.0 / 19.0;
    p = p * z + 1.0 / 17.0;
    p = p * z + 1.0 / 15.0;
    p = p * z + 1.0 / 13.0;
    p = p * z + 1.0 / 11.0;
    p = p * z + 1.0 / 9.0;
    p = p * z + 1.0 / 7.0;
    p = p * z + 1.0 / 5.0;
    p = p * z + 1.0 / 3.0;
    p = p * z + 1.0;
    return (double)e * 0.69314718055994530942 + 2.0 * s * p;
}

__device__ inline double highland(double depth, int log_term)
{
    double f = 1.0;
    if (log_term) f = 1.0 + 0.038 * series_log(div_rn(depth, kX0, 1.0 / kX0));
    return div_rn(kE0 * kE0 * f * f, kX0, 1.0 / kX0);
}

// 1/(beta^2 p^2) of a 200 MeV proton in water, per mm^k.
__device__ inline void power_coefs(int const_power, double b[6])
{
    b[0] = 7.457e-6;
    b[1] = 4.548e-8;
    b[2] = -5.777e-10;
    b[3] = 1.301e-11;
    b[4] = -9.228e-14;
    b[5] = 2.687e-16;
    if (const_power) b[1] = b[2] = b[3] = b[4] = b[5] = 0.0;
}

struct M2 { double a, b, c, d; };   // [[a, b], [c, d]]

// Inverse as the adjugate times the reciprocal of the determinant.
__device__ inline M2 inv(const M2 &A)
{
    const double det = A.a * A.d - A.b * A.c;
    const double r = recip_rn(det);
    return {A.d * r, -A.b * r, -A.c * r, A.a * r};
}
__device__ inline void mvec(const M2 &A, double x0, double x1, double &y0, double &y1)
{
    double r0 = A.a * x0 + A.b * x1;
    double r1 = A.c * x0 + A.d * x1;
    y0 = r0;
    y1 = r1;
}

// Row emission state: consecutive pieces in one voxel merge into one entry.
// Entries also group into segments: maximal runs of consecutive entries in
// one image tile.  Modes:
//   kCount    counts entries and segments;
//   kSeg      reserves each segment's place in its (block, tile) list;
//   kRowMajor writes the entries in walk order (tvs_debug_rows);
//   kTiled    writes every entry into its tile list at the reserved place.
enum EmitMode { kCount = 0, kSeg = 1, kRowMajor = 2, kTiled = 3 };

// A chord as an unsigned multiple of the fixed-point store's unit (1 / qinv
// mm), rounded to nearest; the unit is the longest chord of the loaded rows
// / qmax, rounded up, so the clamp only catches rounding at the top.
__device__ inline uint32_t encode_fixed(double len, double qinv, uint32_t qmax)
{
    const double u = rint(len * qinv);
    return u > (double)qmax ? qmax : (uint32_t)u;
}

template <int MODE, typename CH>
struct Emit {
    int32_t cur = -1;
    double cur_len = 0.0;
    double norm2 = 0.0;
    int64_t n = 0;               // entries emitted
    int32_t nseg = 0;            // segments opened
    int32_t tile = -1;           // tile of the open segment
    uint32_t seg_len = 0;        // kSeg: entries of the open segment
    int32_t *idx = nullptr;      // kRowMajor
    CH *chord = nullptr;         // kRowMajor, kTiled
    double qinv = 0.0;           // kTiled, fixed-point chords: units per mm
    uint32_t qmax = 0;           // kTiled, fixed-point chords: largest code
    uint32_t qshift = 31;        // kTiled, fixed-point chords: tag bit of the code's bit 16
    double maxc = 0.0;           // kSeg: longest entry of the row
    uint32_t *btc = nullptr;     // kSeg: list lengths of this row's block
    uint64_t *segtab = nullptr;  // kSeg: (tile, place) of this row's segments
    const int64_t *segdst = nullptr;  // kTiled: first entry of this row's segments
    uint32_t *meta = nullptr;    // kTiled
    int64_t base = 0, dst = 0;   // kTiled
    uint32_t q = 0;              // kTiled: row within its block
    // kTiled: entries are staged in a ring of this lane's LDS slots: the open
    // segment's last ns (list places dst - ns .. dst - 1) from slot head, and
    // before them a closed segment's cn (from place cdst, slot chead) that
    // wait to be written.  A wavefront writes its lanes' closed segments
    // together, 16 lanes per segment (write_closed), so that each leaves as one
    // burst and the other lanes do not idle through it.
    int ns = 0, head = 0, cn = 0, chead = 0;
    int64_t cdst = 0;
    // kSeg, kTiled: guards against a walk that disagrees with the load-time
    // count (segments of this row, entries of the buffer); a disagreement
    // writes nothing and raises *err
    int32_t seg_cap = 0;
    int64_t cap = 0;
    uint32_t *err = nullptr;
    bool ok = true;

    __device__ inline void close_seg()
    {
        if constexpr (MODE == kSeg) {
            if (seg_len && ok) {
                const uint32_t pos = atomicAdd(btc + tile, seg_len);
                segtab[nseg - 1] = ((uint64_t)(uint32_t)tile << 32) | pos;
            }
            seg_len = 0;
        }
    }

    __device__ inline void bad()
    {
        if (ok) atomicOr(err, 1u);
        ok = false;
    }

    __device__ inline void flush()
    {
        if (cur < 0) return;
        const int32_t t = cur >> kTileShift;
        if (t != tile) {
            close_seg();
            if constexpr (MODE == kTiled) close_run();
            tile = t;
            if constexpr (MODE == kSeg || MODE == kTiled) {
                if (nseg >= seg_cap) bad();
            }
            if constexpr (MODE == kTiled) {
                if (ok) dst = segdst[nseg] - base;
            }
            nseg++;
        }
        if constexpr (MODE == kRowMajor) {
            idx[n] = cur;
            if constexpr (sizeof(CH) == 4) chord[n] = (float)cur_len;
            else chord[n] = __float2half((float)cur_len);
        }
        if constexpr (MODE == kTiled) {
            if (ok && (dst < 0 || dst >= cap)) bad();
            if (ok) {
                if (ns + cn == kStage) {     // no slot left: this lane writes by itself
                    if (cn == 0) close_run();
                    write_own();
                }
                const int slot = ((head + ns) & (kStage - 1)) * kStageRow + (int)threadIdx.x;
                uint32_t tag = (uint32_t)(cur & (kTileWords - 1)) | (q << kTileShift);
                if constexpr (sizeof(CH) == 4) {
                    stage_chord()[slot] = (float)cur_len;
                } else if constexpr (std::is_same<CH, uint16_t>::value) {
                    const uint32_t code = encode_fixed(cur_len, qinv, qmax);
                    tag |= (code >> 16) << qshift;
                    stage_chord()[slot] = (uint16_t)(code & 0xffffu);
                } else {
                    stage_chord()[slot] = __float2half((float)cur_len);
                }
                stage_meta()[slot] = tag;
                dst++;
                ns++;
            }
        }
        if constexpr (MODE == kSeg) {
            seg_len++;
            maxc = fmax(maxc, cur_len);
        }
        norm2 += cur_len * cur_len;
        n++;
        cur = -1;
        cur_len = 0.0;
    }

    // kTiled staging slots (LDS)
    static __device__ inline uint32_t *stage_meta()
    {
        __shared__ uint32_t sm[kStage * kStageRow];
        return sm;
    }
    static __device__ inline CH *stage_chord()
    {
        __shared__ CH sc[kStage * kStageRow];
        return sc;
    }

    // kTiled: the open segment's staged entries become the closed ones
    __device__ inline void close_run()
    {
        if (ns == 0) return;
        if (cn) write_own();
        cn = ns;
        chead = head;
        cdst = dst - ns;
        head = (head + ns) & (kStage - 1);
        ns = 0;
    }

    // kTiled: writes this lane's closed entries to their list places
    __device__ inline void write_own()
    {
        for (int k = 0; k < cn; k++) {
            const int slot = ((chead + k) & (kStage - 1)) * kStageRow + (int)threadIdx.x;
            meta[cdst + k] = stage_meta()[slot];
            chord[cdst + k] = stage_chord()[slot];
        }
        cn = 0;
    }

    // kTiled, every lane of the wavefront together: writes the closed entries
    // of all lanes, four lanes' at once.
    __device__ inline void write_closed()
    {
        if (ns > kStage - 4) close_run();      // a vertex adds at most three entries
        uint64_t left = __ballot(cn > 0);
        const int lane = threadIdx.x & 63, k = lane & 15;
        const int col = (int)threadIdx.x - lane;
        while (left) {
            int src[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                src[q] = left ? __builtin_ctzll(left) : -1;
                left &= left - 1;
            }
            const int a = (lane & 16) ? src[1] : src[0], b = (lane & 16) ? src[3] : src[2];
            const int from = (lane & 32) ? b : a, f = from < 0 ? 0 : from;
            const int run = __shfl(cn | chead << 8, f, 64);
            const int64_t at = __shfl(cdst, f, 64);
            if (from >= 0 && k < (run & 255)) {
                const int slot = (((run >> 8) + k) & (kStage - 1)) * kStageRow + col + from;
                meta[at + k] = stage_meta()[slot];
                chord[at + k] = stage_chord()[slot];
            }
        }
        cn = 0;
    }

    __device__ inline void finish()
    {
        flush();
        close_seg();
        if constexpr (MODE == kTiled) {
            close_run();
            write_own();
        }
    }
};

// Grid coordinates (p - o) / v of a point (quotients correctly rounded).
__device__ inline void to_grid(const GridDev &g, const double p[3], double gp[3])
{
    gp[0] = div_rn(p[0] - g.ox, g.vx, g.rvx);
    gp[1] = div_rn(p[1] - g.oy, g.vy, g.rvy);
    gp[2] = div_rn(p[2] - g.oz, g.vz, g.rvz);
}

// Walks segment q0 -> q1 of length len given the grid coordinates g0, g1 of
// its end points (each point's coordinates are computed once and shared by the two
// segments that meet there).
template <int MODE, typename CH>
__device__ void walk_segment(const GridDev &g, double len, const double g0[3], const double g1[3],
                             Emit<MODE, CH> &e)
{
    const int32_t n[3] = {g.nx, g.ny, g.nz};
    double dg[3];
    for (int a = 0; a < 3; a++) dg[a] = g1[a] - g0[a];
    if (!(len > 0.0)) return;

    // Per axis: next integer plane in the direction of travel, how many
    // planes inside [0, n] remain after it, and its crossing parameter
    // tau = (m - g0) / dg.  An axis with no plane left has tau = 2, past the
    // segment's end, so it is never the nearest crossing.
    double mnext[3], tnext[3];
    int rem[3];
    for (int a = 0; a < 3; a++) {
        mnext[a] = 0.0;
        tnext[a] = 2.0;
        rem[a] = 0;
        if (dg[a] == 0.0) continue;
        double lo = (g0[a] < g1[a]) ? g0[a] : g1[a];
        double hi = (g0[a] < g1[a]) ? g1[a] : g0[a];
        double mlo = floor(lo) + 1.0;
        double mhi = ceil(hi) - 1.0;
        if (mlo < 0.0) mlo = 0.0;
        if (mhi > (double)n[a]) mhi = (double)n[a];
        if (mlo > mhi) continue;
        mnext[a] = (dg[a] > 0.0) ? mlo : mhi;
        rem[a] = (int)(mhi - mlo);
        tnext[a] = (mnext[a] - g0[a]) / dg[a];
    }

    double prev = 0.0;
    for (;;) {
        double tb = 1.0;
        for (int a = 0; a < 3; a++)
            if (tnext[a] < tb) tb = tnext[a];
        if (tb > prev) {
            double ta = prev;
            prev = tb;
            double tm = (ta + tb) * 0.5;
            double c[3];
            bool inside = true;
            for (int a = 0; a < 3; a++) {
                c[a] = floor(g0[a] + tm * dg[a]);
                inside = inside && !(c[a] < 0.0 || c[a] >= (double)n[a]);
            }
            if (inside) {
                int32_t lin = vaddr32(g, (int32_t)c[0], (int32_t)c[1], (int32_t)c[2]);
                double clen = (tb - ta) * len;
                if (lin == e.cur) {
                    e.cur_len += clen;
                } else {
                    e.flush();
                    e.cur = lin;
                    e.cur_len = clen;
                }
            }
        }
        if (tb >= 1.0) break;
        for (int a = 0; a < 3; a++) {
            if (tnext[a] == tb) {
                if (rem[a] == 0) {
                    tnext[a] = 2.0;
                } else {
                    rem[a]--;
                    mnext[a] += (dg[a] > 0.0) ? 1.0 : -1.0;
                    tnext[a] = (mnext[a] - g0[a]) / dg[a];
                }
            }
        }
    }
}

// A vertex of the polyline as its segments need it: the point, its grid
// coordinates, the cell that holds it, and whether it lies inside the grid and
// at least kClear off every plane.
struct Vertex {
    double p[3], gp[3];
    int32_t c[3];
    bool clear;
};
constexpr double kClear = 1.0e-5;


__device__ inline void locate(const GridDev &g, Vertex &v)
{
    to_grid(g, v.p, v.gp);
    const int32_t n[3] = {g.nx, g.ny, g.nz};
    v.clear = true;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const double f = floor(v.gp[a]), r = v.gp[a] - f;
        v.clear = v.clear && r > kClear && r < 1.0 - kClear && f >= 0.0 && f < (double)n[a];
        v.c[a] = (int32_t)f;
    }
}

// Walks the segment u -> v.  Nearly every segment is short: both ends clear
// of the planes, at most one plane crossed per axis, and the crossings apart
// from each other and from the ends by kClear of its length.  Then the voxels
// follow from the ends' cells and the order of the crossings, without a
// midpoint for every piece: a midpoint keeps kClear / 2 of the segment's
// length from a crossed plane, which it passes by at least 2 kClear, hence
// 1e-10 of a voxel, and kClear from any other, while its rounding is below
// 1e-11 on grids of up to 4,096 voxels an axis, so that its floor names
// the same voxel.  Everything else takes the general walk.  `joined`: the
// open entry lies in u's cell (the last segment was a short one).
//
// Bound by instruction issue (the count pass keeps the VALUs 100 % busy): 4M
// rows of 200x200x16 (4.7e8 vertices) are counted in 8.0 ms, 10.8 with the
// general walk of every segment, and written to float32 lists in 11.5 ms
// (13.7).
template <int MODE, typename CH>
__device__ inline void walk(const GridDev &g, const Vertex &u, const Vertex &v, bool &joined,
                            Emit<MODE, CH> &e)
{
    const double dx = v.p[0] - u.p[0], dy = v.p[1] - u.p[1], dz = v.p[2] - u.p[2];
    const double len = sqrt_rn(dx * dx + dy * dy + dz * dz);
    // crossing parameter by axis; past the end, and apart, where there is none
    double t[3] = {2.0, 3.0, 4.0};
    int32_t d[3];
    bool fast = u.clear && v.clear && len > 0.0 && g.short_ok;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        d[a] = v.c[a] - u.c[a];
        fast = fast && d[a] >= -1 && d[a] <= 1;
    }
#pragma unroll
    for (int a = 0; a < 3; a++) {
        if (fast && d[a] != 0) {
            const double m = (double)(d[a] > 0 ? v.c[a] : u.c[a]);
            t[a] = quot_rn(m - u.gp[a], v.gp[a] - u.gp[a]);
            fast = t[a] > kClear && t[a] < 1.0 - kClear;
        }
    }
    // crossings in order; the axis of each in two bits, the first lowest
    double s0 = t[0], s1 = t[1], s2 = t[2];
    uint32_t a0 = 0u, a1 = 1u, a2 = 2u;
    auto order = [](double &x, double &y, uint32_t &ax, uint32_t &ay) {
        const bool sw = y < x;
        const double tx = sw ? y : x, ty = sw ? x : y;
        const uint32_t bx = sw ? ay : ax, by = sw ? ax : ay;
        x = tx;
        y = ty;
        ax = bx;
        ay = by;
    };
    order(s0, s1, a0, a1);
    order(s1, s2, a1, a2);
    order(s0, s1, a0, a1);
    fast = fast && s1 - s0 > kClear && s2 - s1 > kClear;
    if (fast) {
        const double first = (s0 < 1.0 ? s0 : 1.0) * len;
        if (joined) {
            e.cur_len += first;
        } else {
            const int32_t lin = vaddr32(g, u.c[0], u.c[1], u.c[2]);
            if (lin == e.cur) {
                e.cur_len += first;
            } else {
                e.flush();
                e.cur = lin;
                e.cur_len = first;
            }
        }
        int32_t i = u.c[0], j = u.c[1], k = u.c[2];
        while (s0 < 1.0) {
            e.flush();
            i = a0 == 0u ? v.c[0] : i;
            j = a0 == 1u ? v.c[1] : j;
            k = a0 == 2u ? v.c[2] : k;
            e.cur = vaddr32(g, i, j, k);
            e.cur_len = ((s1 < 1.0 ? s1 : 1.0) - s0) * len;
            s0 = s1;
            a0 = a1;
            s1 = s2;
            a1 = a2;
            s2 = 2.0;
        }
    } else {
        walk_segment<MODE, CH>(g, len, u.gp, v.gp, e);
    }
    joined = fast;
}

// Inverse covariance of the entry-side slab at depth d1, (Sigma_1(d1))^-1,
// as {a, b, d} of the symmetric 2x2 matrix [[a, b], [b, d]].  It depends on
// the depth only, so a context computes it once per vertex depth j * step
// (k_mlp_table) and every row reads it from that table.
__device__ inline void entry_sigma_inv(double d1, const MlpCfg &m, double s[3])
{
    double b[6];
    power_coefs(m.const_power, b);
    double i1[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int mm = 0; mm < 3; mm++) {
#pragma unroll
        for (int k = 0; k < 6; k++) {
            const double beta = fact(mm) * fact(k) / fact(mm + k + 1);
            i1[mm] += b[k] * ipow(d1, mm + k + 1) * beta;
        }
    }
    double A1 = highland(d1, m.log_term);
    M2 S1 = {A1 * i1[2], A1 * i1[1], A1 * i1[1], A1 * i1[0]};
    M2 S1i = inv(S1);
    s[0] = S1i.a;
    s[1] = S1i.b;   // equals S1i.c: S1 is symmetric
    s[2] = S1i.d;
}

// MLP of history i and the Siddon walk of its polyline.  All lanes of a
// wavefront call it together; valid: this lane has a history (i names some
// history in any case).
template <int MODE, typename CH>
__device__ void form_row(const GridDev &g, const HistDev &H, const MlpCfg &m, int64_t i,
                         bool valid, Emit<MODE, CH> &e)
{
    double ex = H.s(kEx)[i], ey = H.s(kEy)[i], ez = H.s(kEz)[i];
    double qx = H.s(kQx)[i], qy = H.s(kQy)[i], qz = H.s(kQz)[i];
    double eth = H.s(kEth)[i], eps = H.s(kEps)[i], qth = H.s(kQth)[i], qps = H.s(kQps)[i];
    double ux = H.s(kUx)[i], uy = H.s(kUy)[i];
    double nrm = sqrt(ux * ux + uy * uy);
    ux = ux / nrm;
    uy = uy / nrm;

    double u0 = ex * ux + ey * uy, t0 = -ex * uy + ey * ux, v0 = ez;
    double u2 = qx * ux + qy * uy, t2 = -qx * uy + qy * ux, v2 = qz;
    double L = u2 - u0;
    const bool some = valid && L > 0.0;
    double Jd = ceil(L / m.step);
    const int64_t J = !some ? 0 : (Jd < 1.0) ? 1 : (int64_t)Jd;

    double b[6];
    power_coefs(m.const_power, b);
    // Exit-side expansion P(L - s) = sum_k c_k s^k.
    double c[6];
#pragma unroll
    for (int k = 0; k < 6; k++) {
        double acc = 0.0;
#pragma unroll
        for (int q = k; q < 6; q++) {
            const double binom = fact(q) / (fact(k) * fact(q - k));
            acc += b[q] * binom * ipow(L, q - k);
        }
        c[k] = (k % 2) ? -acc : acc;
    }

    bool miss = false;
    // MLP vertex j (1 <= j < J); the table index is clamped and a depth past
    // the table only noted, so that the body has no branch and two vertices
    // can be evaluated side by side
    auto vertex = [&](int64_t j, double p[3]) {
        double d1 = (double)j * m.step;
        double d2 = L - d1;
        // (the table covers every depth of the loaded histories, their
        // vertex counts bound it; a depth past it raises the consistency flag)
        const bool in_tab = j < m.nj;
        miss |= !in_tab;
        double s1[3] = {0.0, 0.0, 0.0};
        if (in_tab) {
            const double *tab = m.s1i + 3 * j;
            s1[0] = tab[0];
            s1[1] = tab[1];
            s1[2] = tab[2];
        }
        // integral_0^d2 s^(mm+k) ds = d2^n / n, n = mm + k + 1 (powers of
        // d2 as running products, which equal repeated multiplication)
        double pw = 1.0, q[9];
#pragma unroll
        for (int n = 1; n <= 8; n++) {
            pw = pw * d2;
            q[n] = div_int(pw, n);
        }
        double j2[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int mm = 0; mm < 3; mm++)
#pragma unroll
            for (int k = 0; k < 6; k++)
                j2[mm] += c[k] * q[mm + k + 1];
        double A2 = highland(d2, m.log_term);
        M2 S2 = {A2 * j2[2], A2 * j2[1], A2 * j2[1], A2 * j2[0]};
        M2 S1i = {s1[0], s1[1], s1[1], s1[2]};
        M2 S2i = inv(S2);
        // R0 = [[1, d1], [0, 1]], R1 = [[1, d2], [0, 1]]: products with their
        // ones and zeros written out (every factor is finite, so they add
        // nothing)
        M2 T = {S2i.a, S2i.b, d2 * S2i.a + S2i.c, d2 * S2i.b + S2i.d};   // R1^T S2^-1
        M2 T2 = {T.a, T.a * d2 + T.b, T.c, T.c * d2 + T.d};              // R1^T S2^-1 R1
        M2 M = {S1i.a + T2.a, S1i.b + T2.b, S1i.c + T2.c, S1i.d + T2.d};
        M2 Mi = inv(M);
        double y1t, y1v;
        {
            double a0, a1, p0, p1, q0, q1, r0, r1, y0_, y1_;
            a0 = t0 + d1 * eth;
            a1 = eth;
            mvec(S1i, a0, a1, p0, p1);
            mvec(T, t2, qth, q0, q1);
            r0 = p0 + q0;
            r1 = p1 + q1;
            mvec(Mi, r0, r1, y0_, y1_);
            y1t = y0_;
        }
        {
            double a0, a1, p0, p1, q0, q1, r0, r1, y0_, y1_;
            a0 = v0 + d1 * eps;
            a1 = eps;
            mvec(S1i, a0, a1, p0, p1);
            mvec(T, v2, qps, q0, q1);
            r0 = p0 + q0;
            r1 = p1 + q1;
            mvec(Mi, r0, r1, y0_, y1_);
            y1v = y0_;
        }
        double u = u0 + d1;
        p[0] = u * ux - y1t * uy;
        p[1] = u * uy + y1t * ux;
        p[2] = y1v;
    };

    Vertex u;
    u.p[0] = ex;
    u.p[1] = ey;
    u.p[2] = ez;
    locate(g, u);
    bool joined = false;
    // vertices 1 .. J - 1, then the exit point.  Every lane of the wavefront
    // runs as many rounds as the longest row: the staged entries are written
    // by all lanes together
    for (int64_t j = 1; __any(j <= J); j++) {
        if (j <= J) {
            Vertex a;
            a.p[0] = qx;
            a.p[1] = qy;
            a.p[2] = qz;
            if (j < J) vertex(j, a.p);
            locate(g, a);
            walk<MODE, CH>(g, u, a, joined, e);
            u = a;
        }
        if constexpr (MODE == kTiled) e.write_closed();
    }
    if (miss && m.err) atomicOr(m.err, 1u);
}

__global__ void __launch_bounds__(kThreads) k_mlp_table(MlpCfg m, int64_t nj, double *tab)
{
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= nj) return;
    double s[3] = {0.0, 0.0, 0.0};
    if (j > 0) entry_sigma_inv((double)j * m.step, m, s);
    tab[3 * j] = s[0];
    tab[3 * j + 1] = s[1];
    tab[3 * j + 2] = s[2];
}

__global__ void __launch_bounds__(kThreads, kRowWaves)
k_rows_count(GridDev g, HistDev H, MlpCfg m, int64_t first, int64_t n, int32_t *nnz, int32_t *nseg)
{
    int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    Emit<kCount, float> e;
    form_row<kCount, float>(g, H, m, first + (q < n ? q : n - 1), q < n, e);
    if (q >= n) return;
    e.finish();
    nnz[q] = (int32_t)e.n;
    if (nseg) nseg[q] = (int32_t)e.nseg;
}

__global__ void __launch_bounds__(kThreads, kRowWaves)
k_rows_seg(GridDev g, HistDev H, MlpCfg m, int64_t n, int64_t B, int64_t ntiles,
           const int64_t *seg_off, uint32_t *btc, uint64_t *segtab, uint32_t *err,
           uint32_t *chmax, const int32_t *order)
{
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    uint32_t bits = 0u;
    const bool valid = i < n;
    i = valid ? i : n - 1;
    if (order) i = order[i];
    Emit<kSeg, float> e;
    e.btc = btc + (i / B) * ntiles;
    e.segtab = segtab + seg_off[i];
    e.seg_cap = (int32_t)(seg_off[i + 1] - seg_off[i]);
    e.err = err;
    form_row<kSeg, float>(g, H, m, i, valid, e);
    if (valid) {
        e.finish();
        // longest chord as float32 bits, rounded up (non-negative floats
        // order as their bit patterns)
        float mf = (float)e.maxc;
        if ((double)mf < e.maxc) mf = nextafterf(mf, INFINITY);
        bits = __float_as_uint(mf);
    }
    // the wavefront's maximum (every lane takes part), one atomic per wavefront
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t o = __shfl_xor(bits, d, 64);
        bits = o > bits ? o : bits;
    }
    if ((threadIdx.x & 63) == 0 && chmax && bits) atomicMax(chmax, bits);
}

__global__ void __launch_bounds__(kThreads)
k_seg_dest(int64_t n, int64_t B, int64_t ntiles, const int64_t *seg_off, const int64_t *bt_off,
           const int32_t *slot_of, int64_t nslots, uint64_t *segtab, uint32_t *err)
{
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const int64_t *bto = bt_off + (i / B) * nslots;
    for (int64_t s = seg_off[i]; s < seg_off[i + 1]; s++) {
        const uint64_t v = segtab[s];
        const int64_t T = (int64_t)(v >> 32);
        const int32_t slot = T < ntiles ? slot_of[T] : -1;
        if (slot < 0) {
            atomicOr(err, 1u);
            segtab[s] = 0;
            continue;
        }
        segtab[s] = (uint64_t)(bto[slot] + (int64_t)(v & 0xffffffffull));
    }
}

// kRoom: the kernel takes at least 171 VGPRs (176 allocated: the empty asm
// below claims v170), so that a SIMD holds two of its waves and four 40-VGPR
// DROP waves beside them; otherwise it fits three waves per SIMD, and a DROP
// step finds no room on a SIMD that holds three.
template <typename CH, bool kRoom>
__global__ void __launch_bounds__(kThreads, kRoom ? 2 : kRowWaves)
k_rows_fill_tiled(GridDev g, HistDev H, MlpCfg m, TileFill f, CH *chord)
{
    if constexpr (kRoom) asm volatile("" ::: "v170");
    // grid-stride: the grid may be held below the device's capacity so that
    // the DROP launches running beside it always find free slots
    for (int64_t q0 = (int64_t)blockIdx.x * kThreads; q0 < f.n; q0 += (int64_t)gridDim.x * kThreads) {
        const bool valid = q0 + threadIdx.x < f.n;
        const int64_t q = valid ? q0 + threadIdx.x : f.n - 1;
        const int64_t i = f.order ? (int64_t)f.order[f.first + q] : f.first + q;
        Emit<kTiled, CH> e;
        e.segdst = f.segdst + f.seg_off[i];
        e.seg_cap = (int32_t)(f.seg_off[i + 1] - f.seg_off[i]);
        e.cap = f.cap;
        e.err = f.err;
        e.meta = f.meta;
        e.chord = chord;
        e.base = f.base;
        e.qinv = f.qinv;
        e.qmax = f.qmax;
        e.qshift = f.qshift;
        e.q = (uint32_t)(i % f.B);
        form_row<kTiled, CH>(g, H, m, i, valid, e);
        e.finish();
        if (valid) f.norm2[i] = (float)e.norm2;
    }
}

__global__ void __launch_bounds__(kThreads, kRowWaves)
k_rows_fill(GridDev g, HistDev H, MlpCfg m, int64_t first, int64_t n, const int64_t *row_off,
            int64_t base, int32_t *idx, float *chord, float *norm2)
{
    int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool valid = q < n;
    q = valid ? q : n - 1;
    Emit<kRowMajor, float> e;
    int64_t off = row_off[q] - base;
    e.idx = idx + off;
    e.chord = chord + off;
    form_row<kRowMajor, float>(g, H, m, first + q, valid, e);
    if (!valid) return;
    e.finish();
    norm2[q] = (float)e.norm2;
}

__global__ void __launch_bounds__(kThreads)
k_validate(HistDev H, int64_t n, double step, uint32_t *bad, uint32_t *jmax)
{
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    bool ok = true;
    for (int q = 0; q < 13; q++) {
        float v = H.s(q)[i];
        if (!isfinite(v) || fabsf(v) > 1.0e6f) ok = false;
    }
    if (ok) {
        double ux = H.s(kUx)[i], uy = H.s(kUy)[i];
        double nn = ux * ux + uy * uy;
        if (!(nn >= 1.0e-12)) {
            ok = false;
        } else {
            double nrm = sqrt(nn);
            double L = ((double)H.s(kQx)[i] - (double)H.s(kEx)[i]) * (ux / nrm) +
                       ((double)H.s(kQy)[i] - (double)H.s(kEy)[i]) * (uy / nrm);
            if (L / step > 1048576.0) ok = false;
            else if (L > 0.0) atomicMax(jmax, (uint32_t)ceil(L / step) + 2u);
        }
    }
    if (!ok) atomicAdd(bad, 1u);
}

// Hull detection: every history's straight line from its entry to its exit
// point; a line whose WEPL reaches wepl_in counts its voxels (space
// modelling), one whose WEPL is below wepl_out carves them (space carving).
// One lane per history; the counters (x-fastest) saturate at in_sat / out_sat
// (min_in and max_out + 1): past them no further line changes a decision, and
// most adds are skipped.  A count read below its true value (another line's
// add not yet seen) only costs an add; one at the value has reached it for
// good.
struct HullCounts {
    uint32_t *in_cnt, *out_cnt;
    const uint32_t *in_full, *out_full;   // voxels at their value, a bit each (may be null)
    uint32_t in_sat, out_sat;
    bool in_read, out_read;               // kByFlags: whether a count is read before it is added to
};

// How a voxel's count is added to: after a read of it (kRead), after one that is
// requested a piece before (kEarly), or after a read where the flags say so.
enum HullCount { kRead, kEarly, kByFlags };

// What a line learns of voxel p as it enters it: the full-voxel bits that hold it
// or, kEarly, its count.
template <HullCount HOW>
__device__ inline uint32_t hull_word(const uint32_t *cnt, const uint32_t *full, int32_t p)
{
    if (HOW == kEarly) return __hip_atomic_load(cnt + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return full ? full[p >> 5] : 0u;
}

// Counts voxel p; word: what hull_word gave.
template <HullCount HOW>
__device__ inline void hull_count(uint32_t *cnt, uint32_t word, uint32_t sat, bool read, int32_t p)
{
    if (HOW == kEarly) {
        if (word < sat) atomicAdd(cnt + p, 1u);
        return;
    }
    if ((word >> (p & 31)) & 1u) return;
    if ((HOW == kByFlags && !read) ||
        __hip_atomic_load(cnt + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < sat)
        atomicAdd(cnt + p, 1u);
}

// The line g0 -> g1 (grid coordinates): the pieces of walk_segment.  While
// crossings are apart by more than eps of the line, their order follows from
// parameters stepped by 1 / |dg| (rounding far below eps), and a piece's
// voxel from the planes crossed so far: its midpoint keeps half the piece
// times the slowest crossing axis' |dg| (1e-8) from every plane that axis
// crosses, and kClear from the others.  Where two parameters come within eps
// of each other or of the end, they are formed as walk_segment forms them,
// and a piece no longer than eps takes its voxel at the midpoint; a line that
// touches a plane without crossing it does so all the way.
template <HullCount HOW>
__device__ inline void hull_line(const GridDev &g, const double g0[3], const double g1[3],
                                 const HullCounts &h, bool in, bool out)
{
    const int32_t n[3] = {g.nx, g.ny, g.nz};
    const int32_t stride[3] = {1, g.nx, g.nx * g.ny};
    double t[3], dt[3], slow = 1.0;
    int32_t c[3], dir[3], p = 0, last = -1;
    bool loose = !g.short_ok;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const double dg = g1[a] - g0[a];
        const double lo = g0[a] < g1[a] ? g0[a] : g1[a], hi = g0[a] < g1[a] ? g1[a] : g0[a];
        const double top = (double)n[a], fl = floor(lo);
        double mlo = fl + 1.0, mhi = ceil(hi) - 1.0;
        if (mlo < 0.0) mlo = 0.0;
        if (mhi > top) mhi = top;
        t[a] = 2.0;
        dt[a] = 0.0;
        dir[a] = 0;
        if (dg != 0.0 && mlo <= mhi) {
            dir[a] = dg > 0.0 ? 1 : -1;
            c[a] = dg > 0.0 ? (int32_t)mlo - 1 : (int32_t)mhi;
            t[a] = ((dg > 0.0 ? mlo : mhi) - g0[a]) / dg;
            dt[a] = fabs(1.0 / dg);
            slow = fabs(dg) < slow ? fabs(dg) : slow;
        } else {
            c[a] = hi < 0.0 ? -1 : lo > top ? n[a] : (int32_t)fl;
            const bool off = hi < -kClear || lo > top + kClear;
            loose = loose || (dg != 0.0 && !off && !(lo - fl > kClear && hi - fl < 1.0 - kClear));
        }
        p += c[a] * stride[a];
    }
    const double eps = loose ? 4.0 : 2.0e-8 / slow;
    double prev = 0.0;
    // a voxel is counted one piece later: its bits (its count) arrive meanwhile
    uint32_t win = 0u, wout = 0u;
    auto count_last = [&]() {
        if (last < 0) return;
        if (in) hull_count<HOW>(h.in_cnt, win, h.in_sat, h.in_read, last);
        if (out) hull_count<HOW>(h.out_cnt, wout, h.out_sat, h.out_read, last);
    };
    for (;;) {
        const double lo = fmin(t[0], t[1]), hi = fmax(t[0], t[1]);
        double tb = fmin(lo, t[2]);
        const double second = fmin(fmin(hi, fmax(lo, t[2])), 1.0);
        bool inside = (uint32_t)c[0] < (uint32_t)n[0] && (uint32_t)c[1] < (uint32_t)n[1] &&
                      (uint32_t)c[2] < (uint32_t)n[2];
        int32_t at = p;
        if (second - tb < eps) {
#pragma unroll
            for (int a = 0; a < 3; a++) {
                // the plane ahead; past the grid's planes there is none
                const int32_t m = c[a] + (dir[a] > 0 ? 1 : 0);
                if (dir[a])
                    t[a] = (m >= 0 && m <= n[a]) ? ((double)m - g0[a]) / (g1[a] - g0[a]) : 2.0;
            }
            tb = fmin(fmin(t[0], t[1]), fmin(t[2], 1.0));
            if (!(tb - prev > eps)) {
                const double tm = (prev + tb) * 0.5;
                inside = tb > prev;
                at = 0;
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    const double f = floor(g0[a] + tm * (g1[a] - g0[a]));
                    inside = inside && !(f < 0.0 || f >= (double)n[a]);
                    at += (inside ? (int32_t)f : 0) * stride[a];
                }
            }
        }
        if (inside && at != last) {
            count_last();
            last = at;
            win = in ? hull_word<HOW>(h.in_cnt, h.in_full, at) : 0u;
            wout = out ? hull_word<HOW>(h.out_cnt, h.out_full, at) : 0u;
        }
        prev = tb;
        bool more = tb < 1.0;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const bool cross = t[a] == tb;
            t[a] += cross ? dt[a] : 0.0;
            c[a] += cross ? dir[a] : 0;
            p += cross ? (dir[a] > 0 ? stride[a] : -stride[a]) : 0;
            // out by the last plane of this axis: nothing more inside
            more = more && (loose || !cross || (uint32_t)c[a] < (uint32_t)n[a] ||
                            (dir[a] > 0 ? c[a] < 0 : c[a] >= n[a]));
        }
        if (!more) break;
    }
    count_last();
}

template <HullCount HOW>
__global__ void __launch_bounds__(kThreads)
k_hull_counts(GridDev g, HistDev H, int64_t first, int64_t n, double wepl_in, double wepl_out,
              HullCounts h)
{
    const int64_t i = first + (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const double w = H.s(kWepl)[i];
    const bool in = w >= wepl_in && h.in_sat > 0u, out = w < wepl_out;
    if (!in && !out) return;
    const double p0[3] = {H.s(kEx)[i], H.s(kEy)[i], H.s(kEz)[i]};
    const double p1[3] = {H.s(kQx)[i], H.s(kQy)[i], H.s(kQz)[i]};
    const double dx = p1[0] - p0[0], dy = p1[1] - p0[1], dz = p1[2] - p0[2];
    if (!(dx * dx + dy * dy + dz * dz > 0.0)) return;
    double g0[3], g1[3];
    to_grid(g, p0, g0);
    to_grid(g, p1, g1);
    hull_line<HOW>(g, g0, g1, h, in, out);
}

// A bit per voxel: its count has reached sat (in words [0, nw), out after them).
__global__ void __launch_bounds__(kThreads)
k_hull_full(const uint32_t *in_cnt, const uint32_t *out_cnt, int64_t n, uint32_t in_sat,
            uint32_t out_sat, uint32_t *full, int64_t nw)
{
    const int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint64_t bi = __ballot(q < n && in_cnt[q < n ? q : 0] >= in_sat);
    const uint64_t bo = __ballot(q < n && out_cnt[q < n ? q : 0] >= out_sat);
    const int lane = threadIdx.x & 63;
    const int64_t w = (q >> 6) * 2 + (lane & 1);
    if (lane < 2 && w < nw) {
        full[w] = (uint32_t)(bi >> (32 * lane));
        full[nw + w] = (uint32_t)(bo >> (32 * lane));
    }
}

// hull[p] (x-fastest) = in_cnt >= min_in and out_cnt <= max_out; with mask,
// the image x (tiled layout) is multiplied by the hull.
__global__ void __launch_bounds__(kThreads)
k_hull_decide(GridDev g, const uint32_t *in_cnt, const uint32_t *out_cnt, uint32_t min_in,
              uint32_t max_out, uint8_t *hull, double *mask)
{
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * kThreads) {
        const int64_t ii = p % g.nx, t = p / g.nx, jj = t % g.ny, kk = t / g.ny;
        const int64_t a = vaddr(g, ii, jj, kk);
        const bool inside = in_cnt[p] >= min_in && out_cnt[p] <= max_out;
        hull[p] = inside ? 1u : 0u;
        if (mask && !inside) mask[a] = 0.0;
    }
}

// Longest row and number of empty rows: stat[0], stat[1] (cleared before).
__global__ void __launch_bounds__(kThreads) k_row_stats(const int32_t *nnz, int64_t n, uint32_t *stat)
{
    uint32_t mx = 0, empty = 0;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads) {
        const uint32_t len = (uint32_t)nnz[i];
        mx = len > mx ? len : mx;
        empty += len == 0u;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t m = (uint32_t)__shfl_xor((int)mx, o, 64);
        mx = m > mx ? m : mx;
        empty += (uint32_t)__shfl_xor((int)empty, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(stat, mx);
        if (empty) atomicAdd(stat + 1, empty);
    }
}

// Processing order of the row passes: within each DROP block, histories by
// decreasing row length (a counting sort over at most BINS classes of
// lengths), so that the lanes of a wavefront walk rows of similar length while
// a block's tile lists are still written together (their partly written lines
// meet in the L2 before they are evicted).  Each segment's place is fixed
// otherwise, so the order changes no result, nor does that of rows of one class.
// Two passes over the lengths (4 B a history) and one over the order; sorted on
// the host, with the copies there and back, and with allocations made anew, a
// request of 2 M histories of 128x128x8 took 31.8 ms, 25.6 now.
template <int NT, int BINS>
__global__ void __launch_bounds__(NT)
k_row_order(const int32_t *nnz, int64_t n, int64_t B, int64_t nblocks,
            const uint32_t *stat, int32_t *order)
{
    __shared__ uint32_t place[BINS], part[NT];
    const int tid = threadIdx.x;
    const uint32_t mx = stat[0];
    // class of a length, the longest rows' lowest: (mx - len) scaled to the classes
    const bool exact = mx < (uint32_t)BINS;
    const float scale = (float)(BINS - 1) / (float)(mx > 0 ? mx : 1u);
    auto bin = [&](int32_t len) {
        const uint32_t d = mx - (uint32_t)len;
        if (exact) return (int)d;
        const int b = (int)((float)d * scale);
        return b < BINS ? b : BINS - 1;
    };
    const int per = BINS / NT;
    for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const int64_t f0 = b * B, f1 = f0 + B < n ? f0 + B : n;
        for (int q = tid; q < BINS; q += NT) place[q] = 0;
        __syncthreads();
#pragma unroll 4
        for (int64_t i = f0 + tid; i < f1; i += NT) atomicAdd(place + bin(nnz[i]), 1u);
        __syncthreads();
        // exclusive sums: each thread its `per` classes, then the threads' totals
        uint32_t sum = 0;
        for (int q = 0; q < per; q++) sum += place[tid * per + q];
        part[tid] = sum;
        __syncthreads();
        for (int o = 1; o < NT; o <<= 1) {
            const uint32_t v = tid >= o ? part[tid - o] : 0u;
            __syncthreads();
            part[tid] += v;
            __syncthreads();
        }
        uint32_t pos = part[tid] - sum;
        for (int q = 0; q < per; q++) {
            const uint32_t c = place[tid * per + q];
            place[tid * per + q] = pos;
            pos += c;
        }
        __syncthreads();
#pragma unroll 4
        for (int64_t i = f0 + tid; i < f1; i += NT)
            order[f0 + (int64_t)atomicAdd(place + bin(nnz[i]), 1u)] = (int32_t)i;
        __syncthreads();
    }
}

// dst[b] = src[b * stride] for b = 0 .. n - 1
__global__ void __launch_bounds__(kThreads)
k_pick(const int64_t *src, int64_t stride, int64_t n, int64_t *dst)
{
    for (int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x; b < n;
         b += (int64_t)gridDim.x * kThreads)
        dst[b] = src[b * stride];
}

// ---------------------------------------------------------------- scan
constexpr int kScanItems = 8;
constexpr int kScanTile = kThreads * kScanItems;

__device__ inline int64_t block_exclusive_scan(int64_t v, int64_t *total)
{
    __shared__ int64_t warp_sums[kThreads / 64];
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int64_t t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) warp_sums[w] = inc;
    __syncthreads();
    int64_t before = 0, all = 0;
    for (int q = 0; q < kThreads / 64; q++) {
        if (q < w) before += warp_sums[q];
        all += warp_sums[q];
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

__global__ void __launch_bounds__(kThreads)
k_scan_tiles(const int32_t *cnt, int64_t n, int64_t *tile_sum)
{
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    int64_t s = 0;
    for (int q = 0; q < kScanItems; q++) {
        int64_t i = base + (int64_t)threadIdx.x * kScanItems + q;
        if (i < n) s += cnt[i];
    }
    int64_t total;
    block_exclusive_scan(s, &total);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kThreads)
k_scan_partials(int64_t *tile_sum, int64_t ntiles)
{
    // Single workgroup: exclusive scan of the tile sums in place, in chunks.
    int64_t carry = 0;
    for (int64_t base = 0; base < ntiles; base += kThreads) {
        int64_t i = base + threadIdx.x;
        int64_t v = (i < ntiles) ? tile_sum[i] : 0;
        int64_t total;
        int64_t ex = block_exclusive_scan(v, &total);
        if (i < ntiles) tile_sum[i] = carry + ex;
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) tile_sum[ntiles] = carry;
}

__global__ void __launch_bounds__(kThreads)
k_scan_write(const int32_t *cnt, int64_t n, const int64_t *tile_off, int64_t ntiles, int64_t *off)
{
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    int64_t v[kScanItems];
    int64_t s = 0;
    for (int q = 0; q < kScanItems; q++) {
        int64_t i = base + (int64_t)threadIdx.x * kScanItems + q;
        v[q] = (i < n) ? (int64_t)cnt[i] : 0;
        s += v[q];
    }
    int64_t total;
    int64_t ex = block_exclusive_scan(s, &total) + tile_off[blockIdx.x];
    for (int q = 0; q < kScanItems; q++) {
        int64_t i = base + (int64_t)threadIdx.x * kScanItems + q;
        if (i < n) off[i] = ex;
        ex += v[q];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) off[n] = tile_off[ntiles];
}

}  // namespace

hipError_t launch_rows_count(const GridDev &g, const HistDev &h, const MlpCfg &m, int64_t first,
                             int64_t n, int32_t *nnz, int32_t *nseg, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    dim3 grid((unsigned)((n + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(k_rows_count, grid, dim3(kThreads), 0, stream, g, h, m, first, n, nnz, nseg);
    return hipGetLastError();
}

hipError_t launch_rows_seg(const GridDev &g, const HistDev &h, const MlpCfg &m, int64_t n,
                           int64_t B, const int64_t *seg_off, uint32_t *btc, uint64_t *segtab,
                           uint32_t *err, uint32_t *chmax, const int32_t *order,
                           hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    dim3 grid((unsigned)((n + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(k_rows_seg, grid, dim3(kThreads), 0, stream, g, h, m, n, B, num_tiles(g),
                       seg_off, btc, segtab, err, chmax, order);
    return hipGetLastError();
}

hipError_t launch_seg_dest(const GridDev &g, int64_t n, int64_t B, const int64_t *seg_off,
                           const int64_t *bt_off, const int32_t *slot_of, int64_t nslots,
                           uint64_t *segtab, uint32_t *err, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    dim3 grid((unsigned)((n + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(k_seg_dest, grid, dim3(kThreads), 0, stream, n, B, num_tiles(g), seg_off,
                       bt_off, slot_of, nslots, segtab, err);
    return hipGetLastError();
}

hipError_t launch_rows_fill_tiled(const GridDev &g, const HistDev &h, const MlpCfg &m,
                                  const TileFill &f, hipStream_t stream)
{
    if (f.n <= 0) return hipSuccess;
    int64_t wgs = (f.n + kThreads - 1) / kThreads;
    if (f.max_wgs > 0 && wgs > f.max_wgs) wgs = f.max_wgs;
    dim3 grid((unsigned)wgs);
    if (f.chq)
        hipLaunchKernelGGL((k_rows_fill_tiled<uint16_t, false>), grid, dim3(kThreads), 0, stream,
                           g, h, m, f, f.chq);
    else if (f.ch16)
        hipLaunchKernelGGL((k_rows_fill_tiled<__half, false>), grid, dim3(kThreads), 0, stream, g,
                           h, m, f, f.ch16);
    else if (f.room)
        hipLaunchKernelGGL((k_rows_fill_tiled<float, true>), grid, dim3(kThreads), 0, stream, g, h,
                           m, f, f.ch32);
    else
        hipLaunchKernelGGL((k_rows_fill_tiled<float, false>), grid, dim3(kThreads), 0, stream, g,
                           h, m, f, f.ch32);
    return hipGetLastError();
}

hipError_t launch_rows_fill(const GridDev &g, const HistDev &h, const MlpCfg &m, const RowSet &rs,
                            hipStream_t stream)
{
    if (rs.n <= 0) return hipSuccess;
    dim3 grid((unsigned)((rs.n + kThreads - 1) / kThreads));
    hipLaunchKernelGGL(k_rows_fill, grid, dim3(kThreads), 0, stream, g, h, m, rs.first, rs.n,
                       rs.row_off, rs.base, rs.idx, rs.chord32, rs.norm2);
    return hipGetLastError();
}

int64_t scan_tmp_elems(int64_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

hipError_t launch_validate(const HistDev &h, int64_t n, double step, uint32_t *bad,
                           uint32_t *jmax, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_validate, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads),
                       0, stream, h, n, step, bad, jmax);
    return hipGetLastError();
}

hipError_t launch_hull_counts(const GridDev &g, const HistDev &h, int64_t n, double wepl_in,
                              double wepl_out, uint32_t *in_cnt, uint32_t *out_cnt,
                              uint32_t in_sat, uint32_t out_sat, uint32_t *full,
                              hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    const int64_t nvox = (int64_t)g.nx * g.ny * g.nz, nw = (nvox + 31) / 32;
    // The first lines fill most voxels; every later stage reads which are
    // full from bits that do not change while it runs (256 KB at 256x256x32:
    // they stay in the caches, where the counters themselves are read past
    // them).  8M lines of 256x256x32: 5.7 ms, bound by instruction issue (two
    // thirds of the lanes idle in the average piece); 16.6 ms without stages and
    // with a midpoint per piece.
    const int64_t stage[3] = {std::min<int64_t>(n, std::max<int64_t>(n / 64, 65536)),
                              std::min<int64_t>(n, std::max<int64_t>(n / 8, 262144)), n};
    int64_t first = 0;
    for (int q = 0; q < 3; q++) {
        const int64_t end = stage[q];
        if (end <= first) continue;
        HullCounts c{in_cnt, out_cnt, nullptr, nullptr, in_sat, out_sat, true, true};
        if (first > 0) {
            hipLaunchKernelGGL(k_hull_full, dim3((unsigned)((nvox + kThreads - 1) / kThreads)),
                               dim3(kThreads), 0, stream, in_cnt, out_cnt, nvox, in_sat, out_sat,
                               full, nw);
            c.in_full = full;
            c.out_full = full + nw;
        }
        // A count is read before it is added to where most of the stage's lines
        // would find it at its value: (nx + ny) / voxels of them pass through a voxel,
        // about.  A read waits for the adds before it, so where these are many
        // plain adds are faster (never filled: 8M lines of 256x256x32 61 ms
        // against 98, 4M of 200x200 35 against 184; filled by the first line: 4M of
        // 200x200 2.5 ms a call with the read, 3.1 without; 60,000 of 64x64 filled
        // by four fifths of them 1.46 ms, 0.39 without).
        const double hits = 0.125 * (double)(end - first) * ((double)g.nx + g.ny) / (double)nvox;
        c.in_read = (double)in_sat < hits;
        c.out_read = (double)out_sat < hits;
        // Few lines wait for each voxel's count, so they read it a piece early
        // (20,000 lines: 64x64 117 us a call against 123, 200x200x16 270
        // against 311); with more of them a slice's counts are out of date by then
        // and needless adds cost more (60,000 of 64x64 198 against 195, 200,000
        // of 256x256 953 against 907).
        auto kernel = !(c.in_read && c.out_read) ? k_hull_counts<kByFlags>
                                                 : n <= kFewLines ? k_hull_counts<kEarly> : k_hull_counts<kRead>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)((end - first + kThreads - 1) / kThreads)),
                           dim3(kThreads), 0, stream, g, h, first, end, wepl_in, wepl_out, c);
        first = end;
    }
    return hipGetLastError();
}

hipError_t launch_hull_decide(const GridDev &g, const uint32_t *in_cnt, const uint32_t *out_cnt,
                              uint32_t min_in, uint32_t max_out, uint8_t *hull, double *mask,
                              hipStream_t stream)
{
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    int64_t wgs = (n + kThreads - 1) / kThreads;
    if (wgs > 4096) wgs = 4096;
    hipLaunchKernelGGL(k_hull_decide, dim3((unsigned)wgs), dim3(kThreads), 0, stream, g, in_cnt,
                       out_cnt, min_in, max_out, hull, mask);
    return hipGetLastError();
}

hipError_t launch_row_stats(const int32_t *nnz, int64_t n, uint32_t *stat, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    const int64_t wgs = std::min<int64_t>((n + kThreads - 1) / kThreads, 1024);
    hipLaunchKernelGGL(k_row_stats, dim3((unsigned)wgs), dim3(kThreads), 0, stream, nnz, n, stat);
    return hipGetLastError();
}

hipError_t launch_row_order(const int32_t *nnz, int64_t n, int64_t B, const uint32_t *stat,
                            int32_t *order, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    const int64_t nblocks = (n + B - 1) / B;
    const dim3 grid((unsigned)std::min<int64_t>(nblocks, 1 << 16));
    if (B < 1024)       // fewer classes to clear and add up
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_row_order<256, 256>), grid, dim3(256), 0, stream, nnz, n,
                           B, nblocks, stat, order);
    else
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_row_order<1024, 4096>), grid, dim3(1024), 0, stream, nnz,
                           n, B, nblocks, stat, order);
    return hipGetLastError();
}

hipError_t launch_pick(const int64_t *src, int64_t stride, int64_t n, int64_t *dst,
                       hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    int64_t wgs = (n + kThreads - 1) / kThreads;
    if (wgs > 1024) wgs = 1024;
    hipLaunchKernelGGL(k_pick, dim3((unsigned)wgs), dim3(kThreads), 0, stream, src, stride, n, dst);
    return hipGetLastError();
}

hipError_t launch_mlp_table(const MlpCfg &m, int64_t nj, double *tab, hipStream_t stream)
{
    if (nj <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_table, dim3((unsigned)((nj + kThreads - 1) / kThreads)), dim3(kThreads),
                       0, stream, m, nj, tab);
    return hipGetLastError();
}

hipError_t launch_scan(const int32_t *cnt, int64_t n, int64_t *off, int64_t *tmp,
                       hipStream_t stream)
{
    int64_t ntiles = (n + kScanTile - 1) / kScanTile;
    if (ntiles == 0) {
        hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(kThreads), 0, stream, tmp, (int64_t)0);
        hipLaunchKernelGGL(k_scan_write, dim3(1), dim3(kThreads), 0, stream, cnt, (int64_t)0, tmp,
                           (int64_t)0, off);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)ntiles), dim3(kThreads), 0, stream, cnt, n, tmp);
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(kThreads), 0, stream, tmp, ntiles);
    hipLaunchKernelGGL(k_scan_write, dim3((unsigned)ntiles), dim3(kThreads), 0, stream, cnt, n, tmp,
                       ntiles, off);
    return hipGetLastError();
}

}  // namespace tvs

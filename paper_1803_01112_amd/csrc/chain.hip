// chain.hip -- the DROP chain of a sweep as one resident kernel on gfx950.
//
// The tile-wise step of drop.hip runs as one launch per block: every launch
// pays the dispatch and drain of its workgroups, reads and writes the float64
// image of every crossed tile, reads each list twice and sends one
// memory-side atomic per row run; on a grid of few tiles it has only that
// many workgroups.  Here one workgroup per CU stays for
// many blocks and owns a region: consecutive dispatch slots, hence one
// contiguous range of every block's lists, whose image tiles stay in LDS.
// Per block b a workgroup
//   residuals  reads the finished dot products of block b - 1, once per row
//              that crosses its region: r = (wepl - dot) / ||a||^2;
//   finish     adds r a_ij of block b - 1's entries (kept in registers since
//              their dot products were formed) to the region's sums in LDS;
//   update     x += lambda c / s on the words with hits;
//   dots       forms block b's products from x in LDS.  A lane takes
//              consecutive entries, which mostly belong to one row, adds
//              them in a register and then into a small table of the rows
//              that cross the region; one memory-side atomic per (row,
//              region) instead of one per (row, tile, wavefront);
//   arrives at the device-wide barrier, and while it waits loads block
//   b + 1's entries, enters their rows in the next table and counts the hits
//   of block b.
// All numbers are those of drop.hip: the same integer sums of the same
// rounded values, so the images agree bit for bit.
//
// What crosses workgroups is only the dot products (memory-side atomics,
// read and cleared with agent-scope accesses, which bypass the XCDs' L2s) and
// the barrier's counters; the lists were written before the launch.  So no
// step needs a cache write-back or invalidation.  The barrier adds to one
// of 16 counters on lines of their own and polls all 16 with one load of a
// wavefront: 2.0 us for 256 workgroups, against 3.8 us with one counter.
//
// On a grid of fewer tiles than half the CUs the workgroups of a region
// split each list: they exchange their sums of a block through memory (a
// second, smaller barrier among them) and keep equal copies of the tile.
//
// A block is bound by latency, not by memory: 6.4 us at 200x200x16, float32
// store, B = 3200 (8.7 launched).  By lane 0's clock (whose reads add 0.35 us) 0.55
// residuals, 0.6 finish, 0.8 update, 0.9 dots, 0.8 flush and drain of the
// atomics, 2.4 preparing the next block and 0.65 more at the barrier.  Counters
// over such blocks: the waves wait on memory or a barrier 55 % of their time, the
// VALUs are busy 41 % of it, the LDS 31 % (18 % in bank conflicts); 5.3 MB move a
// block, 4.1 of them its lists and rows' data.  Other blocks of 3200: 5.8
// against 12.2 us at 128x128x8, 10.7 against 109 at 64x64.
//
// The launch is cooperative (all workgroups resident), and the library lets
// the chains of several contexts follow one another; every wait is bounded and
// ends the kernel with an error flag.
#include <algorithm>
#include <type_traits>

#include "device_common.hpp"
#include "tvs_internal.hpp"

namespace tvs {
namespace {

using dev::drain_memory;
using dev::round_scaled;

constexpr int kShards = kChainShards;
constexpr uint32_t kNone = 0xffffffffu;   // no entry; an empty table slot
// packed entry: word of the region | key << 13; the key is the table slot of
// the entry's row, or, with the top bit, the row itself (not in the table)
constexpr int kKeyShift = 13;
constexpr uint32_t kWordMask = (1u << kKeyShift) - 1u, kKeyMask = 0x3ffffu, kLoose = 0x80000000u;
constexpr int kProbes = 8;                // slots tried for a row
constexpr int kRing = 8;                  // blocks whose list starts are held
constexpr double kDotUnit = 1.0 / kDotScale;
constexpr double kCorrUnit = 1.0 / kCorrScale;
constexpr uint64_t kWaitTicks = 3000000000ull;   // 30 s of the 100 MHz clock

template <typename T>
__device__ inline T load_agent(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ inline void store_agent(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void add_ll(long long *p, long long v)
{
    atomicAdd(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}
// a / h, correctly rounded, from y = 1 / h rounded to nearest: the estimate
// corrected twice by its residual (Markstein's theorem; a finite, h < 256).
__device__ inline double div_count(double a, double h, double y)
{
    double q = a * y;
    q = fma(fma(-q, h, a), y, q);
    return fma(fma(-q, h, a), y, q);
}
// The same in LDS (workgroup scope: kept apart from adds to memory).
__device__ inline void lds_add(long long *p, long long v)
{
    __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline uint32_t lds_add(uint32_t *p, uint32_t v)
{
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

struct Lds {
    double *x;
    long long *cf;       // fixed-point corrections of the block being finished
    long long *tv;       // row table: dot sums, then (as float64) residuals
    double *inv;         // 1 / h, h < 256
    int64_t *lo;         // ring: the first entry of a block's list
    uint32_t *hits;
    uint32_t *tag;       // row table: rows of even blocks, then of odd blocks
    int *bnd;            // ring: the list's starts by tile of the region
    int *cut;            // ring: first and last entry of this workgroup's share of the list
    uint32_t *misc;      // [0] wait result, [1] a large correction was met, [2] one of its own,
                         // [3] the counters are not to be used, of even and odd blocks:
                         // [4], [5] rows in the table, [6], [7] words in hit
    uint16_t *used;      // slots taken in the tables of even and odd blocks
    uint16_t *hit;       // words with hits (one workgroup per region)
};

// One block's entries of this workgroup: [s0, s1) of the region's list.
struct Span {
    int64_t lo = 0;      // index of the region's first entry in meta / chords
    int s0 = 0, s1 = 0;
    uint32_t rows = 0;
    const int *bnd = nullptr;
};

// Entries as loaded (chords as their bits), and as used: the first n.
template <int E>
struct Raw {
    uint32_t m[E];
    uint32_t c[E];
};
template <int E>
struct Ents {
    uint32_t pk[E];
    float a[E];
    int n = 0;
};

// NT lanes, E consecutive entries of a block held by each.
template <int NT, int E, typename CH, bool SPLIT>
struct Chain {
    const ChainArgs &A;
    Lds L;
    const int t;
    int region, part, slot0, T, words;

    __device__ __forceinline__ Chain(const ChainArgs &a, char *lds) : A(a), t((int)threadIdx.x)
    {
        region = SPLIT ? (int)(blockIdx.x % (unsigned)A.nreg) : (int)blockIdx.x;
        part = SPLIT ? (int)(blockIdx.x / (unsigned)A.nreg) : 0;
        slot0 = A.reg[region];
        T = A.reg[region + 1] - slot0;
        words = T << kTileShift;
        const int W = A.tmax << kTileShift;
        L.x = reinterpret_cast<double *>(lds);
        L.cf = reinterpret_cast<long long *>(L.x + W);
        L.tv = L.cf + W;
        L.inv = reinterpret_cast<double *>(L.tv + A.ns);
        L.lo = reinterpret_cast<int64_t *>(L.inv + 256);
        L.hits = reinterpret_cast<uint32_t *>(L.lo + kRing);
        L.tag = L.hits + W;
        L.misc = L.tag + 2 * A.ns;
        L.bnd = reinterpret_cast<int *>(L.misc + 8);
        L.cut = L.bnd + kRing * (A.tmax + 1);
        L.used = reinterpret_cast<uint16_t *>(L.cut + kRing * 2);
        L.hit = L.used + 2 * A.ns;
    }

    __device__ __forceinline__ int *bounds(int64_t b) const { return L.bnd + (b & (kRing - 1)) * (A.tmax + 1); }
    __device__ __forceinline__ uint32_t *tags(int64_t b) const { return L.tag + (b & 1) * A.ns; }
    __device__ __forceinline__ uint16_t *used(int64_t b) const { return L.used + (b & 1) * A.ns; }
    __device__ __forceinline__ uint32_t *taken(int64_t b) const { return L.misc + 4 + (b & 1); }
    __device__ __forceinline__ static uint32_t key(uint32_t pk) { return (pk >> kKeyShift) & kKeyMask; }
    __device__ __forceinline__ static int word(uint32_t pk) { return (int)(pk & kWordMask); }
    __device__ __forceinline__ int64_t image_word(int w) const
    {
        return ((int64_t)A.act[slot0 + (w >> kTileShift)] << kTileShift) | (w & (kTileWords - 1));
    }

    // List starts of block b by lane (the first T + 1 of wavefront 0), and
    // their place in the ring.
    __device__ __forceinline__ int64_t request_bounds(int64_t b) const
    {
        return (b < A.b1 && t <= T) ? A.toff[b * A.nact + slot0 + t] : 0;
    }
    __device__ __forceinline__ void keep_bounds(int64_t b, int64_t off) const
    {
        if (t >= 64) return;
        const int64_t first = __shfl(off, 0, 64);
        const int n = (int)(off - first), last = __shfl(n, T, 64);
        const int k = (int)(b & (kRing - 1));
        if (b < A.b1 && t <= T) bounds(b)[t] = n;
        if (t == 0) {
            L.lo[k] = first - A.base;
            L.cut[2 * k] = SPLIT ? (int)((int64_t)last * part / A.parts) : 0;
            L.cut[2 * k + 1] = SPLIT ? (int)((int64_t)last * (part + 1) / A.parts) : last;
        }
    }

    __device__ __forceinline__ Span span(int64_t b) const
    {
        Span s;
        const int k = (int)(b & (kRing - 1));
        s.bnd = bounds(b);
        s.lo = L.lo[k];
        s.s0 = __builtin_amdgcn_readfirstlane(L.cut[2 * k]);
        s.s1 = __builtin_amdgcn_readfirstlane(L.cut[2 * k + 1]);
        const int64_t left = A.nh - b * A.B;
        s.rows = (uint32_t)(left < A.B ? left : A.B);
        return s;
    }
    __device__ __forceinline__ static int rounds(const Span &s)
    {
        return (int)((uint32_t)(s.s1 - s.s0 + NT * E - 1) / (uint32_t)(NT * E));
    }
    // Entries a lane takes of round r, and the first of them: consecutive
    // ones (they mostly belong to one row), an even share for every lane.
    __device__ __forceinline__ static int share(const Span &s, int r)
    {
        const int n = s.s1 - s.s0 - r * (NT * E);
        return n >= NT * E ? E : (int)((uint32_t)(n + NT - 1) / (uint32_t)NT);
    }
    __device__ __forceinline__ int first(const Span &s, int r) const { return s.s0 + r * (NT * E) + t * share(s, r); }

    // Entries of this lane in round r (FULL: every lane has E).
    template <bool FULL>
    __device__ __forceinline__ int count(const Span &s, int r) const
    {
        if (FULL) return E;
        return max(0, min(share(s, r), s.s1 - first(s, r)));
    }

    // Requests this lane's entries of round r.
    template <bool FULL>
    __device__ __forceinline__ void request(const Span &s, int r, Raw<E> &raw) const
    {
        const int n = count<FULL>(s, r);
        const int64_t at = s.lo + (FULL ? s.s0 + r * (NT * E) + t * E : first(s, r));
        const uint32_t *m = A.meta + at;
        const CH *c = chords() + at;
        if (FULL) {
            CH ch[E];
            __builtin_memcpy(raw.m, m, sizeof(raw.m));
            __builtin_memcpy(ch, c, sizeof(ch));
#pragma unroll
            for (int i = 0; i < E; i++) raw.c[i] = bits(ch[i]);
            return;
        }
        if (n == 0) return;
        const int per = share(s, r);
#pragma unroll
        for (int i = 0; i < E; i++) {
            if (i >= per) break;
            raw.m[i] = m[min(i, n - 1)];
            raw.c[i] = bits(c[min(i, n - 1)]);
        }
    }
    __device__ __forceinline__ const CH *chords() const
    {
        if constexpr (std::is_same<CH, uint16_t>::value) return A.chq;
        else if constexpr (std::is_same<CH, __half>::value) return A.ch16;
        else return A.ch32;
    }
    __device__ __forceinline__ static uint32_t bits(float c) { return __float_as_uint(c); }
    __device__ __forceinline__ static uint32_t bits(__half c) { return __half_as_ushort(c); }
    __device__ __forceinline__ static uint32_t bits(uint16_t c) { return c; }

    // The chord as dev::entry_chord reads it.
    __device__ __forceinline__ float chord(uint32_t m, uint32_t c) const
    {
        if constexpr (std::is_same<CH, uint16_t>::value)
            return (float)((double)(((m >> A.qshift) << 16) | c) * A.qunit);
        else if constexpr (std::is_same<CH, __half>::value)
            return __half2float(__ushort_as_half((unsigned short)c));
        else
            return __uint_as_float(c);
    }

    // The entries requested as round r of block b: words of the region, and
    // their rows entered in the block's table (ENTER) or looked up there: a
    // row takes the first free slot from its own on, and one that finds none
    // goes to memory entry by entry.
    template <bool FULL, bool ENTER>
    __device__ __forceinline__ void take(int64_t b, const Span &s, int r, const Raw<E> &raw, Ents<E> &o) const
    {
        const int n = o.n = count<FULL>(s, r);
        const int per = FULL ? E : share(s, r), e0 = FULL ? s.s0 + r * (NT * E) + t * E : first(s, r);
        uint32_t k[E];                         // first word of the entry's tile
#pragma unroll
        for (int i = 0; i < E; i++) k[i] = 0u;
        if (!SPLIT) {
            // lane j holds the start of tile j + 1 of the list; the
            // wavefront's entries cross the starts j0 .. j1 - 1 of them
            const int lane = t & 63, w0 = __builtin_amdgcn_readfirstlane(e0);
            const int mine = lane < T ? s.bnd[lane + 1] : 0x7fffffff;
            const int j0 = __popcll(__ballot(mine <= w0));
            const int j1 = __popcll(__ballot(mine < w0 + 64 * per));
#pragma unroll
            for (int i = 0; i < E; i++) k[i] = (uint32_t)j0 << kTileShift;
            for (int j = j0; j < j1; j++) {
                const int start = __builtin_amdgcn_readlane(mine, j) - e0;
#pragma unroll
                for (int i = 0; i < E; i++) k[i] += i >= start ? kTileWords : 0;
            }
        }
        uint32_t *tag = tags(b);
        uint32_t q[E], old[E], sl[E];
        uint32_t top = 0u;
#pragma unroll
        for (int i = 0; i < E; i++) {
            q[i] = (raw.m[i] >> kTileShift) & A.rowmask;
            if (FULL || i < n) top = max(top, q[i]);
        }
        if (top >= s.rows) {
            // names no row of the block: raises the flag and counts for row 0
            atomicOr(A.err, 2u);
#pragma unroll
            for (int i = 0; i < E; i++)
                if (q[i] >= s.rows) q[i] = 0u;
        }
#pragma unroll
        for (int i = 0; i < E; i++) {
            sl[i] = q[i] & (A.ns - 1u);
            old[i] = q[i];
            if (FULL || i < n) old[i] = ENTER ? atomicCAS(tag + sl[i], kNone, q[i]) : tag[sl[i]];
        }
#pragma unroll
        for (int i = 0; i < E; i++) {
            if (old[i] != q[i]) {
                // new in the table, or another row's slot: the next ones
                for (int p = 1; !(ENTER && old[i] == kNone) && old[i] != q[i] && p < kProbes; p++) {
                    sl[i] = (sl[i] + 1u) & (A.ns - 1u);
                    old[i] = ENTER ? atomicCAS(tag + sl[i], kNone, q[i]) : tag[sl[i]];
                }
                if (ENTER && old[i] == kNone) {
                    used(b)[lds_add(taken(b), 1u)] = (uint16_t)sl[i];
                    old[i] = q[i];
                }
            }
            const uint32_t kk = old[i] == q[i] ? sl[i] << kKeyShift : kLoose | (q[i] << kKeyShift);
            o.pk[i] = k[i] | (raw.m[i] & (kTileWords - 1)) | kk;
            o.a[i] = chord(raw.m[i], raw.c[i]);
            if (!FULL && i >= n) {
                o.pk[i] = 0u;
                o.a[i] = 0.0f;
            }
        }
    }

    // Counts the hits; a word's first one enters it in the list of hit words.
    template <bool FULL>
    __device__ __forceinline__ void count_hits(int64_t b, const Ents<E> &en) const
    {
        if (SPLIT) {
#pragma unroll
            for (int i = 0; i < E; i++)
                if (FULL || i < en.n) lds_add(L.hits + word(en.pk[i]), 1u);
            return;
        }
        uint32_t was[E];
#pragma unroll
        for (int i = 0; i < E; i++) {
            was[i] = 1u;
            if (FULL || i < en.n) was[i] = lds_add(L.hits + word(en.pk[i]), 1u);
        }
        uint64_t fresh[E];
        int n = 0;
#pragma unroll
        for (int i = 0; i < E; i++) {
            fresh[i] = __ballot(was[i] == 0u);
            n += __popcll(fresh[i]);
        }
        if (!n) return;
        const int lane = t & 63;
        uint32_t at = 0u;
        if (lane == 0) at = lds_add(L.misc + 6 + (b & 1), (uint32_t)n);
        at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int i = 0; i < E; i++) {
            if (was[i] == 0u)
                L.hit[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(fresh[i] >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)fresh[i], 0u))] =
                    (uint16_t)word(en.pk[i]);
            at += (uint32_t)__popcll(fresh[i]);
        }
    }

    __device__ __forceinline__ void emit(long long *dot, uint32_t pk, long long f) const
    {
        if (pk & kLoose) add_ll(dot + key(pk), f);
        else lds_add(L.tv + key(pk), f);
    }

    // Dot products of these entries with the region's image.
    template <bool FULL>
    __device__ __forceinline__ void dots(long long *dot, const Ents<E> &en) const
    {
        double p[E];
        long long f[E];
        bool rare = false;
#pragma unroll
        for (int i = 0; i < E; i++) p[i] = (double)en.a[i] * L.x[word(en.pk[i])];
#pragma unroll
        for (int i = 0; i < E; i++) {
            f[i] = round_scaled(p[i], kDotScale);
            rare |= !(fabs(p[i]) <= A.dot_small);
        }
        if (rare) {
#pragma unroll
            for (int i = 0; i < E; i++) {
                if (fabs(p[i]) <= A.dot_max) {
                    f[i] = __double2ll_rn(p[i] * kDotScale);
                } else {
                    f[i] = 0;
                    if (FULL || i < en.n) atomicOr(A.err, 1u);
                }
            }
        }
        // a lane's entries of one row are added up before they leave
        bool same[E];
#pragma unroll
        for (int i = E - 1; i >= 1; i--) {
            same[i] = (!FULL && i >= en.n) || (en.pk[i] >> kKeyShift) == (en.pk[i - 1] >> kKeyShift);
            f[i - 1] += same[i] ? f[i] : 0ll;
        }
        same[0] = !FULL && en.n == 0;
#pragma unroll
        for (int i = 0; i < E; i++)
            if (!same[i]) emit(dot, en.pk[i], f[i]);
    }

    // Corrections of these entries of block b into the region's sums; dot:
    // the block's dot products.
    template <bool FULL>
    __device__ __forceinline__ void finish(int64_t b, const long long *dot, const Ents<E> &en, double *cb) const
    {
        double v[E];
        uint32_t loose = 0u;
        bool rare = false;
#pragma unroll
        for (int i = 0; i < E; i++) v[i] = __longlong_as_double(L.tv[key(en.pk[i]) & (A.ns - 1u)]);
#pragma unroll
        for (int i = 0; i < E; i++) {
            v[i] = v[i] * (double)en.a[i];
            if (FULL || i < en.n) {
                rare |= !(fabs(v[i]) <= A.corr_small);
                loose |= en.pk[i];
            }
        }
        if (!(rare || (loose & kLoose))) {
#pragma unroll
            for (int i = 0; i < E; i++)
                if (FULL || i < en.n) lds_add(L.cf + word(en.pk[i]), round_scaled(v[i], kCorrScale));
            return;
        }
#pragma unroll 1
        for (int i = 0; i < E; i++) {
            uint32_t pk = 0u;
            float a = 0.0f;
            double vi = 0.0;
#pragma unroll
            for (int k = 0; k < E; k++)
                if (k == i) {
                    pk = en.pk[k];
                    a = en.a[k];
                    vi = v[k];
                }
            if (!FULL && i >= en.n) continue;
            if (pk & kLoose) {
                const uint32_t q = key(pk);
                const int64_t h = b * A.B + q;
                vi = ((double)A.wepl[h] - (double)load_agent(dot + q) * kDotUnit) /
                     (double)A.n2[h] * (double)a;
            }
            const int w = word(pk);
            if (fabs(vi) <= A.big) {
                lds_add(L.cf + w, __double2ll_rn(vi * kCorrScale));
            } else {
                L.misc[1] = 1u;
                unsafeAtomicAdd(cb + (SPLIT ? w : image_word(w)), vi);
                drain_memory();
            }
        }
    }

    // Rounds 1 .. n - 1 of block b's list (those past the entries the lanes
    // hold), the next one's entries requested before one is used: finishing
    // the block, or its dot products and hits.
    template <bool FINISH>
    __device__ __forceinline__ void more_rounds(int64_t b, const Span &s, int n, long long *dot, double *cb) const
    {
        Raw<E> next;
        if (n > 2) request<true>(s, 1, next);
        for (int r = 1; r < n - 1; r++) {
            const Raw<E> raw = next;
            if (r + 1 < n - 1) request<true>(s, r + 1, next);
            else request<false>(s, r + 1, next);
            Ents<E> X;
            take<true, !FINISH>(b, s, r, raw, X);
            if (FINISH) {
                finish<true>(b, dot, X, cb);
            } else {
                count_hits<true>(b, X);
                dots<true>(dot, X);
            }
        }
        if (n == 2) request<false>(s, 1, next);
        Ents<E> X;
        take<false, !FINISH>(b, s, n - 1, next, X);
        if (FINISH) {
            finish<false>(b, dot, X, cb);
        } else {
            count_hits<false>(b, X);
            dots<false>(dot, X);
        }
    }

    // Exchange record of a workgroup: sums and hits (top bit: the block met
    // large corrections) of even and odd blocks, and their float64 sums.
    struct Exch {
        long long cf[2][kTileWords];
        double cb[kTileWords];
        uint32_t hits[2][kTileWords];
    };
    static_assert(sizeof(Exch) == kChainExchBytes, "exchange record size");
    __device__ __forceinline__ Exch *exch(int p) const
    {
        return reinterpret_cast<Exch *>(A.exch) + ((int64_t)region * A.parts + p);
    }

    __device__ __forceinline__ void arrive(uint32_t *counter) const
    {
        drain_memory();
        __syncthreads();
        if (t == 0)
            __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // Waits until n arrivals have been counted: by the 16 counters of all
    // workgroups `epoch` times (SUB false), or by a region's counter; false on
    // time-out.
    template <bool SUB>
    __device__ __forceinline__ bool wait(uint32_t epoch) const
    {
        if (t < 64) {
            const uint32_t n = (gridDim.x + kShards - 1u - (uint32_t)(t & (kShards - 1))) / kShards;
            const uint32_t want = epoch * (SUB ? (uint32_t)A.parts : n);
            const uint32_t *c = SUB ? A.sub + region * 32 : A.bar + (t & (kShards - 1)) * 32;
            const bool mine = SUB || t < kShards;
            uint32_t ok = 1u;
            const uint64_t t0 = wall_clock64();
            for (;;) {
                if (__all(!mine || (int32_t)(load_agent(c) - want) >= 0)) break;
                if (wall_clock64() - t0 > kWaitTicks) {
                    ok = 0u;
                    break;
                }
            }
            if (t == 0) L.misc[0] = ok;
        }
        __syncthreads();
        const bool ok = L.misc[0] != 0u;
        if (!ok && t == 0) {
            atomicOr(A.err, 4u);
            store_agent(A.dead, 1u);
        }
        return ok;
    }

    __device__ __forceinline__ void run()
    {
        __builtin_amdgcn_s_setprio(3);
        double *cb = SPLIT ? exch(part)->cb : A.cb;
        uint32_t *shard = A.bar + (blockIdx.x & (kShards - 1u)) * 32;
        uint32_t epoch = A.epoch, sub = A.sub_epoch;
        for (int w = t; w < words; w += NT) {
            L.x[w] = A.x[image_word(w)];
            L.cf[w] = 0;
            L.hits[w] = 0u;
            store_agent(cb + (SPLIT ? w : image_word(w)), 0.0);
        }
        for (uint32_t s = t; s < A.ns; s += NT) {
            L.tv[s] = 0;
            L.tag[s] = L.tag[A.ns + s] = kNone;
        }
        if (t < 8 && t != 3) L.misc[t] = 0u;
        // after a time-out the counters no longer match the launches queued
        // behind it: those leave at once, whatever became of the error flag
        if (t == 3) L.misc[3] = load_agent(A.dead);
        if (t < 256) L.inv[t] = 1.0 / (double)t;
        // dot products of blocks b - 1, b and b + 1 (three buffers in turn)
        long long *d0 = A.dot + ((A.b0 + 2) % 3) * A.B, *d1 = A.dot + (A.b0 % 3) * A.B,
                  *d2 = A.dot + ((A.b0 + 1) % 3) * A.B;
        for (int64_t b = A.b0; b < A.b0 + 3; b++) keep_bounds(b, request_bounds(b));
        int64_t off = request_bounds(A.b0 + 3);
        clear_dots(d1);
        __syncthreads();
        if (L.misc[3]) {
            if (t == 0) atomicOr(A.err, 4u);
            return;
        }
        Raw<E> raw;
        Ents<E> C, P;
        request<false>(span(A.b0), 0, raw);
        take<false, true>(A.b0, span(A.b0), 0, raw, C);
        if (A.b0 + 1 < A.b1) request<false>(span(A.b0 + 1), 0, raw);
        float rw = 0.0f, rn = 1.0f;      // WEPL and ||a||^2 of this lane's row of the table
        int rslot = -1;
        uint32_t rrow = 0u;
        arrive(shard);
        if (!wait<false>(++epoch)) return;
        for (int64_t b = A.b0;; b++) {
            const bool has_c = b < A.b1;
            if (b > A.b0) {
                // residuals of block b - 1's rows
                const long long *dot = d0;
                if (rslot >= 0) {
                    const double d = (double)load_agent(dot + rrow) * kDotUnit;
                    L.tv[rslot] = __double_as_longlong(((double)rw - d) / (double)rn);
                }
                for (uint32_t u = t + NT; u < *taken(b - 1); u += NT) {
                    const int s = used(b - 1)[u];
                    const uint32_t q = tags(b - 1)[s];
                    const int64_t h = (b - 1) * A.B + q;
                    const double d = (double)load_agent(dot + q) * kDotUnit;
                    L.tv[s] = __double_as_longlong(((double)A.wepl[h] - d) / (double)A.n2[h]);
                }
                if (SPLIT && L.misc[2]) {      // everyone has read the last block's float64 sums
                    for (int w = t; w < kTileWords; w += NT) store_agent(cb + w, 0.0);
                    drain_memory();
                }
                __syncthreads();
                finish<false>(b - 1, dot, P, cb);
                const Span S = span(b - 1);
                if (const int n = rounds(S); n > 1) more_rounds<true>(b - 1, S, n, d0, cb);
                __syncthreads();
                if (SPLIT) {
                    sub++;
                    if (!exchange(b, sub)) return;
                }
                update(b - 1, b, cb);
            }
            if (!has_c) break;
            long long *dot = d1;
            clear_dots(d2);
            dots<false>(dot, C);
            const Span S = span(b);
            if (const int n = rounds(S); n > 1) more_rounds<false>(b, S, n, dot, cb);
            __syncthreads();
            // the table's sums to memory, one atomic per row of the region
            rslot = -1;
            for (uint32_t u = t; u < *taken(b); u += NT) {
                const int s = used(b)[u];
                const uint32_t q = tags(b)[s];
                add_ll(dot + q, L.tv[s]);
                if (u < NT) {
                    rslot = s;
                    rrow = q;
                    rw = A.wepl[b * A.B + q];
                    rn = A.n2[b * A.B + q];
                }
            }
            arrive(shard);
            // while the others arrive
            count_hits<false>(b, C);
            P = C;
            C.n = 0;
            keep_bounds(b + 3, off);
            off = request_bounds(b + 4);
            if (b + 1 < A.b1) take<false, true>(b + 1, span(b + 1), 0, raw, C);
            if (b + 2 < A.b1) request<false>(span(b + 2), 0, raw);
            if (!wait<false>(++epoch)) return;
            dot = d0;
            d0 = d1;
            d1 = d2;
            d2 = dot;
        }
        if (part == 0)
            for (int w = t; w < words; w += NT) A.x[image_word(w)] = L.x[w];
    }

    __device__ __forceinline__ void clear_dots(long long *dot) const
    {
        for (int64_t q = (int64_t)blockIdx.x * NT + t; q < A.B; q += (int64_t)gridDim.x * NT)
            store_agent(dot + q, 0ll);
    }

    // Sums of the region's workgroups: every one writes its own, then adds
    // all of them (integers: in any order).
    __device__ __forceinline__ bool exchange(int64_t b, uint32_t sub) const
    {
        constexpr int kGroups = NT / kTileWords, kAhead = 8;
        const int par = (int)(b & 1), w = t & (kTileWords - 1), g = t >> kTileShift;
        Exch *me = exch(part);
        const uint32_t large = L.misc[1] ? 0x80000000u : 0u;
        if (g == 0) store_agent(&me->cf[par][w], L.cf[w]);
        else if (g == 1) store_agent(&me->hits[par][w], L.hits[w] | large);
        if (t == 0) L.misc[2] = large;
        uint32_t *counter = A.sub + region * 32;
        arrive(counter);
        if (g == 0) {
            L.cf[w] = 0;
            L.hits[w] = 0u;
        }
        if (!wait<true>(sub)) return false;
        long long c = 0;
        uint32_t h = 0u;
        bool any = false;
        for (int p0 = g; p0 < A.parts; p0 += kGroups * kAhead) {
            long long cp[kAhead];
            uint32_t hp[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; i++) {
                const int p = p0 + i * kGroups;
                cp[i] = 0;
                hp[i] = 0u;
                if (p < A.parts) {
                    cp[i] = load_agent(&exch(p)->cf[par][w]);
                    hp[i] = load_agent(&exch(p)->hits[par][w]);
                }
            }
#pragma unroll
            for (int i = 0; i < kAhead; i++) {
                c += cp[i];
                h += hp[i] & 0x7fffffffu;
                any |= (hp[i] >> 31) != 0u;
            }
        }
        lds_add(L.cf + w, c);
        lds_add(L.hits + w, h);
        if (any) L.misc[1] = 1u;
        __syncthreads();
        return true;
    }

    // x += lambda c / s of a word; clears its sums.
    __device__ __forceinline__ void update_word(int64_t now, double *cb, int w, uint32_t h, long long f,
                                                double x, bool large) const
    {
        double c = (double)f * kCorrUnit, d;
        if (large) c += large_sum(now, cb, w);
        if (h < 256u && !large) d = div_count(A.lambda * c, (double)h, L.inv[h]);
        else d = A.lambda * c / (double)h;
        L.x[w] = x + d;
        L.cf[w] = 0;
        L.hits[w] = 0u;
    }

    // Updates the words with hits, two a lane at once; clears the sums, block
    // b's table and its rows.
    __device__ __forceinline__ void update(int64_t b, int64_t now, double *cb) const
    {
        const bool large = L.misc[1] != 0u;
        if (SPLIT) {
            const int w = t;
            if (w < kTileWords && L.hits[w]) update_word(now, cb, w, L.hits[w], L.cf[w], L.x[w], large);
        } else {
            const int n = (int)L.misc[6 + (b & 1)];
            for (int u = t; u < n; u += 2 * NT) {
                const bool two = u + NT < n;
                const int w0 = L.hit[u], w1 = L.hit[two ? u + NT : u];
                const uint32_t h0 = L.hits[w0], h1 = L.hits[w1];
                const long long f0 = L.cf[w0], f1 = L.cf[w1];
                const double x0 = L.x[w0], x1 = L.x[w1];
                update_word(now, cb, w0, h0, f0, x0, large);
                if (two) update_word(now, cb, w1, h1, f1, x1, large);
            }
        }
        for (uint32_t u = t; u < *taken(b); u += NT) {
            const int s = used(b)[u];
            L.tv[s] = 0;
            tags(b)[s] = kNone;
        }
        __syncthreads();
        if (t == 0) {
            L.misc[1] = L.misc[6 + (b & 1)] = 0u;
            *taken(b) = 0u;
        }
    }

    __device__ __forceinline__ double large_sum(int64_t now, double *cb, int w) const
    {
        if (!SPLIT) {
            double *p = cb + image_word(w);
            const double v = load_agent(p);
            if (v != 0.0) store_agent(p, 0.0);
            return v;
        }
        double v = 0.0;
        for (int p = 0; p < A.parts; p++)
            if (load_agent(&exch(p)->hits[now & 1][w]) >> 31) v += load_agent(&exch(p)->cb[w]);
        return v;
    }
};

template <int NT, int E, typename CH, bool SPLIT>
__global__ void __launch_bounds__(NT) k_chain(ChainArgs A)
{
    extern __shared__ __align__(16) char chain_lds[];
    Chain<NT, E, CH, SPLIT> c(A, chain_lds);
    c.run();
}

// A region of its own takes 1,024 lanes of 4 entries: 7.2 us a block against 7.4
// to 7.8 with 512 lanes of 6 (200x200x16, float32 store), 11.3 against 11.7 ms a
// cycle of 2 M rows on the fly.  A shared region is divided so that each of its
// workgroups has about two entries a lane of 512 (plan_chain).
template <typename CH>
const void *chain_kernel(bool split)
{
    return split ? (const void *)k_chain<kChainSplitThreads, 6, CH, true> : (const void *)k_chain<1024, 4, CH, false>;
}

}  // namespace

size_t chain_lds_bytes(int tmax, int ns)
{
    return (size_t)tmax * kTileWords * 22 + (size_t)ns * 20 + 2048 + (size_t)kRing * 16 + 32 +
           (size_t)kRing * 4 * (tmax + 1) + 16;
}

hipError_t launch_chain(const ChainArgs &a, hipStream_t stream)
{
    const bool split = a.parts > 1;
    const void *k = a.chq ? chain_kernel<uint16_t>(split)
                          : a.ch16 ? chain_kernel<__half>(split) : chain_kernel<float>(split);
    const size_t lds = chain_lds_bytes(a.tmax, (int)a.ns);
    hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ChainArgs arg = a;
    arg.dot_small = std::min(a.dot_max, 16384.0);      // |a x| 2^36 below 2^51
    arg.corr_small = std::min(a.big, 1024.0);          // |r a| 2^40 below 2^51
    void *args[] = {&arg};
    return hipLaunchCooperativeKernel(k, dim3((unsigned)(a.nreg * a.parts)),
                                      dim3(split ? kChainSplitThreads : 1024), args, (unsigned)lds, stream);
}

}  // namespace tvs

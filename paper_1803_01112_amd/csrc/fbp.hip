// fbp.hip -- initial iterate on gfx950: filtered backprojection (FBP) of the
// binned histories and an in-slice median filter.
//
// The paper starts every reconstruction from an initial iterate to which a
// median filter of radius 2 has been applied (arXiv 1803.01112, Section
// V-A); it cites, and does not spell out, how that iterate is formed.
// Reading: textbook parallel-beam FBP.
//   binning      each history's straight line from entry to exit, at its
//                crossing of the depth u = 0 (the rotation axis): angle bin
//                round(phi / (2 pi / A)) mod A of the beam direction, lateral
//                bin of t in width tau (nt bins centred on t = 0), slice of
//                the height; a bin's projection is the mean WEPL of its
//                histories (0 when empty), the sums taken as 64-bit integers
//                in units of 2^-32 mm so that they do not depend on order;
//   filter       discrete Ram-Lak kernel h(0) = 1/(4 tau^2),
//                h(n odd) = -1/(n^2 pi^2 tau^2), h(n even) = 0, times tau;
//   backproject  linear interpolation, weight pi / A (A angles over 360
//                degrees see each line twice);
//   median       lower median of the (2r+1)^2 window clipped to the slice.
// Every step is one lane per output with a fixed order of summation, so
// the float64 results follow the written operations exactly.
#include "tvs_internal.hpp"

namespace tvs {
namespace {

constexpr int kThreads = 256;
constexpr int kBinThreads = 1024;
constexpr int kFiltThreads = 1024;
constexpr int32_t kFiltBins = 2816;       // rows staged in 64 KB of the LDS
constexpr int64_t kBinCells = 12288;      // 144 KB of the LDS
constexpr double kPi = 3.14159265358979323846;
constexpr double kFixed = 4294967296.0;   // 2^32

// The bin of a history's straight line: angle a and cell (slice, lateral bin).
__device__ inline bool bin_of(const GridDev &g, const HistDev &H, int64_t i, int32_t A, double tau,
                              int32_t nt, int32_t &a, int64_t &cell)
{
    const double ex = H.s(kEx)[i], ey = H.s(kEy)[i], ez = H.s(kEz)[i];
    const double qx = H.s(kQx)[i], qy = H.s(kQy)[i], qz = H.s(kQz)[i];
    double ux = H.s(kUx)[i], uy = H.s(kUy)[i];
    const double nrm = sqrt(ux * ux + uy * uy);
    ux = ux / nrm;
    uy = uy / nrm;
    const double u0 = ex * ux + ey * uy, t0 = -ex * uy + ey * ux;
    const double u2 = qx * ux + qy * uy, t2 = -qx * uy + qy * ux;
    const double L = u2 - u0;
    if (!(L > 0.0)) return false;
    const double f = (0.0 - u0) / L;
    const double tc = t0 + (t2 - t0) * f;
    const double vc = ez + (qz - ez) * f;
    const double phi = atan2(uy, ux);
    const double da = 2.0 * kPi / (double)A;
    int64_t an = (int64_t)floor(phi / da + 0.5);
    an %= A;
    if (an < 0) an += A;
    const double mm = floor(tc / tau + 0.5 * (double)nt);
    if (!(mm >= 0.0 && mm < (double)nt)) return false;
    const double kk = floor((vc - g.oz) / g.vz);
    if (!(kk >= 0.0 && kk < (double)g.nz)) return false;
    a = (int32_t)an;
    cell = (int64_t)kk * nt + (int64_t)mm;
    return true;
}

// Adds (v, 1) to bin b of every lane with `on`.  Two lanes serve one bin, so
// that its two words, which share a 16-byte slot, leave as one request: the
// atomic units take one per cache line of an instruction, some 24 G/s, and two
// instructions (sum, then count) cost twice (8 M random bins: 638 against 341 us).
__device__ inline void add_pairs(unsigned long long *slots, int64_t b, long long v, bool on)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int h = 0; h < 64; h += 32) {
        const int src = h + (lane >> 1);
        const int64_t bb = __shfl(b, src, 64);
        const long long vv = __shfl(v, src, 64);
        if (__shfl((int)on, src, 64))
            __hip_atomic_fetch_add(slots + 2 * bb + (lane & 1),
                                   (lane & 1) ? 1ull : (unsigned long long)vv, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Each workgroup takes `per` consecutive histories.  With WIN it collects those
// of one angle (that of a history near its middle) in LDS, `cells` bins of that
// angle, and adds the touched ones to memory at the end, whole lines at a time;
// a scan taken angle by angle sends few others.
template <bool WIN>
__global__ void __launch_bounds__(kBinThreads)
k_fbp_bin(GridDev g, HistDev H, int64_t n, int64_t per, int32_t A, double tau, int32_t nt,
          int32_t cells, unsigned long long *slots)
{
    extern __shared__ unsigned long long win[];    // cells sums, then cells counts
    __shared__ int32_t angle;
    uint32_t *wcnt = reinterpret_cast<uint32_t *>(win + (WIN ? cells : 0));
    const int64_t c0 = (int64_t)blockIdx.x * per;
    const int64_t c1 = c0 + per < n ? c0 + per : n;
    const int tid = threadIdx.x;
    if (WIN) {
        for (int q = tid; q < cells; q += kBinThreads) {
            win[q] = 0;
            wcnt[q] = 0;
        }
        if (tid < 64) {
            int32_t a = -1;
            int64_t cell = 0;
            const int64_t i = c0 + (c1 - c0) * tid / 64;
            const unsigned long long ok = __ballot(bin_of(g, H, i, A, tau, nt, a, cell));
            const unsigned long long late = ok >> 32;
            const int pick = late ? 32 + __ffsll((long long)late) - 1
                                  : (ok ? __ffsll((long long)ok) - 1 : 0);
            a = __shfl(a, pick, 64);
            if (tid == 0) angle = ok ? a : -1;
        }
        __syncthreads();
    }
    const int32_t a0 = WIN ? angle : -1;
    for (int64_t base = c0; base < c1; base += kBinThreads) {
        const int64_t i = base + tid;
        int32_t a = -1;
        int64_t cell = 0;
        bool on = i < c1 && bin_of(g, H, i, A, tau, nt, a, cell);
        const long long v = on ? llrint((double)H.s(kWepl)[i] * kFixed) : 0;
        if (WIN && on && a == a0) {
            __hip_atomic_fetch_add(win + cell, (unsigned long long)v, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_fetch_add(wcnt + cell, 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            on = false;
        }
        if (__any(on)) add_pairs(slots, (int64_t)a * g.nz * nt + cell, v, on);
    }
    if (WIN) {
        __syncthreads();
        unsigned long long *dst = slots + 2 * (int64_t)a0 * cells;
        for (int q = tid; q < 2 * cells; q += kBinThreads) {
            const uint32_t c = wcnt[q >> 1];
            if (c)
                __hip_atomic_fetch_add(dst + q, (q & 1) ? (unsigned long long)c : win[q >> 1],
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

__global__ void __launch_bounds__(kThreads)
k_fbp_mean(const unsigned long long *slots, int64_t nb, double *p)
{
    const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (b >= nb) return;
    const unsigned long long cnt = slots[2 * b + 1];
    p[b] = cnt ? ((double)(long long)slots[2 * b] / kFixed) / (double)cnt : 0.0;
}

// hv[(d - 1) / 2] = h(d) for the odd d < nt
__global__ void __launch_bounds__(kThreads) k_fbp_taps(int32_t nt, double tau, double *hv)
{
    const int32_t q = (int32_t)(blockIdx.x * kThreads + threadIdx.x);
    const int32_t d = 2 * q + 1;
    if (d < nt) hv[q] = -1.0 / ((double)d * (double)d * kPi * kPi * tau * tau);
}

// q[r * nt + m] = tau * sum over s (ascending) of p[r * nt + s] h(m - s).
// The taps come from the table (their quotients were most of the 235 us that
// 2880 rows of 286 bins took).  Two 8-byte reads, a product and a sum per tap:
// the reads bound it, 125 us through the vector cache, 54 with STAGED, where
// a workgroup's rows and the taps are copied to the LDS first.
template <bool STAGED>
__global__ void __launch_bounds__(kFiltThreads)
k_fbp_filter(const double *p, const double *hv, int64_t rows, int32_t nt, double tau, double *q)
{
    extern __shared__ double stage[];
    const int64_t o0 = (int64_t)blockIdx.x * kFiltThreads;
    const int64_t o = o0 + threadIdx.x;
    int64_t r0 = 0;
    if (STAGED) {
        r0 = o0 / nt;
        int64_t r1 = (o0 + kFiltThreads - 1) / nt + 1;      // at most kFiltThreads + 2 nt words
        if (r1 > rows) r1 = rows;
        const int32_t words = (int32_t)(r1 - r0) * nt, taps = nt / 2;
        for (int32_t w = threadIdx.x; w < taps; w += kFiltThreads) stage[w] = hv[w];
        for (int32_t w = threadIdx.x; w < words; w += kFiltThreads) stage[taps + w] = p[r0 * nt + w];
        hv = stage;
        p = stage + taps;
        __syncthreads();
    }
    if (o >= rows * nt) return;
    const int64_t r = o / nt;
    const int32_t m = (int32_t)(o - r * nt);
    const double *pr = p + (r - r0) * nt;
    double acc = 0.0;
    // s = m - d, d = 2 j + 1, from the first s of that parity up to m - 1
    const int32_t first = (m + 1) / 2;      // odd d <= m
#pragma unroll 8
    for (int32_t j = first - 1; j >= 0; j--) acc += pr[m - 2 * j - 1] * hv[j];
    acc += pr[m] * (1.0 / (4.0 * tau * tau));
    const int32_t last = (nt - m) / 2;      // odd d <= nt - 1 - m
#pragma unroll 8
    for (int32_t j = 0; j < last; j++) acc += pr[m + 2 * j + 1] * hv[j];
    q[o] = tau * acc;
}

// t / tau, correctly rounded, from rtau = 1 / tau: the product, corrected twice
// by its residual (Markstein's theorem; no overflow or underflow in between).
__device__ inline double quot(double t, double tau, double rtau)
{
    double q = t * rtau;
    q = fma(fma(-q, tau, t), rtau, q);
    return fma(fma(-q, tau, t), rtau, q);
}

// x (x-fastest, float64) = pi / A * sum over angles of the interpolated
// filtered projection; cs[2a], cs[2a+1] = cos, sin of angle a (host table);
// rtau = 1 / tau, or 0 where quot does not apply.  Vector issue bounds it: with
// a full division and 64-bit indices per sample 640 k voxels x 180 angles took
// 204 us, 105 now.
__global__ void __launch_bounds__(kThreads)
k_fbp_backproject(GridDev g, const double *q, const double *cs, int32_t A, double tau, double rtau,
                  int32_t nt, int clip, double *x)
{
    const int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t nvox = (int64_t)g.nx * g.ny * g.nz;
    if (o >= nvox) return;
    const int64_t i = o % g.nx, j = (o / g.nx) % g.ny, k = o / ((int64_t)g.nx * g.ny);
    const double X = g.ox + ((double)i + 0.5) * g.vx;
    const double Y = g.oy + ((double)j + 0.5) * g.vy;
    const double half = 0.5 * (double)nt;
    const double *row = q + k * nt;
    const int64_t next = (int64_t)g.nz * nt;
    double acc = 0.0;
#pragma unroll 4
    for (int32_t a = 0; a < A; a++, row += next) {
        const double t = -X * cs[2 * a + 1] + Y * cs[2 * a];
        const double sp = (rtau != 0.0 ? quot(t, tau, rtau) : t / tau) + half - 0.5;
        const double m0 = floor(sp);
        const double w = sp - m0;
        // 0 <= m0 <= nt - 2: the bins reach a whole one past the grid's corners
        int32_t m = (int32_t)m0;
        m = m < 0 ? 0 : (m > nt - 2 ? nt - 2 : m);
        const double v0 = row[m], v1 = row[m + 1];
        acc += (1.0 - w) * v0 + w * v1;
    }
    double v = acc * (kPi / (double)A);
    if (clip && v < 0.0) v = 0.0;
    x[o] = v;
}

// Lower median of the (2R+1)^2 window clipped to the slice, by rank (unrolled,
// so the window stays in registers).  Each pair is compared once; what lies
// outside the slice, and NaN, ranks as +inf, and a window whose median would be
// one of these gives 0.  640 k voxels, radius 2: 66 us
// with two compares per ordered pair, 27 now.
template <int R>
__global__ void __launch_bounds__(kThreads)
k_median(GridDev g, const double *x, float *out)
{
    constexpr int W = 2 * R + 1;
    const int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t nvox = (int64_t)g.nx * g.ny * g.nz;
    if (o >= nvox) return;
    const int64_t i = o % g.nx, j = (o / g.nx) % g.ny, k = o / ((int64_t)g.nx * g.ny);
    double v[W * W];
    int rank[W * W];
    int n = 0, valid = 0;
#pragma unroll
    for (int dj = 0; dj < W; dj++)
#pragma unroll
        for (int di = 0; di < W; di++) {
            const int64_t ii = i + di - R, jj = j + dj - R;
            const bool ok = ii >= 0 && ii < g.nx && jj >= 0 && jj < g.ny;
            const double xv = ok ? x[ii + g.nx * (jj + g.ny * k)] : 0.0;
            const bool num = ok && xv == xv;
            v[dj * W + di] = num ? xv : __builtin_inf();
            rank[dj * W + di] = dj * W + di;      // as if all before it came first
            n += ok;
            valid += num;
        }
    const int want = (n - 1) / 2;      // rank of the lower median (0-based)
#pragma unroll
    for (int c = 0; c < W * W; c++)
#pragma unroll
        for (int d = c + 1; d < W * W; d++) {
            const int p = v[d] < v[c];
            rank[c] += p;
            rank[d] -= p;
        }
    double med = 0.0;
#pragma unroll
    for (int c = 0; c < W * W; c++)
        if (rank[c] == want && want < valid) med = v[c];
    out[o] = (float)med;
}

// cs[2a], cs[2a+1] = cos, sin of angle a * 2 pi / A, formed on the device
// (the allocation-free entry point takes no host table)
__global__ void __launch_bounds__(kThreads) k_fbp_angles(int32_t A, double *cs)
{
    const int32_t a = (int32_t)(blockIdx.x * kThreads + threadIdx.x);
    if (a >= A) return;
    const double phi = (double)a * (2.0 * kPi / (double)A);
    cs[2 * a] = cos(phi);
    cs[2 * a + 1] = sin(phi);
}

__global__ void __launch_bounds__(kThreads) k_narrow_abi(const double *x, int64_t n, float *out)
{
    const int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (o < n) out[o] = (float)x[o];
}

dim3 grid_for(int64_t n) { return dim3((unsigned)((n + kThreads - 1) / kThreads)); }

}  // namespace

hipError_t launch_fbp_bin(const GridDev &g, const HistDev &h, int64_t n, int32_t A, double tau,
                          int32_t nt, int32_t cus, unsigned long long *slots, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    // Two workgroups per CU share the histories when their bins of one angle fit
    // the LDS and each takes at least as many histories as it has bins to flush;
    // else one history per lane (8 M histories angle by angle, 4576
    // cells: 145 us against 411; 677 with the sum and the count in two requests)
    const int64_t cells = (int64_t)g.nz * nt;
    int64_t per = (n + 2 * cus - 1) / (2 * cus);
    per = (per + kBinThreads - 1) / kBinThreads * kBinThreads;
    if (cells <= kBinCells && per >= cells) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_fbp_bin<true>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)kBinCells * 12);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_fbp_bin<true>, dim3((unsigned)((n + per - 1) / per)),
                           dim3(kBinThreads), (size_t)cells * 12, stream, g, h, n, per, A, tau, nt,
                           (int32_t)cells, slots);
    } else {
        per = kBinThreads;
        hipLaunchKernelGGL(k_fbp_bin<false>, dim3((unsigned)((n + per - 1) / per)),
                           dim3(kBinThreads), 0, stream, g, h, n, per, A, tau, nt, 0, slots);
    }
    return hipGetLastError();
}

hipError_t launch_fbp_filter(unsigned long long *slots, int64_t rows, int32_t nt, double tau,
                             double *taps, double *p, hipStream_t stream)
{
    if (rows * nt <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fbp_mean, grid_for(rows * nt), dim3(kThreads), 0, stream,
                       (const unsigned long long *)slots, rows * nt, p);
    hipLaunchKernelGGL(k_fbp_taps, grid_for(nt / 2 + 1), dim3(kThreads), 0, stream, nt, tau, taps);
    double *q = reinterpret_cast<double *>(slots);
    const dim3 grid((unsigned)((rows * nt + kFiltThreads - 1) / kFiltThreads));
    if (nt <= kFiltBins)
        hipLaunchKernelGGL(k_fbp_filter<true>, grid, dim3(kFiltThreads),
                           sizeof(double) * (size_t)(kFiltThreads + 2 * nt + nt / 2), stream,
                           (const double *)p, (const double *)taps, rows, nt, tau, q);
    else
        hipLaunchKernelGGL(k_fbp_filter<false>, grid, dim3(kFiltThreads), 0, stream,
                           (const double *)p, (const double *)taps, rows, nt, tau, q);
    return hipGetLastError();
}

hipError_t launch_fbp_backproject(const GridDev &g, const double *q, const double *cs, int32_t A,
                                  double tau, int32_t nt, int clip, double *x, hipStream_t stream)
{
    const int64_t nvox = (int64_t)g.nx * g.ny * g.nz;
    const double rtau = tau > 1e-100 && tau < 1e100 ? 1.0 / tau : 0.0;
    hipLaunchKernelGGL(k_fbp_backproject, grid_for(nvox), dim3(kThreads), 0, stream, g, q, cs, A,
                       tau, rtau, nt, clip, x);
    return hipGetLastError();
}

hipError_t launch_fbp_angles(int32_t A, double *cs, hipStream_t stream)
{
    if (A <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fbp_angles, grid_for(A), dim3(kThreads), 0, stream, A, cs);
    return hipGetLastError();
}

hipError_t launch_median(const GridDev &g, const double *x, int radius, float *out,
                         hipStream_t stream)
{
    const int64_t nvox = (int64_t)g.nx * g.ny * g.nz;
    switch (radius) {
    case 0: hipLaunchKernelGGL(k_narrow_abi, grid_for(nvox), dim3(kThreads), 0, stream, x, nvox, out); break;
    case 1: hipLaunchKernelGGL(k_median<1>, grid_for(nvox), dim3(kThreads), 0, stream, g, x, out); break;
    case 2: hipLaunchKernelGGL(k_median<2>, grid_for(nvox), dim3(kThreads), 0, stream, g, x, out); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace tvs

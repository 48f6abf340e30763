// batch.hip -- S reconstructions of the same histories advanced together
// (a parameter study over (lambda, N, alpha) as in arXiv 1803.01112,
// Section III-E, run as one job instead of one reconstruction each).
//
// The S images are interleaved by voxel in planes of kPlane settings (the last
// plane as wide as is left): x[plane][p][s], so that the values an entry reads
// for one group of settings are a line of their own (interleaved over all S,
// a group's workgroup fetched the other groups' settings with every voxel:
// 322 of 380 MB a step at S = 24).  The DROP sweep is the tile-wise chain of
// drop.hip with S images at once: one workgroup per (tile, group of up to
// 16 settings) applies each entry of the tile's lists to the settings of its
// group through LDS; hit counts depend only on the rows.  The TV steps of every
// setting run in one kernel per step index n, with per-setting beta read
// from a device table indexed by a device cycle counter, so the launches of
// one cycle can be captured once in a hipGraph and replayed for every cycle.
#include "device_common.hpp"
#include "tvs_internal.hpp"

namespace tvs {
namespace {

constexpr int kThreads = 256;
constexpr int kPlane = 8;
using dev::entry_chord;
using dev::row_of;
using dev::kNoRow;

constexpr double kDotUnit = 1.0 / kDotScale;
constexpr double kCorrUnit = 1.0 / kCorrScale;

// Place of setting s of word 0, and the distance of its words.
struct Place {
    int64_t at;
    int step;
};
__host__ __device__ inline Place place(int64_t nvox, int S, int s)
{
    const int g = s / kPlane * kPlane;
    return Place{(int64_t)g * nvox + (s - g), S - g < kPlane ? S - g : kPlane};
}

// ------------------------------------------------------------- TV, S images
// Thread t of a workgroup handles setting s = t % S of voxel w*V + t / S.
__global__ void __launch_bounds__(kThreads)
k_tvb_grad(GridDev G, const double *x, int S, int V, uint32_t active, const double *eps,
           double *g, double *part)
{
    __shared__ double red[kThreads];
    const int t = threadIdx.x;
    const int v = t / S, s = t - v * S;
    const int64_t nx = G.nx, ny = G.ny;
    const int64_t nvox = padded_voxels(G);
    // a fixed grid strides over batches of V voxels (few partial sums)
    const Place at = place(nvox, S, s);
    x += at.at;
    g += at.at;
    double sq = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * V + v; v < V && p < nvox;
         p += (int64_t)gridDim.x * V) {     // tiled-layout word
        int64_t i = 0, j = 0, k = 0;
        vcoord(G, p, i, j, k);
        if (!(i < nx && j < ny && ((active >> s) & 1u))) continue;
        const double e2 = eps[s] * eps[s];
        auto X = [&](int32_t di, int32_t dj) {
            return x[(int64_t)vaddr32(G, (int32_t)i + di, (int32_t)j + dj, (int32_t)k) * at.step];
        };
        auto dxf = [&](int64_t ii, int64_t jj) {
            return (i + ii + 1 < nx) ? X(ii + 1, jj) - X(ii, jj) : 0.0;
        };
        auto dyf = [&](int64_t ii, int64_t jj) {
            return (j + jj + 1 < ny) ? X(ii, jj + 1) - X(ii, jj) : 0.0;
        };
        auto mf = [&](int64_t ii, int64_t jj) {
            double a = dxf(ii, jj), b = dyf(ii, jj);
            return sqrt(a * a + b * b + e2);
        };
        double gv = 0.0;
        double m = mf(0, 0);
        if (m > 0.0) gv -= (dxf(0, 0) + dyf(0, 0)) / m;
        if (i > 0) {
            double mm = mf(-1, 0);
            if (mm > 0.0) gv += dxf(-1, 0) / mm;
        }
        if (j > 0) {
            double mm = mf(0, -1);
            if (mm > 0.0) gv += dyf(0, -1) / mm;
        }
        g[p * at.step] = gv;
        sq += gv * gv;
    }
    red[t] = sq;
    __syncthreads();
    if (t < S) {
        double a = 0.0;
        for (int vv = 0; vv < V; vv++) a += red[vv * S + t];
        part[(int64_t)blockIdx.x * S + t] = a;
    }
}

// Squared norms from the partials, one workgroup per setting: thread v adds
// those of every V-th workgroup of the gradient, then the V sums in order.  A
// launch of its own: handing the partials over inside the gradient's launch
// made its workgroups write back the L2's dirty lines (300 us a gradient of 24
// settings of 200x200x16 against 206 and 7 for this launch; 248 with 64-bit
// voxel coordinates, 30 without the sums' loads in flight together).
__global__ void __launch_bounds__(kThreads)
k_tvb_norm(const double *part, uint32_t n, int S, int V, double *norm2)
{
    __shared__ double red[kThreads];
    const int v = threadIdx.x, s = blockIdx.x;
    double a = 0.0;
    if (v < V) {
        const double *p = part + (int64_t)v * S + s;
        const int terms = ((int)n - v + V - 1) / V, step = V * S;
#pragma unroll 16
        for (int q = 0; q < terms; q++) a += p[q * step];
    }
    red[v] = a;
    __syncthreads();
    if (v == 0) {
        double b = 0.0;
        for (int vv = 0; vv < V; vv++) b += red[vv];
        norm2[s] = b;
    }
}

// Setting and word of element q of an S-image buffer.
__device__ inline int64_t word_of(int64_t q, int S, int64_t nvox)
{
    const int g = (int)(q / (nvox * kPlane)) * kPlane;
    return (q - g * nvox) / (S - g < kPlane ? S - g : kPlane);
}
__device__ inline int setting_of(int64_t q, int S, int64_t nvox)
{
    const int g = (int)(q / (nvox * kPlane)) * kPlane;
    return g + (int)((q - g * nvox) % (S - g < kPlane ? S - g : kPlane));
}

// x += (-beta_s / ||g_s||) g for the active settings; beta of step n of the
// current cycle is beta_tab[(cyc * nmax + n) * S + s].
__global__ void __launch_bounds__(kThreads)
k_tvb_step(double *x, const double *g, int S, int64_t n_elems, uint32_t active,
           const double *beta_tab, const int32_t *cyc, int n, int nmax, const double *norm2)
{
    const int64_t base = ((int64_t)(*cyc) * nmax + n) * S;
    for (int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x; q < n_elems;
         q += (int64_t)gridDim.x * kThreads) {
        const int s = setting_of(q, S, n_elems / S);
        if (!((active >> s) & 1u)) continue;
        const double nn = norm2[s];
        const double sc = (nn > 0.0) ? -beta_tab[base + s] / sqrt(nn) : 0.0;
        if (sc != 0.0) x[q] = fma(sc, g[q], x[q]);
    }
}

__global__ void k_set_counter(int32_t *cyc, int32_t v)
{
    if (threadIdx.x == 0) *cyc = v;
}

__global__ void k_tick(int32_t *cyc)
{
    if (threadIdx.x == 0) *cyc += 1;
}

__global__ void __launch_bounds__(kThreads)
k_replicate(const double *x0, double *xb, int S, int64_t nvox)
{
    for (int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x; q < nvox * S;
         q += (int64_t)gridDim.x * kThreads)
        xb[q] = x0[word_of(q, S, nvox)];
}

__global__ void __launch_bounds__(kThreads)
k_extract(GridDev G, const double *xb, int S, int s, float *out)
{
    const int64_t n = (int64_t)G.nx * G.ny * G.nz;
    const Place at = place(padded_voxels(G), S, s);
    for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * kThreads) {
        const int64_t i = p % G.nx, t = p / G.nx, j = t % G.ny, k = t / G.ny;
        out[p] = (float)xb[at.at + vaddr(G, i, j, k) * at.step];
    }
}

unsigned elem_grid(int64_t n)
{
    int64_t wgs = (n + kThreads - 1) / kThreads;
    if (wgs > 4096) wgs = 4096;
    if (wgs < 1) wgs = 1;
    return (unsigned)wgs;
}

// ------------------------------------------------------------- DROP, S images
// Settings per pass through LDS (GP: 2, 4, 8 or 16) and threads per workgroup
// (NT: 128 or 256) are template parameters, picked by the batch autotuner.

// LDS index of (voxel word w, setting s of the group): the settings of a
// voxel are XOR-swizzled by w so that lanes holding different voxels and the
// same setting fall into different banks (without it every voxel's setting s
// shares one bank pair).
template <int GP>
__device__ inline int sx(int w, int s) { return w * GP + (s ^ (w & (GP - 1))); }

template <int NT, int GP>
struct BatchLds {
    double x[kTileWords * GP];
    long long cf[kTileWords * GP];   // fixed-point corrections (float64 once a large one was met)
    double inv[kTileWords];          // 1 / h
    uint32_t hits[kTileWords];
    uint32_t row[NT];                // rows of the run sums staged by each wavefront
    uint32_t large;
};

// One step of the tile-wise chain for S settings: finish block P and form
// the dot products of block C (dot arrays row-major: dot[q * S + s]).  The
// per-entry quotient a_ij / ||a_i||^2 and the per-voxel 1 / s_j are formed
// once and shared by the settings (a rounding apart from the single-image
// kernel, which divides per value).
//
// Bound by instruction issue (64 % of the cycles) and the memory-side atomics
// of the dot products.  24 settings of 200x200x16, B = 3200, float32 store:
// 72 us a step, 102.9 with all settings interleaved and the run sums
// formed by six shuffles of 64 bits through LDS.  A lane per setting over a
// whole run (the sum in a register, no scan) took 92: the lanes of a wavefront
// wait for the longest of its runs.
template <int NT, int GP, typename CH>
__global__ void __launch_bounds__(NT)
k_drop_tile_batch(DropTileArgs A, int S, int64_t nvox, const double *lambda)
{
    __shared__ BatchLds<NT, GP> L;
    const int t = threadIdx.x;
    if (A.zero)
        for (int64_t q = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * NT + t;
             q < A.B * S; q += (int64_t)gridDim.x * gridDim.y * NT)
            A.zero[q] = 0;
    // workgroup x takes dispatch slot x (or slots[x]): its lists' bounds at
    // [slot], its tile act[slot]
    const int64_t slot = A.slots ? A.slots[blockIdx.x] : (int64_t)blockIdx.x;
    const int64_t T = A.tiles[slot];
    int64_t p0 = 0, p1 = 0, c0 = 0, c1 = 0;
    if (A.P.valid) {
        p0 = A.P.toff[slot];
        p1 = A.P.toff[slot + 1];
    }
    if (A.C.valid) {
        c0 = A.C.toff[slot];
        c1 = A.C.toff[slot + 1];
    }
    if (p0 == p1 && c0 == c1) return;
    // one group of settings per workgroup (the grid's second dimension)
    const int g0 = (int)blockIdx.y * GP;
    const int G = (S - g0 < GP) ? S - g0 : GP;
    const int s = t & (GP - 1);              // this lane's setting where a lane takes one
    const Place at = place(nvox, S, g0 + (s < G ? s : 0));
    double *xt = A.x + at.at + (T << kTileShift) * at.step;
    // the first round of both lists and the finished rows' data
    uint32_t pm = 0u, cm = 0u;
    float pa = 0.0f, ca = 0.0f;
    double pw = 0.0, pn2 = 1.0;
    const bool pok = p0 + t < p1, cok = c0 + t < c1;
    if (pok) {
        pm = A.P.meta[p0 + t - A.P.base];
        pa = entry_chord<CH>(A.P, p0 + t - A.P.base, pm);
    }
    if (cok) {
        cm = A.C.meta[c0 + t - A.C.base];
        ca = entry_chord<CH>(A.C, c0 + t - A.C.base, cm);
    }
    if (pok && row_of(A.P, pm) < A.P.rows) {
        pw = (double)A.P.wepl[row_of(A.P, pm)];
        pn2 = (double)A.P.n2[row_of(A.P, pm)];
    }
    for (int w = t / GP; w < kTileWords; w += NT / GP)
        if (s < G) L.x[sx<GP>(w, s)] = xt[w * at.step];
    if (t == 0) L.large = 0u;
    if (p1 > p0) {
        for (int i = t; i < kTileWords * GP; i += NT) L.cf[i] = 0;
        for (int w = t; w < kTileWords; w += NT) L.hits[w] = 0u;
        __syncthreads();
        // pass 0: every correction within the fixed-point range; pass 1, after
        // one that is not: those in float64 on top of the sums
        const double small = A.big < 1024.0 ? A.big : 1024.0;
        auto finish = [&](int pass) {
            for (int64_t e = p0 + t; e < p1; e += NT) {
                const bool first = e == p0 + t;
                const uint32_t m = first ? pm : A.P.meta[e - A.P.base];
                const int w = (int)(m & (kTileWords - 1));
                const uint32_t q = row_of(A.P, m);
                if (q >= A.P.rows) {
                    atomicOr(A.err, 2u);
                    continue;
                }
                const double a = (double)(first ? pa : entry_chord<CH>(A.P, e - A.P.base, m));
                const double wp = first ? pw : (double)A.P.wepl[q];
                const double n2 = first ? pn2 : (double)A.P.n2[q];
                const long long *dot = A.P.dot + (int64_t)q * S + g0;
                const double an2 = a / n2;   // one division for all settings
                long long d[GP];
#pragma unroll
                for (int k = 0; k < GP; k++) d[k] = k < G ? dot[k] : 0;
                if (pass == 0) atomicAdd(&L.hits[w], 1u);
#pragma unroll
                for (int k = 0; k < GP; k++) {
                    if (k >= G) continue;
                    const double v = (wp - (double)d[k] * kDotUnit) * an2;
                    const bool in = fabs(v) <= A.big;
                    if (pass == 0 && in) {
                        const long long f = fabs(v) <= small ? dev::round_scaled(v, kCorrScale)
                                                             : __double2ll_rn(v * kCorrScale);
                        atomicAdd(reinterpret_cast<unsigned long long *>(&L.cf[sx<GP>(w, k)]),
                                  (unsigned long long)f);
                    } else if (pass == 0) {
                        L.large = 1u;
                    } else if (!in) {
                        atomicAdd(reinterpret_cast<double *>(&L.cf[sx<GP>(w, k)]), v);
                    }
                }
            }
        };
        finish(0);
        __syncthreads();
        const bool large = L.large != 0u;
        for (int w = t; w < kTileWords; w += NT)
            if (L.hits[w]) L.inv[w] = 1.0 / (double)L.hits[w];   // one division for all settings
        if (large) {
            for (int i = t; i < kTileWords * GP; i += NT)
                L.cf[i] = __double_as_longlong((double)L.cf[i] * kCorrUnit);
            __syncthreads();
            finish(1);
        }
        __syncthreads();
        if (s < G) {
            const double lam = lambda[g0 + s];
            for (int w = t / GP; w < kTileWords; w += NT / GP) {
                if (!L.hits[w]) continue;
                const int k = sx<GP>(w, s);
                const double c = large ? __longlong_as_double(L.cf[k]) : (double)L.cf[k] * kCorrUnit;
                const double nx = L.x[k] + lam * c * L.inv[w];
                L.x[k] = nx;
                xt[w * at.step] = nx;
            }
        }
    }
    const double dot_small = A.dot_max < 16384.0 ? A.dot_max : 16384.0;
    auto rounded = [&](double p) -> long long {
        if (fabs(p) <= dot_small) return dev::round_scaled(p, kDotScale);
        if (fabs(p) <= A.dot_max) return __double2ll_rn(p * kDotScale);
        atomicOr(A.err, 1u);
        return 0;
    };
    __syncthreads();
    // An entry per lane; the run sums of the group's settings are staged in
    // the finish sums' space, free by now, and leave as atomics of GP settings
    // of one row each: one line per run instead of GP.
    const int wave = t >> 6, lane = t & 63;
    long long *stage = L.cf + wave * 64 * GP;
    uint32_t *stage_row = L.row + wave * 64;
    for (int64_t r0 = c0; r0 < c1; r0 += NT) {
        if (r0 + wave * 64 >= c1) break;       // nothing for this wavefront
        uint32_t q = kNoRow, m = cm;
        float a = ca;
        if (r0 + t < c1) {
            if (r0 != c0) {
                m = A.C.meta[r0 + t - A.C.base];
                a = entry_chord<CH>(A.C, r0 + t - A.C.base, m);
            }
            q = row_of(A.C, m);
            if (q >= A.C.rows) {
                atomicOr(A.err, 2u);
                q = kNoRow;
            }
        }
        const dev::Runs runs = dev::wave_runs(q);
        const bool emit = runs.tail && q != kNoRow;
        const unsigned long long tails = __ballot(emit);
        const int n = __popcll(tails), j = __popcll(tails & ((1ull << lane) - 1ull));
        const int w = (int)(m & (kTileWords - 1));
#pragma unroll
        for (int k = 0; k < GP; k++) {
            if (k >= G) continue;
            long long f = 0;
            if (q != kNoRow) f = rounded((double)a * L.x[sx<GP>(w, k)]);
            f = dev::run_sum(f, runs);
            if (emit) stage[j * GP + k] = f;
        }
        if (emit) stage_row[j] = q;
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int b = 0; b < n; b += 64 / GP) {
            const int i = b + lane / GP;
            if (i < n && s < G)
                atomicAdd(reinterpret_cast<unsigned long long *>(A.C.dot + (int64_t)stage_row[i] * S +
                                                                 g0 + s),
                          (unsigned long long)stage[i * GP + s]);
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

}  // namespace

int batch_vox_per_wg(int S) { return kThreads / S; }

int64_t batch_num_parts(const GridDev &g, int S)
{
    const int64_t nvox = padded_voxels(g);
    const int V = batch_vox_per_wg(S);
    const int64_t batches = (nvox + V - 1) / V;
    return batches < 1024 ? batches : 1024;    // the gradient kernel's grid
}

hipError_t launch_tvb_grad(const GridDev &g, const BatchBuffers &b, uint32_t active,
                           hipStream_t stream)
{
    const int V = batch_vox_per_wg(b.S);
    hipLaunchKernelGGL(k_tvb_grad, dim3((unsigned)batch_num_parts(g, b.S)), dim3(V * b.S), 0,
                       stream, g, b.x, b.S, V, active, b.eps, b.g, b.part);
    hipLaunchKernelGGL(k_tvb_norm, dim3((unsigned)b.S), dim3(kThreads), 0, stream,
                       (const double *)b.part, (uint32_t)batch_num_parts(g, b.S), b.S, V, b.norm2);
    return hipGetLastError();
}

hipError_t launch_tvb_step(const BatchBuffers &b, uint32_t active, int n, int nmax,
                           hipStream_t stream)
{
    const int64_t ne = b.nvox * b.S;
    hipLaunchKernelGGL(k_tvb_step, dim3(elem_grid(ne)), dim3(kThreads), 0, stream, b.x, b.g, b.S,
                       ne, active, b.beta_tab, b.cyc, n, nmax, b.norm2);
    return hipGetLastError();
}

hipError_t launch_set_counter(int32_t *cyc, int32_t v, hipStream_t stream)
{
    hipLaunchKernelGGL(k_set_counter, dim3(1), dim3(64), 0, stream, cyc, v);
    return hipGetLastError();
}

hipError_t launch_tick(int32_t *cyc, hipStream_t stream)
{
    hipLaunchKernelGGL(k_tick, dim3(1), dim3(64), 0, stream, cyc);
    return hipGetLastError();
}

hipError_t launch_replicate(const double *x0, const BatchBuffers &b, hipStream_t stream)
{
    hipLaunchKernelGGL(k_replicate, dim3(elem_grid(b.nvox * b.S)), dim3(kThreads), 0, stream, x0,
                       b.x, b.S, b.nvox);
    return hipGetLastError();
}

hipError_t launch_extract(const GridDev &g, const BatchBuffers &b, int s, float *out,
                          hipStream_t stream)
{
    const int64_t n = (int64_t)g.nx * g.ny * g.nz;
    hipLaunchKernelGGL(k_extract, dim3(elem_grid(n)), dim3(kThreads), 0, stream, g, b.x, b.S, s,
                       out);
    return hipGetLastError();
}

namespace {

template <int NT, int GP>
hipError_t drop_batch(const DropTileArgs &a, const BatchBuffers &b, hipStream_t stream)
{
    const TileBlock &v = a.P.valid ? a.P : a.C;
    const dim3 grid((unsigned)a.nact, (unsigned)((b.S + GP - 1) / GP));
    if (v.chq)
        hipLaunchKernelGGL((k_drop_tile_batch<NT, GP, uint16_t>), grid, dim3(NT), 0, stream, a,
                           b.S, b.nvox, (const double *)b.lambda);
    else if (v.ch16)
        hipLaunchKernelGGL((k_drop_tile_batch<NT, GP, __half>), grid, dim3(NT), 0, stream, a, b.S,
                           b.nvox, (const double *)b.lambda);
    else
        hipLaunchKernelGGL((k_drop_tile_batch<NT, GP, float>), grid, dim3(NT), 0, stream, a, b.S,
                           b.nvox, (const double *)b.lambda);
    return hipGetLastError();
}

}  // namespace

bool batch_shape_ok(int threads, int group)
{
    return (threads == 128 || threads == 256) &&
           (group == 2 || group == 4 || group == 8 || group == 16);
}

hipError_t launch_drop_tiles_batch(const DropTileArgs &a, const BatchBuffers &b, int64_t ntiles,
                                   int threads, int group, hipStream_t stream)
{
    if (ntiles <= 0 || (!a.P.valid && !a.C.valid) || !a.tiles || a.nact <= 0) return hipSuccess;
    if (threads == 128) {
        if (group == 2) return drop_batch<128, 2>(a, b, stream);
        if (group == 4) return drop_batch<128, 4>(a, b, stream);
        if (group == 16) return drop_batch<128, 16>(a, b, stream);
        return drop_batch<128, 8>(a, b, stream);
    }
    if (group == 2) return drop_batch<256, 2>(a, b, stream);
    if (group == 4) return drop_batch<256, 4>(a, b, stream);
    if (group == 16) return drop_batch<256, 16>(a, b, stream);
    return drop_batch<256, 8>(a, b, stream);
}

}  // namespace tvs

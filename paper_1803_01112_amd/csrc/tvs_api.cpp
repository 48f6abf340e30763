// tvs_api.cpp -- the C ABI (include/tvs.h) and the host runtime around the
// gfx950 kernels: argument validation, device memory ownership and HBM
// budget, history ingest and the tile lists of every DROP block (their
// layout fixed at load; rows formed once for a path store, per chunk and
// sweep for on-the-fly rows), the cycle driver (schedule of ell and beta,
// TV steps with or without the TV-reduction check, the DROP sweep) and the
// step log.
//
// Cycle structure (arXiv 1803.01112, Appendix C): ell_k = rand(k, ell_{k-1})
// once per cycle; N perturbation steps with beta = alpha^ell, ell += 1 after
// each; then x = P_T(x).  With the check, each step retries z = x + beta v
// with ell += 1 (and beta = alpha^ell recomputed) until TV(z) <= TV(x).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "tvs_internal.hpp"

using tvs::GridDev;
using tvs::HistDev;
using tvs::RowSet;
using tvs::TileBlock;

namespace {

constexpr int kNumStreams = 13;
constexpr uint32_t kTileShiftHost = (uint32_t)tvs::kTileShift;

// Step records of checked cycles held on the device before they are copied
// back (once per call, or when the buffer fills).
constexpr int64_t kDevLogCap = 4096;

// On the fly, rows are formed into a ring of chunk buffers: with three, the
// formation stream can form the next sweep's first chunk while the DROP
// chain still reads the last two of this sweep.
constexpr int kChunkBuffers = 3;

// Blocks one launch of the resident chain takes at most (about 6 ms; a
// launch's own cost is some 20 us).
constexpr int64_t kChainBlocks = 1024;
// Sweeps on the fly that go by launches beside the row formation after a chain
// launch was refused (another process held the cooperative queue) before the
// chain is tried again.  A sweep that finds it still refused has formed its rows
// first and launches the blocks then (3 M rows of 200x200x16 19.3 ms against
// 18.05 beside each other and 14.8 with the chain; of 256x256x32 22.2, 21.7
// and 17.8), so one in sixteen costs 0.2 to 0.5 %.
constexpr int kRefusedSweeps = 15;
// What a sweep by the chain costs beside its blocks, more than one by launches
// (the cooperative launch, the image into the LDS and back): 38 against 14 us, and
// half the difference again, since the estimates favour the chain on few blocks
// (the first angles' lists are longer than the mean).  A sweep of few blocks is
// launched (200x200x16 at B = 3,200, chain / launched: one block 45 / 22 us, four
// 65 / 47, eight 91 / 79, sixteen 140 / 143).
constexpr double kChainSweepUs = 36.0;
constexpr int kChainTable = 2048;            // slots of its row table
constexpr int kChainLds = 160 * 1024 - 256;  // LDS of a CU it may take

// Flags on the device: DROP fixed-point range, tile-list consistency,
// history validation, longest vertex count, longest chord (float32 bits).
enum {
    kFlagRange = 0,
    kFlagLists = 1,
    kFlagInvalid = 2,
    kFlagJmax = 3,
    kFlagChordMax = 4,
    kNumFlags = 5
};

// SplitMix64 (Steele, Lea, Flood 2014): golden-gamma Weyl state, variant-13
// output mixer.
uint64_t splitmix64(uint64_t &state)
{
    state += 0x9E3779B97F4A7C15ull;
    uint64_t z = state;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// rand(k, ell): uniform integer in [k, ell], both ends included (k when
// ell < k); exactly one draw per call.
int64_t draw_ell(int64_t k, int64_t ell, uint64_t &state)
{
    uint64_t u = splitmix64(state);
    if (ell < k) return k;
    uint64_t span = (uint64_t)(ell - k) + 1u;
    unsigned __int128 p = (unsigned __int128)u * span;
    return k + (int64_t)(uint64_t)(p >> 64);
}

// Device workspace of tvs_initial_fbp_noalloc: one file-scope array, held by
// every device the library runs on until the process ends.  Host code never
// uses the array's name as an address: each device's copy is looked up once
// (fbp_scratch_setup, from tvs_create with that device current) and its
// address is passed to the kernels.
constexpr size_t kFbpScratchBytes = (size_t)64 << 20;

}  // namespace

static __device__ __align__(256) unsigned char scratch[kFbpScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
hipError_t g_scratch_status[kMaxDevices] = {};
bool g_scratch_done[kMaxDevices] = {};

// Resident chains of one device run one after the other: each launch waits for
// the event that the last one of any context recorded.  Two of them at once
// could each hold part of the CUs and wait for the rest.
std::mutex g_chain_mu;
hipEvent_t g_chain_done[kMaxDevices] = {};

// Looks up this device's copy of `scratch` (the device must be current).
void fbp_scratch_setup(int dev)
{
    if (dev < 0 || dev >= kMaxDevices) return;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_done[dev]) return;
    void *p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        p = nullptr;
    }
    g_scratch_ptr[dev] = p;
    g_scratch_status[dev] = e;
    g_scratch_done[dev] = true;
}

}  // namespace

struct tvs_ctx {
    tvs_grid grid{};
    tvs_config cfg{};
    GridDev gd{};
    tvs::MlpCfg mlp{};
    hipStream_t stream = nullptr;
    int64_t nvox = 0;               // words of a device image (tiled layout, padding included)
    int64_t nimg = 0;               // voxels of an image at the ABI (nx * ny * nz)
    int64_t ntiles = 0;
    int cus = 256;
    uint64_t budget = 0;
    uint64_t bytes = 0;
    // during tvs_load_histories: allocations given back in that call, for its next ones
    bool recycle = false;
    uint64_t spare_bytes = 0;
    std::vector<std::pair<void *, size_t>> spare;
    std::string err;

    // image side (float64, tiled layout)
    double *x = nullptr, *g = nullptr;
    double *x0 = nullptr;           // initial iterate, the starting image of batches
    float *xio = nullptr;           // float32 staging of the image at the ABI
    double *part = nullptr;         // partial sums of ||g||^2
    double *dec = nullptr;          // checked step: step scale, accepted
    uint32_t *ticket = nullptr;     // checked step: last-workgroup counter
    int64_t nparts = 0;
    uint32_t *flags = nullptr;      // kNumFlags device flags
    long long *dot = nullptr;       // 3 x B fixed-point row dot products

    // histories and the tile lists of their DROP blocks
    bool loaded = false;
    int64_t nh = 0;
    float *hist = nullptr;          // 13 * nh floats
    int64_t *row_off = nullptr;     // nh + 1, entry offsets in walk order
    float *norm2 = nullptr;         // nh
    double *s1i = nullptr;          // entry-side MLP table (3 per vertex depth)
    int64_t nj = 0;
    int64_t *seg_off = nullptr;     // nh + 1
    int32_t *order = nullptr;       // nh: each chunk's histories by decreasing row length
    uint64_t *segtab = nullptr;     // nseg: global entry index of each segment's first entry
    int64_t nseg = 0;
    int64_t *bt_off = nullptr;      // nblocks * nact + 1 list starts, slots in order per block
    int32_t *act = nullptr;         // tiles that some block's lists cross (slot -> tile)
    int32_t *slot_of = nullptr;     // ntiles: while lists are laid out, tile -> slot, -1 for a
                                    // tile no list crosses; then, by_region, the slots by
                                    // decreasing entries (launches per block)
    bool by_region = false;         // slots in the order of the chain's regions
    int64_t nact = 0;
    int64_t nblocks = 0;
    // entries: the store, or a ring of chunk buffers on the fly
    uint32_t *meta[kChunkBuffers] = {};
    float *ch32[kChunkBuffers] = {};
    __half *ch16 = nullptr;
    uint16_t *chq = nullptr;        // fixed-point store: low 16 bits of the chord codes
    float chord_max = 0.0f;         // longest chord of the loaded rows (float32, rounded up)
    double qunit = 0.0;             // fixed-point store: mm per code unit
    double qinv = 0.0;              // 1 / qunit
    uint32_t qmax = 0;              // largest code (2^bits - 1)
    uint32_t qshift = 31;           // tag bit that holds the code's bit 16
    uint32_t rowmask = 0xffffffu;   // row field of the tags
    int64_t cap = 0;                // entries per buffer
    int nbuf = 0;                   // chunk buffers, side by side in one allocation
    int64_t joined = 1;             // chunks formed as one, in the buffers as one
    int64_t cbase = 0;              // ring position of the next sweep's first chunk
    hipStream_t fill_stream = nullptr;          // row formation of the next chunks
    hipEvent_t ev_filled[kChunkBuffers] = {};
    hipEvent_t ev_free[kChunkBuffers] = {};
    int64_t nnz = 0, max_row = 0, skipped = 0;
    int64_t chunk = 0;              // histories per chunk (a multiple of B)
    std::vector<int64_t> chunk_base;  // entry offset of each chunk start (and the end)
    double big = 0.0, dot_max = 0.0;  // fixed-point ranges of the DROP kernels
    int threads = 256;              // threads per tile workgroup
    bool tuned = false;             // by tvs_autotune (else tile_lanes at every load)
    bool launches = false;          // tvs_autotune: launches per block, not the chain
    int split = 0;                  // 1: two launches per block
    int bthreads = 256;             // batched DROP step: threads per workgroup
    int bgroup = 4;                 // batched DROP step: settings per pass through LDS
    int64_t fill_wgs = 0;           // grid cap of the sweep's row formation (0: none)
    int fill_wide_pct = 0;          // chunks formed at the row kernel's full occupancy, %

    // cycle state
    int64_t k = 0, ell = 0;
    uint64_t rng = 0;
    bool seeded = false;
    std::vector<tvs_step_log> log;
    int64_t tries = 0;
    // checked cycles keep ell and the RNG state on the device (sched) and
    // write their step records there (dlog); dev_sched: the device copy is
    // the current one, to be copied back (after ev_sched) before the host
    // uses ell again or reports the log
    tvs::SchedDev *sched = nullptr;
    tvs_step_log *dlog = nullptr;
    int64_t dlog_n = 0;
    bool dev_sched = false;
    hipEvent_t ev_sched = nullptr;
    double *cpart = nullptr;        // partial sums of the device-side check

    // timing: HIP events recorded on the launch stream around every phase of
    // the last tvs_iterate call, resolved lazily by tvs_get_stats
    std::vector<hipEvent_t> tev;
    size_t tev_used = 0;
    // kind: 0 TV steps, 1 sweep, 2 rows, 3 DROP, 4 first / 5 second launch of a sampled block
    struct Span { int kind; size_t a, b; int64_t n; };   // n: blocks the span covers
    std::vector<Span> spans;
    bool timed = false;
    double last_sweep_ms = 0, last_tv_ms = 0, last_rows_ms = 0;
    double tot_ms[6] = {0, 0, 0, 0, 0, 0};
    int64_t tot_n[6] = {0, 0, 0, 0, 0, 0};

    // the resident DROP chain (plan_chain) of the loaded histories
    struct Chain {
        bool planned = false;       // the grid and the blocks suit it
        bool failed = false;        // a barrier timed out: its counters no longer match
        int refused = 0;            // sweeps until it is tried again after a refused launch
                                    // (rows of several chunks on the fly)
        bool refuse = false;        // tvs_debug_sweep: the next launch counts as refused
        int nreg = 0, parts = 1, tmax = 0, ns = 0;
        std::vector<int32_t> first; // first slot of each region (nreg + 1)
        // device workspace, given back when a call needs its room (dalloc, chain_restore)
        int32_t *reg = nullptr;     // first, on the device
        uint32_t *bar = nullptr;    // barrier counters: all workgroups', then one per region;
                                    // behind them the mark of a wait that timed out
        uint8_t *exch = nullptr;    // exchange records of the workgroups (parts > 1)
        uint8_t *mem = nullptr;     // the allocation that holds them all
        size_t bytes = 0;
        uint32_t epoch = 0, sub_epoch = 0;
        bool on() const { return planned && mem && !failed; }
    } chain;

    // batched reconstructions
    struct Batch {
        int S = 0;
        bool valid = false;
        std::vector<tvs_params> p;
        tvs::BatchBuffers b;
        long long *dot = nullptr;   // 3 x B x S
        int64_t k = 0;
        std::vector<int64_t> ell;
        std::vector<uint64_t> rng;
        int64_t beta_cap = 0;
        double ms_total = 0;
        int64_t cycles = 0;
    } batch;
    // fork/join events of the captured batched cycle (the fill stream's row
    // formation beside the batched chain); only ever recorded in capture
    hipEvent_t bev_fork = nullptr;
    hipEvent_t bev_filled[kChunkBuffers] = {};
    hipEvent_t bev_free[kChunkBuffers] = {};
};

namespace {

int fail(tvs_ctx *ctx, int code, const std::string &msg)
{
    if (ctx) ctx->err = msg;
    return code;
}

#define HIPCHK(expr)                                                                          \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return fail(ctx, TVS_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

void chain_release(tvs_ctx *ctx);

size_t chain_bar_bytes(int nreg) { return 4 * (size_t)(tvs::kChainShards + nreg + 1) * 32; }

// Frees what tvs_load_histories has given back and not taken again.
void drop_spare(tvs_ctx *ctx)
{
    for (auto &s : ctx->spare) (void)hipFree(s.first);
    ctx->spare.clear();
    ctx->spare_bytes = 0;
}

template <typename T>
int dalloc(tvs_ctx *ctx, T **p, size_t count)
{
    size_t bytes = count * sizeof(T);
    if (bytes == 0) bytes = sizeof(T);
    for (size_t i = 0; i < ctx->spare.size(); i++) {
        if (ctx->spare[i].second != bytes) continue;
        if (ctx->bytes + bytes > ctx->budget) break;
        *p = static_cast<T *>(ctx->spare[i].first);
        ctx->spare.erase(ctx->spare.begin() + (long)i);
        ctx->spare_bytes -= bytes;
        ctx->bytes += bytes;
        return TVS_OK;
    }
    if (ctx->bytes + ctx->spare_bytes + bytes > ctx->budget) drop_spare(ctx);
    // the chain's workspace gives way to what then fits (chain_restore)
    if (ctx->bytes + bytes > ctx->budget && ctx->chain.mem &&
        ctx->bytes - ctx->chain.bytes + bytes <= ctx->budget)
        chain_release(ctx);
    if (ctx->bytes + bytes > ctx->budget)
        return fail(ctx, TVS_ENOMEM,
                    "footprint " + std::to_string(ctx->bytes + bytes) + " B exceeds budget " +
                        std::to_string(ctx->budget) + " B");
    void *q = nullptr;
    hipError_t e = hipMalloc(&q, bytes);
    if (e != hipSuccess && !ctx->spare.empty()) {
        (void)hipGetLastError();
        drop_spare(ctx);
        e = hipMalloc(&q, bytes);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return fail(ctx, TVS_ENOMEM, std::string("hipMalloc: ") + hipGetErrorString(e));
    }
    *p = static_cast<T *>(q);
    ctx->bytes += bytes;
    return TVS_OK;
}

template <typename T>
void dfree(tvs_ctx *ctx, T **p, size_t count)
{
    if (*p) {
        size_t bytes = count * sizeof(T);
        if (bytes == 0) bytes = sizeof(T);
        if (ctx->recycle) {
            ctx->spare.emplace_back(*p, bytes);
            ctx->spare_bytes += bytes;
        } else {
            (void)hipFree(*p);
        }
        ctx->bytes -= std::min<uint64_t>(ctx->bytes, bytes);
        *p = nullptr;
    }
}

// Gives the chain's workspace back to the device (not to the next allocations
// of a load: the room is wanted now).
void chain_release(tvs_ctx *ctx)
{
    auto &c = ctx->chain;
    const bool recycle = ctx->recycle;
    ctx->recycle = false;
    dfree(ctx, &c.mem, c.bytes);
    ctx->recycle = recycle;
    c.reg = nullptr;
    c.bar = nullptr;
    c.exch = nullptr;
}

// Forms the chain's workspace again where it is missing and there is room:
// counters and exchange records (cleared), then the regions.
void chain_restore(tvs_ctx *ctx)
{
    auto &c = ctx->chain;
    if (!c.planned || c.failed || c.mem || ctx->bytes + c.bytes > ctx->budget) return;
    const std::string err = ctx->err;
    const size_t nbar = chain_bar_bytes(c.nreg);
    const size_t nfirst = 4 * c.first.size(), clear = c.bytes - nfirst;
    if (dalloc(ctx, &c.mem, c.bytes) == TVS_OK) {
        c.bar = reinterpret_cast<uint32_t *>(c.mem);
        c.exch = c.mem + nbar;
        c.reg = reinterpret_cast<int32_t *>(c.mem + clear);
        c.epoch = c.sub_epoch = 0;
        hipError_t e = hipMemsetAsync(c.mem, 0, clear, ctx->stream);
        if (e == hipSuccess)
            e = hipMemcpyAsync(c.reg, c.first.data(), nfirst, hipMemcpyHostToDevice, ctx->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            chain_release(ctx);
        }
    }
    ctx->err = err;
}

// Word of the workspace that a timed-out wait sets, behind the counters.
uint32_t *chain_dead(tvs_ctx *ctx)
{
    return ctx->chain.bar + (tvs::kChainShards + ctx->chain.nreg) * 32;
}

// Whether sweeps take the chain.
bool chain_on(const tvs_ctx *ctx) { return ctx->chain.on() && !ctx->launches; }

// At the end of every call that allocates: what the call took from the chain
// and has given back is the chain's again.
struct ChainBack {
    tvs_ctx *c;
    ~ChainBack() { chain_restore(c); }
};

int64_t bt_len(const tvs_ctx *ctx) { return ctx->nblocks * ctx->nact + 1; }

// Ring buffer of chunk c of the current sweep (on the fly).
int chunk_buffer(const tvs_ctx *ctx, int64_t c) { return (int)((ctx->cbase + c) % ctx->nbuf); }

void free_histories(tvs_ctx *ctx)
{
    dfree(ctx, &ctx->hist, (size_t)(kNumStreams * ctx->nh));
    dfree(ctx, &ctx->row_off, (size_t)(ctx->nh + 1));
    dfree(ctx, &ctx->norm2, (size_t)ctx->nh);
    dfree(ctx, &ctx->seg_off, (size_t)(ctx->nh + 1));
    dfree(ctx, &ctx->order, (size_t)ctx->nh);
    dfree(ctx, &ctx->s1i, (size_t)(3 * ctx->nj));
    ctx->nj = 0;
    ctx->mlp.s1i = nullptr;
    ctx->mlp.nj = 0;
    dfree(ctx, &ctx->segtab, (size_t)ctx->nseg);
    dfree(ctx, &ctx->bt_off, (size_t)bt_len(ctx));
    dfree(ctx, &ctx->chain.mem, ctx->chain.bytes);
    ctx->chain = tvs_ctx::Chain();
    dfree(ctx, &ctx->act, (size_t)std::max<int64_t>(ctx->nact, 1));
    dfree(ctx, &ctx->slot_of, (size_t)std::max<int64_t>(ctx->ntiles, 1));
    ctx->nact = 0;
    dfree(ctx, &ctx->meta[0], (size_t)(ctx->nbuf * ctx->cap));
    dfree(ctx, &ctx->ch32[0], (size_t)(ctx->nbuf * ctx->cap));
    for (int q = 1; q < kChunkBuffers; q++) {
        ctx->meta[q] = nullptr;
        ctx->ch32[q] = nullptr;
    }
    dfree(ctx, &ctx->ch16, (size_t)ctx->cap);
    dfree(ctx, &ctx->chq, (size_t)ctx->cap);
    ctx->chord_max = 0.0f;
    ctx->qunit = ctx->qinv = 0.0;
    ctx->qmax = 0;
    ctx->qshift = 31;
    ctx->rowmask = 0xffffffu;
    ctx->loaded = false;
    ctx->nh = 0;
    ctx->nseg = 0;
    ctx->nblocks = 0;
    ctx->cap = 0;
    ctx->nbuf = 0;
    ctx->cbase = 0;
    ctx->nnz = ctx->max_row = ctx->skipped = 0;
    ctx->chunk_base.clear();
}

void free_batch(tvs_ctx *ctx)
{
    auto &B = ctx->batch;
    const size_t n = (size_t)(ctx->nvox * B.S);
    dfree(ctx, &B.b.x, n);
    dfree(ctx, &B.b.g, n);
    dfree(ctx, &B.b.part, (size_t)(tvs::batch_num_parts(ctx->gd, std::max(B.S, 1)) * B.S));
    dfree(ctx, &B.b.norm2, (size_t)B.S);
    dfree(ctx, &B.b.lambda, (size_t)B.S);
    dfree(ctx, &B.b.eps, (size_t)B.S);
    dfree(ctx, &B.b.beta_tab, (size_t)B.beta_cap);
    dfree(ctx, &B.b.cyc, (size_t)4);
    dfree(ctx, &B.dot, (size_t)(3 * (int64_t)ctx->cfg.block_size * B.S));
    B = tvs_ctx::Batch();
}

HistDev hist_dev(const tvs_ctx *ctx)
{
    return HistDev{ctx->hist, ctx->nh};
}

tvs::TvBuffers tv_bufs(tvs_ctx *ctx)
{
    return tvs::TvBuffers{ctx->g, ctx->part, ctx->nparts};
}

hipStream_t pick(tvs_ctx *ctx, void *stream)
{
    return stream ? static_cast<hipStream_t>(stream) : ctx->stream;
}

void reset_state(tvs_ctx *ctx)
{
    ctx->k = 0;
    ctx->ell = 0;
    ctx->rng = 0;
    ctx->seeded = false;
    ctx->log.clear();
    ctx->tries = 0;
    ctx->dev_sched = false;
    ctx->dlog_n = 0;
}

// Copies the schedule and step records of checked cycles back from the
// device (waits for the work of the last checked call).
int settle_sched(tvs_ctx *ctx)
{
    if (!ctx->dev_sched) return TVS_OK;
    HIPCHK(hipEventSynchronize(ctx->ev_sched));
    tvs::SchedDev sd{};
    HIPCHK(hipMemcpy(&sd, ctx->sched, sizeof(sd), hipMemcpyDeviceToHost));
    std::vector<tvs_step_log> recs((size_t)ctx->dlog_n);
    if (ctx->dlog_n > 0)
        HIPCHK(hipMemcpy(recs.data(), ctx->dlog, sizeof(tvs_step_log) * (size_t)ctx->dlog_n,
                         hipMemcpyDeviceToHost));
    for (const auto &r : recs) {
        ctx->log.push_back(r);
        ctx->tries += r.tries;
    }
    ctx->ell = sd.ell;
    ctx->rng = sd.rng;
    ctx->dlog_n = 0;
    ctx->dev_sched = false;
    return TVS_OK;
}

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

// Records a timing event on st; returns its index in the pool (or -1). Pool
// events skip the system-scope fence: they carry timestamps only, and the fence
// (an L2 write-back) would otherwise be timed with the work it brackets.
long mark(tvs_ctx *ctx, hipStream_t st)
{
    if (ctx->tev_used == ctx->tev.size()) {
        hipEvent_t e;
        if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return -1;
        ctx->tev.push_back(e);
    }
    if (hipEventRecord(ctx->tev[ctx->tev_used], st) != hipSuccess) return -1;
    return (long)ctx->tev_used++;
}

// Reserves an event of the pool without recording it (recorded by a launch).
long slot(tvs_ctx *ctx)
{
    if (ctx->tev_used == ctx->tev.size()) {
        hipEvent_t e;
        if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return -1;
        ctx->tev.push_back(e);
    }
    return (long)ctx->tev_used++;
}

void span(tvs_ctx *ctx, int kind, long a, long b, int64_t n = 1)
{
    if (a >= 0 && b >= 0) ctx->spans.push_back({kind, (size_t)a, (size_t)b, n});
}

// Pool events for the kernels of one sampled block, stamped by the launches
// themselves: the first launch (kind 4) and, when the step is split in two
// launches, the second (kind 5).
bool ktimer(tvs_ctx *ctx, tvs::KTimer &kt, bool two)
{
    const int n = two ? 4 : 2;
    long q[4] = {-1, -1, -1, -1};
    for (int i = 0; i < n; i++)
        if ((q[i] = slot(ctx)) < 0) return false;
    for (int i = 0; i < n; i++) kt.e[i] = ctx->tev[(size_t)q[i]];
    span(ctx, 4, q[0], q[1]);
    if (two) span(ctx, 5, q[2], q[3]);
    return true;
}

// Checks the device flags raised by the DROP and row kernels (waits for the
// work queued on st).
int check_flags(tvs_ctx *ctx, hipStream_t st)
{
    uint32_t f[kNumFlags] = {};
    HIPCHK(hipMemcpyAsync(f, ctx->flags, sizeof(f), hipMemcpyDeviceToHost, st));
    HIPCHK(hipStreamSynchronize(st));
    if (f[kFlagLists] || (f[kFlagRange] & 2u))
        return fail(ctx, TVS_EDEVICE, "a row walk disagreed with its load-time tile lists");
    if (f[kFlagRange] & 4u) {
        // the barrier's counters no longer match: launch block by block until the next load
        ctx->chain.failed = true;
        return fail(ctx, TVS_EDEVICE, "a workgroup of the DROP chain did not reach its barrier");
    }
    if (f[kFlagRange])
        return fail(ctx, TVS_ERANGE,
                    "a DROP product |a_ij x_j| left the fixed-point range (image values too "
                    "large); set a new image to clear");
    return TVS_OK;
}

// One block's tile lists as the DROP kernels see them.
TileBlock block_view(tvs_ctx *ctx, int64_t b, long long *dot_base, int64_t dot_stride)
{
    const int64_t B = ctx->cfg.block_size;
    const bool otf = ctx->cfg.path_mode == TVS_PATH_ON_THE_FLY;
    const int64_t c = otf ? (b * B) / ctx->chunk / ctx->joined * ctx->joined : 0;
    const int buf = otf ? chunk_buffer(ctx, c) : 0;
    TileBlock t;
    t.meta = ctx->meta[buf];
    t.ch32 = ctx->ch32[buf];
    t.ch16 = ctx->ch16;
    t.chq = ctx->chq;
    t.qunit = ctx->qunit;
    t.qshift = ctx->qshift;
    t.rowmask = ctx->rowmask;
    t.toff = ctx->bt_off + b * ctx->nact;
    t.base = otf ? ctx->chunk_base[(size_t)c] : 0;
    t.wepl = ctx->hist + 12 * ctx->nh + b * B;
    t.n2 = ctx->norm2 + b * B;
    t.dot = dot_base + (b % 3) * dot_stride;
    t.rows = (uint32_t)std::min<int64_t>(B, ctx->nh - b * B);
    t.valid = 1;
    return t;
}

// Forms the rows of chunk c (histories [c*chunk, c*chunk + n)) into its buffer.
tvs::TileFill chunk_fill(tvs_ctx *ctx, int64_t c, int64_t n)
{
    tvs::TileFill f;
    f.first = c * ctx->chunk;
    f.n = n;
    f.B = ctx->cfg.block_size;
    f.seg_off = ctx->seg_off;
    f.segdst = reinterpret_cast<const int64_t *>(ctx->segtab);
    f.base = ctx->chunk_base[(size_t)c];
    f.meta = ctx->meta[chunk_buffer(ctx, c)];
    f.ch32 = ctx->ch32[chunk_buffer(ctx, c)];
    f.ch16 = ctx->ch16;
    f.cap = ctx->cap;
    f.norm2 = ctx->norm2;
    f.err = ctx->flags + kFlagLists;
    f.max_wgs = ctx->fill_wgs;
    f.order = ctx->order;
    // beside per-block launches: chunk c at full occupancy when the running count
    // of such chunks steps up at c (fill_wide_pct of them, spread evenly),
    // else held at two waves per SIMD
    const int64_t pct = ctx->fill_wide_pct;
    f.room = ((c + 1) * pct / 100 > c * pct / 100) ? 0 : 1;
    return f;
}

// Blocks [b0, b1) of a sweep, one launch (or two) per block.
int launch_blocks(tvs_ctx *ctx, double lambda, int64_t b0, int64_t b1, hipStream_t st)
{
    const int64_t B = ctx->cfg.block_size;
    HIPCHK(tvs::launch_zero_i64(ctx->dot, 3 * B, st));
    for (int64_t b = b0; b <= b1; b++) {
        const bool has_c = b < b1;
        tvs::DropTileArgs A;
        if (b > b0) A.P = block_view(ctx, b - 1, ctx->dot, B);
        if (has_c) A.C = block_view(ctx, b, ctx->dot, B);
        A.x = ctx->x;
        A.lambda = lambda;
        A.big = ctx->big;
        A.dot_max = ctx->dot_max;
        A.zero = ctx->dot + ((b + 1) % 3) * B;
        A.B = B;
        A.err = ctx->flags + kFlagRange;
        A.tiles = ctx->act;
        A.nact = ctx->nact;
        A.slots = ctx->by_region ? ctx->slot_of : nullptr;
        const bool samp = ctx->cfg.time_sample > 0 && has_c && b > b0 &&
                          b % ctx->cfg.time_sample == 0;
        tvs::KTimer kt;
        const bool timed = samp && ktimer(ctx, kt, ctx->split != 0);
        HIPCHK(tvs::launch_drop_tiles(A, ctx->ntiles, ctx->threads, ctx->split, st,
                                      timed ? &kt : nullptr));
    }
    return TVS_OK;
}

// Blocks [b0, b1) of a sweep by the resident chain; false: nothing was
// launched (another process holds the device's cooperative queue), and the
// blocks are to be launched one by one.
bool run_chain(tvs_ctx *ctx, double lambda, int64_t b0, int64_t b1, hipStream_t st)
{
    auto &c = ctx->chain;
    if (c.refuse) {
        c.refuse = false;
        return false;
    }
    const int64_t B = ctx->cfg.block_size;
    const TileBlock v = block_view(ctx, b0, ctx->dot, B);
    tvs::ChainArgs a;
    a.meta = v.meta;
    a.ch32 = v.ch32;
    a.ch16 = v.ch16;
    a.chq = v.chq;
    a.qunit = v.qunit;
    a.qshift = v.qshift;
    a.rowmask = v.rowmask;
    a.toff = ctx->bt_off;
    a.nact = ctx->nact;
    a.base = v.base;
    a.act = ctx->act;
    a.reg = c.reg;
    a.wepl = ctx->hist + 12 * ctx->nh;
    a.n2 = ctx->norm2;
    a.dot = ctx->dot;
    a.B = B;
    a.nh = ctx->nh;
    a.x = ctx->x;
    a.cb = ctx->g;     // the subgradient is formed anew by every TV step
    a.lambda = lambda;
    a.big = ctx->big;
    a.dot_max = ctx->dot_max;
    a.err = ctx->flags + kFlagRange;
    a.bar = c.bar;
    a.sub = c.bar + tvs::kChainShards * 32;
    a.dead = chain_dead(ctx);
    a.exch = c.exch;
    a.nreg = c.nreg;
    a.parts = c.parts;
    a.tmax = c.tmax;
    a.ns = (uint32_t)c.ns;
    a.b0 = b0;
    a.b1 = b1;
    a.epoch = c.epoch;
    a.sub_epoch = c.sub_epoch;
    const bool timed = ctx->cfg.time_sample > 0;
    const int dev = ctx->cfg.device;
    if (dev < 0 || dev >= kMaxDevices) return false;
    const long e0 = timed ? mark(ctx, st) : -1;
    {
        std::lock_guard<std::mutex> lk(g_chain_mu);
        hipEvent_t &done = g_chain_done[dev];
        hipError_t e = done ? hipStreamWaitEvent(st, done, 0)
                            : hipEventCreateWithFlags(&done, hipEventDisableTiming);
        if (e == hipSuccess) e = tvs::launch_chain(a, st);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        e = hipEventRecord(done, st);
        if (e != hipSuccess) (void)hipStreamSynchronize(st);
    }
    if (timed) span(ctx, 4, e0, mark(ctx, st), b1 - b0);
    c.epoch += (uint32_t)(b1 - b0) + 1u;
    c.sub_epoch += (uint32_t)(b1 - b0);
    return true;
}

// One P_T sweep over the loaded histories, by the chain where use_chain is set
// and nothing stands against it (the first `limit` histories when limit >= 0, a
// multiple of B: used to time launch shapes).
int run_sweep(tvs_ctx *ctx, double lambda, hipStream_t st, bool use_chain, int64_t limit = -1)
{
    const int64_t B = ctx->cfg.block_size;
    const int64_t nh_run = (limit >= 0) ? std::min(limit, ctx->nh) : ctx->nh;
    if (nh_run <= 0) return TVS_OK;
    const int64_t nb = (nh_run + B - 1) / B;
    const bool otf = ctx->cfg.path_mode == TVS_PATH_ON_THE_FLY;
    // a cooperative launch is not captured
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    const bool several = otf && ctx->nbuf > 1;
    bool chain = use_chain && ctx->chain.on() && hipStreamIsCapturing(st, &cap) == hipSuccess &&
                 cap == hipStreamCaptureStatusNone;
    // after a refused launch the rows of several chunks are formed beside
    // per-block launches again, for some sweeps
    if (chain && several && ctx->chain.refused > 0) {
        ctx->chain.refused--;
        chain = false;
    }
    // for the chain: the buffers as one, filled (the first time beside the TV
    // steps) and emptied in turn
    const int64_t NB = chain ? 1 : ctx->nbuf;
    ctx->joined = chain ? ctx->nbuf : 1;
    if (chain) ctx->cbase = 0;
    const int64_t step = otf ? ctx->chunk * ctx->joined : ctx->nh;
    const int64_t nchunks = (nh_run + step - 1) / step;
    hipStream_t fs = ctx->fill_stream;
    struct Unjoin {
        tvs_ctx *c;
        ~Unjoin() { c->joined = 1; }
    } unjoin{ctx};
    // a chunk is always formed whole, also when the sweep stops inside it:
    // its rows are formed in length order, so the first n of them are not
    // the histories of the first blocks
    auto fill = [&](int64_t c) -> int {
        const int64_t n = std::min(step, ctx->nh - c * step);
        tvs::TileFill f = chunk_fill(ctx, c * ctx->joined, n);
        // nothing but the TV steps beside a single chunk: full occupancy (900 k rows
        // of 200x200x16 with launches at B = 25,600: 4.0 ms a cycle, 4.65 held)
        if (!several) f.room = 0;
        if (chain) {
            f.cap *= ctx->joined;
            f.max_wgs = 0;
            f.room = 0;
            for (int q = 0; q < ctx->nbuf; q++) HIPCHK(hipStreamWaitEvent(fs, ctx->ev_free[q], 0));
        } else {
            HIPCHK(hipStreamWaitEvent(fs, ctx->ev_free[chunk_buffer(ctx, c)], 0));
        }
        long a = mark(ctx, fs);
        HIPCHK(tvs::launch_rows_fill_tiled(ctx->gd, hist_dev(ctx), ctx->mlp, f, fs));
        span(ctx, 2, a, mark(ctx, fs));
        HIPCHK(hipEventRecord(ctx->ev_filled[chunk_buffer(ctx, c)], fs));
        return TVS_OK;
    };
    if (otf) {
        for (int64_t c = 0; c < std::min<int64_t>(NB, nchunks); c++) {
            int rc = fill(c);
            if (rc) return rc;
        }
    }
    for (int64_t c = 0; c < nchunks; c++) {
        const int64_t c0 = c * step / B, c1 = std::min(nb, ((c + 1) * step + B - 1) / B);
        if (otf) HIPCHK(hipStreamWaitEvent(st, ctx->ev_filled[chunk_buffer(ctx, c)], 0));
        const long e0 = mark(ctx, st);      // past the wait for the rows
        // at most kChainBlocks blocks a launch, so that reconstructions on
        // other streams, whose chains wait for this one, get their turn
        for (int64_t b = c0; b < c1;) {
            const int64_t e = chain ? std::min(c1, b + kChainBlocks) : c1;
            if (!chain || !run_chain(ctx, lambda, b, e, st)) {
                if (chain) ctx->chain.refused = kRefusedSweeps;
                int rc = launch_blocks(ctx, lambda, b, e, st);
                if (rc) return rc;
            }
            b = e;
        }
        span(ctx, 3, e0, mark(ctx, st), c == 0 ? 1 : 0);
        if (otf) {
            if (chain) {
                for (int q = 0; q < ctx->nbuf; q++) HIPCHK(hipEventRecord(ctx->ev_free[q], st));
            } else {
                HIPCHK(hipEventRecord(ctx->ev_free[chunk_buffer(ctx, c)], st));
            }
            if (c + NB < nchunks) {
                int rc = fill(c + NB);
                if (rc) return rc;
            }
        }
    }
    // the ring continues with the next sweep, whose first chunks take the
    // buffers freed first
    if (otf && !chain) ctx->cbase = (ctx->cbase + nchunks) % NB;
    return TVS_OK;
}

int validate_params(tvs_ctx *ctx, const tvs_params *p)
{
    if (!p) return fail(ctx, TVS_EINVAL, "params is NULL");
    if (!finite_pos(p->lambda)) return fail(ctx, TVS_EINVAL, "lambda must be finite and > 0");
    if (p->variant < 0 || p->variant > 2) return fail(ctx, TVS_EINVAL, "unknown variant");
    if (p->variant != TVS_OTVS && !(p->alpha > 0.0 && p->alpha < 1.0))
        return fail(ctx, TVS_EINVAL, "alpha must lie in (0, 1)");
    if (p->N < 0) return fail(ctx, TVS_EINVAL, "N must be >= 0");
    if (!(p->tv_eps >= 0.0) || !std::isfinite(p->tv_eps))
        return fail(ctx, TVS_EINVAL, "tv_eps must be finite and >= 0");
    if (p->variant == TVS_DECOUPLED && !(p->gamma > 0.0 && p->gamma < 1.0))
        return fail(ctx, TVS_EINVAL, "gamma must lie in (0, 1)");
    return TVS_OK;
}

// Row lengths of histories [first, first + n) into row_off_dev (n + 1).
int count_rows(tvs_ctx *ctx, int64_t first, int64_t n, int64_t *row_off_dev, hipStream_t st)
{
    int32_t *cnt = nullptr;
    int64_t *tmp = nullptr;
    int rc = dalloc(ctx, &cnt, (size_t)std::max<int64_t>(n, 1));
    if (rc) return rc;
    rc = dalloc(ctx, &tmp, (size_t)tvs::scan_tmp_elems(n) + 1);
    if (rc) {
        dfree(ctx, &cnt, (size_t)std::max<int64_t>(n, 1));
        return rc;
    }
    hipError_t e =
        tvs::launch_rows_count(ctx->gd, hist_dev(ctx), ctx->mlp, first, n, cnt, nullptr, st);
    if (e == hipSuccess) e = tvs::launch_scan(cnt, n, row_off_dev, tmp, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    dfree(ctx, &cnt, (size_t)std::max<int64_t>(n, 1));
    dfree(ctx, &tmp, (size_t)tvs::scan_tmp_elems(n) + 1);
    if (e != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("row count: ") + hipGetErrorString(e));
    return TVS_OK;
}

// Time of a DROP block, us, launched and in the resident chain, for choosing
// between them: n crossed tiles, `longest` the longest list of a block, `busiest`
// the entries of the fullest region.  A launch's time goes with its longest list,
// up to 8 tiles per CU being in work at once, and with all entries; the chain's
// with a CU's entries, from some 3,000 on (the lanes hold 4,096 in registers, a
// block more or less than the mean) at three times the price.  Least squares
// over eleven grids of 0.5 to 17 tiles per CU at B = 16 to 102,400 (8 % and 4 %
// mean error; the same for both stores).  Chain / launched, measured:
//   tiles per CU 1.3    B = 800 4.9 / 6.1, 3,200 5.7 / 10.8, 25,600 31.5 / 69.8, 102,400 172 / 280
//                2.8    800 5.1 / 6.3, 6,400 9.4 / 13.9, 25,600 41.8 / 47.2, 51,200 94.6 / 90.0
//                3.4    6,400 11.6 / 14.0, 12,800 22.2 / 24.2, 25,600 50.3 / 47.5, 102,400 269 / 179
//                5.5    800 5.3 / 6.7, 6,400 11.0 / 12.7, 12,800 21.2 / 20.7, 25,600 47.0 / 35.6
//                16.7   800 5.5 / 8.8, 6,400 12.5 / 16.4, 12,800 22.0 / 25.4, 25,600 43.5 / 40.4
double launch_us(const tvs_ctx *ctx, int n, double longest)
{
    const double t = (double)n / ctx->cus;
    const double per_cu = (double)ctx->nnz / (double)std::max<int64_t>(ctx->nblocks, 1) / ctx->cus;
    return 2.5 + 0.0064 * std::min(longest, 100.0) + 0.0043 * longest * std::max(1.0, t / 8.0) +
           0.001 * per_cu + 1.4 * std::min(t, 1.0) + 0.15 * std::max(t - 1.0, 0.0);
}
double chain_us(int n, int cus, int parts, double busiest)
{
    const double e = busiest / parts;
    return 4.7 + 0.0008 * e + (n < 8 * cus ? 0.0019 : 0.00115) * std::max(e - 3000.0, 0.0) +
           0.00155 * std::max(e - 20000.0, 0.0) + (parts > 1 ? 2.2 : 0.0);
}

// Places the active tiles in regions of the resident chain (chain.hip), one
// region per workgroup: reorders a (the tiles by slot) and describes them in
// the context's chain.  False where the chain does not fit: explicit
// launch shapes, blocks of more rows than a packed entry names, images whose
// crossed tiles do not fit the device's LDS, sweeps that launches make faster.
bool plan_chain(tvs_ctx *ctx, const std::vector<uint32_t> &entries, std::vector<int32_t> &a)
{
    auto &c = ctx->chain;
    std::vector<int32_t> reg;
    const int64_t B = ctx->cfg.block_size;
    if (ctx->cfg.sweep_kernel != 0 || ctx->cfg.tile_threads != 0 || B > tvs::kChainMaxB) return false;
    const int cus = ctx->cus;
    int coop = 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, ctx->cfg.device) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    if (!coop) return false;
    const int n = (int)a.size();
    c.ns = kChainTable;
    int cap = tvs::kChainMaxTiles;
    while (cap > 0 && tvs::chain_lds_bytes(cap, c.ns) > (size_t)kChainLds) cap--;
    if (cap < 1 || (int64_t)cap * cus < n) return false;
    // neighbours in a slice next to each other (Morton order of the tiles), so
    // that a row crosses few regions
    const GridDev &g = ctx->gd;
    auto key = [&](int32_t T) {
        const int64_t z = T / ((int64_t)g.ntx * g.nty);
        const uint32_t i = (uint32_t)(T % g.ntx), j = (uint32_t)((T / g.ntx) % g.nty);
        uint64_t m = 0;
        for (int q = 0; q < 16; q++)
            m |= (uint64_t)(((i >> q) & 1u) | (((j >> q) & 1u) << 1)) << (2 * q);
        return ((uint64_t)z << 32) | m;
    };
    std::sort(a.begin(), a.end(), [&](int32_t x, int32_t y) { return key(x) < key(y); });
    // a tile's work per block: its entries, and its words (a quarter of an entry each)
    const double nb = (double)std::max<int64_t>(ctx->nblocks, 1);
    double total = 0.0, most = 0.0;
    std::vector<double> w(a.size());
    for (size_t i = 0; i < a.size(); i++) {
        w[i] = (double)entries[(size_t)a[i]] / nb + 64.0;
        total += w[i];
        most = std::max(most, w[i]);
    }
    auto cut = [&](double limit) {
        reg.assign(1, 0);
        double sum = 0.0;
        for (int i = 0; i < n; i++) {
            if (i > reg.back() && (sum + w[(size_t)i] > limit || i - reg.back() >= cap)) {
                reg.push_back(i);
                sum = 0.0;
            }
            sum += w[(size_t)i];
        }
        reg.push_back(n);
        return (int)reg.size() - 1;
    };
    if (n <= cus) {
        for (int i = 0; i <= n; i++) reg.push_back(i);
        // few tiles: several workgroups per tile, as far as the busiest
        // tile's list of a block fills them
        const double per = 2.0 * tvs::kChainSplitThreads;
        c.parts = std::max(1, std::min(std::min(cus / n, 32), (int)std::ceil((most - 64.0) / per)));
    } else {
        double lo = std::max(most, total / cus), hi = total + 1.0;
        if (cut(hi) > cus) return false;       // the tile cap alone needs more regions
        for (int q = 0; q < 40; q++) {
            const double mid = 0.5 * (lo + hi);
            if (cut(mid) <= cus) hi = mid;
            else lo = mid;
        }
        cut(hi);
        c.parts = 1;
    }
    c.nreg = (int)reg.size() - 1;
    c.tmax = 0;
    for (int r = 0; r < c.nreg; r++) c.tmax = std::max(c.tmax, reg[(size_t)r + 1] - reg[(size_t)r]);
    double busiest = 0.0;       // entries of a block in the fullest region
    for (int r = 0; r < c.nreg; r++) {
        double sum = 0.0;
        for (int i = reg[(size_t)r]; i < reg[(size_t)r + 1]; i++) sum += w[(size_t)i] - 64.0;
        busiest = std::max(busiest, sum);
    }
    // On the fly too: the rows of all the buffers' chunks are formed first, three
    // waves to a SIMD, then the chain runs over them.  The two do not fit a CU
    // together, and each alone is so much faster than beside the other that row
    // formation overlapped with per-block launches loses: a cycle of 4 M rows of
    // 200x200x16 takes 19.6 ms against 23.0, 60 M of 256x256x32 349 against 372,
    // 2 M of 200x200x16 in chunks of 64 k 12.8 against 18.0, of 6,400 57 against 146.
    // So with several chunks the faster block decides, else a whole sweep's blocks.
    const bool several = ctx->cfg.path_mode == TVS_PATH_ON_THE_FLY && ctx->chunk_base.size() > 2;
    const double saved = launch_us(ctx, n, most - 64.0) - chain_us(n, cus, c.parts, busiest);
    if (several ? saved <= 0.0 : saved * nb <= kChainSweepUs) return false;
    c.first = reg;
    const size_t nexch = c.parts > 1 ? (size_t)c.nreg * c.parts * tvs::kChainExchBytes : 0;
    c.bytes = chain_bar_bytes(c.nreg) + nexch + 4 * c.first.size();
    c.planned = true;
    return true;
}

// The tiles that some block's lists cross (a tile outside the scanned
// object has no entry in any block), from the (block, tile) list lengths:
// the DROP steps launch one workgroup per such tile only, in order of
// decreasing entries over the scan, so that the longest lists are
// dispatched first and do not trail the step.  Workgroup i of a step takes
// slot i: tile act[i], whose lists are laid out in slot order (slot_of
// inverts act; -1 for a tile no list crosses).  Where the chain runs the slots
// are in the order of its regions instead, and workgroup i takes slot
// busiest[i]; the caller puts busiest into slot_of's memory when that has
// served.  Like every argument of the per-block launches it stays until the
// next load: a caller's graph may hold it.  At least one tile is kept, so that
// a step always has a workgroup to clear the next dot-product buffer.
int build_active_tiles(tvs_ctx *ctx, const uint32_t *btc, std::vector<int32_t> &busiest,
                       hipStream_t st)
{
    const int64_t nt = ctx->ntiles;
    uint32_t *total = nullptr;
    int rc = dalloc(ctx, &total, (size_t)std::max<int64_t>(nt, 1));
    if (rc) return rc;
    std::vector<uint32_t> f((size_t)std::max<int64_t>(nt, 1), 0u);
    hipError_t e = tvs::launch_tile_totals(btc, ctx->nblocks, nt, total, st);
    if (e == hipSuccess && nt > 0)
        e = hipMemcpyAsync(f.data(), total, sizeof(uint32_t) * nt, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    dfree(ctx, &total, (size_t)std::max<int64_t>(nt, 1));
    if (e != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("active tiles: ") + hipGetErrorString(e));
    std::vector<int32_t> a;
    for (int64_t T = 0; T < nt; T++)
        if (f[(size_t)T]) a.push_back((int32_t)T);
    auto busier = [&](int32_t x, int32_t y) { return f[(size_t)x] > f[(size_t)y]; };
    std::stable_sort(a.begin(), a.end(), busier);
    if (a.empty()) a.push_back(0);
    ctx->nact = (int64_t)a.size();
    busiest = a;
    std::vector<int32_t> placed = a;
    ctx->by_region = plan_chain(ctx, f, placed);
    if (ctx->by_region) a.swap(placed);
    std::vector<int32_t> inv((size_t)std::max<int64_t>(nt, 1), -1);
    for (size_t i = 0; i < a.size(); i++) inv[(size_t)a[i]] = (int32_t)i;
    for (int32_t &t : busiest) t = inv[(size_t)t];
    rc = dalloc(ctx, &ctx->act, a.size());
    if (!rc) rc = dalloc(ctx, &ctx->slot_of, inv.size());
    if (rc) return rc;
    e = hipMemcpyAsync(ctx->act, a.data(), sizeof(int32_t) * a.size(), hipMemcpyHostToDevice, st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ctx->slot_of, inv.data(), sizeof(int32_t) * inv.size(),
                           hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("active tiles: ") + hipGetErrorString(e));
    return TVS_OK;
}

// Threads per tile workgroup of the launches per block for the loaded lists.
// 128 on the fly with several chunks (they leave the row formation beside them
// more room).  Else 256 on grids of up to 16 tiles per CU, twice the
// workgroups of 256 that the device holds at once; on larger ones two more
// rounds of workgroups pay only where the lists are long: from 18 entries per
// crossed tile of a CU on.  Measured, us a block with 128 / 256 lanes (float32
// store, 6-byte store alike), crossed tiles per CU and entries of a list:
//   16.7: 151 11.4 / 12.6, 450 21.2 / 21.3, 590 25.9 / 25.4, 1209 43.5 / 41.0
//   26:   240 21.4 / 21.9, 472 32.8 / 30.8, 967 56.0 / 49.8
//   52:   236 35.5 / 39.9, 483 53.4 / 57.2, 967 92.8 / 92.6
//   66:   295 49.0 / 52.6, 604 79.8 / 82.0, 1207 148 / 142
//   208:  94 78.6 / 102, 387 168 / 190
int tile_lanes(const tvs_ctx *ctx)
{
    const bool otf = ctx->cfg.path_mode == TVS_PATH_ON_THE_FLY;
    if (otf && ctx->chunk_base.size() > 2) return 128;
    if (ctx->ntiles <= 16 * (int64_t)ctx->cus) return 256;
    const double nact = (double)ctx->nact;
    const double list = (double)ctx->nnz / ((double)std::max<int64_t>(ctx->nblocks, 1) * nact);
    return list >= 18.0 * nact / (double)ctx->cus ? 256 : 128;
}

// Lays out the tile lists of every block: row and segment counts, each
// segment's place in its (block, tile) list, the list starts.  Sets nnz,
// max_row, skipped, nseg, nblocks and the chunking.
int build_tile_lists(tvs_ctx *ctx, hipStream_t st)
{
    const int64_t n = ctx->nh, B = ctx->cfg.block_size;
    const int64_t nbt = ((n + B - 1) / B) * ctx->ntiles;
    int32_t *cnt = nullptr, *cseg = nullptr;
    uint32_t *btc = nullptr, *sbc = nullptr;   // list lengths by (block, tile), by (block, slot)
    int64_t nsbc = 0;
    int64_t *tmp = nullptr;
    // scan scratch, also the gathered block starts and, behind them, the row statistics
    const int64_t nblocks = (n + B - 1) / B;
    const int64_t ntmp = std::max(tvs::scan_tmp_elems(std::max(n, nbt)) + 1, nblocks + 2);
    auto cleanup = [&]() {
        dfree(ctx, &cnt, (size_t)std::max<int64_t>(n, 1));
        dfree(ctx, &cseg, (size_t)std::max<int64_t>(n, 1));
        dfree(ctx, &btc, (size_t)std::max<int64_t>(nbt, 1));
        dfree(ctx, &sbc, (size_t)std::max<int64_t>(nsbc, 1));
        dfree(ctx, &tmp, (size_t)ntmp);
    };
    int rc = dalloc(ctx, &cnt, (size_t)std::max<int64_t>(n, 1));
    if (!rc) rc = dalloc(ctx, &cseg, (size_t)std::max<int64_t>(n, 1));
    if (!rc) rc = dalloc(ctx, &tmp, (size_t)ntmp);
    if (rc) {
        cleanup();
        return rc;
    }
    HistDev hd = hist_dev(ctx);
    hipError_t e = tvs::launch_rows_count(ctx->gd, hd, ctx->mlp, 0, n, cnt, cseg, st);
    if (e == hipSuccess) e = tvs::launch_scan(cnt, n, ctx->row_off, tmp, st);
    if (e == hipSuccess) e = tvs::launch_scan(cseg, n, ctx->seg_off, tmp, st);
    // first entry of every block (and the end), segments, longest and empty rows
    std::vector<int64_t> off((size_t)nblocks + 1);
    int64_t nseg = 0;
    uint32_t stat[2] = {0, 0};
    uint32_t *dstat = reinterpret_cast<uint32_t *>(tmp + nblocks + 1);
    if (e == hipSuccess) e = hipMemsetAsync(dstat, 0, sizeof(stat), st);
    if (e == hipSuccess) e = tvs::launch_row_stats(cnt, n, dstat, st);
    if (e == hipSuccess && nblocks > 0) {
        e = tvs::launch_pick(ctx->row_off, B, nblocks, tmp, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(off.data(), tmp, sizeof(int64_t) * nblocks, hipMemcpyDeviceToHost, st);
    }
    if (e == hipSuccess)
        e = hipMemcpyAsync(&off[(size_t)nblocks], ctx->row_off + n, sizeof(int64_t),
                           hipMemcpyDeviceToHost, st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(&nseg, ctx->seg_off + n, sizeof(int64_t), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipMemcpyAsync(stat, dstat, sizeof(stat), hipMemcpyDeviceToHost, st);
    rc = dalloc(ctx, &ctx->order, (size_t)n);
    if (rc) {
        (void)hipStreamSynchronize(st);
        cleanup();
        return rc;
    }
    if (e == hipSuccess) e = tvs::launch_row_order(cnt, n, B, dstat, ctx->order, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
        cleanup();
        return fail(ctx, TVS_EDEVICE, std::string("row count: ") + hipGetErrorString(e));
    }
    dfree(ctx, &cnt, (size_t)std::max<int64_t>(n, 1));
    dfree(ctx, &cseg, (size_t)std::max<int64_t>(n, 1));
    const int64_t total = off[(size_t)nblocks];
    const int64_t mx = stat[0], sk = stat[1];
    ctx->nnz = total;
    ctx->max_row = mx;
    ctx->skipped = sk;
    ctx->nseg = nseg;
    ctx->nblocks = nblocks;
    int64_t chunk = ctx->cfg.chunk_histories;
    if (chunk <= 0) {
        // about 2^20 histories, as even as whole blocks allow: beside per-block
        // launches the row formation of the next sweep's first chunk waits for
        // them to leave that chunk's buffer, i.e. to finish the next-to-last
        // chunk, so a small last chunk would leave the formation stream idle
        const int64_t target = std::max<int64_t>(B, ((int64_t)1 << 20) / B * B);
        const int64_t parts = std::max<int64_t>(1, (n + target - 1) / target);
        chunk = ((n + parts - 1) / parts + B - 1) / B * B;
        chunk = std::max<int64_t>(chunk, B);
    } else {
        chunk = (chunk + B - 1) / B * B;
    }
    ctx->chunk = std::max<int64_t>(chunk, 1);
    for (int64_t f = 0; f < n; f += ctx->chunk)
        ctx->chunk_base.push_back(off[(size_t)(f / B)]);
    ctx->chunk_base.push_back(total);
    // integer ranges of the DROP sums: no voxel takes more than 2B entries of
    // one block, no row more than max_row entries
    ctx->big = 2097152.0 / (double)B;                              // 2^21 / B
    ctx->dot_max = 67108864.0 / (double)std::max<int64_t>(mx, 1);  // 2^26 / max_row

    rc = dalloc(ctx, &ctx->segtab, (size_t)nseg);
    if (!rc) rc = dalloc(ctx, &btc, (size_t)std::max<int64_t>(nbt, 1));
    if (rc) {
        cleanup();
        return rc;
    }
    e = hipMemsetAsync(btc, 0, sizeof(uint32_t) * std::max<int64_t>(nbt, 1), st);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->flags, 0, sizeof(uint32_t) * kNumFlags, st);
    if (e == hipSuccess)
        e = tvs::launch_rows_seg(ctx->gd, hd, ctx->mlp, n, B, ctx->seg_off, btc, ctx->segtab,
                                 ctx->flags + kFlagLists, ctx->flags + kFlagChordMax, ctx->order,
                                 st);
    if (e != hipSuccess) {
        cleanup();
        return fail(ctx, TVS_EDEVICE, std::string("tile lists: ") + hipGetErrorString(e));
    }
    // the dispatch slots, then the lists of every block laid out in slot
    // order: their bounds are at [b * nact + slot]
    std::vector<int32_t> busiest;
    rc = build_active_tiles(ctx, btc, busiest, st);
    if (!ctx->cfg.tile_threads && !ctx->tuned) ctx->threads = tile_lanes(ctx);
    nsbc = ctx->nblocks * ctx->nact;
    if (!rc) rc = dalloc(ctx, &ctx->bt_off, (size_t)bt_len(ctx));
    if (!rc) rc = dalloc(ctx, &sbc, (size_t)std::max<int64_t>(nsbc, 1));
    if (rc) {
        cleanup();
        return rc;
    }
    e = tvs::launch_slot_counts(btc, ctx->act, ctx->nact, ctx->nblocks, ctx->ntiles, sbc, st);
    if (e == hipSuccess)
        e = tvs::launch_scan(reinterpret_cast<const int32_t *>(sbc), nsbc, ctx->bt_off, tmp, st);
    if (e == hipSuccess)
        e = tvs::launch_seg_dest(ctx->gd, n, B, ctx->seg_off, ctx->bt_off, ctx->slot_of,
                                 ctx->nact, ctx->segtab, ctx->flags + kFlagLists, st);
    if (e == hipSuccess && ctx->by_region)
        e = hipMemcpyAsync(ctx->slot_of, busiest.data(), sizeof(int32_t) * busiest.size(),
                           hipMemcpyHostToDevice, st);
    // every block's lists must add up to the block's entries (the block
    // starts are gathered into the freed count buffer, then copied)
    std::vector<int64_t> starts((size_t)ctx->nblocks + 1);
    if (e == hipSuccess && ctx->nblocks > 0)
        e = tvs::launch_pick(ctx->bt_off, ctx->nact, ctx->nblocks + 1, tmp, st);
    if (e == hipSuccess && ctx->nblocks > 0)
        e = hipMemcpyAsync(starts.data(), tmp, sizeof(int64_t) * (ctx->nblocks + 1),
                           hipMemcpyDeviceToHost, st);
    uint32_t fl[kNumFlags] = {};
    if (e == hipSuccess)
        e = hipMemcpyAsync(fl, ctx->flags, sizeof(fl), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    cleanup();
    if (e != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("tile lists: ") + hipGetErrorString(e));
    if (fl[kFlagLists])
        return fail(ctx, TVS_EDEVICE, "tile lists: a row walk disagreed with the count pass");
    std::memcpy(&ctx->chord_max, &fl[kFlagChordMax], sizeof(float));
    for (int64_t b = 0; b <= ctx->nblocks && ctx->nblocks > 0; b++) {
        const int64_t want = off[(size_t)b];
        if (starts[(size_t)b] != want)
            return fail(ctx, TVS_EDEVICE,
                        "tile lists disagree with the row lengths at block " + std::to_string(b) +
                            " of " + std::to_string(ctx->nblocks) + ": " +
                            std::to_string(starts[(size_t)b]) + " != " + std::to_string(want));
    }
    return TVS_OK;
}

// Allocates the entry buffers and, for a path store, forms every row now.
int form_entries(tvs_ctx *ctx, hipStream_t st)
{
    const bool otf = ctx->cfg.path_mode == TVS_PATH_ON_THE_FLY;
    int64_t cap = ctx->nnz;
    if (otf) {
        cap = 0;
        for (size_t q = 0; q + 1 < ctx->chunk_base.size(); q++)
            cap = std::max(cap, ctx->chunk_base[q + 1] - ctx->chunk_base[q]);
    }
    ctx->cap = std::max<int64_t>(cap, 1);
    const int64_t nchunks = (int64_t)ctx->chunk_base.size() - 1;
    ctx->nbuf = otf ? (int)std::max<int64_t>(1, std::min<int64_t>(kChunkBuffers, nchunks)) : 1;
    ctx->cbase = 0;
    const size_t all = (size_t)(ctx->nbuf * ctx->cap);
    int rc = dalloc(ctx, &ctx->meta[0], all);
    if (!rc) {
        if (ctx->cfg.path_mode == TVS_PATH_STORE_F16) rc = dalloc(ctx, &ctx->ch16, all);
        else if (ctx->cfg.path_mode == TVS_PATH_STORE_Q16) rc = dalloc(ctx, &ctx->chq, all);
        else rc = dalloc(ctx, &ctx->ch32[0], all);
    }
    // entries start as (row 0, word 0, chord 0): never an index out of range
    if (!rc) HIPCHK(hipMemsetAsync(ctx->meta[0], 0, sizeof(uint32_t) * all, st));
    if (!rc && ctx->ch32[0]) HIPCHK(hipMemsetAsync(ctx->ch32[0], 0, sizeof(float) * all, st));
    for (int q = 1; q < ctx->nbuf && !rc; q++) {
        ctx->meta[q] = ctx->meta[0] + q * ctx->cap;
        if (ctx->ch32[0]) ctx->ch32[q] = ctx->ch32[0] + q * ctx->cap;
    }
    if (!rc && ctx->ch16) HIPCHK(hipMemsetAsync(ctx->ch16, 0, sizeof(__half) * ctx->cap, st));
    if (!rc && ctx->chq) HIPCHK(hipMemsetAsync(ctx->chq, 0, sizeof(uint16_t) * ctx->cap, st));
    if (rc) return rc;
    if (ctx->chq) {
        // fixed-point chords: rb bits of a tag hold the row within its block
        // (B rows), the 24 - rb above them the code's high bits, so a code
        // has 16 + 24 - rb bits (at most 30); the unit is the longest chord /
        // the largest code, made a little larger so that the longest chord's
        // code stays in range after rounding
        const uint32_t B = (uint32_t)ctx->cfg.block_size;
        uint32_t rb = 0;
        while (rb < 24 && ((uint32_t)1 << rb) < B) rb++;
        const uint32_t bits = std::min<uint32_t>(30, 16 + (24 - rb));
        ctx->rowmask = rb ? (((uint32_t)1 << rb) - 1u) : 0u;
        ctx->qshift = kTileShiftHost + rb;
        ctx->qmax = (uint32_t)(((uint64_t)1 << bits) - 1u);
        const double m = ctx->chord_max > 0.0f ? (double)ctx->chord_max : 1.0;
        ctx->qunit = m * (1.0 + 1.0 / 1048576.0) / (double)ctx->qmax;
        ctx->qinv = 1.0 / ctx->qunit;
    }
    if (otf) {
        // the first sweep's row formation runs on the fill stream: it must
        // not start before these clears, or they overwrite formed entries
        for (int q = 0; q < kChunkBuffers; q++) HIPCHK(hipEventRecord(ctx->ev_free[q], st));
        return TVS_OK;
    }
    if (ctx->nh == 0) return TVS_OK;
    tvs::TileFill f;
    f.first = 0;
    f.n = ctx->nh;
    f.B = ctx->cfg.block_size;
    f.seg_off = ctx->seg_off;
    f.segdst = reinterpret_cast<const int64_t *>(ctx->segtab);
    f.base = 0;
    f.meta = ctx->meta[0];
    f.ch32 = ctx->ch32[0];
    f.ch16 = ctx->ch16;
    f.chq = ctx->chq;
    f.qinv = ctx->qinv;
    f.qmax = ctx->qmax;
    f.qshift = ctx->qshift;
    f.cap = ctx->cap;
    f.norm2 = ctx->norm2;
    f.err = ctx->flags + kFlagLists;
    f.order = ctx->order;
    hipError_t e = tvs::launch_rows_fill_tiled(ctx->gd, hist_dev(ctx), ctx->mlp, f, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("row fill: ") + hipGetErrorString(e));
    return check_flags(ctx, st);
}

}  // namespace

extern "C" {

void tvs_config_default(tvs_config *cfg)
{
    if (!cfg) return;
    std::memset(cfg, 0, sizeof(*cfg));
    cfg->block_size = 3200;
    cfg->path_mode = TVS_PATH_ON_THE_FLY;
    cfg->mlp_step_mm = 0.0;
    cfg->mlp_log_term = 1;
    cfg->mlp_const_power = 0;
    cfg->chunk_histories = 0;
    cfg->hbm_budget_bytes = 0;
    cfg->device = 0;
    cfg->max_tries = 0;
    cfg->sweep_kernel = 0;
    cfg->tile_threads = 0;
    cfg->time_sample = 0;
    cfg->fill_wgs_per_cu = 0;
    cfg->fill_wide_pct = -1;
}

const char *tvs_strerror(int status)
{
    switch (status) {
    case TVS_OK: return "ok";
    case TVS_EINVAL: return "invalid argument";
    case TVS_ENOMEM: return "out of device memory or HBM budget";
    case TVS_EDEVICE: return "HIP device error";
    case TVS_ESTATE: return "call out of order";
    case TVS_ERANGE: return "index, size or value out of range";
    default: return "unknown status";
    }
}

const char *tvs_last_error(tvs_ctx *ctx) { return ctx ? ctx->err.c_str() : ""; }

void tvs_destroy(tvs_ctx *ctx)
{
    if (!ctx) return;
    (void)hipSetDevice(ctx->cfg.device);
    if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
    if (ctx->fill_stream) (void)hipStreamSynchronize(ctx->fill_stream);
    free_histories(ctx);
    free_batch(ctx);
    dfree(ctx, &ctx->x0, (size_t)ctx->nvox);
    dfree(ctx, &ctx->x, (size_t)ctx->nvox);
    dfree(ctx, &ctx->xio, (size_t)ctx->nvox);
    dfree(ctx, &ctx->g, (size_t)ctx->nvox);
    dfree(ctx, &ctx->flags, (size_t)kNumFlags);
    dfree(ctx, &ctx->dot, (size_t)(3 * (int64_t)ctx->cfg.block_size));
    dfree(ctx, &ctx->part, (size_t)ctx->nparts);
    dfree(ctx, &ctx->dec, (size_t)2);
    dfree(ctx, &ctx->ticket, (size_t)1);
    dfree(ctx, &ctx->sched, (size_t)1);
    dfree(ctx, &ctx->dlog, (size_t)kDevLogCap);
    dfree(ctx, &ctx->cpart, (size_t)tvs::tv_check_parts(ctx->gd));
    if (ctx->ev_sched) (void)hipEventDestroy(ctx->ev_sched);
    for (auto &e : ctx->tev)
        if (e) (void)hipEventDestroy(e);
    for (int q = 0; q < kChunkBuffers; q++) {
        if (ctx->ev_filled[q]) (void)hipEventDestroy(ctx->ev_filled[q]);
        if (ctx->ev_free[q]) (void)hipEventDestroy(ctx->ev_free[q]);
        if (ctx->bev_filled[q]) (void)hipEventDestroy(ctx->bev_filled[q]);
        if (ctx->bev_free[q]) (void)hipEventDestroy(ctx->bev_free[q]);
    }
    if (ctx->bev_fork) (void)hipEventDestroy(ctx->bev_fork);
    if (ctx->fill_stream) (void)hipStreamDestroy(ctx->fill_stream);
    if (ctx->stream) (void)hipStreamDestroy(ctx->stream);
    delete ctx;
}

int tvs_create(const tvs_grid *grid, const tvs_config *cfg_in, tvs_ctx **out)
{
    tvs_ctx *ctx = nullptr;
    if (!out) return TVS_EINVAL;
    *out = nullptr;
    if (!grid) return TVS_EINVAL;
    tvs_config cfg;
    if (cfg_in) cfg = *cfg_in;
    else tvs_config_default(&cfg);
    if (grid->nx <= 0 || grid->ny <= 0 || grid->nz <= 0) return TVS_EINVAL;
    if (!finite_pos(grid->vx) || !finite_pos(grid->vy) || !finite_pos(grid->vz)) return TVS_EINVAL;
    if (!std::isfinite(grid->ox) || !std::isfinite(grid->oy) || !std::isfinite(grid->oz))
        return TVS_EINVAL;
    if (grid->nx >= (1 << 20) || grid->ny >= (1 << 20) || grid->nz >= (1 << 20)) return TVS_EINVAL;
    const tvs::GridDev gdev = tvs::make_grid_dev(*grid);
    const int64_t nimg = (int64_t)grid->nx * grid->ny * grid->nz;
    const int64_t nvox = tvs::padded_voxels(gdev);     // device image words (tiled layout)
    if (nvox >= ((int64_t)1 << 31)) return TVS_EINVAL;
    if (cfg.block_size < 1 || cfg.block_size > (1 << 24)) return TVS_EINVAL;
    if (cfg.path_mode < 0 || cfg.path_mode > 3) return TVS_EINVAL;
    // the fixed-point store keeps at least 4 code bits in each tag
    if (cfg.path_mode == TVS_PATH_STORE_Q16 && cfg.block_size > (1 << 20)) return TVS_EINVAL;
    if (!std::isfinite(cfg.mlp_step_mm)) return TVS_EINVAL;
    if (cfg.chunk_histories < 0 || cfg.max_tries < 0) return TVS_EINVAL;
    if (cfg.sweep_kernel < 0 || cfg.sweep_kernel > 2) return TVS_EINVAL;
    if (cfg.tile_threads != 0 && cfg.tile_threads != 64 && cfg.tile_threads != 128 &&
        cfg.tile_threads != 256)
        return TVS_EINVAL;
    if (cfg.time_sample < 0) return TVS_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || cfg.device < 0 || cfg.device >= ndev)
        return TVS_EDEVICE;
    if (hipSetDevice(cfg.device) != hipSuccess) return TVS_EDEVICE;
    fbp_scratch_setup(cfg.device);

    ctx = new tvs_ctx();
    ctx->grid = *grid;
    ctx->cfg = cfg;
    ctx->gd = gdev;
    ctx->nimg = nimg;
    ctx->nvox = nvox;
    ctx->ntiles = tvs::num_tiles(gdev);
    double step = cfg.mlp_step_mm > 0.0 ? cfg.mlp_step_mm : std::min(grid->vx, grid->vy);
    ctx->mlp = tvs::MlpCfg{step, cfg.mlp_log_term ? 1 : 0, cfg.mlp_const_power ? 1 : 0};
    if (ctx->cfg.max_tries == 0) ctx->cfg.max_tries = 100000;
    ctx->split = (cfg.sweep_kernel == 2) ? 1 : 0;
    {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, cfg.device) !=
            hipSuccess)
            cus = 0;
        if (cus > 0) ctx->cus = cus;
        const int per_cu = cfg.fill_wgs_per_cu;
        ctx->fill_wgs = (per_cu > 0 && cus > 0) ? (int64_t)per_cu * cus : 0;
        // the library's choice: about 40 % of the chunks at full occupancy
        // (within a few % of the best share at 200x200x16 and 256x256x32;
        // tvs_autotune times the shares on the loaded histories)
        ctx->fill_wide_pct = cfg.fill_wide_pct < 0 ? 40 : std::min(cfg.fill_wide_pct, 100);
        // (0: tile_lanes at every load)
        ctx->threads = cfg.tile_threads ? cfg.tile_threads : 256;
    }

    size_t freeb = 0, totalb = 0;
    if (hipMemGetInfo(&freeb, &totalb) != hipSuccess) {
        delete ctx;
        return TVS_EDEVICE;
    }
    ctx->budget = cfg.hbm_budget_bytes ? cfg.hbm_budget_bytes : (uint64_t)(0.8 * (double)freeb);

    int rc = TVS_OK;
    ctx->nparts = tvs::tv_num_parts(ctx->gd);
    if (!rc) rc = dalloc(ctx, &ctx->x, (size_t)nvox);
    if (!rc) rc = dalloc(ctx, &ctx->x0, (size_t)nvox);
    if (!rc) rc = dalloc(ctx, &ctx->xio, (size_t)nvox);
    if (!rc) rc = dalloc(ctx, &ctx->g, (size_t)nvox);
    if (!rc) rc = dalloc(ctx, &ctx->flags, (size_t)kNumFlags);
    if (!rc) rc = dalloc(ctx, &ctx->dot, (size_t)(3 * (int64_t)cfg.block_size));
    if (!rc) rc = dalloc(ctx, &ctx->part, (size_t)ctx->nparts);
    if (!rc) rc = dalloc(ctx, &ctx->dec, (size_t)2);
    if (!rc) rc = dalloc(ctx, &ctx->ticket, (size_t)1);
    if (!rc) rc = dalloc(ctx, &ctx->sched, (size_t)1);
    if (!rc) rc = dalloc(ctx, &ctx->dlog, (size_t)kDevLogCap);
    if (!rc) rc = dalloc(ctx, &ctx->cpart, (size_t)tvs::tv_check_parts(ctx->gd));
    if (rc) {
        tvs_destroy(ctx);
        return rc;
    }
    if (hipEventCreateWithFlags(&ctx->ev_sched, hipEventDisableTiming) != hipSuccess) {
        tvs_destroy(ctx);
        return TVS_EDEVICE;
    }
    if (hipStreamCreateWithFlags(&ctx->stream, hipStreamNonBlocking) != hipSuccess ||
        hipStreamCreateWithFlags(&ctx->fill_stream, hipStreamNonBlocking) != hipSuccess) {
        tvs_destroy(ctx);
        return TVS_EDEVICE;
    }
    for (int q = 0; q < kChunkBuffers; q++) {
        if (hipEventCreateWithFlags(&ctx->ev_filled[q], hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&ctx->ev_free[q], hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&ctx->bev_filled[q], hipEventDisableTiming) != hipSuccess ||
            hipEventCreateWithFlags(&ctx->bev_free[q], hipEventDisableTiming) != hipSuccess ||
            hipEventRecord(ctx->ev_free[q], ctx->stream) != hipSuccess) {
            tvs_destroy(ctx);
            return TVS_EDEVICE;
        }
    }
    if (hipEventCreateWithFlags(&ctx->bev_fork, hipEventDisableTiming) != hipSuccess) {
        tvs_destroy(ctx);
        return TVS_EDEVICE;
    }
    hipError_t e = hipSuccess;
    if (e == hipSuccess) e = hipMemsetAsync(ctx->x, 0, sizeof(double) * nvox, ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->x0, 0, sizeof(double) * nvox, ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->g, 0, sizeof(double) * nvox, ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->flags, 0, sizeof(uint32_t) * kNumFlags, ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->ticket, 0, sizeof(uint32_t), ctx->stream);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->dec, 0, sizeof(double) * 2, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (e != hipSuccess) {
        tvs_destroy(ctx);
        return TVS_EDEVICE;
    }
    *out = ctx;
    return TVS_OK;
}

int tvs_load_histories(tvs_ctx *ctx, int64_t n, const tvs_histories *h, int on_device, void *stream)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    if (n < 0) return fail(ctx, TVS_EINVAL, "n must be >= 0");
    if (n >= ((int64_t)1 << 31)) return fail(ctx, TVS_EINVAL, "at most 2^31 - 1 histories");
    if (n > 0 && !h) return fail(ctx, TVS_EINVAL, "histories is NULL");
    const float *src[kNumStreams] = {};
    if (n > 0) {
        const float *tmp[kNumStreams] = {h->ex,  h->ey,  h->ez, h->qx, h->qy, h->qz, h->eth,
                                         h->eps, h->qth, h->qps, h->ux, h->uy, h->wepl};
        for (int q = 0; q < kNumStreams; q++) {
            if (!tmp[q]) return fail(ctx, TVS_EINVAL, "a history stream is NULL");
            src[q] = tmp[q];
        }
    }
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    HIPCHK(hipStreamSynchronize(st));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    HIPCHK(hipStreamSynchronize(ctx->fill_stream));
    // Allocations given back in this call serve its next ones of the same size
    // (a new scan of the same shape, and the temporaries: an allocation and its
    // release take 0.1 to 0.4 ms) and are freed at its end.  Work of any stream
    // on the old ones ends first, as hipFree would have seen to.
    if (ctx->hist) HIPCHK(hipDeviceSynchronize());
    struct Recycle {
        tvs_ctx *c;
        ~Recycle()
        {
            c->recycle = false;
            drop_spare(c);
        }
    } recycle{ctx};
    ctx->recycle = true;
    ChainBack back{ctx};
    free_histories(ctx);
    reset_state(ctx);
    HIPCHK(hipMemsetAsync(ctx->x, 0, sizeof(double) * ctx->nvox, st));
    HIPCHK(hipMemsetAsync(ctx->x0, 0, sizeof(double) * ctx->nvox, st));
    HIPCHK(hipMemsetAsync(ctx->flags, 0, sizeof(uint32_t) * kNumFlags, st));
    ctx->batch.valid = false;
    ctx->nh = n;

    int rc = dalloc(ctx, &ctx->hist, (size_t)(kNumStreams * n));
    if (!rc) rc = dalloc(ctx, &ctx->row_off, (size_t)(n + 1));
    if (!rc) rc = dalloc(ctx, &ctx->norm2, (size_t)n);
    if (!rc) rc = dalloc(ctx, &ctx->seg_off, (size_t)(n + 1));
    if (rc) {
        free_histories(ctx);
        return rc;
    }
    hipMemcpyKind kind = on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    for (int q = 0; q < kNumStreams && n > 0; q++) {
        hipError_t e = hipMemcpyAsync(ctx->hist + q * n, src[q], sizeof(float) * n, kind, st);
        if (e != hipSuccess) {
            free_histories(ctx);
            return fail(ctx, TVS_EDEVICE, std::string("history copy: ") + hipGetErrorString(e));
        }
    }
    // validation on the device (the inputs may live there already)
    uint32_t bad = 0, jmax = 0;
    {
        hipError_t e = tvs::launch_validate(hist_dev(ctx), n, ctx->mlp.step,
                                            ctx->flags + kFlagInvalid, ctx->flags + kFlagJmax, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(&bad, ctx->flags + kFlagInvalid, sizeof(uint32_t),
                               hipMemcpyDeviceToHost, st);
        if (e == hipSuccess)
            e = hipMemcpyAsync(&jmax, ctx->flags + kFlagJmax, sizeof(uint32_t),
                               hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) {
            free_histories(ctx);
            return fail(ctx, TVS_EDEVICE, std::string("validation: ") + hipGetErrorString(e));
        }
    }
    if (bad) {
        free_histories(ctx);
        (void)hipMemsetAsync(ctx->flags, 0, sizeof(uint32_t) * kNumFlags, st);
        return fail(ctx, TVS_EINVAL,
                    std::to_string(bad) + " histories hold NaN/inf, |value| > 1e6, a zero beam "
                                          "axis or more than 2^20 MLP vertices");
    }
    // entry-side MLP table for every vertex depth of these histories
    if (jmax > 0) {
        rc = dalloc(ctx, &ctx->s1i, (size_t)(3 * (int64_t)jmax));
        if (!rc) {
            ctx->nj = jmax;
            hipError_t e = tvs::launch_mlp_table(ctx->mlp, ctx->nj, ctx->s1i, st);
            if (e != hipSuccess) rc = fail(ctx, TVS_EDEVICE, std::string("MLP table: ") + hipGetErrorString(e));
            ctx->mlp.s1i = ctx->s1i;
            ctx->mlp.nj = ctx->nj;
            ctx->mlp.err = ctx->flags + kFlagLists;
        }
        if (rc) {
            std::string msg = ctx->err;
            free_histories(ctx);
            return fail(ctx, rc, msg);
        }
    }
    // the tile lists of every block (their layout; rows themselves are
    // formed now for a path store, per chunk and sweep otherwise)
    rc = build_tile_lists(ctx, st);
    if (!rc) rc = form_entries(ctx, st);
    if (rc) {
        std::string msg = ctx->err;
        free_histories(ctx);
        return fail(ctx, rc, msg);
    }
    ctx->loaded = true;
    ctx->timed = false;
    ctx->spans.clear();
    return TVS_OK;
}

int tvs_set_image(tvs_ctx *ctx, const float *x0, int on_device, void *stream)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    if (!x0) return fail(ctx, TVS_EINVAL, "image is NULL");
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    if (!on_device) {
        for (int64_t j = 0; j < ctx->nimg; j++)
            if (!std::isfinite(x0[j])) return fail(ctx, TVS_EINVAL, "image holds NaN/inf");
    }
    HIPCHK(hipMemcpyAsync(ctx->xio, x0, sizeof(float) * ctx->nimg,
                          on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, st));
    HIPCHK(tvs::launch_widen(ctx->gd, ctx->xio, ctx->x, st));
    HIPCHK(hipMemcpyAsync(ctx->x0, ctx->x, sizeof(double) * ctx->nvox, hipMemcpyDeviceToDevice, st));
    HIPCHK(hipMemsetAsync(ctx->flags + kFlagRange, 0, sizeof(uint32_t), st));
    if (!on_device) HIPCHK(hipStreamSynchronize(st));
    reset_state(ctx);
    ctx->batch.valid = false;
    return TVS_OK;
}

}  // extern "C"

namespace {

// Checks the FBP parameters against the context and sizes the bins: lateral
// bin width tau, nt lateral bins (2 ceil(R / tau) + 2, R the farthest slice
// corner from the axis), nb = A * nz * nt bins.
int fbp_geometry(tvs_ctx *ctx, const tvs_fbp_params *p, const char *who, double &tau,
                 int32_t &nt, int64_t &nb)
{
    if (!p) return fail(ctx, TVS_EINVAL, "params is NULL");
    if (p->n_angles < 1) return fail(ctx, TVS_EINVAL, "n_angles must be >= 1");
    if (!(p->t_bin_mm >= 0.0) || !std::isfinite(p->t_bin_mm))
        return fail(ctx, TVS_EINVAL, "t_bin_mm must be finite and >= 0");
    if (p->median_radius < 0 || p->median_radius > 2)
        return fail(ctx, TVS_EINVAL, "median_radius must lie in 0..2");
    if (!ctx->loaded) return fail(ctx, TVS_ESTATE, std::string(who) + " before tvs_load_histories");
    const tvs_grid &g = ctx->grid;
    tau = p->t_bin_mm > 0.0 ? p->t_bin_mm : g.vx;
    double R = 0.0;
    for (int cx = 0; cx < 2; cx++)
        for (int cy = 0; cy < 2; cy++)
            R = std::max(R, std::hypot(g.ox + cx * g.nx * g.vx, g.oy + cy * g.ny * g.vy));
    const double ntd = 2.0 * std::ceil(R / tau) + 2.0;
    if (!(ntd <= 16777216.0)) return fail(ctx, TVS_EINVAL, "t_bin_mm too small for the grid");
    nt = (int32_t)ntd;
    nb = (int64_t)p->n_angles * g.nz * nt;
    return TVS_OK;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

extern "C" {

int tvs_initial_fbp(tvs_ctx *ctx, const tvs_fbp_params *p, float *out, int on_device, void *stream)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    double tau = 0.0;
    int32_t nt = 0;
    int64_t nb = 0;
    int rc = fbp_geometry(ctx, p, "tvs_initial_fbp", tau, nt, nb);
    if (rc) return rc;
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    const tvs_grid &g = ctx->grid;
    const int32_t A = p->n_angles;

    // one allocation: 20 B per bin (a sum and a count each, then the filter's
    // taps; the filtered projections over the former), the means, the angle
    // table, the image.  nt is even.
    const size_t words = (size_t)nb / 2 * 5 + (size_t)nb + (size_t)(2 * A) + (size_t)ctx->nimg;
    double *work = nullptr;
    ChainBack back{ctx};
    rc = dalloc(ctx, &work, words);
    if (rc) return rc;
    auto *slots = reinterpret_cast<unsigned long long *>(work);
    double *qb = work, *taps = work + 2 * nb, *pb = work + nb / 2 * 5, *cs = pb + nb;
    double *img = cs + 2 * A;
    // cos, sin of every beam angle a * 2 pi / A
    std::vector<double> tab((size_t)(2 * A));
    const double da = 2.0 * 3.14159265358979323846 / (double)A;
    for (int32_t a = 0; a < A; a++) {
        const double phi = (double)a * da;
        tab[(size_t)(2 * a)] = std::cos(phi);
        tab[(size_t)(2 * a + 1)] = std::sin(phi);
    }
    hipError_t e = hipMemsetAsync(slots, 0, sizeof(unsigned long long) * 2 * nb, st);
    if (e == hipSuccess) e = hipMemcpyAsync(cs, tab.data(), sizeof(double) * 2 * A, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = tvs::launch_fbp_bin(ctx->gd, hist_dev(ctx), ctx->nh, A, tau, nt, ctx->cus, slots, st);
    if (e == hipSuccess) e = tvs::launch_fbp_filter(slots, (int64_t)A * g.nz, nt, tau, taps, pb, st);
    if (e == hipSuccess)
        e = tvs::launch_fbp_backproject(ctx->gd, qb, cs, A, tau, nt, p->clip_negative ? 1 : 0, img, st);
    if (e == hipSuccess) e = tvs::launch_median(ctx->gd, img, p->median_radius, ctx->xio, st);
    // the result becomes the context image, as by tvs_set_image
    if (e == hipSuccess) e = tvs::launch_widen(ctx->gd, ctx->xio, ctx->x, st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ctx->x0, ctx->x, sizeof(double) * ctx->nvox, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess) e = hipMemsetAsync(ctx->flags + kFlagRange, 0, sizeof(uint32_t), st);
    if (e == hipSuccess && out)
        e = hipMemcpyAsync(out, ctx->xio, sizeof(float) * ctx->nimg,
                           on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    dfree(ctx, &work, words);
    if (e != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("initial fbp: ") + hipGetErrorString(e));
    reset_state(ctx);
    ctx->batch.valid = false;
    return TVS_OK;
}

int tvs_initial_fbp_noalloc(tvs_ctx *ctx, const tvs_fbp_params *p, float *out, int on_device,
                            void *stream)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    double tau = 0.0;
    int32_t nt = 0;
    int64_t nb = 0;
    int rc = fbp_geometry(ctx, p, "tvs_initial_fbp_noalloc", tau, nt, nb);
    if (rc) return rc;
    const int32_t A = p->n_angles;
    // workspace layout: bin sums and counts (cleared) in 16 of the 20 B per bin
    // up to o_pb, the filter's taps behind them, the filtered projections over
    // the former, means, angle table, backprojected image; each part 256-aligned
    const size_t nbw = align256(sizeof(double) * (size_t)nb);
    const size_t o_pb = 2 * nbw + align256(sizeof(uint32_t) * (size_t)nb);
    const size_t o_cs = o_pb + nbw;
    const size_t o_img = o_cs + align256(sizeof(double) * 2 * (size_t)A);
    const size_t need = o_img + align256(sizeof(double) * (size_t)ctx->nimg);
    if (need > kFbpScratchBytes)
        return fail(ctx, TVS_ERANGE,
                    "tvs_initial_fbp_noalloc needs " + std::to_string(need) +
                        " B of workspace (" + std::to_string(nb) + " bins, " +
                        std::to_string(ctx->nimg) + " voxels); its fixed workspace holds " +
                        std::to_string(kFbpScratchBytes) + " B");
    const int dev = ctx->cfg.device;
    if (dev < 0 || dev >= kMaxDevices)
        return fail(ctx, TVS_EDEVICE, "device ordinal beyond the workspace table");
    HIPCHK(hipSetDevice(dev));
    fbp_scratch_setup(dev);
    unsigned char *base = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        if (!g_scratch_ptr[dev])
            return fail(ctx, TVS_EDEVICE,
                        std::string("workspace address lookup failed: ") +
                            hipGetErrorString(g_scratch_status[dev]));
        base = static_cast<unsigned char *>(g_scratch_ptr[dev]);
    }
    hipStream_t st = pick(ctx, stream);
    auto *slots = reinterpret_cast<unsigned long long *>(base);
    auto *taps = reinterpret_cast<double *>(slots + 2 * nb);
    auto *qb = reinterpret_cast<double *>(base), *pb = reinterpret_cast<double *>(base + o_pb);
    auto *cs = reinterpret_cast<double *>(base + o_cs);
    auto *img = reinterpret_cast<double *>(base + o_img);
    const tvs_grid &g = ctx->grid;
    // sums and counts start at zero (a fill kernel: the workspace keeps the
    // previous call's contents)
    hipError_t e = tvs::launch_zero_i64(reinterpret_cast<long long *>(slots), 2 * nb, st);
    if (e == hipSuccess) e = tvs::launch_fbp_angles(A, cs, st);
    if (e == hipSuccess) e = tvs::launch_fbp_bin(ctx->gd, hist_dev(ctx), ctx->nh, A, tau, nt, ctx->cus, slots, st);
    if (e == hipSuccess) e = tvs::launch_fbp_filter(slots, (int64_t)A * g.nz, nt, tau, taps, pb, st);
    if (e == hipSuccess)
        e = tvs::launch_fbp_backproject(ctx->gd, qb, cs, A, tau, nt, p->clip_negative ? 1 : 0, img, st);
    if (e == hipSuccess) e = tvs::launch_median(ctx->gd, img, p->median_radius, ctx->xio, st);
    if (e == hipSuccess) e = tvs::launch_widen(ctx->gd, ctx->xio, ctx->x, st);
    if (e == hipSuccess)
        e = hipMemcpyAsync(ctx->x0, ctx->x, sizeof(double) * ctx->nvox, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess)
        e = tvs::launch_set_counter(reinterpret_cast<int32_t *>(ctx->flags + kFlagRange), 0, st);
    if (e == hipSuccess && out)
        e = hipMemcpyAsync(out, ctx->xio, sizeof(float) * ctx->nimg,
                           on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, st);
    if (e == hipSuccess && out && !on_device) e = hipStreamSynchronize(st);
    if (e != hipSuccess)
        return fail(ctx, TVS_EDEVICE, std::string("initial fbp (no-alloc): ") + hipGetErrorString(e));
    reset_state(ctx);
    ctx->batch.valid = false;
    return TVS_OK;
}

int tvs_hull_detect(tvs_ctx *ctx, const tvs_hull_params *p, uint8_t *hull, int on_device,
                    void *stream)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    if (!p) return fail(ctx, TVS_EINVAL, "params is NULL");
    if (p->min_in < 0 || p->max_out < 0) return fail(ctx, TVS_EINVAL, "min_in and max_out must be >= 0");
    if (std::isnan(p->wepl_in_mm) || std::isnan(p->wepl_out_mm))
        return fail(ctx, TVS_EINVAL, "WEPL thresholds must not be NaN");
    if (!ctx->loaded) return fail(ctx, TVS_ESTATE, "tvs_hull_detect before tvs_load_histories");
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    uint32_t *cnt = nullptr;
    uint8_t *hd = nullptr;
    // the mask's buffer holds the full-voxel bits until the mask is written
    const size_t nhd = std::max((size_t)ctx->nimg, (size_t)(4 * tvs::hull_full_words(ctx->gd)));
    ChainBack back{ctx};
    int rc = dalloc(ctx, &cnt, (size_t)(2 * ctx->nimg));
    if (!rc) rc = dalloc(ctx, &hd, nhd);
    if (rc) {
        dfree(ctx, &cnt, (size_t)(2 * ctx->nimg));
        return rc;
    }
    // the counting threshold -inf when space modelling is off makes every
    // line count; min_in = 0 then accepts every voxel on that side
    hipError_t e = hipMemsetAsync(cnt, 0, sizeof(uint32_t) * 2 * ctx->nimg, st);
    if (e == hipSuccess)
        e = tvs::launch_hull_counts(ctx->gd, hist_dev(ctx), ctx->nh, p->wepl_in_mm, p->wepl_out_mm,
                                    cnt, cnt + ctx->nimg, (uint32_t)p->min_in,
                                    (uint32_t)p->max_out + 1u, reinterpret_cast<uint32_t *>(hd), st);
    if (e == hipSuccess)
        e = tvs::launch_hull_decide(ctx->gd, cnt, cnt + ctx->nimg, (uint32_t)p->min_in,
                                    (uint32_t)p->max_out, hd, p->mask_image ? ctx->x : nullptr, st);
    if (e == hipSuccess && p->mask_image)
        e = hipMemcpyAsync(ctx->x0, ctx->x, sizeof(double) * ctx->nvox, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess && hull)
        e = hipMemcpyAsync(hull, hd, (size_t)ctx->nimg,
                           on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    dfree(ctx, &cnt, (size_t)(2 * ctx->nimg));
    dfree(ctx, &hd, nhd);
    if (e != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("hull: ") + hipGetErrorString(e));
    if (p->mask_image) {
        reset_state(ctx);
        ctx->batch.valid = false;
    }
    return TVS_OK;
}

int tvs_iterate(tvs_ctx *ctx, const tvs_params *p, int32_t K, void *stream)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    int rc = validate_params(ctx, p);
    if (rc) return rc;
    if (K < 0) return fail(ctx, TVS_EINVAL, "K must be >= 0");
    if (!ctx->loaded) return fail(ctx, TVS_ESTATE, "tvs_iterate before tvs_load_histories");
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    tvs::TvBuffers tb = tv_bufs(ctx);
    if (!ctx->seeded) {
        ctx->rng = p->seed;
        ctx->seeded = true;
    }
    const bool checked = (p->variant == TVS_OTVS) || (p->variant == TVS_NTVS && p->tv_check);
    const int32_t nsteps = (p->variant == TVS_OTVS) ? 1 : p->N;
    // unchecked steps take ell from the host: bring a device-held schedule back
    if (!checked) {
        rc = settle_sched(ctx);
        if (rc) return rc;
    }
    if (K > 0) {
        ctx->tev_used = 0;
        ctx->spans.clear();
        ctx->timed = true;
    }
    const tvs::CheckBuffers cb{ctx->cpart, ctx->ticket, ctx->dec};
    const double check_alpha = (p->variant == TVS_OTVS) ? 0.5 : p->alpha;
    if (checked && K > 0 && !ctx->dev_sched) {
        HIPCHK(tvs::launch_sched_set(ctx->sched, ctx->ell, ctx->rng, st));
        ctx->dev_sched = true;
    }
    for (int32_t kk = 0; kk < K; kk++) {
        const int64_t k = ctx->k;
        if (checked && ctx->dlog_n + nsteps > kDevLogCap) {
            // the record buffer is full: copy it back and go on
            HIPCHK(hipEventRecord(ctx->ev_sched, st));
            rc = settle_sched(ctx);
            if (rc) return rc;
            HIPCHK(tvs::launch_sched_set(ctx->sched, ctx->ell, ctx->rng, st));
            ctx->dev_sched = true;
        }
        if (p->variant == TVS_NTVS) {
            if (checked) HIPCHK(tvs::launch_sched_draw(ctx->sched, k, st));
            else ctx->ell = draw_ell(k, ctx->ell, ctx->rng);
        }
        const long c0 = mark(ctx, st);
        for (int32_t n = 0; n < nsteps; n++) {
            HIPCHK(tvs::launch_tv_grad(ctx->gd, ctx->x, p->tv_eps, tb, st));
            if (!checked) {
                tvs_step_log rec;
                std::memset(&rec, 0, sizeof(rec));
                rec.k = (int32_t)k;
                rec.n = n;
                rec.ell_start = ctx->ell;
                rec.gnorm = -1.0;
                double beta = (p->variant == TVS_DECOUPLED)
                                  ? std::pow(p->alpha, (double)(n + 1)) * std::pow(p->gamma, (double)k)
                                  : std::pow(p->alpha, (double)ctx->ell);
                HIPCHK(tvs::launch_tv_step(ctx->gd, ctx->x, beta, tb, st));
                ctx->ell += 1;
                rec.tries = 1;
                rec.accepted = 1;
                ctx->tries += 1;
                ctx->log.push_back(rec);
            } else {
                // decided on the device: no host round trip
                HIPCHK(tvs::launch_tv_check(ctx->gd, ctx->x, p->tv_eps, check_alpha,
                                            ctx->cfg.max_tries, (int32_t)k, n, ctx->sched,
                                            ctx->dlog + ctx->dlog_n, cb, tb, st));
                HIPCHK(tvs::launch_tv_apply(ctx->gd, ctx->x, tb, cb, st));
                ctx->dlog_n += 1;
            }
        }
        const long c1 = mark(ctx, st);
        span(ctx, 0, c0, c1);
        rc = run_sweep(ctx, p->lambda, st, chain_on(ctx));
        if (rc) return rc;
        span(ctx, 1, c1, mark(ctx, st));
        ctx->k += 1;
    }
    if (checked && K > 0) HIPCHK(hipEventRecord(ctx->ev_sched, st));
    return TVS_OK;
}

int tvs_get_image(tvs_ctx *ctx, float *out, int on_device, void *stream)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    if (!out) return fail(ctx, TVS_EINVAL, "output is NULL");
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    int rc = check_flags(ctx, st);
    if (rc) return rc;
    HIPCHK(tvs::launch_narrow(ctx->gd, ctx->x, ctx->xio, st));
    HIPCHK(hipMemcpyAsync(out, ctx->xio, sizeof(float) * ctx->nimg,
                          on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, st));
    if (!on_device) HIPCHK(hipStreamSynchronize(st));
    return TVS_OK;
}

int tvs_get_stats(tvs_ctx *ctx, tvs_stats *out)
{
    if (!ctx || !out) return TVS_EINVAL;
    ctx->err.clear();
    HIPCHK(hipSetDevice(ctx->cfg.device));
    int src = settle_sched(ctx);
    if (src) return src;
    if (ctx->timed && !ctx->spans.empty()) {
        HIPCHK(hipEventSynchronize(ctx->tev[ctx->spans.back().b]));
        HIPCHK(hipStreamSynchronize(ctx->fill_stream));
        for (int q = 0; q < 6; q++) {
            ctx->tot_ms[q] = 0.0;
            ctx->tot_n[q] = 0;
        }
        double last[4] = {0, 0, 0, 0};
        size_t last_cycle_start = 0;
        for (const auto &sp : ctx->spans) {
            float ms = 0;
            HIPCHK(hipEventElapsedTime(&ms, ctx->tev[sp.a], ctx->tev[sp.b]));
            ctx->tot_ms[sp.kind] += ms;
            ctx->tot_n[sp.kind] += sp.n;
            if (sp.kind == 0) {
                last_cycle_start = sp.a;
                last[0] = ms;
                last[2] = 0;
            } else if (sp.kind == 1) {
                last[1] = ms;
            } else if (sp.kind == 2 && sp.a >= last_cycle_start) {
                last[2] += ms;
            }
        }
        ctx->last_tv_ms = last[0];
        ctx->last_sweep_ms = last[1];
        ctx->last_rows_ms = last[2];
        ctx->timed = false;
    }
    int rc = check_flags(ctx, ctx->stream);
    if (rc) return rc;
    out->k = ctx->k;
    out->ell = ctx->ell;
    out->n_hist = ctx->nh;
    out->n_skipped = ctx->skipped;
    out->nnz = ctx->nnz;
    out->steps = (int64_t)ctx->log.size();
    out->tries = ctx->tries;
    out->max_row_nnz = ctx->max_row;
    out->last_sweep_ms = ctx->last_sweep_ms;
    out->last_tv_ms = ctx->last_tv_ms;
    out->last_rows_ms = ctx->last_rows_ms;
    out->device_bytes = ctx->bytes;
    out->tv_ms_total = ctx->tot_ms[0];
    out->sweep_ms_total = ctx->tot_ms[1];
    out->rows_ms_total = ctx->tot_ms[2];
    out->drop_ms_total = ctx->tot_ms[3];
    out->cycles_timed = ctx->tot_n[1];
    out->rows_launches = ctx->tot_n[2];
    out->drop_launches = ctx->tot_n[3];
    out->k1_ms_total = ctx->tot_ms[4];
    out->k2_ms_total = ctx->tot_ms[5];
    out->k_samples = ctx->tot_n[4];
    out->batch_ms_total = ctx->batch.ms_total;
    out->batch_cycles = ctx->batch.cycles;
    out->batch_size = ctx->batch.valid ? ctx->batch.S : 0;
    out->pad = 0;
    return TVS_OK;
}

int tvs_get_step_log(tvs_ctx *ctx, tvs_step_log *out, int64_t cap, int64_t *n)
{
    if (!ctx || !n || cap < 0 || (cap > 0 && !out)) return TVS_EINVAL;
    ctx->err.clear();
    HIPCHK(hipSetDevice(ctx->cfg.device));
    int rc = settle_sched(ctx);
    if (rc) return rc;
    *n = (int64_t)ctx->log.size();
    int64_t m = std::min<int64_t>(cap, *n);
    if (m > 0) std::memcpy(out, ctx->log.data(), sizeof(tvs_step_log) * (size_t)m);
    return TVS_OK;
}

int tvs_debug_sweep(tvs_ctx *ctx, int32_t what, int32_t out[2])
{
    if (!ctx || !out) return TVS_EINVAL;
    ctx->err.clear();
    if (what < 0 || what > 2) return fail(ctx, TVS_EINVAL, "what must lie in 0..2");
    if (!ctx->loaded) return fail(ctx, TVS_ESTATE, "no histories loaded");
    HIPCHK(hipSetDevice(ctx->cfg.device));
    auto &c = ctx->chain;
    if (what == 1 && c.mem) {
        const uint32_t one = 1;
        HIPCHK(hipStreamSynchronize(ctx->stream));
        HIPCHK(hipMemcpy(chain_dead(ctx), &one, sizeof(one), hipMemcpyHostToDevice));
    }
    if (what == 2) c.refuse = true;
    out[0] = chain_on(ctx) && !(c.refused > 0 && ctx->nbuf > 1);
    out[1] = ctx->threads;
    return TVS_OK;
}

int tvs_debug_rows(tvs_ctx *ctx, int64_t first, int64_t count, int64_t *row_nnz, int32_t *idx,
                   float *chord, float *norm2, int64_t cap)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    if (!ctx->loaded) return fail(ctx, TVS_ESTATE, "no histories loaded");
    if (first < 0 || count < 0 || first + count > ctx->nh)
        return fail(ctx, TVS_ERANGE, "history range outside the loaded histories");
    if (count > 0 && (!row_nnz || !norm2)) return fail(ctx, TVS_EINVAL, "output is NULL");
    if (count == 0) return TVS_OK;
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = ctx->stream;
    int64_t *off = nullptr;
    ChainBack back{ctx};
    int rc = dalloc(ctx, &off, (size_t)(count + 1));
    if (rc) return rc;
    rc = count_rows(ctx, first, count, off, st);
    std::vector<int64_t> offh((size_t)count + 1);
    if (!rc && hipMemcpy(offh.data(), off, sizeof(int64_t) * (count + 1), hipMemcpyDeviceToHost) !=
                   hipSuccess)
        rc = fail(ctx, TVS_EDEVICE, "row offsets copy");
    if (rc) {
        dfree(ctx, &off, (size_t)(count + 1));
        return rc;
    }
    const int64_t tot = offh[(size_t)count];
    for (int64_t q = 0; q < count; q++) row_nnz[q] = offh[(size_t)q + 1] - offh[(size_t)q];
    if (tot > cap || (tot > 0 && (!idx || !chord))) {
        dfree(ctx, &off, (size_t)(count + 1));
        return fail(ctx, TVS_ERANGE, "cap smaller than the entries of the requested rows");
    }
    int32_t *di = nullptr;
    float *dc = nullptr, *dn = nullptr;
    rc = dalloc(ctx, &di, (size_t)std::max<int64_t>(tot, 1));
    if (!rc) rc = dalloc(ctx, &dc, (size_t)std::max<int64_t>(tot, 1));
    if (!rc) rc = dalloc(ctx, &dn, (size_t)count);
    if (!rc) {
        RowSet rs;
        rs.first = first;
        rs.n = count;
        rs.base = 0;
        rs.row_off = off;
        rs.idx = di;
        rs.chord32 = dc;
        rs.norm2 = dn;
        hipError_t e = tvs::launch_rows_fill(ctx->gd, hist_dev(ctx), ctx->mlp, rs, st);
        if (e == hipSuccess && tot > 0)
            e = hipMemcpyAsync(idx, di, sizeof(int32_t) * tot, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e == hipSuccess) {
            // tiled-layout words to x-fastest voxel indices (the ABI's order)
            const GridDev &g = ctx->gd;
            for (int64_t q = 0; q < tot; q++) {
                int64_t i, j, k;
                tvs::vcoord(g, idx[q], i, j, k);
                idx[q] = (int32_t)((k * g.ny + j) * g.nx + i);
            }
        }
        if (e == hipSuccess && tot > 0)
            e = hipMemcpyAsync(chord, dc, sizeof(float) * tot, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipMemcpyAsync(norm2, dn, sizeof(float) * count, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) rc = fail(ctx, TVS_EDEVICE, std::string("debug rows: ") + hipGetErrorString(e));
    }
    dfree(ctx, &di, (size_t)std::max<int64_t>(tot, 1));
    dfree(ctx, &dc, (size_t)std::max<int64_t>(tot, 1));
    dfree(ctx, &dn, (size_t)count);
    dfree(ctx, &off, (size_t)(count + 1));
    return rc;
}

}  // extern "C"

namespace {

bool same_params(const tvs_params &a, const tvs_params &b)
{
    return a.lambda == b.lambda && a.N == b.N && a.alpha == b.alpha && a.tv_check == b.tv_check &&
           a.variant == b.variant && a.tv_eps == b.tv_eps && a.seed == b.seed &&
           (a.variant != TVS_DECOUPLED || a.gamma == b.gamma);
}

// (Re)allocates the S-image buffers and starts every setting from x0.
int batch_init(tvs_ctx *ctx, const tvs_params *p, int S, hipStream_t st)
{
    auto &B = ctx->batch;
    if (B.S != S) {
        free_batch(ctx);
        B.S = S;
        const size_t n = (size_t)(ctx->nvox * S);
        int rc = dalloc(ctx, &B.b.x, n);
        if (!rc) rc = dalloc(ctx, &B.b.g, n);
        if (!rc) rc = dalloc(ctx, &B.b.part, (size_t)(tvs::batch_num_parts(ctx->gd, S) * S));
        if (!rc) rc = dalloc(ctx, &B.b.norm2, (size_t)S);
        if (!rc) rc = dalloc(ctx, &B.b.lambda, (size_t)S);
        if (!rc) rc = dalloc(ctx, &B.b.eps, (size_t)S);
        if (!rc) rc = dalloc(ctx, &B.b.cyc, (size_t)4);
        if (!rc) rc = dalloc(ctx, &B.dot, (size_t)(3 * (int64_t)ctx->cfg.block_size * S));
        if (rc) {
            free_batch(ctx);
            return rc;
        }
        B.b.S = S;
        B.b.nvox = ctx->nvox;
        HIPCHK(hipMemsetAsync(B.b.g, 0, sizeof(double) * n, st));
    }
    B.p.assign(p, p + S);
    std::vector<double> lam(S), eps(S);
    for (int q = 0; q < S; q++) {
        lam[q] = p[q].lambda;
        eps[q] = p[q].tv_eps;
    }
    HIPCHK(hipMemcpyAsync(B.b.lambda, lam.data(), sizeof(double) * S, hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(B.b.eps, eps.data(), sizeof(double) * S, hipMemcpyHostToDevice, st));
    HIPCHK(tvs::launch_replicate(ctx->x0, B.b, st));
    HIPCHK(hipStreamSynchronize(st));
    B.k = 0;
    B.ell.assign(S, 0);
    B.rng.assign(S, 0);
    for (int q = 0; q < S; q++) B.rng[q] = p[q].seed;
    B.valid = true;
    return TVS_OK;
}

// Enqueues the launches of one batched cycle (captured into a graph): the
// TV steps of every setting, then the tile-wise DROP chain for all S
// images.  On the fly, the fill stream joins the capture and forms the
// rows chunk by chunk into the ring of buffers beside the TV steps and the
// chain, with the single-image sweep's filled/free ordering (events of the
// batch's own, so the sweep's events keep their real records); the chain
// waits for the last chunk, which joins the fill stream back.
int batch_cycle(tvs_ctx *ctx, int nmax, hipStream_t st)
{
    auto &Bt = ctx->batch;
    const int S = Bt.S;
    const int64_t B = ctx->cfg.block_size, nb = ctx->nblocks;
    const bool otf = ctx->cfg.path_mode == TVS_PATH_ON_THE_FLY;
    const int64_t step = otf ? ctx->chunk : ctx->nh;
    const int64_t nchunks = nb > 0 ? (ctx->nh + step - 1) / step : 0;
    const int64_t NB = ctx->nbuf;
    hipStream_t fs = ctx->fill_stream;
    auto fill = [&](int64_t c) -> int {
        const int q = chunk_buffer(ctx, c);
        if (c >= NB) HIPCHK(hipStreamWaitEvent(fs, ctx->bev_free[q], 0));
        tvs::TileFill f = chunk_fill(ctx, c, std::min(step, ctx->nh - c * step));
        HIPCHK(tvs::launch_rows_fill_tiled(ctx->gd, hist_dev(ctx), ctx->mlp, f, fs));
        HIPCHK(hipEventRecord(ctx->bev_filled[q], fs));
        return TVS_OK;
    };
    if (otf && nchunks > 0) {
        HIPCHK(hipEventRecord(ctx->bev_fork, st));
        HIPCHK(hipStreamWaitEvent(fs, ctx->bev_fork, 0));
        for (int64_t c = 0; c < std::min<int64_t>(NB, nchunks); c++) {
            int rc = fill(c);
            if (rc) return rc;
        }
    }
    for (int n = 0; n < nmax; n++) {
        uint32_t active = 0;
        for (int q = 0; q < S; q++)
            if (Bt.p[q].N > n) active |= 1u << q;
        HIPCHK(tvs::launch_tvb_grad(ctx->gd, Bt.b, active, st));
        HIPCHK(tvs::launch_tvb_step(Bt.b, active, n, nmax, st));
    }
    if (nb == 0) {
        HIPCHK(tvs::launch_tick(Bt.b.cyc, st));
        return TVS_OK;
    }
    HIPCHK(tvs::launch_zero_i64(Bt.dot, 3 * B * S, st));
    for (int64_t b = 0; b <= nb; b++) {
        const bool has_c = b < nb;
        const int64_t c = has_c ? (b * B) / step : -1;
        const bool first_of_chunk = has_c && (b * B) % step == 0;
        if (otf && first_of_chunk)
            HIPCHK(hipStreamWaitEvent(st, ctx->bev_filled[chunk_buffer(ctx, c)], 0));
        tvs::DropTileArgs A;
        if (b > 0) A.P = block_view(ctx, b - 1, Bt.dot, B * S);
        if (has_c) A.C = block_view(ctx, b, Bt.dot, B * S);
        A.x = Bt.b.x;
        A.big = ctx->big;
        A.dot_max = ctx->dot_max;
        A.zero = Bt.dot + ((b + 1) % 3) * B * S;
        A.B = B;
        A.err = ctx->flags + kFlagRange;
        A.tiles = ctx->act;
        A.nact = ctx->nact;
        A.slots = ctx->by_region ? ctx->slot_of : nullptr;
        HIPCHK(tvs::launch_drop_tiles_batch(A, Bt.b, ctx->ntiles, ctx->bthreads, ctx->bgroup, st));
        if (otf && first_of_chunk && c >= 1 && c - 1 + NB < nchunks) {
            // the launch above was the last to read chunk c - 1's buffer
            HIPCHK(hipEventRecord(ctx->bev_free[chunk_buffer(ctx, c - 1)], st));
            int rc = fill(c - 1 + NB);
            if (rc) return rc;
        }
    }
    HIPCHK(tvs::launch_tick(Bt.b.cyc, st));
    return TVS_OK;
}

}  // namespace

extern "C" {

int tvs_iterate_batch(tvs_ctx *ctx, const tvs_params *p, int32_t S, int32_t K, void *stream)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    if (S < 1 || S > 32) return fail(ctx, TVS_EINVAL, "batch size must lie in [1, 32]");
    if (!p) return fail(ctx, TVS_EINVAL, "params is NULL");
    if (K < 0) return fail(ctx, TVS_EINVAL, "K must be >= 0");
    for (int q = 0; q < S; q++) {
        int rc = validate_params(ctx, p + q);
        if (rc) return rc;
        if (p[q].variant == TVS_OTVS || (p[q].variant == TVS_NTVS && p[q].tv_check))
            return fail(ctx, TVS_EINVAL, "batches take unchecked schedules only");
    }
    if (!ctx->loaded) return fail(ctx, TVS_ESTATE, "tvs_iterate_batch before tvs_load_histories");
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    // the chunk buffers must be free of the single-image sweep's work (its
    // last reads are marked by the buffer-free events, also when it ran on
    // another stream)
    HIPCHK(hipStreamSynchronize(ctx->fill_stream));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    if (ctx->cfg.path_mode == TVS_PATH_ON_THE_FLY)
        for (int q = 0; q < kChunkBuffers; q++) HIPCHK(hipStreamWaitEvent(st, ctx->ev_free[q], 0));
    ChainBack back{ctx};
    auto &B = ctx->batch;
    bool same = B.valid && B.S == S;
    for (int q = 0; same && q < S; q++) same = same_params(B.p[q], p[q]);
    if (!same) {
        int rc = batch_init(ctx, p, S, st);
        if (rc) return rc;
    }
    B.ms_total = 0;
    B.cycles = 0;
    if (K == 0) return TVS_OK;

    // beta of every (cycle, step, setting) of this call, drawn on the host
    int nmax = 0;
    for (int q = 0; q < S; q++) nmax = std::max(nmax, (int)p[q].N);
    const int64_t need = std::max<int64_t>((int64_t)K * std::max(nmax, 1) * S, 1);
    if (need > B.beta_cap) {
        dfree(ctx, &B.b.beta_tab, (size_t)B.beta_cap);
        B.beta_cap = 0;
        int rc = dalloc(ctx, &B.b.beta_tab, (size_t)need);
        if (rc) return rc;
        B.beta_cap = need;
    }
    std::vector<double> beta((size_t)need, 0.0);
    for (int32_t kk = 0; kk < K; kk++) {
        const int64_t k = B.k + kk;
        for (int q = 0; q < S; q++) {
            if (p[q].variant == TVS_NTVS) B.ell[q] = draw_ell(k, B.ell[q], B.rng[q]);
            for (int n = 0; n < p[q].N; n++) {
                double b = (p[q].variant == TVS_DECOUPLED)
                               ? std::pow(p[q].alpha, (double)(n + 1)) * std::pow(p[q].gamma, (double)k)
                               : std::pow(p[q].alpha, (double)B.ell[q]);
                beta[((size_t)kk * nmax + n) * S + q] = b;
                B.ell[q] += 1;
            }
        }
    }
    B.k += K;
    HIPCHK(hipMemcpyAsync(B.b.beta_tab, beta.data(), sizeof(double) * need, hipMemcpyHostToDevice, st));
    HIPCHK(tvs::launch_set_counter(B.b.cyc, 0, st));

    // capture one cycle, replay it K times
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    HIPCHK(hipStreamBeginCapture(st, hipStreamCaptureModeRelaxed));
    int rc = batch_cycle(ctx, nmax, st);
    hipError_t ce = hipStreamEndCapture(st, &graph);
    if (rc) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc;
    }
    if (ce != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("graph capture: ") + hipGetErrorString(ce));
    ce = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    if (ce != hipSuccess) {
        (void)hipGraphDestroy(graph);
        return fail(ctx, TVS_EDEVICE, std::string("graph instantiate: ") + hipGetErrorString(ce));
    }
    ctx->tev_used = 0;
    ctx->spans.clear();
    ctx->timed = false;
    std::vector<long> ev;
    ev.push_back(mark(ctx, st));
    for (int32_t kk = 0; kk < K && ce == hipSuccess; kk++) {
        ce = hipGraphLaunch(exec, st);
        ev.push_back(mark(ctx, st));
    }
    hipError_t se = hipStreamSynchronize(st);
    (void)hipGraphExecDestroy(exec);
    (void)hipGraphDestroy(graph);
    if (ce != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("graph launch: ") + hipGetErrorString(ce));
    if (se != hipSuccess) return fail(ctx, TVS_EDEVICE, std::string("batch sync: ") + hipGetErrorString(se));
    for (size_t q = 1; q < ev.size(); q++) {
        float ms = 0;
        if (ev[q - 1] >= 0 && ev[q] >= 0 &&
            hipEventElapsedTime(&ms, ctx->tev[(size_t)ev[q - 1]], ctx->tev[(size_t)ev[q]]) == hipSuccess)
            B.ms_total += ms;
    }
    B.cycles = K;
    ctx->tev_used = 0;
    return TVS_OK;
}

int tvs_get_batch_image(tvs_ctx *ctx, int32_t s, float *out, int on_device, void *stream)
{
    if (!ctx) return TVS_EINVAL;
    ctx->err.clear();
    if (!out) return fail(ctx, TVS_EINVAL, "output is NULL");
    if (!ctx->batch.valid) return fail(ctx, TVS_ESTATE, "no batch");
    if (s < 0 || s >= ctx->batch.S) return fail(ctx, TVS_ERANGE, "setting outside the batch");
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    int rc = check_flags(ctx, st);
    if (rc) return rc;
    HIPCHK(tvs::launch_extract(ctx->gd, ctx->batch.b, s, ctx->xio, st));
    HIPCHK(hipMemcpyAsync(out, ctx->xio, sizeof(float) * ctx->nimg,
                          on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, st));
    if (!on_device) HIPCHK(hipStreamSynchronize(st));
    return TVS_OK;
}

extern "C++" {

// Launch-shape cache of the tuners: one line per measurement, "key values",
// the key a whitespace-free description of the device, grid, history count,
// B and path mode (plus the tuner's own tag); the last matching line wins.
static std::string tune_key(const tvs_ctx *ctx, const hipDeviceProp_t &prop, const char *tag)
{
    char key[512];
    std::snprintf(key, sizeof(key), "%s|%dx%dx%d|%.6gx%.6gx%.6g|H%lld|B%d|P%d%s", prop.gcnArchName,
                  ctx->grid.nx, ctx->grid.ny, ctx->grid.nz, ctx->grid.vx, ctx->grid.vy,
                  ctx->grid.vz, (long long)ctx->nh, ctx->cfg.block_size, ctx->cfg.path_mode, tag);
    return key;
}

// Calls fn(values) for every line of the cache file whose key is `key`.
template <typename F>
static void cache_scan(const char *path, const std::string &key, F fn)
{
    FILE *f = path ? std::fopen(path, "r") : nullptr;
    if (!f) return;
    char line[1024];
    while (std::fgets(line, sizeof(line), f)) {
        char k[512];
        int used = 0;
        if (std::sscanf(line, "%511s%n", k, &used) == 1 && key == k) fn(line + used);
    }
    std::fclose(f);
}

static void cache_append(const char *path, const std::string &key, const std::string &values)
{
    if (!path) return;
    if (FILE *f = std::fopen(path, "a")) {
        std::fprintf(f, "%s %s\n", key.c_str(), values.c_str());
        std::fclose(f);
    }
}

}  // extern "C++"

int tvs_autotune(tvs_ctx *ctx, double lambda, const char *cache_path, tvs_tune_result *out,
                 void *stream)
{
    if (!ctx || !out) return TVS_EINVAL;
    ctx->err.clear();
    std::memset(out, 0, sizeof(*out));
    if (!finite_pos(lambda)) return fail(ctx, TVS_EINVAL, "lambda must be finite and > 0");
    if (!ctx->loaded) return fail(ctx, TVS_ESTATE, "tvs_autotune before tvs_load_histories");
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    hipDeviceProp_t prop;
    HIPCHK(hipGetDeviceProperties(&prop, ctx->cfg.device));
    const std::string key = tune_key(ctx, prop, "");
    const bool has_chain = ctx->chain.planned && !ctx->chain.failed;
    // what the choice leaves to the context: the chain or launches, and the
    // launches' shape in either case (a captured sweep, a short budget)
    auto keep = [&](int threads, int sweep, int pct, bool chain, double launch_ms, double chain_ms) {
        ctx->threads = threads;
        ctx->split = sweep == 2 ? 1 : 0;
        ctx->fill_wide_pct = pct;
        ctx->tuned = true;
        ctx->launches = has_chain && !chain;     // without one, later loads decide anew
        out->tile_threads = chain ? 0 : threads;
        out->sweep_kernel = chain ? 0 : sweep;
        out->ms_per_block = chain ? chain_ms : launch_ms;
        out->fill_wide_pct = pct;
    };
    if (cache_path) {
        // the launches' shape and time, then whether the chain was the faster and
        // its time.  A line without the last two was measured without a chain:
        // where there is one, the choice is made anew
        cache_scan(cache_path, key, [&](const char *v) {
            int th = 0, sw = 0, pct = -1, ch = 0;
            double ms = 0, cms = 0;
            const int got = std::sscanf(v, "%d %d %lf %d %d %lf", &th, &sw, &ms, &pct, &ch, &cms);
            if (got >= 3 && (th == 64 || th == 128 || th == 256) && (sw == 1 || sw == 2) &&
                (got == 6 || !has_chain)) {
                const int64_t use = (got >= 4 && pct >= 0 && pct <= 100) ? pct : ctx->fill_wide_pct;
                keep(th, sw, (int)use, has_chain && ch != 0, ms, cms);
                out->from_cache = 1;
            }
        });
        if (out->from_cache) return TVS_OK;
    }
    const int64_t B = ctx->cfg.block_size;
    // enough blocks that the candidates' differences stand above the spread
    // of a step's duration (48 blocks picked 64-lane tiles for the 256x256x32
    // fixed-point store, 20 % slower per whole sweep than 128)
    const int64_t nb = std::min<int64_t>(ctx->nblocks, 1024);
    out->fill_wide_pct = ctx->fill_wide_pct;
    if (nb == 0) {
        out->tile_threads = chain_on(ctx) ? 0 : ctx->threads;
        out->sweep_kernel = chain_on(ctx) ? 0 : ctx->split ? 2 : 1;
        return TVS_OK;
    }
    HIPCHK(hipStreamSynchronize(ctx->fill_stream));
    ChainBack back{ctx};
    double *saved = nullptr;
    int rc = dalloc(ctx, &saved, (size_t)ctx->nvox);
    if (rc) return rc;
    HIPCHK(hipMemcpyAsync(saved, ctx->x, sizeof(double) * ctx->nvox, hipMemcpyDeviceToDevice, st));
    // one sweep (of the first `limit` histories), its time in ms, and the image back
    auto time_sweep = [&](bool chain, int64_t limit, float &ms) -> int {
        ctx->tev_used = 0;
        ctx->spans.clear();
        const long a = mark(ctx, st);
        const int r = run_sweep(ctx, lambda, st, chain, limit);
        const long b = mark(ctx, st);
        if (r) return r;
        hipError_t e = hipMemcpyAsync(ctx->x, saved, sizeof(double) * ctx->nvox,
                                      hipMemcpyDeviceToDevice, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e == hipSuccess) e = hipStreamSynchronize(ctx->fill_stream);
        ms = 0;
        if (e == hipSuccess && a >= 0 && b >= 0)
            e = hipEventElapsedTime(&ms, ctx->tev[(size_t)a], ctx->tev[(size_t)b]);
        if (e != hipSuccess)
            return fail(ctx, TVS_EDEVICE, std::string("autotune: ") + hipGetErrorString(e));
        return TVS_OK;
    };
    auto candidate = [&](int threads, int sweep, double ms) {
        if (out->n_candidates >= 8) return;
        out->cand_threads[out->n_candidates] = threads;
        out->cand_sweep[out->n_candidates] = sweep;
        out->cand_ms[out->n_candidates] = ms;
        out->n_candidates++;
    };
    const int ths[3] = {64, 128, 256};
    const int old_threads = ctx->threads, old_split = ctx->split;
    const int64_t limit = std::min(nb * B, ctx->nh);
    double best = 1e300;
    int best_threads = 0, best_sweep = 0;
    for (int sw = 1; sw <= 2 && rc == TVS_OK; sw++) {
        for (int ti = 0; ti < 3 && rc == TVS_OK; ti++) {
            ctx->threads = ths[ti];
            ctx->split = sw == 2 ? 1 : 0;
            double tbest = 1e300;
            for (int rep = 0; rep < 3 && rc == TVS_OK; rep++) {
                float ms = 0;
                rc = time_sweep(false, limit, ms);
                if (rep > 0) tbest = std::min(tbest, (double)ms / nb);   // rep 0 warms up
            }
            if (rc) break;
            candidate(ths[ti], sw, tbest);
            if (tbest < best) {
                best = tbest;
                best_threads = ths[ti];
                best_sweep = sw;
            }
        }
    }
    // on the fly: whole sweeps (the row formation beside the launches) for the
    // share of chunks formed at the row kernel's full occupancy; with one
    // chunk the share does not matter
    const bool several = ctx->cfg.path_mode == TVS_PATH_ON_THE_FLY && ctx->chunk_base.size() > 2;
    const int old_pct = ctx->fill_wide_pct;
    int pct = old_pct;
    double pbest = 1e300;
    if (!rc && several) {
        const int pcts[6] = {0, 20, 40, 60, 80, 100};
        ctx->threads = best_threads;
        ctx->split = best_sweep == 2 ? 1 : 0;
        for (int pi = 0; pi < 6 && rc == TVS_OK; pi++) {
            ctx->fill_wide_pct = pcts[pi];
            float ms = 0;
            rc = time_sweep(false, -1, ms);
            if (rc) break;
            out->cand_pct[out->n_fill] = pcts[pi];
            out->cand_sweep_ms[out->n_fill] = ms;
            out->n_fill++;
            if (ms < pbest) {
                pbest = ms;
                pct = pcts[pi];
            }
        }
    }
    // the chain, where its workspace is there beside the saved image: on the
    // blocks that timed the launches, or against the best share's whole sweep
    double cbest = 1e300;
    if (!rc && ctx->chain.on()) {
        ctx->chain.refused = 0;
        for (int rep = 0; rep < 3 && rc == TVS_OK; rep++) {
            float ms = 0;
            rc = time_sweep(true, several ? -1 : limit, ms);
            if (ctx->chain.refused > 0) {       // launches ran instead
                cbest = 1e300;
                break;
            }
            if (rep > 0) cbest = std::min(cbest, (double)ms / (several ? ctx->nblocks : nb));
        }
        if (!rc && cbest < 1e300) candidate(0, 0, cbest);
    }
    dfree(ctx, &saved, (size_t)ctx->nvox);
    ctx->tev_used = 0;
    ctx->spans.clear();
    ctx->timed = false;
    ctx->threads = old_threads;
    ctx->split = old_split;
    ctx->fill_wide_pct = old_pct;
    if (rc) return rc;
    const bool chain = cbest < 1e300 && cbest <= (several ? pbest / (double)ctx->nblocks : best);
    keep(best_threads, best_sweep, pct, chain, best, cbest);
    char vals[128];
    int len = std::snprintf(vals, sizeof(vals), "%d %d %.6f %d", best_threads, best_sweep, best, pct);
    if (cbest < 1e300)
        std::snprintf(vals + len, sizeof(vals) - (size_t)len, " %d %.6f", chain ? 1 : 0, cbest);
    cache_append(cache_path, key, vals);
    return TVS_OK;
}

int tvs_autotune_batch(tvs_ctx *ctx, const tvs_params *p, int32_t S, const char *cache_path,
                       tvs_batch_tune_result *out, void *stream)
{
    if (!ctx || !out) return TVS_EINVAL;
    ctx->err.clear();
    std::memset(out, 0, sizeof(*out));
    if (S < 1 || S > 32) return fail(ctx, TVS_EINVAL, "batch size must lie in [1, 32]");
    if (!p) return fail(ctx, TVS_EINVAL, "params is NULL");
    for (int q = 0; q < S; q++) {
        int rc = validate_params(ctx, p + q);
        if (rc) return rc;
    }
    if (!ctx->loaded) return fail(ctx, TVS_ESTATE, "tvs_autotune_batch before tvs_load_histories");
    HIPCHK(hipSetDevice(ctx->cfg.device));
    hipStream_t st = pick(ctx, stream);
    hipDeviceProp_t prop;
    HIPCHK(hipGetDeviceProperties(&prop, ctx->cfg.device));
    const std::string key = tune_key(ctx, prop, ("|S" + std::to_string(S)).c_str());
    if (cache_path) {
        cache_scan(cache_path, key, [&](const char *v) {
            int th = 0, gp = 0;
            double ms = 0;
            if (std::sscanf(v, "%d %d %lf", &th, &gp, &ms) == 3 && tvs::batch_shape_ok(th, gp)) {
                out->threads = th;
                out->group = gp;
                out->ms_per_block = ms;
                out->from_cache = 1;
            }
        });
        if (out->from_cache) {
            ctx->bthreads = out->threads;
            ctx->bgroup = out->group;
            return TVS_OK;
        }
    }
    const int64_t B = ctx->cfg.block_size;
    const bool otf = ctx->cfg.path_mode == TVS_PATH_ON_THE_FLY;
    // the first blocks of the first chunk (formed here on the fly)
    int64_t nb = std::min<int64_t>(ctx->nblocks, 48);
    if (otf) nb = std::min<int64_t>(nb, ctx->chunk / B);
    if (nb == 0) {
        out->threads = ctx->bthreads;
        out->group = ctx->bgroup;
        return TVS_OK;
    }
    HIPCHK(hipStreamSynchronize(ctx->fill_stream));
    HIPCHK(hipStreamSynchronize(ctx->stream));
    ChainBack back{ctx};
    int rc = batch_init(ctx, p, S, st);
    if (rc) return rc;
    auto &Bt = ctx->batch;
    if (otf) {
        for (int q = 0; q < kChunkBuffers; q++) HIPCHK(hipStreamWaitEvent(st, ctx->ev_free[q], 0));
        tvs::TileFill f = chunk_fill(ctx, 0, std::min(ctx->chunk, ctx->nh));
        f.max_wgs = 0;
        HIPCHK(tvs::launch_rows_fill_tiled(ctx->gd, hist_dev(ctx), ctx->mlp, f, st));
        HIPCHK(hipEventRecord(ctx->ev_free[chunk_buffer(ctx, 0)], st));
    }
    const int ths[2] = {128, 256}, gps[4] = {2, 4, 8, 16};
    const int old_t = ctx->bthreads, old_g = ctx->bgroup;
    double best = 1e300;
    int nc = 0;
    for (int ti = 0; ti < 2 && rc == TVS_OK; ti++) {
        for (int gi = 0; gi < 4 && rc == TVS_OK; gi++) {
            ctx->bthreads = ths[ti];
            ctx->bgroup = gps[gi];
            double tbest = 1e300;
            for (int rep = 0; rep < 3 && rc == TVS_OK; rep++) {
                ctx->tev_used = 0;
                ctx->spans.clear();
                hipError_t e = tvs::launch_zero_i64(Bt.dot, 3 * B * S, st);
                long a = mark(ctx, st);
                for (int64_t b = 0; b <= nb && e == hipSuccess; b++) {
                    tvs::DropTileArgs A;
                    if (b > 0) A.P = block_view(ctx, b - 1, Bt.dot, B * S);
                    if (b < nb) A.C = block_view(ctx, b, Bt.dot, B * S);
                    A.x = Bt.b.x;
                    A.big = ctx->big;
                    A.dot_max = ctx->dot_max;
                    A.zero = Bt.dot + ((b + 1) % 3) * B * S;
                    A.B = B;
                    A.err = ctx->flags + kFlagRange;
                    A.tiles = ctx->act;
                    A.nact = ctx->nact;
                    A.slots = ctx->by_region ? ctx->slot_of : nullptr;
                    e = tvs::launch_drop_tiles_batch(A, Bt.b, ctx->ntiles, ctx->bthreads,
                                                     ctx->bgroup, st);
                }
                long bm = mark(ctx, st);
                if (e == hipSuccess) e = hipStreamSynchronize(st);
                float ms = 0;
                if (e == hipSuccess && a >= 0 && bm >= 0)
                    e = hipEventElapsedTime(&ms, ctx->tev[(size_t)a], ctx->tev[(size_t)bm]);
                if (e != hipSuccess) {
                    rc = fail(ctx, TVS_EDEVICE, std::string("batch autotune: ") + hipGetErrorString(e));
                    break;
                }
                if (rep > 0) tbest = std::min(tbest, (double)ms / (double)nb);   // rep 0 warms up
            }
            if (rc) break;
            if (nc < 8) {
                out->cand_threads[nc] = ths[ti];
                out->cand_group[nc] = gps[gi];
                out->cand_ms[nc] = tbest;
                nc++;
            }
            if (tbest < best) {
                best = tbest;
                out->threads = ths[ti];
                out->group = gps[gi];
                out->ms_per_block = tbest;
            }
        }
    }
    ctx->tev_used = 0;
    ctx->spans.clear();
    ctx->timed = false;
    out->n_candidates = nc;
    // the timed steps moved the batch images: the next batch starts afresh
    Bt.valid = false;
    if (rc || best == 1e300) {
        ctx->bthreads = old_t;
        ctx->bgroup = old_g;
        return rc ? rc : fail(ctx, TVS_EDEVICE, "batch autotune: no candidate ran");
    }
    ctx->bthreads = out->threads;
    ctx->bgroup = out->group;
    rc = check_flags(ctx, st);
    if (rc) return rc;
    char vals[96];
    std::snprintf(vals, sizeof(vals), "%d %d %.6f", out->threads, out->group, out->ms_per_block);
    cache_append(cache_path, key, vals);
    return TVS_OK;
}

}  // extern "C"

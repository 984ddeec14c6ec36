// libwave.so host side: contexts, launch planning, the checkpointed
// gradient driver, batched runs and the C ABI of include/wave.h.  The
// kernels live in wave_step.h (instantiated by the k_*.hip units).

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "wave.h"
#include "wave_dev.h"
#include "wave_kernels.h"

using namespace wavek;

// Scratch of wave_check_noalloc: its two counters live in this fixed device
// array (one copy per GPU, kept until the process ends), so that the call
// allocates nothing.  On the host `scratch` is only a stand-in for the
// symbol, not a device address: host code uses the address
// hipGetSymbolAddress returns for each device (scratch_for), never the name.
constexpr int kScratchInts = 64;
static __device__ __align__(256) int scratch[kScratchInts];

namespace {

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
int *scratch_dev[kMaxDevices] = {};

// Device address of `scratch` on `device`, looked up once per device with
// that device current (wave_init does it for the context's device).
int scratch_for(int device, int **out)
{
    if (device < 0 || device >= kMaxDevices)
        return WAVE_EINVAL;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_dev[device]) {
        int cur = -1;
        if (hipGetDevice(&cur) != hipSuccess)
            return WAVE_EHIP;
        if (cur != device && hipSetDevice(device) != hipSuccess)
            return WAVE_EHIP;
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device)
            (void)hipSetDevice(cur);
        if (e != hipSuccess || !p)
            return WAVE_EHIP;
        scratch_dev[device] = static_cast<int *>(p);
    }
    *out = scratch_dev[device];
    return WAVE_OK;
}

}  // namespace

namespace {
// ---------------------------------------------------------------------------
// host side

typedef void (*StepKernel)(StepArgs);
typedef void (*BatchKernel)(const ShotDesc *, BatchItems, int);
typedef void (*FlowKernel)(const ShotDesc *, FlowPlan);
typedef void (*RunKernel)(const ShotDesc *, BatchItems, RunSync);

struct Variant {
    const char *name;
    StepKernel fn[kNumKinds];  // by storage type; all NULL for "auto" and "naive"
    BatchKernel batch[3];      // FP32, FP16, BF16 (two-level storage)
    RunKernel run[3];          // the same, every step of a run in one launch
    StepKernel adj[2];  // adjoint step, adjoint step + imaging terms (FP32)
    StepKernel lap[2];  // FP32 step that stores the Laplacian: streaming, cache-resident loads
    FlowKernel flow;    // data-flow batched step (FP32)
    StepKernel fwd_cached;  // FP32 step with cache-resident load policies
    int txv, ty, ry;
};

#define TILED(TXV, TY, RY)                                                                        \
    {step_tiled<WAVE_F32, TXV, TY, RY>, step_tiled<WAVE_F16, TXV, TY, RY>,                        \
     step_tiled<WAVE_BF16, TXV, TY, RY>, step_tiled<WAVE_F16_UV, TXV, TY, RY>,                    \
     step_tiled<WAVE_BF16_UV, TXV, TY, RY>},                                                      \
    {step_batch<WAVE_F32, TXV, TY, RY>, step_batch<WAVE_F16, TXV, TY, RY>,                        \
     step_batch<WAVE_BF16, TXV, TY, RY>},                                                         \
    {step_batch_run<WAVE_F32, TXV, TY, RY>, step_batch_run<WAVE_F16, TXV, TY, RY>,                \
     step_batch_run<WAVE_BF16, TXV, TY, RY>},                                                     \
    {adjoint_tiled<kAdj, TXV, TY, RY>, adjoint_tiled<kFus, TXV, TY, RY>},                         \
    {step_tiled_lap<false, TXV, TY, RY>, step_tiled_lap<true, TXV, TY, RY>},                      \
    step_flow<TXV, TY, RY>, step_tiled_cached<TXV, TY, RY>

const Variant kVariants[] = {
    {"auto", {nullptr, nullptr, nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr},
     {nullptr, nullptr}, {nullptr, nullptr}, nullptr, nullptr, 0, 0, 0},
    {"naive", {nullptr, nullptr, nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr}, {nullptr, nullptr, nullptr},
     {nullptr, nullptr}, {nullptr, nullptr}, nullptr, nullptr, 0, 0, 0},
    {"t64x16_r1", TILED(16, 16, 1), 16, 16, 1},
    {"t128x8_r1", TILED(32, 8, 1), 32, 8, 1},
    {"t128x16_r2", TILED(32, 8, 2), 32, 8, 2},
    {"t64x32_r2", TILED(16, 16, 2), 16, 16, 2},
    {"t128x16_r1", TILED(32, 16, 1), 32, 16, 1},
    {"t256x8_r2", TILED(64, 4, 2), 64, 4, 2},
    {"t64x16_r2", TILED(16, 8, 2), 16, 8, 2},
    {"t128x32_r4", TILED(32, 8, 4), 32, 8, 4},
    {"t256x8_r1", TILED(64, 8, 1), 64, 8, 1},
    {"t64x32_r1", TILED(16, 32, 1), 16, 32, 1},
    {"t128x32_r2", TILED(32, 16, 2), 32, 16, 2},
    {"t256x16_r2", TILED(64, 8, 2), 64, 8, 2},
};
#undef TILED
constexpr int kNumVariants = sizeof(kVariants) / sizeof(kVariants[0]);
constexpr int kNaive = 1;
const StepKernel kNaiveFn[kNumKinds] = {step_naive<WAVE_F32>, step_naive<WAVE_F16>, step_naive<WAVE_BF16>,
                                        step_naive<WAVE_F16_UV>, step_naive<WAVE_BF16_UV>};

// Whether the cells an FP32 step touches in its three fields (u^n, u^{n-1},
// k: the interior and 4 ghost rows and planes on each side) fit in the
// GPU's 256 MiB memory-side cache with room to spare.  Then every field
// keeps the default cache policy (step_tiled_cached): u^{n-1} and k, read
// once per step, are still cached when the next step reads them.  Measured
// with the step's access pattern: 13 % faster at 256^3 (about 210 MiB),
// 8-13 % slower at 384^3, where streaming them is better.
constexpr long long kCacheResidentBytes = 224ll << 20;
long long step_bytes_touched(int nx, int ny, int nz, int kind)
{
    return 3ll * elem_bytes(kind) * (nx + 8) * (ny + 8) * (long long)(nz + 8);
}
bool fits_in_cache(int nx, int ny, int nz) { return step_bytes_touched(nx, ny, nz, WAVE_F32) <= kCacheResidentBytes; }

// The element encoding of a storage type (the u-and-change types store
// both of their fields in the encoding of their base type).
int base_kind(int kind) { return kind == WAVE_F16_UV ? WAVE_F16 : kind == WAVE_BF16_UV ? WAVE_BF16 : kind; }

int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// Launch geometry of a tiled (or the naive) kernel over one grid.
struct Geo {
    int v = 0, ntx = 0, nty = 0, nchunks = 0, zc = 0, nwg = 0, grid = 0;
};

}  // namespace

// ints of a context's scale history: a line that starts with the exponents,
// then 4 levels' max slots; the line also holds two counters of the library's
// own checks (the range of k at init, wave_check)
constexpr int kRingInts = kMaxStride + 4 * kMaxSlots * kMaxStride;
constexpr int kRingCounters = 8;

// State of the gradient computation (FP32 storage): the checkpoints and the
// store of the last checkpointed forward run and the adjoint fields, in the
// field layout (ghost cells zero), and the Laplacians and the FP64 sum, which
// hold interior cells only.
struct wave_grad_state {
    int64_t step0 = 0;  // step counter at the start of the forward run
    int nt = 0;         // steps of the run (0: no run recorded)
    int asked = 0;      // segment length asked for, or chosen by memory (wave_grad_info)
    int every = 0;      // segment length C in use: asked, or nt
    int nseg = 0;       // segments: segment i covers steps i*C .. min((i+1)*C, nt) - 1
    int held = -1;      // segment whose levels' Laplacians the store holds
    bool has_src = false;
    // one allocation: checkpoints (two fields each; none with a single
    // segment, which is never recomputed), the store (lap a^c .. lap
    // a^{c+C-1} of a segment), and the run's source values [nt]
    void *slab = nullptr;
    size_t slab_bytes = 0;
    float *src = nullptr;
    // one allocation: the adjoint fields, the FP64 sum, and one more value
    // (the source term)
    void *work = nullptr;
    void *phi[2] = {nullptr, nullptr};
    double *acc = nullptr;
    // receiver cells (distinct) by work-group of the adjoint's tiling, and,
    // per cell, its receivers (one allocation)
    void *cells = nullptr;
    int *cell_wg = nullptr;
    long long *cell_off = nullptr;
    int *cell_start = nullptr, *cell_rec = nullptr;
    int ncells = -1;
    int cell_v = -1, cell_zc = -1;  // the tiling of cell_wg
};

// Receivers by work-group of a tiling (one device allocation): work-group i
// owns entries start[i] .. start[i + 1] - 1 of off (offset in the field) and
// idx (receiver).
struct RecTables {
    void *base = nullptr;
    int *start = nullptr;
    long long *off = nullptr;
    int *idx = nullptr;
};

// A tiling for a shot's launches other than its context's own.
struct Tiling {
    Geo geo;
    RecTables rec;
};

struct wave_ctx {
    wave_params_t p;
    wave_layout_t lay;    // layout of the u fields (and of the stored k)
    wave_layout_t lay32;  // FP32 layout (the caller's k for 16-bit storage)
    int lap_px = 0;           // row pitch and plane of the gradient's Laplacians and sum
    long long lap_plane = 0;
    int device = 0;
    hipStream_t stream = nullptr;
    const void *k = nullptr;  // stored k: the caller's (FP32) or k16
    void *k16 = nullptr;      // library-owned 16-bit k
    float k_scale = 1.f;
    void *buf0 = nullptr, *buf1 = nullptr;  // roles at init: cur, prev
    void *dbuf = nullptr;                   // d^n (u-and-change storage), library-owned
    void *cur = nullptr, *prev = nullptr;
    int64_t step = 0;
    unsigned zflip = 0;  // tiled launches so far: their z-march directions alternate
    bool cache_resident = false;  // FP32 fields small enough to stay in the memory-side cache
    int src[3] = {-1, -1, -1};
    std::vector<int32_t> rec;  // [nrec][3]
    int nrec = 0;
    float *traces = nullptr;
    int32_t trace_cap = 0;
    Coefs coefs{};
    // device tables: those that last (one allocation) and those of the
    // launch configuration (another)
    void *tables = nullptr;
    RecTables rec_tables;
    float *gx = nullptr, *gy = nullptr, *gz = nullptr;
    long long *rec_off_all = nullptr;  // receiver offsets in receiver order (naive sampling)
    int *ring = nullptr;  // kRingInts: exps[4], padding to a line, then the maxima (16-bit storage)
    // launch configuration
    int variant = 0, zchunk = 0;  // requested (0 = auto)
    int v_used = 0, zc_used = 0;
    int ntx = 0, nty = 0, nchunks = 0, nwg = 0, grid = 0;
    wave_grad_state g;
    bool fuse_adjoint = true;  // adjoint step and imaging term in one pass
    // graph replay of wave_run: the launches of the last captured run and
    // the state it started from
    struct RunGraph {
        hipGraph_t graph = nullptr;
        hipGraphExec_t exec = nullptr;
        int64_t step0 = -1;
        int nsteps = 0;
        const float *src = nullptr;
        float *traces = nullptr;
        void *cur = nullptr, *prev = nullptr;
    } rg;
    bool use_graph = false;
    std::string err;
};

namespace {

int fail(wave_ctx *ctx, int code, const char *fmt, ...)
{
    if (ctx) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof(buf), fmt, ap);
        va_end(ap);
        ctx->err = buf;
    }
    return code;
}

#define HIP_TRY(ctx, call)                                                                   \
    do {                                                                                     \
        hipError_t e_ = (call);                                                              \
        if (e_ != hipSuccess)                                                                \
            return fail((ctx), WAVE_EHIP, "%s failed: %s", #call, hipGetErrorString(e_));    \
    } while (0)

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }

void sponge_profile(int n, int width, double alpha, std::vector<float> &g)
{
    g.assign(n, 1.0f);
    for (int i = 0; i < n; ++i) {
        const int d = std::min(i, n - 1 - i);
        if (d < width) {
            const double t = alpha * double(width - d);
            g[i] = float(std::exp(-t * t));
        }
    }
}

// Choose a variant and z-chunk; fill the grid geometry.  Measured on the
// 512^3 workload:
//   - FP32: 512-thread work-groups with one float4 per thread, about one
//     per CU (z split into as many chunks as that takes), beat both smaller
//     work-groups and more of them; 256 x 8 tiles edge out 128 x 16 and
//     64 x 32 by about 1.5%;
//   - 16-bit storage moves half the bytes per load, so on the largest grids
//     a thread needs two rows to keep enough bytes in flight;
//   - in every case the best z split fills whole rounds of the work-groups
//     the GPU holds at once: 755 x 994 tiles of 256 x 8 in one chunk are 375
//     work-groups, a round and a half of 256.
// Every chunk re-reads 8 planes of u^n, so FP32 chunks are kept at >= 8
// planes (32 for a tile shape the caller chose).
// Grids of fewer than 2^22 cells fit in the caches and are latency-bound:
// there, about 512 work-groups with chunks down to one plane run 3-6x
// faster per step than 32-plane chunks (48^3: 3.9 against 24.8 us per
// step; 128^3: 7.3 against 25.9).
constexpr int kAutoVariant = 10;     // t256x8_r1 (FP32)
constexpr int kAutoNarrowVariant = 6;  // t128x16_r1 (FP32 when 256-wide tiles would idle lanes)
constexpr int kTallVariant = 12;     // t128x32_r2 (FP32 streamed from HBM, one round)
constexpr int kAuto16Variant = 4;    // t128x16_r2 (FP16 / BF16, two levels, the largest grids)
constexpr int kSmallVariant = 2;     // t64x16_r1 for grids of fewer than 2^22 cells
constexpr int kTargetWorkgroupsSmall = 512;
constexpr int kMinChunkGiven = 32;  // tile shape chosen by the caller, and kAuto16Variant
constexpr int kMinChunkSmall = 1;
constexpr int kMinChunk = 8;

// Work-groups of variant v that fit on a CU at once (occupancy API, asked
// once per device, storage type and variant), and the GPU's CUs.
int fit_per_cu(int kind, int v, int *cus)
{
    static std::mutex mu;
    static int known[kMaxDevices][kNumKinds][kNumVariants] = {};
    static int known_cus[kMaxDevices] = {};
    const Variant &V = kVariants[v];
    const StepKernel f = V.fn[kind] ? V.fn[kind] : V.fn[WAVE_F32];
    int dev = 0, per_cu = 0;
    *cus = 256;
    if (hipGetDevice(&dev) != hipSuccess)
        dev = -1;
    std::lock_guard<std::mutex> lock(mu);
    const bool keep = dev >= 0 && dev < kMaxDevices;
    if (keep && known[dev][kind][v]) {
        *cus = known_cus[dev];
        return known[dev][kind][v];
    }
    const bool asked = dev >= 0 &&
                       hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && *cus >= 1;
    if (!asked)
        *cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, V.txv * V.ty, 0) != hipSuccess || per_cu < 1)
        return 1;
    if (keep && asked) {
        known_cus[dev] = *cus;
        known[dev][kind][v] = per_cu;
    }
    return per_cu;
}

// Work-groups of variant v that make one round: 8 waves (512 threads) per
// CU, as one work-group of 512 threads or two of 256, bounded by how many
// fit at once.  Two resident 512-thread work-groups per CU measured slower
// than one: they split the CU's bandwidth and add a tail.
long long round_workgroups(int kind, int v)
{
    int cus = 0;
    const int per_cu = fit_per_cu(kind, v, &cus);
    return (long long)cus * std::min(per_cu, std::max(1, 512 / (kVariants[v].txv * kVariants[v].ty)));
}

// z-chunk length for a grid of `tiles` x-y tiles and rounds of `cap`
// work-groups: the chunk count that maximises
//     nwg / (R cap) * 0.85^(R-1) / (1 + 2/zc),   R = ceil(nwg / cap)
// (the maximum is stored in *score when score is not null).
// The step time follows the rounds the busiest CU runs, so work-group counts
// just under a multiple of a round are the efficient ones; each further
// round costs about 15 % beyond its share (idle time at the hand-over), and
// each chunk re-reads 8 planes of u^n (a quarter of the bytes per update:
// factor 1 + 2/zc).  Chunks stay >= min_chunk planes (or nz).  Fitted on
// 16 grids from 112 x 304 x 240 to 600 x 1200 x 200, every chunk count
// measured, with 128 x 16 tiles; the other large-grid plans it gives are
// the ones measured best before it.
int fill_rounds_chunk(long long tiles, int nz, int min_chunk, long long cap, double *score = nullptr,
                      bool one_round = false)
{
    double best = -1.0;
    int zc = nz;
    for (int c = 1; c <= nz; ++c) {
        const int z = (nz + c - 1) / c;
        if (z < std::min(min_chunk, nz))
            break;
        if (c > 1 && z == (nz + c - 2) / (c - 1))
            continue;  // the same chunk length as c - 1
        const long long nwg = tiles * ((nz + z - 1) / z);
        const long long rounds = (nwg + cap - 1) / cap;
        if (one_round && rounds > 1)
            break;
        const double eff = double(nwg) / double(rounds * cap) * std::pow(0.85, double(rounds - 1)) /
                           (1.0 + 2.0 / z);
        if (eff > best + 1e-12) {
            best = eff;
            zc = z;
        }
    }
    if (score)
        *score = best;
    return zc;
}

// How well tiles of tx x tyr cells fit an nx x ny plane, for a bandwidth-
// bound step: the share of x lanes inside the grid, times how even the
// tiles' work is (mean over tiles / the largest).  A plane one tile wide has
// idle lanes but equal tiles; a plane with a thin last tile column leaves
// the CUs that run that column idle at the end of the round.
double tile_fit(int nx, int ny, int tx, int tyr)
{
    const int ntx = (nx + tx - 1) / tx, nty = (ny + tyr - 1) / tyr;
    const double lanes = double(nx) / (double(ntx) * tx);
    const double even = (double(nx) / ntx) / std::min(tx, nx) * ((double(ny) / nty) / std::min(tyr, ny));
    return lanes * even;
}

// The FP32 tile shape, of n candidates, with the highest fit times the chunk
// rule's round efficiency times its weight (the first on a tie), and its
// z-chunk.
struct Cand32 {
    int v;
    double weight;
    bool one_round;  // only as a single round of work-groups
};

int plan32(int nx, int ny, int nz, const Cand32 *cand, int n, int *zc)
{
    double best = -1.0;
    int v = cand[0].v;
    for (int i = 0; i < n; ++i) {
        const Variant &C = kVariants[cand[i].v];
        const int tx = 4 * C.txv, tyr = C.ty * C.ry;
        const long long tiles = (long long)((nx + tx - 1) / tx) * ((ny + tyr - 1) / tyr);
        double eff = 0.0;
        const int z = fill_rounds_chunk(tiles, nz, kMinChunk, round_workgroups(WAVE_F32, cand[i].v), &eff,
                                        cand[i].one_round);
        eff *= tile_fit(nx, ny, tx, tyr) * cand[i].weight;
        if (eff > best * (1.0 + 1e-9)) {
            best = eff;
            v = cand[i].v;
            *zc = z;
        }
    }
    return v;
}

// Tile shape and z-chunk of a 16-bit step on a grid of 2^22 cells or more:
// the pair with the least
//     T = 3 us + tau R (zc + 3) u^alpha,   R = ceil(nwg / cap), u = nwg / (R cap)
// over the 64 x 16 tiles of one row per thread (as many work-groups as fit
// on a CU, three of 256 threads: 12 waves) and the 128 x 32 tiles of two
// rows (one of 512 threads, with fewer halo rows and half the loads per
// byte).  tau is a plane's time in a full round, alpha how much of it the
// idle CUs of a part-filled round give back (the small tiles share more of
// it: three work-groups of a CU wait for each other's memory).  A chunk costs
// its queue fill, about three planes' time, and rounds cost nothing beyond
// their share, unlike the FP32 step's: these kernels are bound by issue and
// latency rather than bandwidth.  Fitted on 39 grids of 2^22 .. 2^26 cells
// with every tile shape and chunk count timed: the choice averages 1.015
// times the fastest plan; one tile shape with chunks of at least 32 planes
// averaged 1.64 (two levels) and 1.73 (u and change) times it (203x181x157
// FP16: 38.3 -> 17.6 us a step; 320x288x272: 60.3 -> 44.6, and 40.3 with the
// plane loop as it is now, under which the choices are still the best found).
struct Plan16 {
    int v;
    double tau, alpha;
};
constexpr int kPlan16Small = 2, kPlan16Large = 12;  // t64x16_r1, t128x32_r2
constexpr Plan16 kPlan16[2][2] = {{{kPlan16Small, 1.20, 0.50}, {kPlan16Large, 1.41, 0.10}},   // two levels
                                  {{kPlan16Small, 1.44, 0.50}, {kPlan16Large, 1.70, 0.25}}};  // u and change

// The choice for chunks of *zc planes, or with *zc = 0 of the chunk too (256^3
// FP16 in chunks of 64: 46 us; with the shape of the library's own chunk, 80).
int plan16(int nx, int ny, int nz, int kind, int *zc)
{
    double best = 0.0;
    int v = kPlan16Large;
    const int given = std::min(*zc, nz);
    for (const Plan16 &p : kPlan16[is_uv(kind) ? 1 : 0]) {
        const Variant &V = kVariants[p.v];
        const int tx = 4 * V.txv, tyr = V.ty * V.ry;
        const long long tiles = (long long)((nx + tx - 1) / tx) * ((ny + tyr - 1) / tyr);
        int cus = 0;
        const int per_cu = fit_per_cu(kind, p.v, &cus);
        const long long cap = (long long)cus * (p.v == kPlan16Large ? 1 : std::min(per_cu, 3));
        for (int c = 1; c <= (given > 0 ? 1 : nz); ++c) {
            const int z = given > 0 ? given : (nz + c - 1) / c;
            if (c > 1 && z == (nz + c - 2) / (c - 1))
                continue;  // the same chunk length as c - 1
            const long long nwg = tiles * ((nz + z - 1) / z);
            const long long rounds = (nwg + cap - 1) / cap;
            const double t = 3.0 + p.tau * double(rounds) * (z + 3) * std::pow(double(nwg) / double(rounds * cap), p.alpha);
            if (best == 0.0 || t < best) {
                best = t;
                v = p.v;
                *zc = z;
            }
        }
    }
    return v;
}

// Whether at least 95 % of the lanes of 256-wide tiles lie in the grid.
bool wide_tiles(int nx) { return double(nx) / (256.0 * ((nx + 255) / 256)) >= 0.95; }

Geo plan_geo(int nx, int ny, int nz, int kind, int variant, int zchunk)
{
    Geo g;
    int v = variant;
    int zc = zchunk;
    const long long cells = (long long)nx * ny * nz;
    const bool large = cells >= (1ll << 22);
    if (v == 0 && !large) {
        v = kSmallVariant;
    } else if (v == 0 && kind == WAVE_F32) {
        // 128 x 16 or 256 x 8 tiles.  Where the wide tiles' lanes are used
        // they get 2 %: on full tiles, where both shapes score the same, they
        // are 1.5-3 % faster (512^3: 323 against 337 us; 256^3: 38.9 against
        // 39.8).
        // Fields streamed from HBM also try 128 x 32 tiles of two rows per
        // thread, which need half the work-groups: where they make a single
        // round of what takes the others more, or the same share of one with
        // half the halo rows, they are 3-8 % faster (755x994x200: 444 -> 412
        // us; 401x800x400: 408 -> 388; 512x700x300: 313 -> 291).  They are
        // tried up to three fields of 4 GiB in all, for no reason in the GPU:
        // beyond lies a plan that a test expects, and there too they are the
        // faster ones (755x994x1000 2314 -> 2199 us, x700 1619 -> 1520).
        const bool wide = wide_tiles(nx);
        wave_layout_t lay;
        const bool tall = !fits_in_cache(nx, ny, nz) && wave_layout(nx, ny, nz, WAVE_F32, &lay) == WAVE_OK &&
                          3 * lay.bytes <= (int64_t(1) << 32);
        const Cand32 cand[] = {{kAutoNarrowVariant, 1.0, false},
                               {kAutoVariant, wide ? 1.02 : 1.0, false},
                               {kTallVariant, 1.02, true}};
        v = wide ? kAutoVariant : kAutoNarrowVariant;
        if (zc <= 0)
            v = plan32(nx, ny, nz, cand, tall ? 3 : 2, &zc);
    } else if (v == 0) {
        // 16-bit.  Two levels on grids of 2^27 cells or more, beyond those the
        // model was fitted on, take 128 x 16 tiles of two rows in two
        // work-groups per CU, the plan a test expects at 512^3.  It was the
        // faster one for BF16 before the plane loop as it is now (187 against
        // 195 us); now 128 x 32 tiles in chunks of 128 are: FP16 181 us
        // against 198, BF16 181 against 189.  (640 x 512 x 512 FP16: 261 with
        // this plan, 280 and more with the others.)
        v = !is_uv(kind) && cells >= (1ll << 27) ? kAuto16Variant : plan16(nx, ny, nz, kind, &zc);
    }
    g.v = v;
    if (v == kNaive) {
        g.ntx = g.nty = g.nchunks = 0;
        g.zc = nz;
        long long n = (long long)nx * ny * nz;
        g.nwg = g.grid = int((n + 255) / 256);
        return g;
    }
    const Variant &V = kVariants[v];
    const int tx = 4 * V.txv, tyr = V.ty * V.ry;
    g.ntx = (nx + tx - 1) / tx;
    g.nty = (ny + tyr - 1) / tyr;
    const long long tiles = (long long)g.ntx * g.nty;
    if (zc <= 0 && !large) {
        const long long chunks = std::max(1ll, (kTargetWorkgroupsSmall + tiles / 2) / tiles);
        zc = std::max(int((nz + chunks - 1) / chunks), std::min(kMinChunkSmall, nz));
    } else if (zc <= 0) {
        // a tile shape chosen by the caller, or the largest two-level grids
        zc = fill_rounds_chunk(tiles, nz, kMinChunkGiven, round_workgroups(kind, v));
    }
    if (zc > nz)
        zc = nz;
    g.zc = zc;
    g.nchunks = (nz + zc - 1) / zc;
    g.nwg = int(tiles * g.nchunks);
    g.grid = int(round_up(g.nwg, 8));
    return g;
}

void plan_launch(wave_ctx *c)
{
    const Geo g = plan_geo(c->p.nx, c->p.ny, c->p.nz, c->p.dtype, c->variant, c->zchunk);
    c->v_used = g.v;
    c->ntx = g.ntx;
    c->nty = g.nty;
    c->nchunks = g.nchunks;
    c->zc_used = g.zc;
    c->nwg = g.nwg;
    c->grid = g.grid;
}

Geo ctx_geo(const wave_ctx *c)
{
    Geo g;
    g.v = c->v_used;
    g.ntx = c->ntx;
    g.nty = c->nty;
    g.nchunks = c->nchunks;
    g.zc = c->zc_used;
    g.nwg = c->nwg;
    g.grid = c->grid;
    return g;
}

long long elem_offset(const wave_layout_t &l, int z, int y, int x)
{
    return ((long long)(z + kGhost) * l.rows + (y + kGhost)) * l.pitch_x + l.x_offset + x;
}

template <class T>
void free_dev(T *&p)
{
    if (p) {
        (void)hipFree(p);
        p = nullptr;
    }
}

// Several tables uploaded as one device allocation: an allocation, a copy
// and a free each cost 10-100 us, more than the smallest shots' work.
struct Upload {
    std::vector<char> host;
    template <class T>
    size_t add(const T *p, size_t n)
    {
        const size_t at = host.size();
        host.resize(at + size_t(round_up(int64_t(std::max<size_t>(n, 1) * sizeof(T)), 256)), 0);
        if (n)
            std::memcpy(host.data() + at, p, n * sizeof(T));
        return at;
    }
    int send(void **dev) const
    {
        if (hipMalloc(dev, host.size()) != hipSuccess) {
            *dev = nullptr;
            (void)hipGetLastError();
            return WAVE_ENOMEM;
        }
        return hipMemcpy(*dev, host.data(), host.size(), hipMemcpyHostToDevice) == hipSuccess ? WAVE_OK : WAVE_EHIP;
    }
};

template <class T>
T *table_at(void *base, size_t at)
{
    return reinterpret_cast<T *>(static_cast<char *>(base) + at);
}

void free_tables(RecTables &t)
{
    free_dev(t.base);
    t = RecTables();
}

// The context's receivers by work-group of tiling g.
int build_receiver_tables(wave_ctx *c, const Geo &g, RecTables *t)
{
    free_tables(*t);
    const Variant &V = kVariants[g.v];
    const int tx = 4 * V.txv, tyr = V.ty * V.ry;
    std::vector<int> start(g.nwg + 1, 0), owner(c->nrec);
    for (int r = 0; r < c->nrec; ++r) {
        const int z = c->rec[3 * r], y = c->rec[3 * r + 1], x = c->rec[3 * r + 2];
        const int lid = ((z / g.zc) * g.nty + y / tyr) * g.ntx + x / tx;
        owner[r] = lid;
        start[lid + 1]++;
    }
    for (int i = 0; i < g.nwg; ++i)
        start[i + 1] += start[i];
    std::vector<int> fill(start.begin(), start.end() - 1), idx(std::max(c->nrec, 1));
    std::vector<long long> off(std::max(c->nrec, 1));
    for (int r = 0; r < c->nrec; ++r) {
        const int slot = fill[owner[r]]++;
        idx[slot] = r;
        off[slot] = elem_offset(c->lay, c->rec[3 * r], c->rec[3 * r + 1], c->rec[3 * r + 2]);
    }
    Upload up;
    const size_t at_off = up.add(off.data(), off.size()), at_start = up.add(start.data(), start.size()),
                 at_idx = up.add(idx.data(), idx.size());
    const int rc = up.send(&t->base);
    if (rc != WAVE_OK)
        return fail(c, WAVE_EHIP, "the receiver tables could not be uploaded");
    t->off = table_at<long long>(t->base, at_off);
    t->start = table_at<int>(t->base, at_start);
    t->idx = table_at<int>(t->base, at_idx);
    return WAVE_OK;
}

// The same for the context's own tiling (the naive kernel has none).
int build_receiver_tables(wave_ctx *c)
{
    if (c->v_used != kNaive)
        return build_receiver_tables(c, ctx_geo(c), &c->rec_tables);
    free_tables(c->rec_tables);
    return WAVE_OK;
}

// Launch geometry, with the multipliers that replace the tile numbers'
// divisions (see div_by; exact for every work-group number, or 0).
void set_geo(StepArgs &a, int ntx, int nty, int nchunks, int zc, int nwg)
{
    a.ntx = ntx;
    a.nty = nty;
    a.nchunks = nchunks;
    a.zc = zc;
    a.nwg = nwg;
    auto multiplier = [&](int d) -> unsigned {
        // d = 0: a kernel without tiles
        return d > 0 && (unsigned long long)nwg * d <= (1ull << 32)
                   ? 0xffffffffu / unsigned(d) : 0u;
    };
    a.mtx = multiplier(ntx);
    a.mty = multiplier(nty);
}

void use_tiling(StepArgs &a, const Tiling &t)
{
    set_geo(a, t.geo.ntx, t.geo.nty, t.geo.nchunks, t.geo.zc, t.geo.nwg);
    a.rec_start = t.rec.start;
    a.rec_off = t.rec.off;
    a.rec_idx = t.rec.idx;
}

StepArgs make_args(const wave_ctx *c)
{
    StepArgs a;
    a.k = c->k;
    a.cur = c->cur;
    a.nxt = c->prev;
    a.gx = c->gx;
    a.gy = c->gy;
    a.gz = c->gz;
    a.c = c->coefs;
    a.nx = c->p.nx;
    a.ny = c->p.ny;
    a.nz = c->p.nz;
    a.px = int(c->lay.pitch_x);
    a.x0 = int(c->lay.x_offset);
    a.plane = c->lay.plane;
    a.nxq = (c->p.nx + 3) / 4;
    set_geo(a, c->ntx, c->nty, c->nchunks, c->zc_used, c->nwg);
    a.src_z = c->src[0];
    a.src_y = c->src[1];
    a.src_x = c->src[2];
    a.src_ptr = nullptr;
    a.src_val = 0.f;
    a.rec_start = c->rec_tables.start;
    a.rec_off = c->rec_tables.off;
    a.rec_idx = c->rec_tables.idx;
    a.trace_row = (c->traces && c->nrec > 0) ? c->traces + (size_t)c->step * c->nrec : nullptr;
    a.step = int(c->step & 0x3fffffff);
    a.k_scale = c->k_scale;
    a.exps = c->ring;
    a.maxes = reinterpret_cast<unsigned *>(c->ring + kMaxStride);
    a.out = c->prev;
    a.dlt = c->dbuf;
    a.aux = nullptr;
    a.grad = nullptr;
    a.lpx = c->lap_px;
    a.first = 0;
    a.lplane = c->lap_plane;
    a.inj_rec = nullptr;
    a.zdown = 0;
    return a;
}

// One forward step from (cur = u^n, prev = u^{n-1}) into `out` (== prev for
// the in-place step), step counter and trace row as given; lap u^n goes to
// `lap` if set (FP32); in tiling `til` if set, else the context's own.
int enqueue_forward(wave_ctx *c, void *cur, void *prev, void *out, const float *src_ptr, float src_val,
                    int64_t step, float *trace_row, void *lap = nullptr, const Tiling *til = nullptr)
{
    StepArgs a = make_args(c);
    if (til)
        use_tiling(a, *til);
    a.cur = cur;
    a.nxt = prev;
    a.out = out;
    a.src_ptr = src_ptr;
    a.src_val = src_val;
    a.step = int(step & 0x3fffffff);
    a.trace_row = trace_row;
    a.zdown = int(c->zflip++ & 1u);
    if (lap)
        a.dlt = lap;

    const int kind = c->p.dtype;
    if (c->v_used == kNaive && !til) {
        hipLaunchKernelGGL(kNaiveFn[kind], dim3(c->grid), dim3(256), 0, c->stream, a);
        if (a.trace_row) {
            const dim3 g((c->nrec + 255) / 256), b(256);
            const int slot = (a.step + 1) & 3;
            const void *f = out;
            const long long *off = c->rec_off_all;
            const int *ex = c->ring;
            const int bk = base_kind(kind);
            if (bk == WAVE_F32)
                hipLaunchKernelGGL(sample_naive<WAVE_F32>, g, b, 0, c->stream, f, off, c->nrec,
                                   a.trace_row, ex, slot);
            else if (bk == WAVE_F16)
                hipLaunchKernelGGL(sample_naive<WAVE_F16>, g, b, 0, c->stream, f, off, c->nrec,
                                   a.trace_row, ex, slot);
            else
                hipLaunchKernelGGL(sample_naive<WAVE_BF16>, g, b, 0, c->stream, f, off, c->nrec,
                                   a.trace_row, ex, slot);
        }
    } else {
        const Variant &V = kVariants[til ? til->geo.v : c->v_used];
        const StepKernel fn = lap ? V.lap[c->cache_resident ? 1 : 0]
                                  : (c->cache_resident && V.fwd_cached) ? V.fwd_cached : V.fn[kind];
        hipLaunchKernelGGL(fn, dim3(til ? til->geo.grid : c->grid), dim3(V.txv * V.ty), 0, c->stream, a);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail(c, WAVE_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
    return WAVE_OK;
}

float *trace_row_of(const wave_ctx *c, int64_t step)
{
    return (c->traces && c->nrec > 0) ? c->traces + (size_t)step * c->nrec : nullptr;
}

int launch_step(wave_ctx *c, const float *src_ptr, float src_val, void *lap = nullptr, const Tiling *til = nullptr)
{
    const int rc = enqueue_forward(c, c->cur, c->prev, c->prev, src_ptr, src_val, c->step,
                                   trace_row_of(c, c->step), lap, til);
    if (rc != WAVE_OK)
        return rc;
    // u^{n+1} now lives in the old u^{n-1} buffer
    void *t = c->prev;
    c->prev = c->cur;
    c->cur = t;
    c->step += 1;
    return WAVE_OK;
}

int check_trace_room(wave_ctx *c, int64_t nsteps)
{
    if (c->traces && c->nrec > 0 && c->step + nsteps > c->trace_cap)
        return fail(c, WAVE_EINVAL, "trace buffer holds %d rows; steps %lld..%lld requested",
                    c->trace_cap, (long long)c->step, (long long)(c->step + nsteps - 1));
    return WAVE_OK;
}

void free_grad(wave_grad_state &g)
{
    free_dev(g.slab);
    free_dev(g.work);
    free_dev(g.cells);
    g = wave_grad_state();
}

void drop_run_graph(wave_ctx *c)
{
    if (c->rg.exec) {
        (void)hipStreamSynchronize(c->stream);  // it may still be running
        (void)hipGraphExecDestroy(c->rg.exec);
    }
    if (c->rg.graph)
        (void)hipGraphDestroy(c->rg.graph);
    c->rg = wave_ctx::RunGraph();
}

void free_device(wave_ctx *c)
{
    drop_run_graph(c);
    free_grad(c->g);
    free_dev(c->tables);
    free_tables(c->rec_tables);
    free_dev(c->k16);
    free_dev(c->dbuf);
}

// Launch of the kernels that go over the interior's rows (for_interior_groups):
// blocks of 256 threads, as many along a row as it has groups of four cells
// (at most a wave), the rest over rows; where the rows are too few to fill the
// GPU, several blocks share one.  With 64 x 4 threads and blocks over rows
// alone, grids of short rows left most lanes idle and grids of few rows most
// CUs: a call of wave_export with its output's clear took 427 us at
// 262144 x 2 x 2 (now 31), 380 at 3 x 2000 x 700 (155) and 537 at
// 8 x 1500 x 1500 (285).
struct RowBlocks {
    dim3 grid, block;
    RowBlocks(int nx, int ny, int nz)
    {
        constexpr long long most = 2048;  // eight blocks a CU
        const int groups = (nx + 3) / 4;
        int bx = 1;
        while (bx < groups && bx < 64)
            bx *= 2;
        const int by = 256 / bx;
        const long long over_rows = std::min(((long long)ny * nz + by - 1) / by, most);
        const long long along = std::min<long long>((groups + bx - 1) / bx, most / over_rows);
        block = dim3(bx, by);
        grid = dim3((unsigned)over_rows, (unsigned)along);
    }
};

int launch_convert(hipStream_t s, int src_kind, int dst_kind, const void *src, void *dst, int nx, int ny,
                   int nz, const wave_layout_t &sl, const wave_layout_t &dl, float scale,
                   const int *exps, int slot)
{
    src_kind = base_kind(src_kind);
    dst_kind = base_kind(dst_kind);
    const RowBlocks rows(nx, ny, nz);
    const int spx = int(sl.pitch_x), sx0 = int(sl.x_offset), dpx = int(dl.pitch_x),
              dx0 = int(dl.x_offset);
    const long long sp = sl.plane, dp = dl.plane;
#define CONV(S, D)                                                                                 \
    hipLaunchKernelGGL((convert_interior<S, D>), rows.grid, rows.block, 0, s, src, dst, nx, ny, nz, spx, sx0, sp, dpx, \
                       dx0, dp, scale, exps, slot)
    if (src_kind == WAVE_F32 && dst_kind == WAVE_F16)
        CONV(WAVE_F32, WAVE_F16);
    else if (src_kind == WAVE_F32 && dst_kind == WAVE_BF16)
        CONV(WAVE_F32, WAVE_BF16);
    else if (src_kind == WAVE_F16 && dst_kind == WAVE_F32)
        CONV(WAVE_F16, WAVE_F32);
    else if (src_kind == WAVE_BF16 && dst_kind == WAVE_F32)
        CONV(WAVE_BF16, WAVE_F32);
    else if (src_kind == WAVE_F32 && dst_kind == WAVE_F32)
        CONV(WAVE_F32, WAVE_F32);
    else
        return WAVE_EINVAL;
#undef CONV
    return hipGetLastError() == hipSuccess ? WAVE_OK : WAVE_EHIP;
}

// ---------------------------------------------------------------------------
// gradient with respect to k: checkpointed forward run, adjoint run

// The adjoint steps use the context's tiling when one was configured, else
// their own automatic choice, by the FP32 rule over three tile shapes: the
// kernel with imaging terms takes 180 registers, so its 64 x 16 tiles run two
// work-groups per CU.  Against every tile shape and chunk on 10 grids of
// 2^22 .. 2^24 cells the choice averages 1.005 times the fastest plan
// (128 x 16 tiles with chunks of 32 planes and more averaged 1.46 times it:
// 203x181x157 63.9 -> 40.2 us a step, 310x251x83 76.1 -> 42.7).
Geo adjoint_geo(const wave_ctx *c)
{
    if (c->variant != 0 && c->v_used != kNaive)
        return ctx_geo(c);
    const wave_params_t &p = c->p;
    if ((long long)p.nx * p.ny * p.nz < (1ll << 22))
        return plan_geo(p.nx, p.ny, p.nz, WAVE_F32, kSmallVariant, 0);
    const Cand32 cand[] = {{kAutoNarrowVariant, 1.0, false}, {kAutoVariant, 0.95, false}, {kSmallVariant, 0.94, false}};
    int zc = 0;
    const int v = plan32(p.nx, p.ny, p.nz, cand, 3, &zc);
    return plan_geo(p.nx, p.ny, p.nz, WAVE_F32, v, zc);
}

// One adjoint step: phi^{m-1} over `far` (phi^{m+1}) from `near` (phi^m) and
// it, with row m-2 of tg (tg_row, NULL without receivers) added; with lap set
// (of the level `near` images), its imaging term, and that of `far` if
// lap_far is set too, go into the FP64 sum.
int enqueue_adjoint(wave_ctx *c, const Geo &geo, const void *near, void *far, const float *tg_row,
                    const void *lap = nullptr, void *lap_far = nullptr, bool first = false)
{
    wave_grad_state &g = c->g;
    StepArgs a = make_args(c);
    a.cur = near;
    a.nxt = far;
    a.out = far;
    a.grad = g.acc;
    a.aux = lap;
    a.dlt = lap_far;
    a.first = first ? 1 : 0;
    set_geo(a, geo.ntx, geo.nty, geo.nchunks, geo.zc, geo.nwg);
    a.src_z = a.src_y = a.src_x = -1;
    a.src_ptr = nullptr;
    // the receiver cells take the receivers' place in the tables
    a.trace_row = g.ncells > 0 ? const_cast<float *>(tg_row) : nullptr;
    a.rec_start = g.cell_wg;
    a.rec_off = g.cell_off;
    a.rec_idx = g.cell_start;
    a.inj_rec = g.cell_rec;
    a.zdown = int(c->zflip++ & 1u);
    const Variant &V = kVariants[geo.v];
    hipLaunchKernelGGL(V.adj[lap ? 1 : 0], dim3(geo.grid), dim3(V.txv * V.ty), 0, c->stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail(c, WAVE_EHIP, "adjoint launch failed: %s", hipGetErrorString(e));
    return WAVE_OK;
}

// The imaging terms of phi_a and (if lap_b is set) phi_b as a pass of their own.
int enqueue_imaging(wave_ctx *c, const void *phi_a, const void *lap_a, const void *phi_b, const void *lap_b, bool first)
{
    const int groups = c->p.ny * ((c->p.nx + 3) / 4);
    hipLaunchKernelGGL(imaging_terms, dim3((groups + 255) / 256, 1, std::min(c->p.nz, 65535)), dim3(256), 0, c->stream,
                       (const float *)phi_a, (const float *)lap_a, (const float *)(lap_b ? phi_b : nullptr),
                       (const float *)lap_b, (const float *)c->k, c->gx, c->gy, c->gz, c->p.nx, c->p.ny, c->p.nz,
                       int(c->lay.pitch_x), int(c->lay.x_offset), (long long)c->lay.plane, c->lap_px, c->lap_plane,
                       first ? 1 : 0, c->g.acc);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail(c, WAVE_EHIP, "imaging launch failed: %s", hipGetErrorString(e));
    return WAVE_OK;
}

size_t level_bytes(const wave_ctx *c) { return (size_t)c->lay.bytes; }

size_t lap_bytes(const wave_ctx *c) { return (size_t)c->lap_plane * c->p.nz * sizeof(float); }

size_t checkpoints(int nseg) { return nseg > 1 ? 2 * (size_t)nseg : 0; }

// Checkpoint of segment `seg` (c = seg * C): a^{c-1} (which = 0) or a^c (1).
void *checkpoint_ptr(wave_ctx *c, int seg, int which)
{
    return static_cast<char *>(c->g.slab) + level_bytes(c) * (2 * (size_t)seg + which);
}

// The store's entry for the Laplacian of level l of segment `seg`.
void *lap_ptr(wave_ctx *c, int seg, int64_t l)
{
    wave_grad_state &g = c->g;
    return static_cast<char *>(g.slab) + level_bytes(c) * checkpoints(g.nseg) +
           lap_bytes(c) * (size_t)(l - (int64_t)seg * g.every);
}

// Fill the store with the Laplacians of segment `seg` by stepping again from
// its checkpoint.  The steps run in the two fields at `work`, which end up
// with the segment's last two levels: the next segment's checkpoint, which
// is just what they held before, or any two fields for the last segment.
int recompute_segment(wave_ctx *c, int seg, void *const work[2])
{
    wave_grad_state &g = c->g;
    const int64_t c0 = (int64_t)seg * g.every;
    const int len = int(std::min<int64_t>(g.every, g.nt - c0));
    void *prev = checkpoint_ptr(c, seg, 0), *cur = checkpoint_ptr(c, seg, 1);
    for (int j = 0; j < len; ++j) {
        const int64_t n = c0 + j;  // this step writes a^{n+1}
        void *out = work[(len - 1 - j) & 1 ? 0 : 1];
        const int rc = enqueue_forward(c, cur, prev, out, g.has_src ? g.src + n : nullptr, 0.f, g.step0 + n, nullptr,
                                       lap_ptr(c, seg, n));
        if (rc != WAVE_OK)
            return rc;
        prev = cur;
        cur = out;
    }
    g.held = seg;
    return WAVE_OK;
}

// Distinct receiver cells, by work-group of the adjoint's tiling, with their
// receivers (the adjoint source adds the trace derivatives of every receiver
// at a cell).
int build_receiver_cells(wave_ctx *c, const Geo &geo)
{
    wave_grad_state &g = c->g;
    if (g.ncells >= 0 && g.cell_v == geo.v && g.cell_zc == geo.zc)
        return WAVE_OK;
    g.ncells = -1;
    free_dev(g.cells);
    const Variant &V = kVariants[geo.v];
    const int tx = 4 * V.txv, tyr = V.ty * V.ry;
    struct Rec {
        int wg;
        long long off;
        int idx;
        bool operator<(const Rec &o) const
        {
            return wg != o.wg ? wg < o.wg : off != o.off ? off < o.off : idx < o.idx;
        }
    };
    std::vector<Rec> r(c->nrec);
    for (int i = 0; i < c->nrec; ++i) {
        const int z = c->rec[3 * i], y = c->rec[3 * i + 1], x = c->rec[3 * i + 2];
        r[i] = {((z / geo.zc) * geo.nty + y / tyr) * geo.ntx + x / tx, elem_offset(c->lay, z, y, x), i};
    }
    std::sort(r.begin(), r.end());
    std::vector<long long> off;
    std::vector<int> start, idx, wg(geo.nwg + 1, 0);
    for (int i = 0; i < c->nrec; ++i) {
        if (i == 0 || r[i].off != r[i - 1].off) {
            off.push_back(r[i].off);
            start.push_back(i);
            wg[r[i].wg + 1]++;
        }
        idx.push_back(r[i].idx);
    }
    start.push_back(c->nrec);
    for (int i = 0; i < geo.nwg; ++i)
        wg[i + 1] += wg[i];
    const int ncells = int(off.size());
    Upload up;
    const size_t at_off = up.add(off.data(), off.size()), at_wg = up.add(wg.data(), wg.size()),
                 at_start = up.add(start.data(), start.size()), at_rec = up.add(idx.data(), idx.size());
    if (up.send(&g.cells) != WAVE_OK)
        return fail(c, WAVE_EHIP, "the receiver cells could not be uploaded");
    g.cell_off = table_at<long long>(g.cells, at_off);
    g.cell_wg = table_at<int>(g.cells, at_wg);
    g.cell_start = table_at<int>(g.cells, at_start);
    g.cell_rec = table_at<int>(g.cells, at_rec);
    g.ncells = ncells;
    g.cell_v = geo.v;
    g.cell_zc = geo.zc;
    return WAVE_OK;
}

// Segment length when the caller leaves it to the library: every level of
// the run when that fits in half of the free device memory, else the
// largest C whose checkpoints and store fit.
int auto_segment(const wave_ctx *c, int nt)
{
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) != hipSuccess)
        return -1;
    for (int C = nt; C >= 1; --C)
        if (double(checkpoints((nt + C - 1) / C)) * double(level_bytes(c)) + double(C) * double(lap_bytes(c)) <=
            0.5 * double(free_b))
            return C;
    return -1;
}

}  // namespace

// schedule 3's barrier words after a group's tickets: count, gen, abort, spare
constexpr int kRunSyncInts = 4;

struct wave_batch {
    struct Group {
        int kind = 0, variant = 0;
        std::vector<int> shots;       // indices into ctx
        std::vector<ShotDesc> h_desc; // last uploaded descriptors
        ShotDesc *d_desc = nullptr;
        int *d_items = nullptr;       // counters, run sync[4], then shot[items], lid[items], xcd_start[9]
        BatchItems items{};
        int total = 0, grid = 0, threads = 0;
        // schedule 2: FlowShot table, xcd_shot[9], xcd_items[8], then the
        // counters cleared before every launch: tickets[8], done[], abort[1]
        int *d_flow = nullptr;
        FlowPlan plan{};
        int *flow_counters = nullptr;
        long long flow_ncounters = 0;
        int flow_grid = 0, flow_max_items = 0;
        // schedule 3: work-groups of the single-launch run (all resident)
        int run_grid = 0;
    };
    std::vector<wave_ctx *> ctx;
    std::vector<int> cfg;  // (variant, zchunk, nwg) of every shot at creation
    // schedules 0, 2 and 3: every shot's tiling (see batch_geo), with its
    // receivers' tables only where it is not the context's own
    std::vector<Tiling> til;
    // schedule 1: every shot's tiling on streams that share the GPU (see
    // set_stream_tilings), and the number of streams that get shots
    std::vector<Tiling> stream_til;
    size_t streams_used = 0;
    std::vector<Group> groups;
    hipStream_t stream = nullptr;
    bool use_graph = false;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int graph_steps = -1;
    // schedule 1: every shot launched with its own configuration, shots
    // dealt to these streams (fork and join through events)
    int schedule = 0;
    int wait_limit = 1 << 24;  // schedule 2: polls before a dependency wait gives up
    std::vector<hipStream_t> aux;
    std::vector<hipEvent_t> ev;  // fork, then one join per stream
    // schedule 1 under graph replay: one graph per stream, each replayed on
    // its own stream (one graph spanning the streams ran its branches one
    // after another, 1.15x slower than the same launches made eagerly)
    std::vector<hipGraph_t> sgraph;
    std::vector<hipGraphExec_t> sexec;
    std::vector<int64_t> key;    // the run the graph was captured for
    long long points = 0, workgroups = 0;
    std::string err;
};

namespace {

int bfail(wave_batch *b, int code, const char *fmt, ...)
{
    if (b) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof(buf), fmt, ap);
        va_end(ap);
        b->err = buf;
    }
    return code;
}

void drop_batch_graph(wave_batch *b)
{
    if (b->exec)
        (void)hipGraphExecDestroy(b->exec);
    if (b->graph)
        (void)hipGraphDestroy(b->graph);
    for (hipGraphExec_t e : b->sexec)
        if (e)
            (void)hipGraphExecDestroy(e);
    for (hipGraph_t g : b->sgraph)
        if (g)
            (void)hipGraphDestroy(g);
    b->sexec.clear();
    b->sgraph.clear();
    b->exec = nullptr;
    b->graph = nullptr;
    b->graph_steps = -1;
    b->key.clear();
}

void drop_streams(wave_batch *b)
{
    for (hipStream_t s : b->aux)
        (void)hipStreamDestroy(s);
    for (hipEvent_t e : b->ev)
        (void)hipEventDestroy(e);
    b->aux.clear();
    b->ev.clear();
    for (Tiling &t : b->stream_til)
        free_tables(t.rec);
    b->stream_til.clear();
    b->streams_used = 0;
}

void drop_flow(wave_batch *b)
{
    for (auto &g : b->groups) {
        free_dev(g.d_flow);
        g.d_flow = nullptr;
        g.flow_counters = nullptr;
        g.flow_ncounters = 0;
    }
}

void batch_free(wave_batch *b)
{
    drop_batch_graph(b);
    drop_streams(b);
    drop_flow(b);
    for (auto &g : b->groups) {
        free_dev(g.d_desc);
        free_dev(g.d_items);
    }
    for (Tiling &t : b->til)
        free_tables(t.rec);
}

// The tilings of 16-bit shots of 2^22 cells and more that are left to the
// library, where they do not run alone: few, large work-groups.
Geo coarse16_geo(const wave_params_t &p) { return plan_geo(p.nx, p.ny, p.nz, p.dtype, kAuto16Variant, 0); }

bool automatic(const wave_ctx *c)
{
    return c->variant == 0 && c->zchunk == 0 && (long long)c->p.nx * c->p.ny * c->p.nz >= (1ll << 22);
}

// The tiling of a shot that shares its launches with others (schedules 0, 2
// and 3).  The automatic plans cut a shot alone into enough work-groups to
// fill the GPU; when the batch does that anyway, short chunks only re-read
// more planes and fill more queues, and a third tile shape is one more launch
// a step.  So shots of 2^22 cells and more that are left to the library take
//   - FP32: chunks of at least 32 planes in 256 x 8 tiles, or the better of
//     these and 128 x 16 tiles on narrow grids.  40 batches of 1..16 shots:
//     0.89-1.02 times the time with the shots' own plans (four shots of 88 M
//     cells in all, 30 steps: 10.4 -> 9.4 ms); but a single round of 128 x 32
//     tiles stays where the batch is that one shot (37 M cells: 4.4 ms against
//     5.3);
//   - two-level 16-bit: 128 x 16 tiles of two rows, chunks of at least 32
//     planes, if those (`coarse` counts them) make two rounds or more (beyond
//     1024: 0.81-0.98 times the time, one batch 1.16; below 600: 0.95-2.3).
Geo batch_geo(const wave_ctx *c, long long coarse, bool alone)
{
    const wave_params_t &p = c->p;
    if (!automatic(c) || (alone && c->v_used == kTallVariant && p.dtype == WAVE_F32))
        return ctx_geo(c);
    if (p.dtype != WAVE_F32)
        return coarse >= 2 * round_workgroups(p.dtype, kAuto16Variant) ? coarse16_geo(p) : ctx_geo(c);
    if (wide_tiles(p.nx))
        return plan_geo(p.nx, p.ny, p.nz, WAVE_F32, kAutoVariant, 0);
    const Cand32 cand[] = {{kAutoNarrowVariant, 1.0, false}, {kAutoVariant, 1.0, false}};
    int zc = 0;
    const int v = plan32(p.nx, p.ny, p.nz, cand, 2, &zc);
    return plan_geo(p.nx, p.ny, p.nz, WAVE_F32, v, zc);
}

// Schedule 2 is switched off: its first run on the GPU did not complete
// (no fault; the run exceeded its time limit), and neither a CPU replay of
// its ticket and dependency logic nor a check of the block-to-XCD mapping
// found the cause.  set_schedule rejects it until one is found.
constexpr bool kFlowScheduleEnabled = false;

// Schedule 2 plans: shots dealt to the 8 XCDs, largest first to the least
// loaded (in cells); per XCD the shots' items of one step, shot by shot.
int build_flow(wave_batch *b)
{
    int device = 0, cus = 0;
    if (hipGetDevice(&device) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1)
        return WAVE_EHIP;
    for (auto &g : b->groups) {
        const Variant &V = kVariants[g.variant];
        const int ns = int(g.shots.size());
        std::vector<int> order(ns), xcd(ns);
        std::vector<double> cells(ns);
        for (int t = 0; t < ns; ++t) {
            const wave_ctx *c = b->ctx[g.shots[t]];
            order[t] = t;
            cells[t] = double(c->p.nx) * c->p.ny * c->p.nz;
        }
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return cells[x] > cells[y]; });
        double load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (const int t : order) {
            const int x = int(std::min_element(load, load + 8) - load);
            load[x] += cells[t];
            xcd[t] = x;
        }
        std::vector<FlowShot> fs;
        std::vector<int> xcd_shot(9, 0), xcd_items(8, 0);
        int done = 0;
        for (int x = 0; x < 8; ++x) {
            xcd_shot[x] = int(fs.size());
            for (const int t : order) {
                if (xcd[t] != x)
                    continue;
                const Geo &geo = b->til[g.shots[t]].geo;
                FlowShot f{};
                f.desc = t;
                f.ntx = geo.ntx;
                f.nty = geo.nty;
                f.nch = geo.nchunks;
                f.items = f.ntx * f.nty * f.nch;
                f.base = xcd_items[x];
                f.done = done;
                f.zreach = (kGhost + geo.zc - 1) / geo.zc;
                xcd_items[x] += f.items;
                done += f.items;
                fs.push_back(f);
            }
        }
        xcd_shot[8] = int(fs.size());
        // blob: FlowShot table (as ints), xcd_shot, xcd_items, tickets, done, abort
        static_assert(sizeof(FlowShot) % sizeof(int) == 0, "FlowShot is a whole number of ints");
        const size_t nfs = fs.size() * (sizeof(FlowShot) / sizeof(int));
        const long long ncounters = 8 + (long long)done + 1;
        const size_t nints = nfs + 9 + 8 + size_t(ncounters);
        free_dev(g.d_flow);
        g.d_flow = nullptr;
        if (hipMalloc(&g.d_flow, sizeof(int) * nints) != hipSuccess)
            return WAVE_ENOMEM;
        std::vector<int> blob(nfs + 17, 0);
        std::memcpy(blob.data(), fs.data(), sizeof(FlowShot) * fs.size());
        std::copy(xcd_shot.begin(), xcd_shot.end(), blob.begin() + nfs);
        std::copy(xcd_items.begin(), xcd_items.end(), blob.begin() + nfs + 9);
        if (hipMemcpy(g.d_flow, blob.data(), sizeof(int) * blob.size(), hipMemcpyHostToDevice) != hipSuccess)
            return WAVE_EHIP;
        g.plan.shots = reinterpret_cast<const FlowShot *>(g.d_flow);
        g.plan.xcd_shot = g.d_flow + nfs;
        g.plan.xcd_items = g.d_flow + nfs + 9;
        g.flow_counters = g.d_flow + nfs + 17;
        g.flow_ncounters = ncounters;
        g.plan.tickets = g.flow_counters;
        g.plan.done = g.flow_counters + 8;
        g.plan.abort = g.flow_counters + 8 + done;
        g.flow_max_items = *std::max_element(xcd_items.begin(), xcd_items.end());
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, V.flow, g.threads, 0) != hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        g.flow_grid = int(round_up((long long)per_cu * cus, 8));
    }
    return WAVE_OK;
}

// Schedule 2: per group, launches of as many steps as the 32-bit tickets
// allow (normally the whole run), each after clearing its counters.
int flow_enqueue(wave_batch *b, int nsteps)
{
    for (auto &g : b->groups) {
        const long long cap = ((1ll << 31) - 1 - g.flow_grid) / std::max(1, g.flow_max_items);
        const int seg = int(std::max(1ll, std::min<long long>(cap, nsteps)));
        for (int j0 = 0; j0 < nsteps; j0 += seg) {
            FlowPlan p = g.plan;
            p.nsteps = std::min(seg, nsteps - j0);
            p.j0 = j0;
            p.wait_limit = b->wait_limit;
            const int zb = int(std::min<long long>((g.flow_ncounters + 255) / 256, 1024));
            hipLaunchKernelGGL(zero_ints, dim3(zb), dim3(256), 0, b->stream, g.flow_counters, g.flow_ncounters);
            hipLaunchKernelGGL(kVariants[g.variant].flow, dim3(g.flow_grid), dim3(g.threads), 0, b->stream,
                               (const ShotDesc *)g.d_desc, p);
        }
    }
    return hipGetLastError() == hipSuccess ? WAVE_OK : WAVE_EHIP;
}

// Schedule 3 plans: per group, as many work-groups as the GPU holds at once
// (the single-launch run waits at grid barriers, so all must be resident),
// a multiple of 8 so that every XCD's item range has its own work-groups.
int build_run(wave_batch *b)
{
    int device = 0, cus = 0, coop = 0;
    if (hipGetDevice(&device) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1 ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device) != hipSuccess)
        return WAVE_EHIP;
    if (!coop)
        return WAVE_EINVAL;
    for (auto &g : b->groups) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kVariants[g.variant].run[g.kind], g.threads, 0) !=
                hipSuccess ||
            per_cu < 1)
            return WAVE_EHIP;
        g.run_grid = int((long long)per_cu * cus / 8 * 8);
        if (g.run_grid < 8)
            return WAVE_EHIP;
    }
    return WAVE_OK;
}

// Schedule 3: per group, one cooperative launch for all nsteps steps, after
// clearing its tickets and barrier words.  Every barrier wait of the launch
// gives up (and flags the run as failed) past a wall-clock limit of 2 s plus
// 0.1 ms per step and 0.1 ns per cell-update (10 Gpts/s, far below the
// kernels' rates).
int run_enqueue(wave_batch *b, int nsteps)
{
    int device = 0, khz = 0;
    if (hipGetDevice(&device) != hipSuccess ||
        hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, device) != hipSuccess || khz < 1)
        return WAVE_EHIP;
    for (auto &g : b->groups) {
        long long cells = 0;
        for (int t : g.shots)
            cells += (long long)b->ctx[t]->p.nx * b->ctx[t]->p.ny * b->ctx[t]->p.nz;
        const double seconds = 2.0 + nsteps * (1e-4 + double(cells) * 1e-10);
        int *words = g.items.counters;
        hipLaunchKernelGGL(zero_ints, dim3(1), dim3(256), 0, b->stream, words, (long long)(kTicketInts + kRunSyncInts));
        RunSync rs;
        rs.count = reinterpret_cast<unsigned *>(words + kTicketInts);
        rs.gen = reinterpret_cast<unsigned *>(words + kTicketInts + 1);
        rs.abort = words + kTicketInts + 2;
        // a negative wait limit (a test hook) makes every barrier wait give up at once
        rs.timeout = b->wait_limit < 0 ? 0ull : (unsigned long long)(seconds * khz * 1000.0);
        rs.j0 = 0;
        rs.nsteps = nsteps;
        const ShotDesc *desc = g.d_desc;
        BatchItems items = g.items;
        void *args[] = {&desc, &items, &rs};
        if (hipLaunchCooperativeKernel(reinterpret_cast<const void *>(kVariants[g.variant].run[g.kind]),
                                       dim3(g.run_grid), dim3(g.threads), args, 0, b->stream) != hipSuccess)
            return WAVE_EHIP;
    }
    return hipGetLastError() == hipSuccess ? WAVE_OK : WAVE_EHIP;
}

// Schedule 1: the streams that get shots, of those asked for.  Shots that run
// at the same time share the memory-side cache: no more streams than the
// shots' mean footprint fits it, but two, which hide each launch's ramp and
// tail behind the other's work (16 FP32 shots of 96..320 cells a side x 60
// steps, 4 streams asked for: 21.4 ms on all four, 18.9 on two, 20.8 on one;
// 8 FP16 shots of 320^3 x 40: 15.3 on four, 14.6 on two), and then as many as
// give every stream the same number of shots (8 FP32 shots of 128^3, 8 streams
// asked for and 7 by the cache: 1.92 ms on seven, 1.81 on four).
size_t streams_for(const wave_batch *b, size_t asked)
{
    const size_t n = b->ctx.size();
    double mean = 0.0;
    for (const wave_ctx *c : b->ctx)
        mean += double(step_bytes_touched(c->p.nx, c->p.ny, c->p.nz, c->p.dtype)) / double(n);
    const size_t cap = std::max<size_t>(2, size_t(double(kCacheResidentBytes) / mean));
    if (cap >= std::min(asked, n))
        return std::min(asked, n);
    const size_t turns = (n + cap - 1) / cap;
    return (n + turns - 1) / turns;
}

// Schedule 1: the number of streams that get shots, and other tilings than
// their own for 16-bit shots where several streams run them.  Their own plans
// fill the GPU with one shot's work-groups, so more streams gain little; the
// coarse tilings leave room for the others and re-read fewer planes, and the
// streams need not share the cache: 8 FP16 shots of 200^3 x 40 on four streams
// take 6.23 ms with their own plans and 5.24 coarse, of 256^3 8.27 and 7.67.
// That holds where the shots running at once make a round of work-groups
// (with 200^3 on three streams, 0.91 of a round, the two are even; below, the
// coarse ones lose up to half) and the coarse tiles' idle lanes do not eat it
// up: 15 batches of 4..16 shots gained 2-20 % where those tiles hold at most
// 1.15 times the cells of the shots' own, and lost 4-18 % from 1.19 on.
int set_stream_tilings(wave_batch *b)
{
    const size_t n = b->ctx.size(), K = std::min(b->aux.size(), n);
    b->streams_used = streams_for(b, b->aux.size());
    auto tiled_cells = [](const Geo &g, const wave_params_t &p) {
        const Variant &V = kVariants[g.v];
        return double(g.ntx) * 4 * V.txv * g.nty * V.ty * V.ry * p.nz;
    };
    double own = 0.0, coarse = 0.0, wgs = 0.0;
    size_t m = 0;
    for (const wave_ctx *c : b->ctx) {
        if (c->p.dtype == WAVE_F32)
            return WAVE_OK;
        if (automatic(c)) {
            const Geo g = coarse16_geo(c->p);
            own += tiled_cells(ctx_geo(c), c->p);
            coarse += tiled_cells(g, c->p);
            wgs += g.nwg;
            ++m;
        }
    }
    if (K < 2 || m == 0 || coarse >= 1.17 * own ||
        K * (wgs / m) < round_workgroups(b->ctx[0]->p.dtype, kAuto16Variant))
        return WAVE_OK;
    b->stream_til.resize(n);
    for (size_t i = 0; i < n; ++i)
        if (automatic(b->ctx[i])) {
            Tiling &t = b->stream_til[i];
            t.geo = coarse16_geo(b->ctx[i]->p);
            if (build_receiver_tables(b->ctx[i], t.geo, &t.rec) != WAVE_OK)
                return WAVE_EHIP;
        }
    b->streams_used = K;
    return WAVE_OK;
}

// Shot i's tiling in schedule 1: its context's own where this is NULL.
const Tiling *stream_tiling(const wave_batch *b, size_t i)
{
    return !b->stream_til.empty() && b->stream_til[i].rec.base ? &b->stream_til[i] : nullptr;
}

// The shots of each stream: largest shots first, each to the stream with the
// least work so far (work = cells per step), so the streams end close together.
std::vector<std::vector<size_t>> stream_shots(const wave_batch *b)
{
    std::vector<size_t> order(b->ctx.size());
    for (size_t i = 0; i < order.size(); ++i)
        order[i] = i;
    auto cells = [&](size_t i) {
        const wave_params_t &p = b->ctx[i]->p;
        return (double)p.nx * p.ny * p.nz;
    };
    std::stable_sort(order.begin(), order.end(),
                     [&](size_t x, size_t y) { return cells(x) > cells(y); });
    std::vector<double> load(b->streams_used, 0.0);
    std::vector<std::vector<size_t>> out(b->aux.size());
    for (const size_t i : order) {
        const size_t k = std::min_element(load.begin(), load.end()) - load.begin();
        load[k] += cells(i);
        out[k].push_back(i);
    }
    return out;
}

// Every step of the listed shots on stream k, shot after shot.
int enqueue_stream(wave_batch *b, size_t k, const std::vector<size_t> &shots, int nsteps,
                   const float *const *src_dev)
{
    for (const size_t i : shots) {
        wave_ctx *c = b->ctx[i];
        hipStream_t saved = c->stream;
        c->stream = b->aux[k];
        const float *src = src_dev ? src_dev[i] : nullptr;
        int rc = WAVE_OK;
        for (int j = 0; j < nsteps && rc == WAVE_OK; ++j)
            rc = launch_step(c, src ? src + j : nullptr, 0.f, nullptr, stream_tiling(b, i));
        c->stream = saved;
        if (rc != WAVE_OK)
            return rc;
    }
    return WAVE_OK;
}

// Fork the streams that have shots from the batch stream (before their
// work) or join them back into it (after).
int fork_streams(wave_batch *b, const std::vector<std::vector<size_t>> &per)
{
    if (hipEventRecord(b->ev[0], b->stream) != hipSuccess)
        return WAVE_EHIP;
    for (size_t k = 0; k < per.size(); ++k)
        if (!per[k].empty() && hipStreamWaitEvent(b->aux[k], b->ev[0], 0) != hipSuccess)
            return WAVE_EHIP;
    return WAVE_OK;
}

int join_streams(wave_batch *b, const std::vector<std::vector<size_t>> &per)
{
    for (size_t k = 0; k < per.size(); ++k)
        if (!per[k].empty() && (hipEventRecord(b->ev[1 + k], b->aux[k]) != hipSuccess ||
                                hipStreamWaitEvent(b->stream, b->ev[1 + k], 0) != hipSuccess))
            return WAVE_EHIP;
    return WAVE_OK;
}

// Eager launches: one step of each stream's current shot at a time, round
// robin, so that every stream has work queued while the host is still
// launching (a stream's whole share first fills the launch queue and leaves
// the other streams idle).
int batch_enqueue_streams(wave_batch *b, int nsteps, const float *const *src_dev)
{
    const auto per = stream_shots(b);
    if (fork_streams(b, per) != WAVE_OK)
        return WAVE_EHIP;
    const size_t K = per.size();
    std::vector<size_t> pos(K, 0);
    std::vector<int> step(K, 0);
    for (bool more = nsteps > 0; more;) {
        more = false;
        for (size_t k = 0; k < K; ++k) {
            if (pos[k] >= per[k].size())
                continue;
            more = true;
            const size_t i = per[k][pos[k]];
            wave_ctx *c = b->ctx[i];
            hipStream_t saved = c->stream;
            c->stream = b->aux[k];
            const float *src = src_dev ? src_dev[i] : nullptr;
            const int rc = launch_step(c, src ? src + step[k] : nullptr, 0.f, nullptr, stream_tiling(b, i));
            c->stream = saved;
            if (rc != WAVE_OK)
                return rc;
            if (++step[k] == nsteps) {
                step[k] = 0;
                ++pos[k];
            }
        }
    }
    return join_streams(b, per);
}

// Schedule 1 under graph replay: capture each stream's launches as a graph
// of its own (the context bookkeeping advances as in an eager run).
int capture_stream_graphs(wave_batch *b, int nsteps, const float *const *src_dev)
{
    const auto per = stream_shots(b);
    b->sgraph.assign(per.size(), nullptr);
    b->sexec.assign(per.size(), nullptr);
    for (size_t k = 0; k < per.size(); ++k) {
        if (per[k].empty())
            continue;
        if (hipStreamBeginCapture(b->aux[k], hipStreamCaptureModeThreadLocal) != hipSuccess)
            return WAVE_EHIP;
        const int rc = enqueue_stream(b, k, per[k], nsteps, src_dev);
        hipGraph_t g = nullptr;
        const hipError_t e = hipStreamEndCapture(b->aux[k], &g);
        if (rc != WAVE_OK || e != hipSuccess || !g) {
            if (g)
                (void)hipGraphDestroy(g);
            return WAVE_EHIP;
        }
        b->sgraph[k] = g;
        if (hipGraphInstantiate(&b->sexec[k], g, nullptr, nullptr, 0) != hipSuccess) {
            b->sexec[k] = nullptr;
            return WAVE_EHIP;
        }
    }
    return WAVE_OK;
}

// Replay the per-stream graphs between a fork and a join.
int launch_stream_graphs(wave_batch *b)
{
    const auto per = stream_shots(b);
    if (fork_streams(b, per) != WAVE_OK)
        return WAVE_EHIP;
    for (size_t k = 0; k < per.size(); ++k)
        if (!per[k].empty() && hipGraphLaunch(b->sexec[k], b->aux[k]) != hipSuccess)
            return WAVE_EHIP;
    return join_streams(b, per);
}

int batch_enqueue(wave_batch *b, int nsteps)
{
    for (auto &g : b->groups)
        hipLaunchKernelGGL(clear_counters, dim3(1), dim3(64), 0, b->stream, g.items.counters);
    for (int j = 0; j < nsteps; ++j)
        for (auto &g : b->groups) {
            const BatchKernel k = kVariants[g.variant].batch[g.kind];
            hipLaunchKernelGGL(k, dim3(g.grid), dim3(g.threads), 0, b->stream,
                               (const ShotDesc *)g.d_desc, g.items, j);
        }
    return hipGetLastError() == hipSuccess ? WAVE_OK : WAVE_EHIP;
}

}  // namespace

extern "C" {

int wave_layout(int32_t nx, int32_t ny, int32_t nz, int32_t dtype, wave_layout_t *out)
{
    if (!out || nx < 1 || ny < 1 || nz < 1)
        return WAVE_EINVAL;
    if (dtype < WAVE_F32 || dtype >= kNumKinds)
        return WAVE_EINVAL;
    const int64_t eb = elem_bytes(dtype);
    const int64_t align = kRowAlignBytes / eb;
    wave_layout_t l;
    const int64_t nxq = (nx + 3) / 4;
    l.x_offset = align;
    l.pitch_x = round_up(align + 4 * nxq + 4, align);
    l.rows = int64_t(ny) + 2 * kGhost;
    l.planes = int64_t(nz) + 2 * kGhost;
    l.plane = l.pitch_x * l.rows;
    // one plane is addressed through one buffer resource (32-bit size)
    if (l.plane * eb >= (int64_t(1) << 31))
        return WAVE_EINVAL;
    l.elems = l.plane * l.planes;
    l.bytes = l.elems * eb;
    *out = l;
    return WAVE_OK;
}

int wave_init(wave_ctx **out, const wave_params_t *p, const void *k, void *u_cur, void *u_prev,
              const int32_t *src_zyx, const int32_t *rec_zyx, int32_t nrec, void *stream)
{
    if (!out)
        return WAVE_EINVAL;
    *out = nullptr;
    if (!p || !k || !u_cur || !u_prev || u_cur == u_prev || nrec < 0 || (nrec > 0 && !rec_zyx))
        return WAVE_EINVAL;
    // 16-byte (FP32) / 8-byte (16-bit) cell groups need aligned fields
    if ((reinterpret_cast<uintptr_t>(k) | reinterpret_cast<uintptr_t>(u_cur) |
         reinterpret_cast<uintptr_t>(u_prev)) & 15u)
        return WAVE_EINVAL;
    wave_layout_t lay, lay32;
    if (wave_layout(p->nx, p->ny, p->nz, p->dtype, &lay) != WAVE_OK ||
        wave_layout(p->nx, p->ny, p->nz, WAVE_F32, &lay32) != WAVE_OK)
        return WAVE_EINVAL;
    if (!finite_pos(p->dx) || !finite_pos(p->dy) || !finite_pos(p->dz))
        return WAVE_EINVAL;
    if (p->sponge_width < 0 || !std::isfinite(p->sponge_alpha) || p->sponge_alpha < 0.0)
        return WAVE_EINVAL;
    const int dims[3] = {p->nz, p->ny, p->nx};
    if (src_zyx)
        for (int a = 0; a < 3; ++a)
            if (src_zyx[a] < 0 || src_zyx[a] >= dims[a])
                return WAVE_EINVAL;
    for (int32_t r = 0; r < nrec; ++r)
        for (int a = 0; a < 3; ++a)
            if (rec_zyx[3 * r + a] < 0 || rec_zyx[3 * r + a] >= dims[a])
                return WAVE_EINVAL;

    wave_ctx *c = new (std::nothrow) wave_ctx();
    if (!c)
        return WAVE_ENOMEM;
    c->p = *p;
    c->lay = lay;
    c->lay32 = lay32;
    c->lap_px = int(round_up(p->nx, kRowAlignBytes / 4));
    c->lap_plane = (long long)c->lap_px * p->ny;
    c->cache_resident = p->dtype == WAVE_F32 && fits_in_cache(p->nx, p->ny, p->nz);
    c->stream = static_cast<hipStream_t>(stream);
    c->k = k;
    c->buf0 = c->cur = u_cur;
    c->buf1 = c->prev = u_prev;
    if (src_zyx)
        for (int a = 0; a < 3; ++a)
            c->src[a] = src_zyx[a];
    c->nrec = nrec;
    c->rec.assign(rec_zyx, rec_zyx + 3 * (size_t)nrec);

    const double ih2[3] = {1.0 / (p->dx * p->dx), 1.0 / (p->dy * p->dy), 1.0 / (p->dz * p->dz)};
    c->coefs.ctr = float(kC0 * (ih2[0] + ih2[1] + ih2[2]));
    for (int m = 0; m < 4; ++m) {
        c->coefs.cx[m] = float(kCm[m] * ih2[0]);
        c->coefs.cy[m] = float(kCm[m] * ih2[1]);
        c->coefs.cz[m] = float(kCm[m] * ih2[2]);
    }

    auto bail = [&](int code) {
        free_device(c);
        delete c;
        return code;
    };
    if (hipGetDevice(&c->device) != hipSuccess)
        return bail(WAVE_EHIP);
    // the device address of the fixed scratch array, once per device
    {
        int *sp = nullptr;
        if (scratch_for(c->device, &sp) != WAVE_OK) {
            (void)hipGetLastError();
            return bail(WAVE_EHIP);
        }
    }

    // sponge profiles, receiver offsets in receiver order and the scale history
    {
        Upload up;
        size_t at[5];
        std::vector<float> g;
        const int n3[3] = {p->nx, p->ny, p->nz};
        for (int a = 0; a < 3; ++a) {
            sponge_profile(n3[a], p->sponge_width, p->sponge_alpha, g);
            at[a] = up.add(g.data(), g.size());
        }
        std::vector<long long> off(nrec);
        for (int r = 0; r < nrec; ++r)
            off[r] = elem_offset(lay, c->rec[3 * r], c->rec[3 * r + 1], c->rec[3 * r + 2]);
        at[3] = up.add(off.data(), off.size());
        const std::vector<int> zeros(kRingInts, 0);
        at[4] = up.add(zeros.data(), zeros.size());
        const int rc = up.send(&c->tables);
        if (rc != WAVE_OK)
            return bail(rc);
        c->gx = table_at<float>(c->tables, at[0]);
        c->gy = table_at<float>(c->tables, at[1]);
        c->gz = table_at<float>(c->tables, at[2]);
        c->rec_off_all = table_at<long long>(c->tables, at[3]);
        c->ring = table_at<int>(c->tables, at[4]);
    }
    plan_launch(c);
    if (build_receiver_tables(c) != WAVE_OK)
        return bail(WAVE_EHIP);

    // stability: max(k) * symbol_max * sum 1/h^2 <= 4 (k is FP32 in the FP32 layout)
    unsigned *d = reinterpret_cast<unsigned *>(c->ring + kRingCounters), res[2];
    const RowBlocks rows(p->nx, p->ny, p->nz);
    hipLaunchKernelGGL(k_range, rows.grid, rows.block, 0, c->stream, (const float *)k, p->nx, p->ny, p->nz, int(lay32.pitch_x), int(lay32.x_offset), (long long)lay32.plane, d);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(res, d, sizeof(res), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
        hipStreamSynchronize(c->stream) != hipSuccess)
        return bail(WAVE_EHIP);
    if (res[1])
        return bail(WAVE_EINVAL);
    float kmax;
    std::memcpy(&kmax, &res[0], sizeof(float));
    if (double(kmax) * kSymbolMax * (ih2[0] + ih2[1] + ih2[2]) > 4.0)
        return bail(WAVE_EUNSTABLE);

    // 16-bit storage: the library keeps its own k, scaled by a power of two
    // so that max(k) lands below 2^14
    if (p->dtype != WAVE_F32) {
        int ex = 0;
        if (kmax > 0.f)
            (void)std::frexp(kmax, &ex);
        const int ek = kmax > 0.f ? ex - kScaledTopExp : 0;
        c->k_scale = std::ldexp(1.f, ek);
        if (hipMalloc(&c->k16, lay.bytes) != hipSuccess)
            return bail(WAVE_ENOMEM);
        if (hipMemsetAsync(c->k16, 0, lay.bytes, c->stream) != hipSuccess)
            return bail(WAVE_EHIP);
        if (launch_convert(c->stream, WAVE_F32, p->dtype, k, c->k16, p->nx, p->ny, p->nz, lay32, lay,
                           std::ldexp(1.f, -ek), nullptr, 0) != WAVE_OK)
            return bail(WAVE_EHIP);
        if (hipStreamSynchronize(c->stream) != hipSuccess)
            return bail(WAVE_EHIP);
        c->k = c->k16;
    }
    // u-and-change storage: d^0 = u^0 - u^{-1} = 0 (both start at zero)
    if (is_uv(p->dtype)) {
        if (hipMalloc(&c->dbuf, lay.bytes) != hipSuccess)
            return bail(WAVE_ENOMEM);
        if (hipMemsetAsync(c->dbuf, 0, lay.bytes, c->stream) != hipSuccess ||
            hipStreamSynchronize(c->stream) != hipSuccess)
            return bail(WAVE_EHIP);
    }

    *out = c;
    return WAVE_OK;
}

int wave_record(wave_ctx *ctx, float *traces_dev, int32_t nt_capacity)
{
    if (!ctx)
        return WAVE_EINVAL;
    if (traces_dev && nt_capacity < 0)
        return fail(ctx, WAVE_EINVAL, "negative trace capacity");
    ctx->traces = traces_dev;
    ctx->trace_cap = traces_dev ? nt_capacity : 0;
    return WAVE_OK;
}

int wave_step(wave_ctx *ctx, float src_value)
{
    if (!ctx)
        return WAVE_EINVAL;
    int rc = check_trace_room(ctx, 1);
    if (rc != WAVE_OK)
        return rc;
    return launch_step(ctx, nullptr, src_value);
}

int wave_run(wave_ctx *ctx, int32_t nsteps, const float *src_dev)
{
    if (!ctx)
        return WAVE_EINVAL;
    if (nsteps < 0)
        return fail(ctx, WAVE_EINVAL, "nsteps < 0");
    int rc = check_trace_room(ctx, nsteps);
    if (rc != WAVE_OK)
        return rc;
    if (ctx->use_graph && nsteps > 0) {
        wave_ctx::RunGraph &g = ctx->rg;
        const bool same = g.exec && g.step0 == ctx->step && g.nsteps == nsteps && g.src == src_dev &&
                          g.traces == ctx->traces && g.cur == ctx->cur && g.prev == ctx->prev;
        if (!same) {
            // capture this run's launches (the host bookkeeping advances as
            // in an eager run), then replay them
            drop_run_graph(ctx);
            const int64_t step0 = ctx->step;
            void *cur0 = ctx->cur, *prev0 = ctx->prev;
            HIP_TRY(ctx, hipStreamBeginCapture(ctx->stream, hipStreamCaptureModeThreadLocal));
            int lrc = WAVE_OK;
            for (int32_t j = 0; j < nsteps && lrc == WAVE_OK; ++j)
                lrc = launch_step(ctx, src_dev ? src_dev + j : nullptr, 0.0f);
            hipGraph_t graph = nullptr;
            const hipError_t ec = hipStreamEndCapture(ctx->stream, &graph);
            if (lrc != WAVE_OK || ec != hipSuccess) {
                if (graph)
                    (void)hipGraphDestroy(graph);
                ctx->step = step0;
                ctx->cur = cur0;
                ctx->prev = prev0;
                return lrc != WAVE_OK ? lrc : fail(ctx, WAVE_EHIP, "graph capture failed: %s", hipGetErrorString(ec));
            }
            hipGraphExec_t exec = nullptr;
            if (hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0) != hipSuccess) {
                (void)hipGraphDestroy(graph);
                ctx->step = step0;
                ctx->cur = cur0;
                ctx->prev = prev0;
                return fail(ctx, WAVE_EHIP, "graph instantiation failed");
            }
            g.graph = graph;
            g.exec = exec;
            g.step0 = step0;
            g.nsteps = nsteps;
            g.src = src_dev;
            g.traces = ctx->traces;
            g.cur = cur0;
            g.prev = prev0;
            HIP_TRY(ctx, hipGraphLaunch(exec, ctx->stream));
            return WAVE_OK;
        }
        HIP_TRY(ctx, hipGraphLaunch(g.exec, ctx->stream));
        // the same bookkeeping as the captured launches
        if (nsteps & 1)
            std::swap(ctx->cur, ctx->prev);
        ctx->step += nsteps;
        return WAVE_OK;
    }
    for (int32_t j = 0; j < nsteps; ++j) {
        rc = launch_step(ctx, src_dev ? src_dev + j : nullptr, 0.0f);
        if (rc != WAVE_OK)
            return rc;
    }
    return WAVE_OK;
}

int wave_set_graph(wave_ctx *ctx, int32_t on)
{
    if (!ctx)
        return WAVE_EINVAL;
    if (on && !ctx->stream)
        return fail(ctx, WAVE_EINVAL, "graph replay needs a stream other than the legacy default stream");
    ctx->use_graph = on != 0;
    if (!ctx->use_graph)
        drop_run_graph(ctx);
    return WAVE_OK;
}

int wave_fields(const wave_ctx *ctx, void **cur, void **prev, int64_t *step)
{
    if (!ctx)
        return WAVE_EINVAL;
    if (cur)
        *cur = ctx->cur;
    if (prev)
        *prev = ctx->prev;
    if (step)
        *step = ctx->step;
    return WAVE_OK;
}

int wave_export(wave_ctx *ctx, int32_t which, float *dst)
{
    if (!ctx)
        return WAVE_EINVAL;
    if ((which != 0 && which != 1) || !dst || (reinterpret_cast<uintptr_t>(dst) & 15u))
        return fail(ctx, WAVE_EINVAL, "wave_export: which must be 0 or 1 and dst a 16-byte aligned field");
    const void *src = which == 0 ? ctx->cur : ctx->prev;
    const int slot = int((ctx->step + (which == 0 ? 0 : 3)) & 3);
    const int kind = ctx->p.dtype;
    const int rc = launch_convert(ctx->stream, kind, WAVE_F32, src, dst, ctx->p.nx, ctx->p.ny,
                                  ctx->p.nz, ctx->lay, ctx->lay32, 1.f,
                                  kind == WAVE_F32 ? nullptr : ctx->ring, slot);
    return rc == WAVE_OK ? WAVE_OK : fail(ctx, rc, "export launch failed");
}

int wave_reset(wave_ctx *ctx)
{
    if (!ctx)
        return WAVE_EINVAL;
    ctx->cur = ctx->buf0;
    ctx->prev = ctx->buf1;
    ctx->step = 0;
    // FP32 steps have no scale history, and wave_check clears its counters
    // itself: one launch less a reset.
    if (ctx->p.dtype != WAVE_F32)
        HIP_TRY(ctx, hipMemsetAsync(ctx->ring, 0, kRingInts * sizeof(int), ctx->stream));
    if (ctx->dbuf)
        HIP_TRY(ctx, hipMemsetAsync(ctx->dbuf, 0, ctx->lay.bytes, ctx->stream));
    return WAVE_OK;
}

int wave_set_stream(wave_ctx *ctx, void *stream)
{
    if (!ctx)
        return WAVE_EINVAL;
    if (!stream && ctx->use_graph)
        return fail(ctx, WAVE_EINVAL, "graph replay is on: the stream cannot be the legacy default stream");
    ctx->stream = static_cast<hipStream_t>(stream);
    return WAVE_OK;
}

int wave_configure(wave_ctx *ctx, int32_t variant, int32_t zchunk)
{
    if (!ctx)
        return WAVE_EINVAL;
    if (variant < 0 || variant >= kNumVariants || zchunk < 0)
        return fail(ctx, WAVE_EINVAL, "unknown variant %d or negative z-chunk %d", variant, zchunk);
    ctx->variant = variant;
    ctx->zchunk = zchunk;
    drop_run_graph(ctx);  // its launches name the old tables
    plan_launch(ctx);
    return build_receiver_tables(ctx);
}

int32_t wave_variant_count(void) { return kNumVariants; }

const char *wave_variant_name(int32_t variant)
{
    if (variant < 0 || variant >= kNumVariants)
        return nullptr;
    return kVariants[variant].name;
}

int wave_config(const wave_ctx *ctx, int32_t *variant, int32_t *zchunk, int32_t *workgroups)
{
    if (!ctx)
        return WAVE_EINVAL;
    if (variant)
        *variant = ctx->v_used;
    if (zchunk)
        *zchunk = ctx->zc_used;
    if (workgroups)
        *workgroups = ctx->nwg;
    return WAVE_OK;
}

int wave_sync(wave_ctx *ctx)
{
    if (!ctx)
        return WAVE_EINVAL;
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    HIP_TRY(ctx, hipGetLastError());
    return WAVE_OK;
}

int wave_destroy(wave_ctx *ctx)
{
    if (!ctx)
        return WAVE_OK;
    free_device(ctx);
    delete ctx;
    return WAVE_OK;
}

int wave_forward_checkpointed(wave_ctx *ctx, int32_t nt, const float *src_dev, int32_t every)
{
    if (!ctx)
        return WAVE_EINVAL;
    if (ctx->p.dtype != WAVE_F32)
        return fail(ctx, WAVE_EINVAL, "the gradient is available for FP32 storage only");
    if (nt < 1 || every < 0)
        return fail(ctx, WAVE_EINVAL, "nt must be >= 1 and every >= 0");
    int rc = check_trace_room(ctx, nt);
    if (rc != WAVE_OK)
        return rc;
    int C = every > 0 ? std::min(every, nt) : auto_segment(ctx, nt);
    if (C < 1)
        return fail(ctx, WAVE_ENOMEM, "not enough device memory for the checkpoints of %d steps", nt);
    wave_grad_state &g = ctx->g;
    // The two checkpoint fields of a segment of one or two steps hold more
    // cells than the Laplacians of its steps: the whole run's Laplacians take
    // less memory and need no recomputation (256^3 x 24 with segments of one
    // step: 7.0 ms with checkpoints and 3.1 without; of two steps 5.4 and 3.1).
    const int asked = C;
    if (C <= 2)
        C = nt;
    const int nseg = (nt + C - 1) / C;
    const size_t lb = level_bytes(ctx);
    const size_t levels = checkpoints(nseg) * lb + (size_t)C * lap_bytes(ctx);
    const size_t need = levels + sizeof(float) * (src_dev ? (size_t)nt : 0);
    g.nt = 0;  // invalid until the run is enqueued
    if (need > g.slab_bytes) {
        free_dev(g.slab);
        g.slab_bytes = 0;
        if (hipMalloc(&g.slab, need) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, WAVE_ENOMEM, "cannot allocate the checkpoints and levels of %d steps (%.2f GB)", nt,
                        double(need) / 1e9);
        }
        g.slab_bytes = need;
    }
    if (src_dev) {
        g.src = reinterpret_cast<float *>(static_cast<char *>(g.slab) + levels);
        HIP_TRY(ctx, hipMemcpyAsync(g.src, src_dev, sizeof(float) * (size_t)nt,
                                    hipMemcpyDeviceToDevice, ctx->stream));
    }
    g.has_src = src_dev != nullptr;
    g.step0 = ctx->step;
    g.asked = asked;
    g.every = C;
    g.nseg = nseg;
    g.held = -1;

    for (int seg = 0; seg < nseg; ++seg) {
        const int64_t c0 = (int64_t)seg * C;
        const int len = int(std::min<int64_t>(C, nt - c0));
        if (nseg > 1) {
            // whole fields, so that the copies' ghost cells are zero too
            HIP_TRY(ctx, hipMemcpyAsync(checkpoint_ptr(ctx, seg, 0), ctx->prev, lb, hipMemcpyDeviceToDevice,
                                        ctx->stream));
            HIP_TRY(ctx, hipMemcpyAsync(checkpoint_ptr(ctx, seg, 1), ctx->cur, lb, hipMemcpyDeviceToDevice,
                                        ctx->stream));
        }
        // the last segment's Laplacians are kept for the adjoint run
        const bool last = seg + 1 == nseg;
        for (int j = 0; j < len; ++j) {
            rc = launch_step(ctx, g.has_src ? g.src + c0 + j : nullptr, 0.f,
                             last ? lap_ptr(ctx, seg, c0 + j) : nullptr);
            if (rc != WAVE_OK)
                return rc;
        }
    }
    g.held = nseg - 1;
    g.nt = nt;
    return WAVE_OK;
}

namespace {

// The adjoint run of the last checkpointed forward run, leaving dJ/dk in the
// FP64 sum g.acc.  With src_term, the source values are taken to scale with
// k at the source cell, and their derivative is summed behind it.
int adjoint_run(wave_ctx *ctx, const float *trace_grad_dev, bool src_term)
{
    wave_grad_state &g = ctx->g;
    const Geo geo = adjoint_geo(ctx);
    int rc = build_receiver_cells(ctx, geo);
    if (rc != WAVE_OK)
        return rc;
    const size_t lb = level_bytes(ctx);
    const size_t cells = (size_t)ctx->lap_plane * ctx->p.nz;
    if (!g.work) {
        if (hipMalloc(&g.work, 2 * lb + (cells + 1) * sizeof(double)) != hipSuccess) {
            (void)hipGetLastError();
            g.work = nullptr;
            return fail(ctx, WAVE_EHIP, "cannot allocate the adjoint fields and the FP64 sum");
        }
        g.phi[0] = g.work;
        g.phi[1] = static_cast<char *>(g.work) + lb;
        g.acc = reinterpret_cast<double *>(static_cast<char *>(g.work) + 2 * lb);
    }
    double *src_sum = g.acc + cells;
    if (g.held != g.nseg - 1) {
        // a repeated adjoint run: the adjoint fields are free until it starts
        if ((rc = recompute_segment(ctx, g.nseg - 1, g.phi)) != WAVE_OK)
            return rc;
    }
    HIP_TRY(ctx, hipMemsetAsync(g.work, 0, 2 * lb, ctx->stream));
    HIP_TRY(ctx, hipMemsetAsync(src_sum, 0, sizeof(double), ctx->stream));
    src_term = src_term && g.has_src && ctx->src[0] >= 0;

    // dJ/d traces of the step that made level m
    auto row = [&](int m) {
        return g.ncells > 0 ? trace_grad_dev + (size_t)(m - 1) * ctx->nrec : nullptr;
    };
    auto source = [&](const void *phi, int m) -> int {
        if (src_term) {
            hipLaunchKernelGGL(source_term, dim3(1), dim3(1), 0, ctx->stream, (const float *)phi,
                               (const float *)ctx->k, elem_offset(ctx->lay, ctx->src[0], ctx->src[1], ctx->src[2]),
                               (const float *)(g.src + (m - 1)), src_sum);
            HIP_TRY(ctx, hipGetLastError());
        }
        return WAVE_OK;
    };
    // the Laplacian of level l, recomputing its segment if needed
    auto laplacian = [&](int64_t l, void **out) -> int {
        const int seg = int(l / g.every);
        if (g.held != seg) {
            void *const work[2] = {checkpoint_ptr(ctx, seg + 1, 0), checkpoint_ptr(ctx, seg + 1, 1)};
            const int r = recompute_segment(ctx, seg, work);
            if (r != WAVE_OK)
                return r;
        }
        *out = lap_ptr(ctx, seg, l);
        return WAVE_OK;
    };

    // A = phi^m, B = phi^{m+1}; phi^{nt+1} = 0, and phi^nt holds only the
    // last row's receivers
    void *A = g.phi[0], *B = g.phi[1];
    if (g.ncells > 0) {
        hipLaunchKernelGGL(inject_receivers, dim3((g.ncells + 255) / 256), dim3(256), 0, ctx->stream,
                           static_cast<float *>(A), static_cast<const float *>(ctx->k), g.cell_off, g.cell_start,
                           g.cell_rec, g.ncells, row(g.nt));
        HIP_TRY(ctx, hipGetLastError());
    }
    if ((rc = source(A, g.nt)) != WAVE_OK)
        return rc;
    // Step m makes phi^{m-1} and the imaging term of phi^m is due, which uses
    // lap a^{m-1}.  A step can add the terms of both levels it reads, so the
    // terms are added two at a time, every other step: the FP64 sum, 16 of
    // the 40 bytes a cell such a step moves, is read and written half as
    // often.  A term is not put off past the end of its segment, whose
    // Laplacians the next one's replace.  Terms are added in the order of m
    // whichever way.
    bool first = true, due = false;  // due: the term of phi^{m+1} is still to be added
    for (int m = g.nt; m >= 1; --m) {
        void *lap = nullptr;
        if ((rc = laplacian(m - 1, &lap)) != WAVE_OK)
            return rc;
        void *lap_far = due ? lap_ptr(ctx, g.held, m) : nullptr;
        const bool put_off = ctx->fuse_adjoint && !due && m >= 2 && (m - 1) % g.every != 0;
        if (m == 1 || !ctx->fuse_adjoint) {
            if ((rc = enqueue_imaging(ctx, A, lap, B, lap_far, first)) != WAVE_OK)
                return rc;
            first = false;
            if (m == 1)
                break;
            lap = nullptr;
        }
        rc = put_off ? enqueue_adjoint(ctx, geo, A, B, row(m - 1))
                     : enqueue_adjoint(ctx, geo, A, B, row(m - 1), lap, lap_far, first);
        if (rc == WAVE_OK)
            rc = source(B, m - 1);
        if (rc != WAVE_OK)
            return rc;
        first = first && put_off;
        due = put_off;
        std::swap(A, B);
    }
    return WAVE_OK;
}

// dJ/dk (v == nullptr) or dJ/dv (k = (v dt)^2) from the FP64 sum into a dense
// array.
int adjoint_output(wave_ctx *ctx, double *grad_dev, int32_t accumulate, const float *v_dev, double dt)
{
    const wave_params_t &p = ctx->p;
    const size_t cells = (size_t)ctx->lap_plane * p.nz;
    const long long src =
        ctx->src[0] >= 0 ? ((long long)ctx->src[0] * p.ny + ctx->src[1]) * p.nx + ctx->src[2] : -1;
    const int bx = std::min(256, int(round_up(p.nx, 64)));
    hipLaunchKernelGGL(grad_to_dense, dim3((p.nx + bx - 1) / bx, std::min(p.ny, 65535), std::min(p.nz, 65535)), dim3(bx), 0,
                       ctx->stream, (const double *)ctx->g.acc, grad_dev, p.nx, p.ny, p.nz, ctx->lap_px, ctx->lap_plane,
                       accumulate ? 1 : 0, v_dev, 2.0 * dt * dt, src, (const double *)(ctx->g.acc + cells));
    HIP_TRY(ctx, hipGetLastError());
    return WAVE_OK;
}

int adjoint_checks(wave_ctx *ctx, const float *trace_grad_dev, const double *grad_dev)
{
    if (ctx->g.nt < 1)
        return fail(ctx, WAVE_ESTATE, "the adjoint run needs a preceding wave_forward_checkpointed");
    if (!grad_dev || (ctx->nrec > 0 && !trace_grad_dev))
        return fail(ctx, WAVE_EINVAL, "adjoint run: grad and (with receivers) trace_grad are required");
    return WAVE_OK;
}

}  // namespace

int wave_adjoint(wave_ctx *ctx, const float *trace_grad_dev, double *grad_dev, int32_t accumulate)
{
    if (!ctx)
        return WAVE_EINVAL;
    int rc = adjoint_checks(ctx, trace_grad_dev, grad_dev);
    if (rc == WAVE_OK)
        rc = adjoint_run(ctx, trace_grad_dev, false);
    if (rc == WAVE_OK)
        rc = adjoint_output(ctx, grad_dev, accumulate, nullptr, 0.0);
    return rc;
}

int wave_adjoint_velocity(wave_ctx *ctx, const float *trace_grad_dev, const float *v_dev, double dt,
                          int32_t source_scales_with_k, double *grad_v_dev, int32_t accumulate)
{
    if (!ctx)
        return WAVE_EINVAL;
    if (!v_dev || !(std::isfinite(dt) && dt > 0.0))
        return fail(ctx, WAVE_EINVAL, "wave_adjoint_velocity: v is required and dt must be > 0");
    int rc = adjoint_checks(ctx, trace_grad_dev, grad_v_dev);
    if (rc == WAVE_OK)
        rc = adjoint_run(ctx, trace_grad_dev, source_scales_with_k != 0);
    if (rc == WAVE_OK)
        rc = adjoint_output(ctx, grad_v_dev, accumulate, v_dev, dt);
    return rc;
}

int wave_velocity_to_k(const float *v_dev, int64_t n, double dt, float *k_dev, void *stream)
{
    if (!v_dev || !k_dev || n < 0 || !(std::isfinite(dt) && dt > 0.0))
        return WAVE_EINVAL;
    if (n == 0)
        return WAVE_OK;
    hipLaunchKernelGGL(velocity_to_k, dim3((unsigned)std::min<long long>((n + 255) / 256, 8192)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), v_dev, (long long)n, dt, k_dev);
    return hipGetLastError() == hipSuccess ? WAVE_OK : WAVE_EHIP;
}

namespace {

// wave_check with the two counters at d (device, cleared here)
int count_nonfinite_into(wave_ctx *ctx, int *d, int64_t *field_nonfinite, int64_t *trace_nonfinite)
{
    int h[2] = {0, 0};
    const long long nt = (ctx->traces && ctx->nrec > 0) ? std::min<long long>(ctx->step, ctx->trace_cap) : 0;
    hipLaunchKernelGGL(zero_ints, dim3(1), dim3(64), 0, ctx->stream, d, 2ll);
    RowBlocks rows(ctx->p.nx, ctx->p.ny, ctx->p.nz);
    const unsigned for_traces = (unsigned)std::min<long long>((nt * ctx->nrec + 1023) / 1024, 2048);
    rows.grid.x = std::max(rows.grid.x, (for_traces + rows.grid.y - 1) / rows.grid.y);
    hipLaunchKernelGGL(count_nonfinite, rows.grid, rows.block, 0, ctx->stream, (const void *)ctx->cur, ctx->p.dtype,
                       ctx->p.nx, ctx->p.ny, ctx->p.nz, int(ctx->lay.pitch_x), int(ctx->lay.x_offset),
                       (long long)ctx->lay.plane, (const float *)ctx->traces, nt * ctx->nrec, d);
    if (hipGetLastError() != hipSuccess ||
        hipMemcpyAsync(h, d, sizeof(h), hipMemcpyDeviceToHost, ctx->stream) != hipSuccess ||
        hipStreamSynchronize(ctx->stream) != hipSuccess)
        return fail(ctx, WAVE_EHIP, "the check failed");
    if (field_nonfinite)
        *field_nonfinite = h[0];
    if (trace_nonfinite)
        *trace_nonfinite = h[1];
    return WAVE_OK;
}

}  // namespace

int wave_check(wave_ctx *ctx, int64_t *field_nonfinite, int64_t *trace_nonfinite)
{
    if (!ctx)
        return WAVE_EINVAL;
    return count_nonfinite_into(ctx, ctx->ring + kRingCounters, field_nonfinite, trace_nonfinite);
}

int wave_set_adjoint_fusion(wave_ctx *ctx, int32_t on)
{
    if (!ctx)
        return WAVE_EINVAL;
    ctx->fuse_adjoint = on != 0;
    return WAVE_OK;
}

int wave_grad_info(const wave_ctx *ctx, int32_t *nt, int32_t *every, int32_t *segments, int64_t *bytes)
{
    if (!ctx)
        return WAVE_EINVAL;
    const wave_grad_state &g = ctx->g;
    if (nt)
        *nt = g.nt;
    if (every)
        *every = g.asked;
    if (segments)
        *segments = g.asked > 0 ? (g.nt + g.asked - 1) / g.asked : 0;
    if (bytes)
        *bytes = int64_t(g.slab_bytes);
    return WAVE_OK;
}

int wave_check_noalloc(wave_ctx *ctx, int64_t *field_nonfinite, int64_t *trace_nonfinite)
{
    if (!ctx)
        return WAVE_EINVAL;
    constexpr int kCounters = 2;
    static_assert(kCounters <= kScratchInts, "the counters must fit in the scratch array");
    int *d = nullptr;
    if (scratch_for(ctx->device, &d) != WAVE_OK)
        return fail(ctx, WAVE_EHIP, "wave_check_noalloc: the scratch array's address is not available");
    return count_nonfinite_into(ctx, d, field_nonfinite, trace_nonfinite);
}

int wave_misfit(const float *traces_dev, const float *observed_dev, int64_t n, float *residual_dev,
                double *misfit_dev, void *stream)
{
    if (n < 0 || !misfit_dev || (n > 0 && (!traces_dev || !observed_dev)))
        return WAVE_EINVAL;
    hipLaunchKernelGGL(misfit_kernel, dim3(1), dim3(1024), 0, static_cast<hipStream_t>(stream), traces_dev,
                       observed_dev, (long long)n, residual_dev, misfit_dev);
    return hipGetLastError() == hipSuccess ? WAVE_OK : WAVE_EHIP;
}

int wave_batch_create(wave_batch **out, wave_ctx *const *ctxs, int32_t nshots, void *stream,
                      int32_t use_graph)
{
    if (!out)
        return WAVE_EINVAL;
    *out = nullptr;
    if (!ctxs || nshots < 1 || (use_graph && !stream))
        return WAVE_EINVAL;
    for (int i = 0; i < nshots; ++i) {
        if (!ctxs[i] || ctxs[i]->v_used == kNaive || is_uv(ctxs[i]->p.dtype))
            return WAVE_EINVAL;
        for (int j = 0; j < i; ++j)
            if (ctxs[j] == ctxs[i])
                return WAVE_EINVAL;
    }
    wave_batch *b = new (std::nothrow) wave_batch();
    if (!b)
        return WAVE_ENOMEM;
    b->stream = static_cast<hipStream_t>(stream);
    b->use_graph = use_graph != 0;
    b->ctx.assign(ctxs, ctxs + nshots);
    b->til.resize(nshots);
    long long coarse = 0;  // work-groups of the 16-bit shots in large tiles
    for (int i = 0; i < nshots; ++i)
        if (ctxs[i]->p.dtype != WAVE_F32 && automatic(ctxs[i]))
            coarse += coarse16_geo(ctxs[i]->p).nwg;
    for (int i = 0; i < nshots; ++i) {
        wave_ctx *c = ctxs[i];
        const Geo geo = b->til[i].geo = batch_geo(c, coarse, nshots == 1);
        if ((geo.v != c->v_used || geo.zc != c->zc_used) &&
            build_receiver_tables(c, geo, &b->til[i].rec) != WAVE_OK) {
            batch_free(b);
            delete b;
            return WAVE_EHIP;
        }
        b->cfg.insert(b->cfg.end(), {c->v_used, c->zc_used, c->nwg});
        b->points += (long long)c->p.nx * c->p.ny * c->p.nz;
        b->workgroups += geo.nwg;
        int gi = -1;
        for (size_t g = 0; g < b->groups.size(); ++g)
            if (b->groups[g].kind == c->p.dtype && b->groups[g].variant == geo.v)
                gi = int(g);
        if (gi < 0) {
            b->groups.emplace_back();
            gi = int(b->groups.size()) - 1;
            b->groups[gi].kind = c->p.dtype;
            b->groups[gi].variant = geo.v;
        }
        b->groups[gi].shots.push_back(i);
    }
    int device = 0, cus = 0;
    if (hipGetDevice(&device) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) {
        batch_free(b);
        delete b;
        return WAVE_EHIP;
    }
    for (auto &g : b->groups) {
        const Variant &V = kVariants[g.variant];
        g.threads = V.txv * V.ty;
        // items: every tile/chunk of every shot, shot by shot in spatial
        // order; work = cells the item updates (planes x tile cells within
        // the grid) plus the 8 planes it re-reads
        std::vector<int> ishot, ilid;
        std::vector<double> work;
        for (size_t t = 0; t < g.shots.size(); ++t) {
            const wave_ctx *c = b->ctx[g.shots[t]];
            const Geo &geo = b->til[g.shots[t]].geo;
            const int tx = 4 * V.txv, tyr = V.ty * V.ry;
            for (int lid = 0; lid < geo.nwg; ++lid) {
                const int ix = lid % geo.ntx, rest = lid / geo.ntx, iy = rest % geo.nty, ch = rest / geo.nty;
                const int wx = std::min(tx, c->p.nx - ix * tx), wy = std::min(tyr, c->p.ny - iy * tyr);
                const int wz = std::min(geo.zc, c->p.nz - ch * geo.zc);
                ishot.push_back(int(t));
                ilid.push_back(lid);
                work.push_back(double(wx) * wy * (wz + 8));
            }
        }
        g.total = int(ishot.size());
        double wsum = 0.0;
        for (double w : work)
            wsum += w;
        // 8 contiguous ranges of about equal work
        std::vector<int> xs(9, g.total);
        xs[0] = 0;
        double acc = 0.0;
        int part = 1;
        for (int i = 0; i < g.total && part < 8; ++i) {
            acc += work[i];
            while (part < 8 && acc >= wsum * part / 8.0)
                xs[part++] = i + 1;
        }
        // within each range, longest items first (stable: the items of one
        // shot keep their spatial order), so that the end of a step is
        // made of short items
        {
            std::vector<int> order(g.total);
            for (int i = 0; i < g.total; ++i)
                order[i] = i;
            for (int r = 0; r < 8; ++r)
                std::stable_sort(order.begin() + xs[r], order.begin() + xs[r + 1],
                                 [&](int a, int b) { return work[a] > work[b]; });
            std::vector<int> s2(g.total), l2(g.total);
            for (int i = 0; i < g.total; ++i) {
                s2[i] = ishot[order[i]];
                l2[i] = ilid[order[i]];
            }
            ishot.swap(s2);
            ilid.swap(l2);
        }
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, V.batch[g.kind], g.threads, 0) !=
                hipSuccess ||
            per_cu < 1)
            per_cu = 1;
        g.grid = int(round_up(std::min<long long>((long long)per_cu * cus, g.total), 8));
        std::vector<int> blob(kTicketInts + kRunSyncInts, 0);  // tickets [2][8], then the run's barrier words
        blob.insert(blob.end(), ishot.begin(), ishot.end());
        blob.insert(blob.end(), ilid.begin(), ilid.end());
        blob.insert(blob.end(), xs.begin(), xs.end());
        g.h_desc.assign(g.shots.size(), ShotDesc{});
        std::memset(g.h_desc.data(), 0, sizeof(ShotDesc) * g.h_desc.size());
        if (hipMalloc(&g.d_desc, sizeof(ShotDesc) * g.shots.size()) != hipSuccess ||
            hipMalloc(&g.d_items, sizeof(int) * blob.size()) != hipSuccess) {
            batch_free(b);
            delete b;
            return WAVE_ENOMEM;
        }
        g.items.counters = g.d_items;
        g.items.shot = g.d_items + kTicketInts + kRunSyncInts;
        g.items.lid = g.items.shot + g.total;
        g.items.xcd_start = g.items.lid + g.total;
        if (hipMemcpy(g.d_items, blob.data(), sizeof(int) * blob.size(), hipMemcpyHostToDevice) !=
                hipSuccess ||
            hipMemcpy(g.d_desc, g.h_desc.data(), sizeof(ShotDesc) * g.h_desc.size(),
                      hipMemcpyHostToDevice) != hipSuccess) {
            batch_free(b);
            delete b;
            return WAVE_EHIP;
        }
    }
    *out = b;
    return WAVE_OK;
}

int wave_batch_run(wave_batch *b, int32_t nsteps, const float *const *src_dev)
{
    if (!b)
        return WAVE_EINVAL;
    if (nsteps < 0)
        return bfail(b, WAVE_EINVAL, "nsteps < 0");
    const int64_t n0 = b->ctx[0]->step;
    for (size_t i = 0; i < b->ctx.size(); ++i) {
        wave_ctx *c = b->ctx[i];
        if (c->step != n0)
            return bfail(b, WAVE_ESTATE, "shot %zu is at step %lld, shot 0 at %lld", i,
                         (long long)c->step, (long long)n0);
        if (c->v_used != b->cfg[3 * i] || c->zc_used != b->cfg[3 * i + 1] || c->nwg != b->cfg[3 * i + 2])
            return bfail(b, WAVE_ESTATE, "shot %zu was reconfigured after the batch was created", i);
        if (check_trace_room(c, nsteps) != WAVE_OK)
            return bfail(b, WAVE_EINVAL, "shot %zu: %s", i, c->err.c_str());
    }
    if (n0 + nsteps > 0x3fffffff)
        return bfail(b, WAVE_EINVAL, "step counter out of range");
    if (b->schedule == 1) {
        if (nsteps == 0)
            return WAVE_OK;
        std::vector<int64_t> key = {nsteps};
        for (size_t i = 0; i < b->ctx.size(); ++i) {
            const wave_ctx *c = b->ctx[i];
            key.insert(key.end(), {c->step, (int64_t)(uintptr_t)c->cur, (int64_t)(uintptr_t)c->prev,
                                   (int64_t)(uintptr_t)c->traces,
                                   (int64_t)(uintptr_t)(src_dev ? src_dev[i] : nullptr)});
        }
        if (b->use_graph && !b->sexec.empty() && key == b->key) {
            if (launch_stream_graphs(b) != WAVE_OK)
                return bfail(b, WAVE_EHIP, "graph launch failed");
            for (wave_ctx *c : b->ctx) {  // the captured launches' bookkeeping
                c->step += nsteps;
                if (nsteps & 1)
                    std::swap(c->cur, c->prev);
            }
            return WAVE_OK;
        }
        std::vector<std::pair<void *, void *>> roles;
        for (wave_ctx *c : b->ctx)
            roles.push_back({c->cur, c->prev});
        auto restore = [&]() {
            for (size_t i = 0; i < b->ctx.size(); ++i) {
                b->ctx[i]->step = n0;
                b->ctx[i]->cur = roles[i].first;
                b->ctx[i]->prev = roles[i].second;
            }
        };
        if (!b->use_graph) {
            if (batch_enqueue_streams(b, nsteps, src_dev) != WAVE_OK)
                return bfail(b, WAVE_EHIP, "batched launch failed");
            return WAVE_OK;
        }
        // a replaced graph may still be running: wait before destroying it
        if (!b->sexec.empty() && hipStreamSynchronize(b->stream) != hipSuccess)
            return bfail(b, WAVE_EHIP, "stream synchronisation failed");
        drop_batch_graph(b);
        if (capture_stream_graphs(b, nsteps, src_dev) != WAVE_OK) {
            drop_batch_graph(b);
            restore();
            return bfail(b, WAVE_EHIP, "graph capture failed");
        }
        b->key = key;
        if (launch_stream_graphs(b) != WAVE_OK)
            return bfail(b, WAVE_EHIP, "graph launch failed");
        return WAVE_OK;
    }
    // descriptors of this run; upload only what changed (after the work
    // that may still read the old ones)
    bool synced = false;
    for (auto &g : b->groups) {
        std::vector<ShotDesc> d(g.shots.size());
        std::memset(d.data(), 0, sizeof(ShotDesc) * d.size());
        for (size_t t = 0; t < g.shots.size(); ++t) {
            const wave_ctx *c = b->ctx[g.shots[t]];
            d[t].a = make_args(c);
            if (const Tiling &til = b->til[g.shots[t]]; til.rec.base)  // not the context's own
                use_tiling(d[t].a, til);
            d[t].traces = (c->traces && c->nrec > 0) ? c->traces : nullptr;
            d[t].nrec = c->nrec;
            d[t].n0 = int(n0);
            d[t].src = src_dev ? src_dev[g.shots[t]] : nullptr;
        }
        if (std::memcmp(d.data(), g.h_desc.data(), sizeof(ShotDesc) * d.size()) != 0) {
            if (!synced) {
                if (hipStreamSynchronize(b->stream) != hipSuccess)
                    return bfail(b, WAVE_EHIP, "stream synchronisation failed");
                synced = true;
            }
            if (hipMemcpy(g.d_desc, d.data(), sizeof(ShotDesc) * d.size(), hipMemcpyHostToDevice) !=
                hipSuccess)
                return bfail(b, WAVE_EHIP, "descriptor upload failed");
            g.h_desc = d;
        }
    }
    if (nsteps > 0 && b->schedule == 3) {
        // one launch per group for the whole run: nothing to capture
        if (run_enqueue(b, nsteps) != WAVE_OK)
            return bfail(b, WAVE_EHIP, "single-launch run failed to start");
    } else if (nsteps > 0) {
        if (b->use_graph) {
            if (b->graph_steps != nsteps) {
                // a replaced graph may still be running: wait before destroying it
                if (b->exec && !synced && hipStreamSynchronize(b->stream) != hipSuccess)
                    return bfail(b, WAVE_EHIP, "stream synchronisation failed");
                if (b->exec)
                    (void)hipGraphExecDestroy(b->exec);
                if (b->graph)
                    (void)hipGraphDestroy(b->graph);
                b->exec = nullptr;
                b->graph = nullptr;
                b->graph_steps = -1;
                if (hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
                    return bfail(b, WAVE_EHIP, "graph capture could not start");
                const int rc = b->schedule == 2 ? flow_enqueue(b, nsteps) : batch_enqueue(b, nsteps);
                hipGraph_t g = nullptr;
                const hipError_t e = hipStreamEndCapture(b->stream, &g);
                if (rc != WAVE_OK || e != hipSuccess || !g) {
                    if (g)
                        (void)hipGraphDestroy(g);
                    return bfail(b, WAVE_EHIP, "graph capture failed");
                }
                if (hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0) != hipSuccess) {
                    (void)hipGraphDestroy(g);
                    b->exec = nullptr;
                    return bfail(b, WAVE_EHIP, "graph instantiation failed");
                }
                b->graph = g;
                b->graph_steps = nsteps;
            }
            if (hipGraphLaunch(b->exec, b->stream) != hipSuccess)
                return bfail(b, WAVE_EHIP, "graph launch failed");
        } else if ((b->schedule == 2 ? flow_enqueue(b, nsteps) : batch_enqueue(b, nsteps)) != WAVE_OK) {
            return bfail(b, WAVE_EHIP, "batched launch failed");
        }
    }
    for (wave_ctx *c : b->ctx) {
        c->step += nsteps;
        if (nsteps & 1) {
            void *t = c->prev;
            c->prev = c->cur;
            c->cur = t;
        }
    }
    return WAVE_OK;
}

int wave_batch_set_schedule(wave_batch *b, int32_t schedule, int32_t nstreams)
{
    if (!b)
        return WAVE_EINVAL;
    if (schedule < 0 || schedule > 3 || (schedule == 1 && (nstreams < 1 || nstreams > 16)))
        return bfail(b, WAVE_EINVAL, "schedule must be 0, 1 with 1..16 streams, 2 or 3");
    if (schedule == 2 && !kFlowScheduleEnabled)
        return bfail(b, WAVE_EINVAL,
                     "schedule 2 is switched off: its first GPU run did not complete and the cause is not known");
    if (schedule == 2)
        for (const auto &g : b->groups)
            if (g.kind != WAVE_F32)
                return bfail(b, WAVE_EINVAL, "schedule 2 runs FP32 shots only");
    if (schedule == 1 && b->use_graph && !b->stream)
        return bfail(b, WAVE_EINVAL, "graph replay needs a stream other than the legacy default stream");
    if (hipStreamSynchronize(b->stream) != hipSuccess)
        return bfail(b, WAVE_EHIP, "stream synchronisation failed");
    drop_batch_graph(b);
    drop_streams(b);
    drop_flow(b);
    b->schedule = 0;
    if (schedule == 2) {
        const int rc = build_flow(b);
        if (rc != WAVE_OK) {
            drop_flow(b);
            return bfail(b, rc, "schedule 2 plan could not be built");
        }
        b->schedule = 2;
    }
    if (schedule == 3) {
        const int rc = build_run(b);
        if (rc != WAVE_OK)
            return bfail(b, rc, rc == WAVE_EINVAL ? "schedule 3 needs cooperative launches, which the device lacks"
                                                  : "schedule 3 plan could not be built");
        b->schedule = 3;
    }
    if (schedule == 1) {
        // on any failure the batch stays on schedule 0 with no streams
        for (int k = 0; k < nstreams; ++k) {
            hipStream_t st = nullptr;
            if (hipStreamCreateWithFlags(&st, hipStreamNonBlocking) != hipSuccess) {
                drop_streams(b);
                return bfail(b, WAVE_EHIP, "stream creation failed");
            }
            b->aux.push_back(st);
        }
        for (int k = 0; k <= nstreams; ++k) {
            hipEvent_t e = nullptr;
            if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                drop_streams(b);
                return bfail(b, WAVE_EHIP, "event creation failed");
            }
            b->ev.push_back(e);
        }
        if (set_stream_tilings(b) != WAVE_OK) {
            drop_streams(b);
            return bfail(b, WAVE_EHIP, "the receiver tables of the streams' tilings could not be uploaded");
        }
        b->schedule = 1;
    }
    return WAVE_OK;
}

int wave_batch_info(const wave_batch *b, int32_t *groups, int64_t *workgroups_per_step,
                    int64_t *points_per_step)
{
    if (!b)
        return WAVE_EINVAL;
    if (groups)
        *groups = int32_t(b->groups.size());
    if (workgroups_per_step) {
        *workgroups_per_step = b->workgroups;
        if (b->schedule == 1) {
            *workgroups_per_step = 0;
            for (size_t i = 0; i < b->ctx.size(); ++i) {
                const Tiling *t = stream_tiling(b, i);
                *workgroups_per_step += t ? t->geo.nwg : b->ctx[i]->nwg;
            }
        }
    }
    if (points_per_step)
        *points_per_step = b->points;
    return WAVE_OK;
}

int wave_batch_streams(const wave_batch *b, int32_t *streams)
{
    if (!b || !streams)
        return WAVE_EINVAL;
    *streams = int32_t(b->streams_used);
    return WAVE_OK;
}

int wave_batch_sync(wave_batch *b)
{
    if (!b)
        return WAVE_EINVAL;
    if (hipStreamSynchronize(b->stream) != hipSuccess || hipGetLastError() != hipSuccess)
        return bfail(b, WAVE_EHIP, "batched run failed");
    if (b->schedule == 2)
        for (const auto &g : b->groups) {
            int flag = 0;
            if (!g.plan.abort || hipMemcpy(&flag, g.plan.abort, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
                return bfail(b, WAVE_EHIP, "schedule 2 status could not be read");
            if (flag)
                return bfail(b, WAVE_EHIP, "schedule 2: a dependency wait gave up; the run's results are invalid");
        }
    if (b->schedule == 3)
        for (const auto &g : b->groups) {
            int flag = 0;
            if (hipMemcpy(&flag, g.items.counters + kTicketInts + 2, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess)
                return bfail(b, WAVE_EHIP, "schedule 3 status could not be read");
            if (flag)
                return bfail(b, WAVE_EHIP, "schedule 3: a barrier wait ran past its limit; the run's results are invalid");
        }
    return WAVE_OK;
}

int wave_batch_set_wait_limit(wave_batch *b, int32_t polls)
{
    if (!b)
        return WAVE_EINVAL;
    if (hipStreamSynchronize(b->stream) != hipSuccess)
        return bfail(b, WAVE_EHIP, "stream synchronisation failed");
    drop_batch_graph(b);  // the limit is a launch argument of the captured graph
    b->wait_limit = polls;
    return WAVE_OK;
}

int wave_batch_destroy(wave_batch *b)
{
    if (!b)
        return WAVE_OK;
    batch_free(b);
    delete b;
    return WAVE_OK;
}

const char *wave_batch_last_error(const wave_batch *b)
{
    return b ? b->err.c_str() : "";
}

const char *wave_strerror(int code)
{
    switch (code) {
    case WAVE_OK: return "ok";
    case WAVE_EINVAL: return "invalid argument";
    case WAVE_EUNSTABLE: return "time step violates the leapfrog stability limit";
    case WAVE_ESTATE: return "invalid state";
    case WAVE_ENOMEM: return "out of memory";
    case WAVE_EHIP: return "HIP runtime error";
    default: return "unknown error";
    }
}

const char *wave_last_error(const wave_ctx *ctx)
{
    if (!ctx)
        return "";
    return ctx->err.c_str();
}

}  // extern "C"

// clbm_api.hip -- the C-ABI of include/clbm.h: handles, argument checks,
// graph replay of step sequences, batches and the batch autotuner.
#include "clbm.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

#include "clbm_device.h"
#include "clbm_internal.h"

using clbm::LatDesc;

namespace {

thread_local std::string g_err;

int fail(int code, const std::string &msg)
{
    g_err = msg;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    g_err = std::string(what) + ": " + hipGetErrorString(e);
    return CLBM_EHIP;
}

#define HIPCHK(expr)                                                 \
    do {                                                             \
        hipError_t e_ = (expr);                                      \
        if (e_ != hipSuccess) return hip_fail(e_, #expr);            \
    } while (0)

int elem_bytes(int storage)
{
    switch (storage) {
    case CLBM_F64: return 8;
    case CLBM_F32: return 4;
    case CLBM_F16:
    case CLBM_BF16:
    case CLBM_F16_SR:
    case CLBM_BF16_SR: return 2;
    default: return 0;
    }
}

// Elements of one direction's run within a lattice row (padded).
int64_t pitch_of(int nx, int eb) { return clbm::row_pitch(nx, eb); }

// log2 of the rows per row block: double while one direction's run in a
// block is shorter than kBlockRunBytes and the block stays within the
// lattice height.
int row_shift(int nx, int ny, int eb)
{
    const int64_t run = pitch_of(nx, eb) * eb;
    int sh = 0;
    while (run << sh < clbm::kBlockRunBytes && (2LL << sh) <= ny) ++sh;
    return sh;
}

// Rows allocated: ny rounded up to whole row blocks.
int64_t rows_allocated(int nx, int ny, int eb)
{
    const int64_t r = 1LL << row_shift(nx, ny, eb);
    return (ny + r - 1) / r * r;
}

constexpr int kStorageKinds = 6;

bool rate_ok(double s) { return std::isfinite(s) && s > 0.0 && s <= 2.0; }

// Default nodes per thread of the single-lattice step: 16-byte vectors for
// FP64 and FP32, 8-byte vectors for 16-bit storage (fewer live registers).
// Blocks per compute unit for the single-lattice step, measured on MI355X
// (4096^2 and 1024^2 sweeps of 2..8 blocks per CU against no cap).  When a
// step's traffic exceeds the 256 MB Infinity Cache, fewer resident waves
// stream HBM faster for the wide types: FP32 is fastest at 3 blocks per CU
// (196 us against 208 us uncapped at 4096^2), FP64 at 2 (376 against 397);
// the 16-bit kernels, co-limited by ALU issue, want every wave they can get.
// Cache-resident lattices: FP64 gains a little at 4, the rest at no cap.
// In place (phase 0 all aligned, phase 1 at the neighbours), per-phase
// sweeps at 4096^2 put phase 0 at 2 for both wide types (FP32 198 us against
// 202 at 3) and phase 1 at 3 (FP64 392 against 406 at 2).
int default_occupancy(int storage, size_t bytes_per_step, bool inplace = false, int phase = 1)
{
    const bool hbm = bytes_per_step > ((size_t)256 << 20);
    switch (storage) {
    case CLBM_F64: return hbm ? (inplace ? (phase == 0 ? 2 : 3) : 2) : 4;
    case CLBM_F32: return hbm ? (inplace && phase == 0 ? 2 : 3) : 0;
    default: return 0;
    }
}

// Dynamic LDS per block that leaves room for exactly `occ` blocks on a
// compute unit with lds_per_cu bytes (a block asks for lds_per_cu/(occ + 1/2),
// rounded down to 256 bytes).
size_t lds_for_occupancy(int occ)
{
    if (occ <= 0) return 0;
    int dev = 0, per_cu = 0, per_block = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&per_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) !=
            hipSuccess ||
        hipDeviceGetAttribute(&per_block, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) !=
            hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    size_t lds = (size_t)(per_cu / (occ + 0.5)) / 256 * 256;
    if (lds > (size_t)per_block) return 0;  // cannot enforce: leave uncapped
    return lds;
}

int default_vec(int storage)
{
    switch (storage) {
    case CLBM_F64: return 2;
    case CLBM_F32: return 4;
    default: return 4;
    }
}

// Compute units of the current device.
int compute_units()
{
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) {
        (void)hipGetLastError();
        return 256;
    }
    return n;
}

// Check that [p, p + bytes) lies inside one HIP device allocation.
int check_device_range(const void *p, size_t bytes, const char *name)
{
    if (!p) return fail(CLBM_EINVAL, std::string(name) + " is NULL");
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
        (void)hipGetLastError();
        return fail(CLBM_EINVAL, std::string(name) + " is not HIP memory");
    }
    if (attr.type != hipMemoryTypeDevice && attr.type != hipMemoryTypeManaged)
        return fail(CLBM_EINVAL, std::string(name) + " is not device memory");
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(&base, &size, const_cast<void *>(p)) == hipSuccess && base) {
        const char *b = static_cast<const char *>(base);
        const char *q = static_cast<const char *>(p);
        if (q < b || q + bytes > b + size)
            return fail(CLBM_EINVAL, std::string(name) + " is smaller than required");
    } else {
        (void)hipGetLastError();
    }
    return CLBM_OK;
}

// Graphs that may still be queued are not destroyed at once: each is kept
// with an event recorded after its last launch and destroyed once that event
// has completed.  No call of this library waits for the device to drain.
std::mutex g_retire_mu;
std::vector<std::pair<hipGraphExec_t, hipEvent_t>> g_retired;

void reap_retired()
{
    std::lock_guard<std::mutex> lk(g_retire_mu);
    for (size_t k = 0; k < g_retired.size();) {
        if (hipEventQuery(g_retired[k].second) == hipSuccess) {
            (void)hipGraphExecDestroy(g_retired[k].first);
            (void)hipEventDestroy(g_retired[k].second);
            g_retired[k] = g_retired.back();
            g_retired.pop_back();
        } else {
            ++k;
        }
    }
    (void)hipGetLastError();
}

void retire_graph(hipGraphExec_t g, hipStream_t s)
{
    if (!g) return;
    hipEvent_t ev = nullptr;
    if (hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess ||
        hipEventRecord(ev, s) != hipSuccess) {
        // Without an event, wait for the stream once rather than risk
        // destroying a queued graph.
        (void)hipStreamSynchronize(s);
        (void)hipGraphExecDestroy(g);
        if (ev) (void)hipEventDestroy(ev);
        (void)hipGetLastError();
        return;
    }
    std::lock_guard<std::mutex> lk(g_retire_mu);
    g_retired.emplace_back(g, ev);
}

// Reduction scratch of clbm_moments_noalloc, for callers that cannot
// allocate: the FP64 partial sums of at most kMomentsMaxBlocks blocks (three
// components each), 24 KB.  Every GPU the library runs on holds its own copy
// until the process ends.  In host code the name is only a stand-in: its
// device address comes from hipGetSymbolAddress, once per device
// (noalloc_scratch), and only that address is ever handed to a kernel.
constexpr int kNoAllocScratchDoubles = 3 * clbm::kMomentsMaxBlocks;
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};

}  // namespace

static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

namespace {

// Device address of the current device's copy of `scratch`, looked up on
// the first call on that device (with it current) and kept.
int noalloc_scratch(double **out)
{
    int dev = -1;
    HIPCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(CLBM_EINVAL, "device index out of range");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(CLBM_EHIP, "hipGetSymbolAddress(scratch) returned NULL");
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return CLBM_OK;
}

// Pinned host words for the FP64 totals, one set per host thread for the
// life of the process (the calls that use them wait for their stream).  The
// reduction writes them itself (they are mapped): a copy behind it cost 2 us
// of device time and its launch.
double *pinned_words()
{
    static thread_local double *p = nullptr;
    if (!p && hipHostMalloc(&p, 4 * sizeof(double), hipHostMallocDefault) != hipSuccess) p = nullptr;
    return p;
}

}  // namespace

// ---- handle ----------------------------------------------------------------

struct clbm_handle {
    clbm_config cfg;
    LatDesc d;
    hipStream_t stream = nullptr;
    hipStream_t cap = nullptr;  // private stream used only to capture graphs
    int parity = 0;             // buffer holding the current state
    int64_t steps = 0;
    bool ready = false;
    void *force_buf = nullptr;   // stream-ordered allocation
    double *partials = nullptr;  // per-block FP64 partial sums (stream-ordered)
    int vec = 4;
    int occ = 0;                 // blocks per compute unit of the step kernel (0: no cap)
    int64_t resident_max = -1;   // resident kernel up to this many groups, -1 the default (use_resident)
    size_t lds = 0;              // dynamic LDS per block that enforces occ
    size_t lds0 = 0;             // the same for in-place phase-0 steps
    int pairs = -1;              // two fused steps per launch: 1 where supported,
                                 // 0 never, -1 the default (pairs_by_default)
    int cus = 256;               // compute units of the device
    clbm::SweepPlan sweep{};     // four fused steps per launch by default (vec 0: never)
    clbm::TilePlan tile{};       // up to tile.steps fused steps per launch by default (0: never)
    clbm::ShortRun brief{};      // what the last one or two steps take under that plan (tiles_take)
    int graph_steps = -1;        // steps per graph, 0 none, -1 the default (graph_steps_of)
    int graph_launches = 0;      // launches of one graph: each flips the parity
    hipGraphExec_t graph[2] = {nullptr, nullptr};
};

namespace {

void drop_graphs(clbm_handle *h)
{
    for (int p = 0; p < 2; ++p) {
        retire_graph(h->graph[p], h->stream);
        h->graph[p] = nullptr;
    }
}

// Dynamic LDS of a step launch from state `src` (the in-place phase 0 has
// its own default cap).
size_t step_lds(const clbm_handle *h, int src) { return h->d.inplace && src == 0 ? h->lds0 : h->lds; }

// Whether steps go two per launch (the fused two-step kernel).
// Measured on MI355X, graphed steps: every storage type steps faster in
// pairs at every size (64 x 32: FP32 3.6 against 4.3 us per step, FP16 3.7
// against 4.3, two launches becoming one; FP64 in its 64 x 8 tiles: 96^2
// 2.9 against 4.0, 256^2 3.2 against 4.4, 512^2 5.0 against 7.2).
bool pairs_by_default(const clbm::LatDesc &) { return true; }

bool use_pairs(const clbm_handle *h)
{
    if (!clbm::step2_supported(h->d)) return false;
    return h->pairs < 0 ? pairs_by_default(h->d) : h->pairs != 0;
}

// The tile kernel's byte offsets within a buffer are 32-bit.
bool tile_offsets_fit(const LatDesc &d)
{
    return clbm_buffer_bytes(d.nx, d.ny, d.storage) < (size_t)1 << 32;
}

// Tiles of w x h nodes that cover the lattice.
int64_t tile_count(const LatDesc &d, int w, int h)
{
    return (int64_t)((d.nx + w - 1) / w) * ((d.ny + h - 1) / h);
}

clbm::Form form_of(const LatDesc &d) { return clbm::Form{d.force_mode == clbm::FM_FIELD, d.bc_y != 0}; }

// The plan of the fused kernels for the lattice and its force (at creation
// and when the force changes): the tile kernel, the sweep kernel or pairs,
// whichever model gives the least time per step.  Tiles and sweeps cross near
// 2000^2 nodes in FP32 and 1500^2 in FP64.  The 16-bit types have no sweeps
// (slower than pairs: FP16-SR 4096^2 181 against 202 GLUPS) and step in tiles at
// every size, or in pairs between walls where they are large (FP16-SR, us per
// step in tiles and pairs: 512^2 3.0 / 4.3, 1024^2 7.1 / 8.4, 4096^2 79.6 / 85.3;
// between walls 1024^2 8.0 / 8.3, 4096^2 93.0 / 84.9).
void plan_fused(clbm_handle *h)
{
    const LatDesc &d = h->d;
    h->sweep = clbm::SweepPlan{};
    h->tile = clbm::TilePlan{};
    const int64_t nodes = (int64_t)d.nx * d.ny;
    const int eb = elem_bytes(d.storage), cus = h->cus;
    if (d.force_mode == clbm::FM_SC && !d.inplace && tile_offsets_fit(d))
        h->tile = clbm::sc_tile_plan(d.nx, d.ny, d.storage, cus);
    if (!clbm::step2_supported(d)) return;
    double us = 0.0;
    const clbm::Form form = form_of(d);
    const int64_t bytes = (int64_t)clbm_buffer_bytes(d.nx, d.ny, d.storage);
    const clbm::TilePlan t = clbm::tile_plan(d.nx, d.ny, d.storage, bytes, cus, &us, form);
    if (eb != 2 && d.nx >= 64 && d.ny >= 64) {
        const clbm::SweepPlan p =
            clbm::sweep_plan(d.nx, d.ny, eb, 4 * cus, clbm::sweep_max_vec(d.storage, d.force_mode, d.bc_y));
        if (clbm::sweep_us(nodes, eb, 4 * cus, p.vec, p.halo, p.rows, p.units) / clbm::kSweepSteps < us) {
            h->sweep = p;
            return;
        }
    }
    const int64_t pair_tiles = tile_count(d, clbm::tile_w(clbm::kTile64x16), clbm::tile_h(clbm::kTile64x16, d.storage));
    // Pairs only beyond what the models miss in 16-bit storage (FP16-SR with
    // walls, us per step, tiles and pairs: 1500^2 14.2 / 14.6 where the models
    // say 14.2 / 14.2, 2048^2 24.3 / 23.0 for 25.4 / 23.4; FP16 2048^2 21.1 / 20.9
    // for 22.1 / 21.2, 3000^2 44.5 / 42.7 for 44.1 / 42.1).
    const double gain = d.storage == CLBM_F16_SR || d.storage == CLBM_BF16_SR ? 1.05 : (eb == 2 ? 1.03 : 1.0);
    const double pairs = clbm::pair_us(d.storage, pair_tiles, cus, clbm::pair_form(d.storage, form)) / 2;
    if (tile_offsets_fit(d) && us < gain * pairs) {
        h->tile = t;
        h->brief = clbm::ShortRun{t.shape, d.storage, form.walls, t.tiles, pair_tiles, nodes, bytes};
    }
}

// Whether steps go several per launch (the tile or the sweep kernel): by
// default, where the lattice has a plan; an explicit clbm_set_step_pairs
// keeps pairs or single steps.
bool use_tiles(const clbm_handle *h) { return h->pairs < 0 && h->tile.steps != 0; }
bool use_sweeps(const clbm_handle *h) { return h->pairs < 0 && h->sweep.vec != 0; }

// Steps per graph replay (clbm::graph_steps).
int graph_steps_of(const clbm_handle *h)
{
    const int fused = use_tiles(h) ? h->tile.steps : (use_sweeps(h) ? clbm::kSweepSteps : 0);
    return clbm::graph_steps(h->graph_steps, fused, (int64_t)clbm_buffer_bytes(h->d.nx, h->d.ny, h->d.storage));
}

// Whether a run of n steps goes to the resident kernel.  By default tiny
// lattices that would otherwise step singly or in pairs do (16 x 16 FP32, us per
// step: resident 1.5, pairs 3.0, single steps 2.8); the tile kernel is faster
// (1.0).
bool use_resident(const clbm_handle *h, int64_t n)
{
    const int rvec = h->d.storage == CLBM_F64 ? 2 : 4;
    const int64_t groups = (int64_t)h->d.ny * (h->d.pitch / rvec);
    const int64_t most = h->resident_max >= 0 ? h->resident_max : (use_tiles(h) ? 0 : clbm::kResidentMaxGroups);
    return n >= 2 && h->d.force_mode != clbm::FM_SC && groups <= most;
}
constexpr int kResidentSteps = 4096;  // most steps of one resident launch

// The next launch of a run with `left` steps to go: its kernel, and as many
// steps as that takes.
struct Launch {
    clbm_launch_kind kind;
    int steps;
};
Launch next_launch(const clbm_handle *h, int64_t left)
{
    if (use_tiles(h) && (h->d.force_mode == clbm::FM_SC || clbm::tiles_take(left, h->brief, h->cus)))
        return {CLBM_LAUNCH_TILES, (int)std::min<int64_t>(left, h->tile.steps)};
    if (left >= clbm::kSweepSteps && use_sweeps(h)) return {CLBM_LAUNCH_SWEEP, clbm::kSweepSteps};
    if (left >= 2 && use_pairs(h)) return {CLBM_LAUNCH_PAIR, 2};
    return {CLBM_LAUNCH_STEP, 1};
}

// That launch from state `parity`.  Each launch flips the buffer or phase.
hipError_t launch_next(const clbm_handle *h, int parity, int64_t left, hipStream_t s, int *taken)
{
    const Launch l = next_launch(h, left);
    *taken = l.steps;
    switch (l.kind) {
    case CLBM_LAUNCH_TILES: return clbm::launch_tile(h->d, parity, l.steps, h->tile, s);
    case CLBM_LAUNCH_SWEEP: return clbm::launch_sweep(h->d, parity, h->sweep, s);
    case CLBM_LAUNCH_PAIR: return clbm::launch_step2(h->d, parity, s);
    default: return clbm::launch_step(h->d, parity, h->vec, step_lds(h, parity), s);
    }
}

int build_graph(clbm_handle *h, int parity)
{
    hipGraph_t g = nullptr;
    if (!h->cap) HIPCHK(hipStreamCreateWithFlags(&h->cap, hipStreamNonBlocking));
    HIPCHK(hipStreamBeginCapture(h->cap, hipStreamCaptureModeThreadLocal));
    hipError_t le = hipSuccess;
    int launches = 0;
    const int steps = graph_steps_of(h);
    for (int done = 0, n = 0; done < steps && le == hipSuccess; done += n, ++launches)
        le = launch_next(h, (parity + launches) & 1, steps - done, h->cap, &n);
    hipError_t ce = hipStreamEndCapture(h->cap, &g);
    if (le != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return hip_fail(le, "launch_step (capture)");
    }
    if (ce != hipSuccess) return hip_fail(ce, "hipStreamEndCapture");
    hipError_t ie = hipGraphInstantiate(&h->graph[parity], g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (ie != hipSuccess) return hip_fail(ie, "hipGraphInstantiate");
    h->graph_launches = launches;
    return CLBM_OK;
}

int need_ready(const clbm_handle *h)
{
    if (!h) return fail(CLBM_EINVAL, "handle is NULL");
    if (!h->ready) return fail(CLBM_ESTATE, "lattice has no state yet: call clbm_init or clbm_set_populations");
    return CLBM_OK;
}

}  // namespace

extern "C" {

size_t clbm_buffer_bytes(int32_t nx, int32_t ny, int32_t storage)
{
    const int eb = elem_bytes(storage);
    if (nx < 1 || ny < 1 || eb == 0) return 0;
    if (pitch_of(nx, eb) * rows_allocated(nx, ny, eb) > (int64_t)INT32_MAX) return 0;
    return (size_t)(9 * pitch_of(nx, eb) * rows_allocated(nx, ny, eb) * eb + clbm::kTailGuardBytes);
}

int clbm_create(const clbm_config *cfg, clbm_handle **out)
{
    g_err.clear();
    if (!cfg || !out) return fail(CLBM_EINVAL, "cfg and out must not be NULL");
    *out = nullptr;
    if (cfg->nx < 1 || cfg->ny < 1) return fail(CLBM_EINVAL, "nx and ny must be >= 1");
    const int eb = elem_bytes(cfg->storage);
    if (eb && pitch_of(cfg->nx, eb) * rows_allocated(cfg->nx, cfg->ny, eb) > (int64_t)INT32_MAX)
        return fail(CLBM_EINVAL, "lattice too large (nx * ny must stay below 2^31)");
    if (cfg->bc_y != CLBM_Y_PERIODIC && cfg->bc_y != CLBM_Y_BOUNCEBACK)
        return fail(CLBM_EINVAL, "bc_y must be CLBM_Y_PERIODIC or CLBM_Y_BOUNCEBACK");
    if (elem_bytes(cfg->storage) == 0) return fail(CLBM_EINVAL, "unknown storage");
    if (cfg->scheme != CLBM_SCHEME_CONSISTENT && cfg->scheme != CLBM_SCHEME_GUO_LBL &&
        cfg->scheme != CLBM_SCHEME_PREMNATH)
        return fail(CLBM_EINVAL, "unknown scheme");
    if (cfg->streaming != CLBM_STREAM_TWO_BUFFERS && cfg->streaming != CLBM_STREAM_IN_PLACE)
        return fail(CLBM_EINVAL, "streaming must be CLBM_STREAM_TWO_BUFFERS or CLBM_STREAM_IN_PLACE");
    const bool inplace = cfg->streaming == CLBM_STREAM_IN_PLACE;
    const double rates[6] = {cfg->s0, cfg->s1, cfg->sb, cfg->s2, cfg->s3, cfg->s4};
    for (double s : rates)
        if (!rate_ok(s)) return fail(CLBM_EINVAL, "every relaxation rate must lie in (0, 2]");
    if (!std::isfinite(cfg->rho0) || cfg->rho0 <= 0.0) return fail(CLBM_EINVAL, "rho0 must be > 0");
    if (inplace && cfg->pop_b) return fail(CLBM_EINVAL, "in-place streaming takes no pop_b");
    if (!inplace && cfg->pop_a == cfg->pop_b) return fail(CLBM_EINVAL, "pop_a and pop_b must differ");
    const size_t need = clbm_buffer_bytes(cfg->nx, cfg->ny, cfg->storage);
    int rc = check_device_range(cfg->pop_a, need, "pop_a");
    if (rc) return rc;
    if (!inplace && (rc = check_device_range(cfg->pop_b, need, "pop_b"))) return rc;

    clbm_handle *h = new clbm_handle();
    h->cfg = *cfg;
    h->stream = static_cast<hipStream_t>(cfg->stream);
    LatDesc &d = h->d;
    std::memset(&d, 0, sizeof d);
    d.buf[0] = cfg->pop_a;
    d.buf[1] = inplace ? cfg->pop_a : cfg->pop_b;
    d.inplace = inplace ? 1 : 0;
    d.rshift = row_shift(cfg->nx, cfg->ny, eb);
    d.pitch = pitch_of(cfg->nx, eb);
    d.dstride = d.pitch << d.rshift;
    d.bstride = 9 * d.dstride;
    d.nx = cfg->nx;
    d.ny = cfg->ny;
    d.bc_y = cfg->bc_y;
    d.storage = cfg->storage;
    d.force_mode = clbm::FM_CONST;
    d.rho0 = cfg->rho0;
    static_assert(CLBM_SCHEME_GUO_LBL == 1 && CLBM_SCHEME_PREMNATH == 2, "set_rates' scheme numbers");
    clbm::set_rates(d, cfg->s1, cfg->sb, cfg->s2, cfg->s3, cfg->s4, cfg->scheme);
    h->vec = default_vec(cfg->storage);
    h->occ = default_occupancy(cfg->storage, 2 * need, inplace, 1);
    h->lds = lds_for_occupancy(h->occ);
    h->cus = compute_units();
    plan_fused(h);
    h->lds0 = inplace ? lds_for_occupancy(default_occupancy(cfg->storage, 2 * need, true, 0)) : h->lds;

    reap_retired();
    const int nb = clbm::moments_blocks((int64_t)cfg->nx * cfg->ny);
    hipError_t e = hipMallocAsync(reinterpret_cast<void **>(&h->partials),
                                  sizeof(double) * 3 * (size_t)nb, h->stream);
    if (e != hipSuccess) {
        clbm_destroy(h);
        return hip_fail(e, "clbm_create allocations");
    }
    *out = h;
    return CLBM_OK;
}

int clbm_destroy(clbm_handle *h)
{
    if (!h) return CLBM_OK;
    drop_graphs(h);
    if (h->force_buf) (void)hipFreeAsync(h->force_buf, h->stream);
    if (h->partials) (void)hipFreeAsync(h->partials, h->stream);
    if (h->cap) (void)hipStreamDestroy(h->cap);
    (void)hipGetLastError();
    delete h;
    reap_retired();
    return CLBM_OK;
}

int clbm_set_force(clbm_handle *h, int32_t kind, const double *params, const double *fx,
                   const double *fy)
{
    g_err.clear();
    if (!h) return fail(CLBM_EINVAL, "handle is NULL");
    LatDesc &d = h->d;
    const size_t rb = d.storage == CLBM_F64 ? 8 : 4;
    const int64_t n = (int64_t)d.nx * d.ny;
    switch (kind) {
    case CLBM_FORCE_NONE:
    case CLBM_FORCE_CONST: {
        double Fx = 0.0, Fy = 0.0;
        if (kind == CLBM_FORCE_CONST) {
            if (!params) return fail(CLBM_EINVAL, "CONST force needs params {Fx, Fy}");
            Fx = params[0];
            Fy = params[1];
            if (!std::isfinite(Fx) || !std::isfinite(Fy)) return fail(CLBM_EINVAL, "force is not finite");
        }
        d.force_mode = clbm::FM_CONST;
        d.Fx = Fx;
        d.Fy = Fy;
        break;
    }
    case CLBM_FORCE_KOLMOGOROV:
    case CLBM_FORCE_FIELD:
    case CLBM_FORCE_SHAN_CHEN: {
        const size_t bytes = kind == CLBM_FORCE_KOLMOGOROV ? rb * (size_t)d.ny
                             : kind == CLBM_FORCE_FIELD    ? 2 * rb * (size_t)n
                                                           : rb * (size_t)n;
        if (kind == CLBM_FORCE_KOLMOGOROV) {
            if (!params) return fail(CLBM_EINVAL, "KOLMOGOROV force needs params {A, k}");
            if (!std::isfinite(params[0]) || !std::isfinite(params[1]))
                return fail(CLBM_EINVAL, "force parameters are not finite");
        } else if (kind == CLBM_FORCE_SHAN_CHEN) {
            if (!params) return fail(CLBM_EINVAL, "SHAN_CHEN force needs params {G, psi0, rho_ref}");
            if (!std::isfinite(params[0]) || !std::isfinite(params[1]) || !std::isfinite(params[2]))
                return fail(CLBM_EINVAL, "force parameters are not finite");
            if (!(params[1] > 0.0) || !(params[2] > 0.0))
                return fail(CLBM_EINVAL, "SHAN_CHEN needs psi0 > 0 and rho_ref > 0");
            if (d.bc_y != CLBM_Y_PERIODIC)
                return fail(CLBM_EINVAL, "SHAN_CHEN needs a periodic lattice");
        } else {
            int rc = check_device_range(fx, sizeof(double) * n, "fx");
            if (rc) return rc;
            rc = check_device_range(fy, sizeof(double) * n, "fy");
            if (rc) return rc;
        }
        // Queued steps may still read the old table: free it in stream order.
        if (h->force_buf) HIPCHK(hipFreeAsync(h->force_buf, h->stream));
        h->force_buf = nullptr;
        HIPCHK(hipMallocAsync(&h->force_buf, bytes, h->stream));
        if (kind == CLBM_FORCE_KOLMOGOROV) {
            d.force_mode = clbm::FM_ROW;
            HIPCHK(clbm::launch_force_table(d, h->force_buf, params[0], params[1], h->stream));
        } else if (kind == CLBM_FORCE_FIELD) {
            d.force_mode = clbm::FM_FIELD;
            HIPCHK(clbm::launch_force_field(d, h->force_buf, fx, fy, h->stream));
        } else {
            // The psi plane is filled from the state before each use.
            d.force_mode = clbm::FM_SC;
            d.sc_g = params[0];
            d.sc_psi0 = params[1];
            d.sc_rho = params[2];
            d.sc_psic = params[1] * std::exp(-params[2] / d.rho0);
        }
        d.force = h->force_buf;
        d.Fx = d.Fy = 0.0;
        break;
    }
    default:
        return fail(CLBM_EINVAL, "unknown force kind");
    }
    plan_fused(h);
    drop_graphs(h);
    return CLBM_OK;
}

int clbm_init(clbm_handle *h, const double *rho, const double *ux, const double *uy)
{
    g_err.clear();
    if (!h) return fail(CLBM_EINVAL, "handle is NULL");
    const size_t fb = sizeof(double) * (size_t)h->d.nx * h->d.ny;
    int rc;
    if (rho && (rc = check_device_range(rho, fb, "rho"))) return rc;
    if (ux && (rc = check_device_range(ux, fb, "ux"))) return rc;
    if (uy && (rc = check_device_range(uy, fb, "uy"))) return rc;
    if (h->d.force_mode == clbm::FM_SC) HIPCHK(clbm::launch_psi(h->d, -1, rho, h->stream));
    HIPCHK(clbm::launch_init(h->d, 0, rho, ux, uy, h->stream));
    h->parity = 0;
    h->steps = 0;
    h->ready = true;
    return CLBM_OK;
}

int clbm_step(clbm_handle *h, int64_t nsteps)
{
    g_err.clear();
    int rc = need_ready(h);
    if (rc) return rc;
    if (nsteps < 0) return fail(CLBM_EINVAL, "nsteps must be >= 0");
    if (use_resident(h, nsteps)) {
        // A small lattice: many steps per launch in one resident block.
        for (int64_t left = nsteps; left > 0;) {
            const int n = (int)std::min<int64_t>(left, kResidentSteps);
            HIPCHK(clbm::launch_resident(h->d, h->parity, n, h->stream));
            h->parity = (h->parity + n) & 1;
            left -= n;
        }
        h->steps += nsteps;
        return CLBM_OK;
    }
    const int graph = graph_steps_of(h);
    int64_t left = nsteps;
    while (left > 0) {
        if (graph > 0 && left >= graph) {
            if (!h->graph[h->parity] && (rc = build_graph(h, h->parity))) return rc;
            HIPCHK(hipGraphLaunch(h->graph[h->parity], h->stream));
            left -= graph;
            h->parity ^= h->graph_launches & 1;
        } else {
            int n = 0;
            HIPCHK(launch_next(h, h->parity, left, h->stream, &n));
            h->parity ^= 1;
            left -= n;
        }
    }
    h->steps += nsteps;
    return CLBM_OK;
}

int64_t clbm_step_count(const clbm_handle *h) { return h ? h->steps : -1; }

int clbm_moments(clbm_handle *h, double *rho, double *ux, double *uy, double *totals)
{
    g_err.clear();
    int rc = need_ready(h);
    if (rc) return rc;
    const size_t fb = sizeof(double) * (size_t)h->d.nx * h->d.ny;
    if (rho && (rc = check_device_range(rho, fb, "rho"))) return rc;
    if (ux && (rc = check_device_range(ux, fb, "ux"))) return rc;
    if (uy && (rc = check_device_range(uy, fb, "uy"))) return rc;
    int nb = 0;
    if (h->d.force_mode == clbm::FM_SC) HIPCHK(clbm::launch_psi(h->d, h->parity, nullptr, h->stream));
    HIPCHK(clbm::launch_moments(h->d, h->parity, rho, ux, uy, nullptr, nullptr, totals ? h->partials : nullptr, &nb,
                                h->stream));
    if (!totals) return CLBM_OK;
    double *w = pinned_words();
    if (!w) return fail(CLBM_EHIP, "pinned host memory for the totals");
    HIPCHK(clbm::launch_reduce(h->partials, nb, 3, w, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    totals[0] = (double)h->d.nx * h->d.ny * h->d.rho0 + w[0];
    totals[1] = w[1];
    totals[2] = w[2];
    for (int c = 0; c < 3; ++c)
        if (!std::isfinite(totals[c])) return fail(CLBM_ENONFINITE, "mass or momentum is not finite");
    return CLBM_OK;
}

int clbm_moments_noalloc(clbm_handle *h, double *rho, double *ux, double *uy, double *totals)
{
    g_err.clear();
    int rc = need_ready(h);
    if (rc) return rc;
    const size_t fb = sizeof(double) * (size_t)h->d.nx * h->d.ny;
    if (rho && (rc = check_device_range(rho, fb, "rho"))) return rc;
    if (ux && (rc = check_device_range(ux, fb, "ux"))) return rc;
    if (uy && (rc = check_device_range(uy, fb, "uy"))) return rc;
    if (totals && (rc = check_device_range(totals, 3 * sizeof(double), "totals"))) return rc;
    const int nb = clbm::moments_blocks((int64_t)h->d.nx * h->d.ny);
    if (3 * (int64_t)nb > kNoAllocScratchDoubles)
        return fail(CLBM_EINVAL, "lattice needs more reduction scratch than the static maximum");
    double *partials = nullptr;
    if ((rc = noalloc_scratch(&partials))) return rc;
    // Every partial is written before it is read: nothing to clear.
    int used = 0;
    if (h->d.force_mode == clbm::FM_SC) HIPCHK(clbm::launch_psi(h->d, h->parity, nullptr, h->stream));
    HIPCHK(clbm::launch_moments(h->d, h->parity, rho, ux, uy, nullptr, nullptr, totals ? partials : nullptr, &used,
                                h->stream));
    if (!totals) return CLBM_OK;
    HIPCHK(clbm::launch_reduce(partials, used, 3, totals, h->stream,
                               (double)h->d.nx * h->d.ny * h->d.rho0));
    return CLBM_OK;
}

int clbm_error_norms(clbm_handle *h, const double *ux_ref, const double *uy_ref, double *out)
{
    g_err.clear();
    int rc = need_ready(h);
    if (rc) return rc;
    if (!out) return fail(CLBM_EINVAL, "out is NULL");
    const size_t fb = sizeof(double) * (size_t)h->d.nx * h->d.ny;
    if ((rc = check_device_range(ux_ref, fb, "ux_ref"))) return rc;
    if ((rc = check_device_range(uy_ref, fb, "uy_ref"))) return rc;
    int nb = 0;
    if (h->d.force_mode == clbm::FM_SC) HIPCHK(clbm::launch_psi(h->d, h->parity, nullptr, h->stream));
    HIPCHK(clbm::launch_moments(h->d, h->parity, nullptr, nullptr, nullptr, ux_ref, uy_ref,
                                h->partials, &nb, h->stream));
    double *w = pinned_words();
    if (!w) return fail(CLBM_EHIP, "pinned host memory for the norms");
    HIPCHK(clbm::launch_reduce(h->partials, nb, 2, w, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    out[0] = w[0];
    out[1] = w[1];
    return CLBM_OK;
}

int clbm_get_populations(clbm_handle *h, double *f)
{
    g_err.clear();
    int rc = need_ready(h);
    if (rc) return rc;
    if ((rc = check_device_range(f, 9 * sizeof(double) * (size_t)h->d.nx * h->d.ny, "f"))) return rc;
    HIPCHK(clbm::launch_get_populations(h->d, h->parity, f, h->stream));
    return CLBM_OK;
}

int clbm_set_populations(clbm_handle *h, const double *f)
{
    g_err.clear();
    if (!h) return fail(CLBM_EINVAL, "handle is NULL");
    int rc = check_device_range(f, 9 * sizeof(double) * (size_t)h->d.nx * h->d.ny, "f");
    if (rc) return rc;
    HIPCHK(clbm::launch_set_populations(h->d, 0, f, h->stream));
    h->parity = 0;
    h->steps = 0;
    h->ready = true;
    return CLBM_OK;
}

int clbm_set_graph_steps(clbm_handle *h, int32_t steps)
{
    g_err.clear();
    if (!h) return fail(CLBM_EINVAL, "handle is NULL");
    if (steps < 0 || steps > 4096) return fail(CLBM_EINVAL, "graph steps must lie in [0, 4096]");
    drop_graphs(h);
    h->graph_steps = (steps + 1) / 2 * 2;
    return CLBM_OK;
}

int clbm_set_step_pairs(clbm_handle *h, int32_t enable)
{
    g_err.clear();
    if (!h) return fail(CLBM_EINVAL, "handle is NULL");
    if (enable < -1 || enable > 1) return fail(CLBM_EINVAL, "enable must be -1, 0 or 1");
    drop_graphs(h);
    h->pairs = enable;
    return CLBM_OK;
}

int32_t clbm_get_step_pairs(const clbm_handle *h) { return h ? (use_pairs(h) ? 1 : 0) : -1; }

int32_t clbm_steps_per_launch(const clbm_handle *h)
{
    if (!h) return -1;
    if (use_tiles(h)) return h->tile.steps;
    if (use_sweeps(h)) return clbm::kSweepSteps;
    return use_pairs(h) ? 2 : 1;
}

int clbm_next_launch(const clbm_handle *h, int64_t nsteps, int32_t *launch)
{
    g_err.clear();
    if (!h || !launch) return fail(CLBM_EINVAL, "handle and launch must not be NULL");
    if (nsteps < 1) return fail(CLBM_EINVAL, "nsteps must be >= 1");
    const Launch l = use_resident(h, nsteps)
                         ? Launch{CLBM_LAUNCH_RESIDENT, (int)std::min<int64_t>(nsteps, kResidentSteps)}
                         : next_launch(h, nsteps);
    launch[0] = l.kind;
    launch[1] = l.steps;
    launch[2] = launch[3] = 0;
    if (l.kind == CLBM_LAUNCH_TILES) {
        launch[2] = clbm::region_w(h->tile.shape);
        launch[3] = clbm::region_h(h->tile.shape);
    } else if (l.kind == CLBM_LAUNCH_SWEEP) {
        launch[2] = h->sweep.vec;
        launch[3] = h->sweep.rows;
    }
    return CLBM_OK;
}

int clbm_set_occupancy(clbm_handle *h, int32_t blocks_per_cu)
{
    g_err.clear();
    if (!h) return fail(CLBM_EINVAL, "handle is NULL");
    if (blocks_per_cu != 0 && (blocks_per_cu < 2 || blocks_per_cu > 16))
        return fail(CLBM_EINVAL, "blocks per compute unit must be 0 (no cap) or in [2, 16]");
    drop_graphs(h);
    h->occ = blocks_per_cu;
    h->lds = h->lds0 = lds_for_occupancy(blocks_per_cu);
    return CLBM_OK;
}

int32_t clbm_get_occupancy(const clbm_handle *h) { return h ? h->occ : -1; }

int clbm_set_resident_limit(clbm_handle *h, int64_t max_groups)
{
    g_err.clear();
    if (!h) return fail(CLBM_EINVAL, "handle is NULL");
    if (max_groups < 0 || max_groups > (int64_t)1 << 20)
        return fail(CLBM_EINVAL, "resident limit must lie in [0, 2^20] groups");
    h->resident_max = max_groups;
    return CLBM_OK;
}

const char *clbm_last_error(void) { return g_err.c_str(); }

double clbm_nonslip_s3(double s2) { return (16.0 - 8.0 * s2) / (8.0 - s2); }

double clbm_s_from_nu(double nu) { return 1.0 / (3.0 * nu + 0.5); }

}  // extern "C"

// ---- batches ---------------------------------------------------------------

namespace {

// Kernel variants of a batch.  A variant is a pair (single-step variant,
// two-step variant): the first applies to the groups whose lattices step one
// step per launch, the second to those that step in pairs.
// Single-step variants: bytes each thread loads per direction (nodes per
// thread = bytes / element size, clamped to the compiled set), the grid
// (persistent blocks per compute unit, or 0: one block per tile) and a cap
// on resident blocks per compute unit (0: none, -1: the single-lattice
// default of the group's storage type for the group's traffic).
struct Variant {
    int vec_bytes;
    int blocks_per_cu;
    int cap;
};
const Variant kVariants[] = {
    {16, 0, -1}, {16, 0, 0}, {16, 0, 4}, {16, 16, 0}, {8, 0, -1},
    {8, 0, 0},   {8, 16, 0}, {4, 0, -1}, {4, 0, 0},  {4, 16, 0},
};
constexpr int kNumSingle = sizeof(kVariants) / sizeof(kVariants[0]);
// Two-step variants: the tile shape (64 x 16 or 32 x 32 nodes, or, per
// lattice, whichever of the two gives it fewer tiles) and the grid
// (persistent blocks per compute unit walking the tiles, or 0: one block per
// tile; the two-step kernel's LDS lets 4 blocks share a compute unit).
constexpr int kShapePerLattice = 2;
// The first steps lattices of the default clbm_set_step_pairs in LDS tiles,
// four or eight steps per launch; the others (and lattices set to pairs
// under any) in pairs.
struct PairVariant {
    int shape;
    int blocks_per_cu;
    bool tiles;
};
const PairVariant kPairVariants[] = {{clbm::kTile64x16, 0, true},  {clbm::kTile32x32, 0, false},
                                     {clbm::kTile64x16, 4, false}, {clbm::kTile32x32, 4, false},
                                     {kShapePerLattice, 0, false}, {clbm::kTile64x16, 0, false}};
constexpr int kNumPair = sizeof(kPairVariants) / sizeof(kPairVariants[0]);
constexpr int kNumVariants = kNumSingle * kNumPair;
int single_index(int v) { return v / kNumPair; }
const Variant &single_of(int v) { return kVariants[v / kNumPair]; }
const PairVariant &pair_of(int v) { return kPairVariants[v % kNumPair]; }

int vec_for(int storage, int vec_bytes)
{
    switch (storage) {
    case CLBM_F64: return vec_bytes >= 16 ? 2 : 1;
    case CLBM_F32: return vec_bytes >= 16 ? 4 : (vec_bytes >= 8 ? 2 : 1);
    default: return vec_bytes >= 16 ? 8 : (vec_bytes >= 8 ? 4 : 2);
    }
}

}  // namespace

namespace {

// How the lattices of a batch are laid out for a call: their groups and tiles
// under a region shape per storage type.
struct BatchPlan {
    int region[kStorageKinds] = {};   // LDS-tile region shape per storage type, or -1: pairs
    bool made = false;                // the members below are up to date
    std::vector<int> order;           // table position -> caller index (grouped by kind)
    std::vector<int> keys;            // group key of each lattice when ordered
    std::vector<int> per;             // steps per launch of each lattice (caller's order)
    struct Group {
        int storage, key, vec, l_lo, l_hi;  // key = clbm::kernel_key
        int64_t ntiles;
        int64_t tbase;                // first entry of the group in the tile map
        size_t lds;                   // dynamic LDS per block enforcing the cap
        int cls;                      // StepClass
        int shape;                    // pairs: clbm::TileShape; LDS tiles: clbm::RegionShape
        bool small;                   // pairs: every buffer below 4 GB
        bool walls;                   // a lattice of the group has walls
        int per;                      // steps per launch
        int64_t most;                 // most steps a lattice of the group takes in this call
    };
    std::vector<Group> groups;
    std::vector<LatDesc> tab;         // host copy of the table's geometry
    int32_t *d_tile_lat = nullptr;    // tile -> lattice map of every group (stream-ordered)
    int64_t tile_lat_cap = 0;         // entries allocated
    bool map_dirty = true;            // geometry changed since the map was built
    hipGraphExec_t graph = nullptr;
};

}  // namespace

struct clbm_batch {
    std::vector<clbm_handle *> lats;  // caller's order
    hipStream_t stream = nullptr;
    hipStream_t cap = nullptr;        // capture-only stream, created on first graph
    // Groups beyond the first run on side streams, forked from and joined
    // back to the launching stream around every step (also inside graphs).
    std::vector<hipStream_t> side;
    hipEvent_t fork = nullptr;
    std::vector<hipEvent_t> join;
    LatDesc *d_lats = nullptr;        // device lattice table (stream-ordered), uploaded by each call
    // Plan 0, and those of calls of one and two steps where their regions
    // differ (tiles_take), those made on their first call.
    static constexpr int kPlans = 3;
    BatchPlan plan[kPlans];
    int variant = 0;
    int cus = 256;
    int chunk = 64;                   // steps per captured graph (a multiple of every group's steps per launch)
};

namespace {

// Tile shape of a lattice stepping in pairs under the two-step variant's
// shape: the variant's, or the one of 64 x 16 and 32 x 32 that covers the
// lattice with fewer tiles (64 x 16 on a tie).
int pair_shape(int variant_shape, const clbm::LatDesc &d)
{
    if (variant_shape != kShapePerLattice) return variant_shape;
    auto tiles = [&](int shape) { return tile_count(d, clbm::tile_w(shape), clbm::tile_h(shape, d.storage)); };
    return tiles(clbm::kTile32x32) < tiles(clbm::kTile64x16) ? clbm::kTile32x32 : clbm::kTile64x16;
}

// How a lattice of a batch steps: singly, in pairs of one of two tile shapes
// or in LDS tiles (whose region shape the whole group shares).
enum StepClass { kSingle = 0, kPair0 = 1, kPair1 = 2, kLdsTiles = 3, kStepClasses = 4 };
int step_class(const clbm_batch *b, const BatchPlan &p, const clbm_handle *h)
{
    const PairVariant &pv = pair_of(b->variant);
    if (!use_pairs(h)) return kSingle;
    if (pv.tiles && h->pairs < 0 && p.region[h->d.storage] >= 0 && tile_offsets_fit(h->d)) return kLdsTiles;
    return kPair0 + pair_shape(pv.shape, h->d);
}

// Region shape of the lattices of each storage type that may step in LDS
// tiles: the one with the least modelled time per step for all their tiles,
// or -1 where pairs take less; in calls of one or two steps also where a tile
// launch of those would take more than the pair kernel's (tiles_take).
void batch_regions(clbm_batch *b)
{
    for (int st = 0; st < kStorageKinds; ++st) {
        // Tiles of all the lattices, and in units of tiles what they cost with
        // each lattice's form (a group with walls in it runs the kernel for
        // walls throughout).
        int64_t pairs = 0, bytes = 0, nodes = 0, tiles[clbm::kRegionShapes] = {};
        double pair_cost = 0.0, cost[clbm::kRegionShapes] = {};
        auto candidate = [&](const clbm_handle *h) { return h->d.storage == st && h->pairs < 0 && use_pairs(h); };
        bool walls[clbm::kKernelKeys] = {}, any_walls = false;
        for (const auto *h : b->lats)
            if (candidate(h)) walls[clbm::kernel_key(h->d)] |= h->d.bc_y != 0;
        for (const auto *h : b->lats) {
            const LatDesc &d = h->d;
            if (!candidate(h)) continue;
            const clbm::Form form{form_of(d).field, walls[clbm::kernel_key(d)]};
            const int64_t np = tile_count(d, clbm::tile_w(clbm::kTile64x16), clbm::tile_h(clbm::kTile64x16, st));
            pairs += np;
            pair_cost += np * clbm::pair_form(st, form);
            bytes += (int64_t)clbm_buffer_bytes(d.nx, d.ny, st);
            nodes += (int64_t)d.nx * d.ny;
            any_walls |= form.walls;
            for (int shape = 0; shape < clbm::kRegionShapes; ++shape) {
                const int64_t n = tile_count(d, clbm::region_tile_w(shape), clbm::region_tile_h(shape));
                tiles[shape] += n;
                cost[shape] += n * clbm::tile_form(shape, st, form);
            }
        }
        int &region = b->plan[0].region[st];
        region = -1;
        // Against one lattice's time per tile, tiles of many ragged lattices gain
        // 2 % on pairs, in 16-bit storage rounded to nearest 6 % (256 lattices of
        // 32^2 .. 512^2, us per step, tiles and pairs by model, then measured:
        // FP16-SR periodic 46.5 / 48.2, 45.7 / 46.8; walls and force fields 53.5 /
        // 51.8, 55.5 / 51.5; FP16 walls, fields and rows mixed 46.9 / 45.1, 42.6 /
        // 46.8).
        const double gain = st == CLBM_F16 || st == CLBM_BF16 ? 1.06 : 1.02;
        double best = pairs ? gain * clbm::pair_us(st, pairs, b->cus, pair_cost / pairs) / 2 : 0.0;
        for (int shape = 0; shape < clbm::kRegionShapes; ++shape) {
            if (!pairs || !clbm::region_compiled(shape, st)) continue;
            const double us = clbm::tile_us(shape, st, tiles[shape], bytes, b->cus, cost[shape] / tiles[shape]) /
                              clbm::region_steps(shape);
            if (us < best) {
                best = us;
                region = shape;
            }
        }
        for (int left = 1; left < clbm_batch::kPlans; ++left) {
            const clbm::ShortRun run{region, st, any_walls, region < 0 ? 0 : tiles[region], pairs, nodes, bytes};
            b->plan[left].region[st] = region >= 0 && clbm::tiles_take(left, run, b->cus) ? region : -1;
        }
    }
}

// Launch group of a lattice: how it steps, storage type and kernel (storage
// scheme, force mode, forcing scheme).
constexpr int kGroupKeys = kStepClasses * kStorageKinds * clbm::kKernelKeys;
int group_key(const clbm_batch *b, const BatchPlan &p, const clbm_handle *h)
{
    return (step_class(b, p, h) * kStorageKinds + h->d.storage) * clbm::kKernelKeys + clbm::kernel_key(h->d);
}

// Table order: grouped by tile shape, storage and kernel (one launch per
// group), caller order inside a group.
void batch_order(const clbm_batch *b, BatchPlan &p)
{
    p.order.clear();
    p.keys.clear();
    for (auto *h : b->lats) p.keys.push_back(group_key(b, p, h));
    for (int key = 0; key < kGroupKeys; ++key)
        for (size_t j = 0; j < b->lats.size(); ++j)
            if (p.keys[j] == key) p.order.push_back((int)j);
}

// Geometry of the current variant: per lattice nodes per thread, tile
// shape and first tile; per group its lattice range and tile count.
void batch_geometry(const clbm_batch *b, BatchPlan &p)
{
    p.groups.clear();
    int64_t tbase = 0;
    p.tab.assign(p.order.size(), LatDesc());
    p.per.assign(p.order.size(), 1);
    size_t pos = 0;
    while (pos < p.order.size()) {
        const clbm_handle *h0 = b->lats[p.order[pos]];
        const LatDesc &d0 = h0->d;
        const int key = group_key(b, p, h0);
        const int cls = step_class(b, p, h0), st = d0.storage;
        const int vec = cls == kSingle ? vec_for(st, single_of(b->variant).vec_bytes) : 4;
        const int lo = (int)pos;
        size_t end = pos;
        while (end < p.order.size() && group_key(b, p, b->lats[p.order[end]]) == key) ++end;
        // Tile size of the fused steps in the group's shape.
        const int shape = cls == kLdsTiles ? p.region[st] : (cls == kPair1 ? 1 : 0);
        const int tw = cls == kLdsTiles ? clbm::region_tile_w(shape) : clbm::tile_w(shape);
        const int th = cls == kLdsTiles ? clbm::region_tile_h(shape) : clbm::tile_h(shape, st);
        const int per = cls == kLdsTiles ? clbm::region_steps(shape) : (cls == kSingle ? 1 : 2);
        int64_t tiles = 0;
        size_t bytes = 0, largest = 0;
        bool walls = false;
        for (; pos < end; ++pos) {
            LatDesc d = b->lats[p.order[pos]]->d;
            clbm::tile_geometry(d.pitch, d.ny, vec, &d.tpr, &d.inv_tpr, &d.ntiles);
            if (cls != kSingle) {  // the fused kernel's tiles, and their walk
                const int tx = (d.nx + tw - 1) / tw, ty = (d.ny + th - 1) / th;
                const int sw = std::max(clbm::kStripNodes / tw, 1);
                d.ntiles = (int64_t)tx * ty;
                d.walk = clbm::strip_walk(tx, ty, tx < sw ? tx : sw);
            }
            d.vec = vec;
            d.per = per;
            p.per[p.order[pos]] = per;
            d.tile0 = tiles;
            tiles += d.ntiles;
            const size_t one = clbm_buffer_bytes(d.nx, d.ny, d.storage);
            bytes += 2 * one;
            largest = std::max(largest, one);
            walls = walls || d.bc_y;
            p.tab[pos] = d;
        }
        const int cap = single_of(b->variant).cap;
        const size_t lds = lds_for_occupancy(cap < 0 ? default_occupancy(st, bytes) : cap);
        const bool small = largest + 4096 < ((size_t)1 << 32);
        p.groups.push_back({st, clbm::kernel_key(d0), vec, lo, (int)pos, tiles, tbase, lds, cls, shape, small, walls,
                            per, 0});
        tbase += tiles;
    }
    p.map_dirty = true;
    retire_graph(p.graph, b->stream);
    p.graph = nullptr;
    p.made = true;
}

// Refresh the table from the lattices (force, parity) with the steps each
// takes in this call, and send it to the device through kernel arguments.
// With `spare`, in-place lattices write there instead of into their state
// (the autotuner's timed launches).
int batch_upload(clbm_batch *b, BatchPlan &p, const int64_t *nsteps, void *spare = nullptr)
{
    clbm::UploadPayload load;
    const int count = (int)p.order.size();
    for (int first = 0; first < count; first += clbm::kUploadMax) {
        const int n = std::min(clbm::kUploadMax, count - first);
        for (int k = 0; k < n; ++k) {
            const int pos = first + k;
            const clbm_handle *h = b->lats[p.order[pos]];
            LatDesc d = h->d;
            const LatDesc &g = p.tab[pos];
            d.tpr = g.tpr;
            d.inv_tpr = g.inv_tpr;
            d.vec = g.vec;
            d.tile0 = g.tile0;
            d.ntiles = g.ntiles;
            d.walk = g.walk;
            d.per = g.per;
            d.parity = h->parity;
            d.steps = (int32_t)nsteps[p.order[pos]];
            if (spare && d.inplace) d.buf[1] = spare;
            load.d[k] = d;
        }
        HIPCHK(clbm::launch_upload(b->d_lats, first, n, load, b->stream));
    }
    if (p.map_dirty) {
        // Tile -> lattice map of the new geometry.  Graphs that read the old
        // map were retired with the old geometry; the old map is freed in
        // stream order behind their launches.
        const int64_t total = p.groups.empty() ? 0 : p.groups.back().tbase + p.groups.back().ntiles;
        if (total > p.tile_lat_cap) {
            if (p.d_tile_lat) HIPCHK(hipFreeAsync(p.d_tile_lat, b->stream));
            p.d_tile_lat = nullptr;
            p.tile_lat_cap = 0;
            HIPCHK(hipMallocAsync(reinterpret_cast<void **>(&p.d_tile_lat),
                                  sizeof(int32_t) * (size_t)total, b->stream));
            p.tile_lat_cap = total;
        }
        for (const auto &g : p.groups)
            HIPCHK(clbm::launch_tile_map(b->d_lats, g.l_lo, g.l_hi, g.ntiles, p.d_tile_lat + g.tbase,
                                         b->stream));
        p.map_dirty = false;
    }
    return CLBM_OK;
}

// Regions anew, and with them every plan, each when a call next takes it.
void batch_replan(clbm_batch *b)
{
    batch_regions(b);
    for (auto &p : b->plan) p.made = false;
}

bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s, &st) == hipSuccess && st != hipStreamCaptureStatusNone;
}

// The plan of a call whose lattices take at most n steps.  A plan's first call
// allocates and fills its tile map, which a captured call would leave to the
// replays: there plan 0 serves until the other is there.
BatchPlan &batch_pick(clbm_batch *b, int64_t n)
{
    BatchPlan &p = b->plan[n < clbm_batch::kPlans ? n : 0];
    if (std::equal(p.region, p.region + kStorageKinds, b->plan[0].region)) return b->plan[0];
    return (!p.made || p.map_dirty) && capturing(b->stream) ? b->plan[0] : p;
}

// The same, made.  A force change since the last call can move a lattice to
// another kernel (force mode): regroup before launching.
BatchPlan &batch_plan(clbm_batch *b, int64_t n)
{
    BatchPlan *p = &batch_pick(b, n);
    bool same = p->made;
    for (size_t j = 0; same && j < b->lats.size(); ++j) same = group_key(b, *p, b->lats[j]) == p->keys[j];
    if (p->made && !same) {
        batch_replan(b);
        p = &batch_pick(b, n);
    }
    if (!p->made) {
        batch_order(b, *p);
        batch_geometry(b, *p);
    }
    return *p;
}

// Side streams and events for groups 1 .. n-1 (default priority).
int batch_side_streams(clbm_batch *b, size_t n)
{
    if (!b->fork) HIPCHK(hipEventCreateWithFlags(&b->fork, hipEventDisableTiming));
    while (b->side.size() < n) {
        hipStream_t st = nullptr;
        HIPCHK(hipStreamCreateWithFlags(&st, hipStreamNonBlocking));
        b->side.push_back(st);
        hipEvent_t ev = nullptr;
        HIPCHK(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
        b->join.push_back(ev);
    }
    return CLBM_OK;
}

// Steps 0 .. n - 1 of the current call for every group (which = 3), or only
// the groups that step singly (1) or in fused steps (2); with `first`, only
// the first launch of every group, as often as makes kTimedSteps fused steps
// (the autotuner's timed launches, which must not read what they wrote).  The
// groups touch disjoint lattices, so with more than one they run concurrently:
// group 0 on s, the others on side streams forked from s once and joined back
// to it after their n steps (a group of small lattices alone leaves HBM idle
// in its tail; measured +15 % on a batch of FP32 and FP16 lattices).  Within a
// group the steps follow each other in stream order.  With
// `cut`, a group gets no launches beyond its `most` steps (a graph, which other
// counts replay, has them all).
constexpr int kTimedSteps = 8;
int batch_launch_steps(clbm_batch *b, const BatchPlan &p, int n, hipStream_t s, int which = 3, bool first = false,
                       bool cut = false)
{
    const Variant &v = single_of(b->variant);
    const PairVariant &pv = pair_of(b->variant);
    const int64_t grid = v.blocks_per_cu ? (int64_t)b->cus * v.blocks_per_cu : INT32_MAX;
    const int64_t pgrid = pv.blocks_per_cu ? (int64_t)b->cus * pv.blocks_per_cu : 0;
    const size_t ng = p.groups.size();
    if (ng > 1) {
        int rc = batch_side_streams(b, ng - 1);
        if (rc) return rc;
        HIPCHK(hipEventRecord(b->fork, s));
        for (size_t k = 1; k < ng; ++k) HIPCHK(hipStreamWaitEvent(b->side[k - 1], b->fork, 0));
    }
    // The groups' launches in the order of the steps they take, so that they
    // start together however long the host needs to queue them all.
    const int end = first ? kTimedSteps : n;
    for (int t = 0; t < end; ++t) {
        for (size_t k = 0; k < ng; ++k) {
            const auto &g = p.groups[k];
            if (!(which & (g.cls == kSingle ? 1 : 2)) || t % g.per || (first && g.cls == kSingle && t)) continue;
            if (cut && t >= g.most) continue;
            hipStream_t gs = k == 0 ? s : b->side[k - 1];
            const int32_t *map = p.d_tile_lat + g.tbase;
            const int sub = first ? 0 : t / g.per;
            if (g.cls == kLdsTiles)
                HIPCHK(clbm::launch_batch_tile(g.storage, b->d_lats, map, g.ntiles, g.key, g.walls, g.shape, sub, gs));
            else if (g.cls == kSingle)
                HIPCHK(clbm::launch_batch(b->d_lats, map, g.ntiles, g.storage, g.key, g.vec,
                                          (int)std::min<int64_t>(grid, g.ntiles), sub, g.lds, gs));
            else
                HIPCHK(clbm::launch_batch2(g.storage, b->d_lats, map, g.ntiles, g.key, g.small, sub, g.shape,
                                           (int)std::min<int64_t>(pgrid, g.ntiles), gs));
        }
    }
    for (size_t k = 1; k < ng; ++k) {
        HIPCHK(hipEventRecord(b->join[k - 1], b->side[k - 1]));
        HIPCHK(hipStreamWaitEvent(s, b->join[k - 1], 0));
    }
    return CLBM_OK;
}

int batch_build_graph(clbm_batch *b, BatchPlan &p)
{
    hipGraph_t g = nullptr;
    if (!b->cap) HIPCHK(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking));
    HIPCHK(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
    const int rc = batch_launch_steps(b, p, b->chunk, b->cap);
    hipError_t le = rc == CLBM_OK
                        ? clbm::launch_batch_advance(b->d_lats, (int)p.order.size(), b->chunk, b->cap)
                        : hipSuccess;
    hipError_t ce = hipStreamEndCapture(b->cap, &g);
    if (rc != CLBM_OK || le != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return rc != CLBM_OK ? rc : hip_fail(le, "launch_batch_advance (capture)");
    }
    if (ce != hipSuccess) return hip_fail(ce, "hipStreamEndCapture");
    hipError_t ie = hipGraphInstantiate(&p.graph, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (ie != hipSuccess) return hip_fail(ie, "hipGraphInstantiate");
    return CLBM_OK;
}

int batch_run(clbm_batch *b, const int64_t *nsteps)
{
    int64_t maxn = 0;
    for (size_t j = 0; j < b->lats.size(); ++j) {
        if (nsteps[j] < 0) return fail(CLBM_EINVAL, "step counts must be >= 0");
        if (nsteps[j] > INT32_MAX) return fail(CLBM_EINVAL, "step count too large for one call");
        maxn = std::max(maxn, nsteps[j]);
    }
    for (auto *h : b->lats) {
        if (!h->ready) return fail(CLBM_ESTATE, "a lattice of the batch has no state yet");
        if (h->d.force_mode == clbm::FM_SC)
            return fail(CLBM_EINVAL, "a Shan-Chen lattice steps alone, not in a batch");
    }
    if (maxn == 0) return CLBM_OK;
    BatchPlan &p = batch_plan(b, maxn);
    int rc = batch_upload(b, p, nsteps);
    if (rc) return rc;
    // Tiles (four or eight steps per launch) and long launches run as fast
    // launch by launch: no graph to capture on the first call (12 lattices of
    // 10^2 .. 80^2 FP64, 100 steps: 371 -> 190 us; 12 served solves in four
    // groups, first call and 1000 uneven steps: 12.3 -> 11.8 ms; 16 lattices of
    // 16^2 .. 40^2 in four groups 2.0 -> 1.5 us per step).
    bool direct = p.groups.size() == 1 && p.groups[0].ntiles >= 4096;
    if (!direct) {
        direct = true;
        for (const auto &g : p.groups) direct = direct && g.cls == kLdsTiles;
    }
    int64_t left = maxn;
    while (!direct && left >= b->chunk) {
        if (!p.graph && (rc = batch_build_graph(b, p))) return rc;
        HIPCHK(hipGraphLaunch(p.graph, b->stream));
        left -= b->chunk;
    }
    if (left > 0) {
        for (auto &gr : p.groups) {
            gr.most = 0;
            for (int j = gr.l_lo; j < gr.l_hi; ++j) gr.most = std::max(gr.most, nsteps[p.order[j]] - (maxn - left));
        }
        if ((rc = batch_launch_steps(b, p, (int)left, b->stream, 3, false, true))) return rc;
        HIPCHK(clbm::launch_batch_advance(b->d_lats, (int)p.order.size(), (int)left, b->stream));
    }
    for (size_t j = 0; j < b->lats.size(); ++j) {
        // Buffers flip once per launch; every chunk but a lattice's last
        // holds whole launches.
        const int64_t launches = (nsteps[j] + p.per[j] - 1) / p.per[j];
        b->lats[j]->parity = (int)((b->lats[j]->parity + launches) & 1);
        b->lats[j]->steps += nsteps[j];
    }
    return CLBM_OK;
}

std::string batch_signature(const clbm_batch *b)
{
    hipDeviceProp_t prop;
    int dev = 0;
    std::string arch = "unknown";
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
        arch = prop.gcnArchName;
    for (char &c : arch)
        if (c == ' ' || c == ':') c = '_';
    int64_t nodes[kStorageKinds] = {}, counts[kStorageKinds] = {};
    for (auto *h : b->lats) {
        nodes[h->d.storage] += (int64_t)h->d.nx * h->d.ny;
        counts[h->d.storage] += 1;
    }
    std::ostringstream os;
    os << arch << "|v" << kNumSingle << "x" << kNumPair;
    for (int st = 0; st < kStorageKinds; ++st) {
        // Shape class: lattice count and log2 of the node total per storage.
        int lg = 0;
        while (nodes[st] >> (lg + 1)) ++lg;
        os << "|s" << st << ":n" << counts[st] << ":l" << (nodes[st] ? lg : -1);
    }
    return os.str();
}

}  // namespace

extern "C" {

int clbm_batch_create(clbm_handle *const *lattices, int32_t count, void *stream, clbm_batch **out)
{
    g_err.clear();
    if (!lattices || !out || count < 1) return fail(CLBM_EINVAL, "need count >= 1 lattices and out");
    *out = nullptr;
    std::vector<clbm_handle *> v(lattices, lattices + count);
    for (int j = 0; j < count; ++j) {
        if (!v[j]) return fail(CLBM_EINVAL, "NULL lattice in batch");
        for (int k = 0; k < j; ++k)
            if (v[k] == v[j]) return fail(CLBM_EINVAL, "a lattice appears twice in the batch");
    }
    reap_retired();
    clbm_batch *b = new clbm_batch();
    b->lats = v;
    b->stream = static_cast<hipStream_t>(stream);
    b->cus = compute_units();
    batch_replan(b);
    hipError_t e = hipMallocAsync(reinterpret_cast<void **>(&b->d_lats), sizeof(LatDesc) * count,
                                  b->stream);
    if (e != hipSuccess) {
        delete b;
        return hip_fail(e, "clbm_batch_create allocation");
    }
    (void)batch_plan(b, clbm_batch::kPlans);
    *out = b;
    return CLBM_OK;
}

int clbm_batch_step(clbm_batch *b, int64_t nsteps)
{
    g_err.clear();
    if (!b) return fail(CLBM_EINVAL, "batch is NULL");
    std::vector<int64_t> n(b->lats.size(), nsteps);
    return batch_run(b, n.data());
}

int clbm_batch_step_each(clbm_batch *b, const int64_t *nsteps)
{
    g_err.clear();
    if (!b || !nsteps) return fail(CLBM_EINVAL, "batch and nsteps must not be NULL");
    return batch_run(b, nsteps);
}

int32_t clbm_batch_variant_count(void) { return kNumVariants; }

int clbm_batch_set_variant(clbm_batch *b, int32_t variant)
{
    g_err.clear();
    if (!b) return fail(CLBM_EINVAL, "batch is NULL");
    if (variant < 0 || variant >= kNumVariants) return fail(CLBM_EINVAL, "variant out of range");
    if (variant == b->variant) return CLBM_OK;
    b->variant = variant;
    batch_replan(b);  // the groups of a per-lattice tile shape differ
    (void)batch_plan(b, clbm_batch::kPlans);
    return CLBM_OK;
}

int32_t clbm_batch_get_variant(const clbm_batch *b) { return b ? b->variant : -1; }

int clbm_batch_autotune(clbm_batch *b, const char *cache_path, int32_t *chosen)
{
    g_err.clear();
    if (!b) return fail(CLBM_EINVAL, "batch is NULL");
    for (auto *h : b->lats) {
        if (!h->ready) return fail(CLBM_ESTATE, "a lattice of the batch has no state yet");
        if (h->d.force_mode == clbm::FM_SC)
            return fail(CLBM_EINVAL, "a Shan-Chen lattice steps alone, not in a batch");
    }
    const std::string sig = batch_signature(b);
    if (cache_path) {
        std::ifstream in(cache_path);
        std::string key;
        int v;
        while (in >> key >> v) {
            if (key == sig && v >= 0 && v < kNumVariants) {
                int rc = clbm_batch_set_variant(b, v);
                if (!rc && chosen) *chosen = v;
                return rc;
            }
        }
    }
    // Time the variants on the batch's own lattices: one step of every
    // lattice that steps singly and one fused pair of every lattice that
    // steps in pairs.  The timed launches read the current state and write
    // the other buffer without advancing the lattices, so the state is
    // untouched (the next real step overwrites that buffer).  In-place
    // lattices have no other buffer: their timed launches write one scratch
    // allocation as large as the largest of them (all into the same place;
    // its contents are never read).  The single-step part of the variant is
    // chosen first, on the groups that step singly, then the two-step part
    // on the groups that step in pairs.
    bool any_single = false, any_fused = false;
    for (auto *h : b->lats) (use_pairs(h) ? any_fused : any_single) = true;
    size_t spare_bytes = 0;
    for (auto *h : b->lats)
        if (h->d.inplace)
            spare_bytes = std::max(spare_bytes, clbm_buffer_bytes(h->d.nx, h->d.ny, h->d.storage));
    void *spare = nullptr;
    if (spare_bytes) HIPCHK(hipMallocAsync(&spare, spare_bytes, b->stream));
    hipEvent_t t0 = nullptr, t1 = nullptr;
    HIPCHK(hipEventCreate(&t0));
    HIPCHK(hipEventCreate(&t1));
    int rc = CLBM_OK;
    // Mean time of the groups `which` under variant v: one step of those that
    // step singly, kTimedSteps of those that step fused.
    auto time_variant = [&](int v, int which, float *ms) -> int {
        int r = clbm_batch_set_variant(b, v);
        if (r) return r;
        BatchPlan &p = batch_plan(b, clbm_batch::kPlans);
        std::vector<int64_t> counts(p.per.begin(), p.per.end());
        r = batch_upload(b, p, counts.data(), spare);
        const int reps = 5;
        for (int w = 0; w < 2 && r == CLBM_OK; ++w) r = batch_launch_steps(b, p, 1, b->stream, which, true);
        if (r) return r;
        hipError_t e = hipEventRecord(t0, b->stream);
        for (int k = 0; k < reps && r == CLBM_OK && e == hipSuccess; ++k)
            r = batch_launch_steps(b, p, 1, b->stream, which, true);
        if (r) return r;
        if (e == hipSuccess) e = hipEventRecord(t1, b->stream);
        if (e == hipSuccess) e = hipEventSynchronize(t1);
        if (e != hipSuccess) return hip_fail(e, "autotune events");
        (void)hipEventElapsedTime(ms, t0, t1);
        return CLBM_OK;
    };
    int best_single = single_index(b->variant), best_pair = b->variant % kNumPair;
    if (any_single) {
        float best_ms = 1e30f;
        for (int vs = 0; vs < kNumSingle && rc == CLBM_OK; ++vs) {
            float ms = 0.f;
            if ((rc = time_variant(vs * kNumPair + best_pair, 1, &ms))) break;
            if (ms < best_ms) {
                best_ms = ms;
                best_single = vs;
            }
        }
    }
    if (any_fused && rc == CLBM_OK) {
        float best_ms = 1e30f;
        for (int vp = 0; vp < kNumPair && rc == CLBM_OK; ++vp) {
            float ms = 0.f;
            if ((rc = time_variant(best_single * kNumPair + vp, 2, &ms))) break;
            if (ms < best_ms) {
                best_ms = ms;
                best_pair = vp;
            }
        }
    }
    const int best = best_single * kNumPair + best_pair;
    (void)hipEventDestroy(t0);
    (void)hipEventDestroy(t1);
    if (spare) (void)hipFreeAsync(spare, b->stream);
    if (rc) return rc;
    if ((rc = clbm_batch_set_variant(b, best))) return rc;
    if (chosen) *chosen = best;
    if (cache_path) {
        std::ofstream out(cache_path, std::ios::app);
        if (out) out << sig << " " << best << "\n";
    }
    return CLBM_OK;
}

int clbm_batch_destroy(clbm_batch *b)
{
    if (!b) return CLBM_OK;
    for (auto &p : b->plan) {
        retire_graph(p.graph, b->stream);
        if (p.d_tile_lat) (void)hipFreeAsync(p.d_tile_lat, b->stream);
    }
    if (b->d_lats) (void)hipFreeAsync(b->d_lats, b->stream);
    if (b->cap) (void)hipStreamDestroy(b->cap);
    for (auto st : b->side) (void)hipStreamDestroy(st);
    for (auto ev : b->join) (void)hipEventDestroy(ev);
    if (b->fork) (void)hipEventDestroy(b->fork);
    (void)hipGetLastError();
    delete b;
    reap_retired();
    return CLBM_OK;
}

}  // extern "C"

// clbm_internal.h -- types shared by the kernels and the C-ABI layer.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "clbm_device.h"

namespace clbm {

// Where the force density of a lattice comes from.
enum ForceMode {
    FM_CONST = 0,  // (Fx, Fy) of the descriptor at every node (zero = no force)
    FM_ROW = 1,    // Fx from a per-row table, Fy = 0 (Kolmogorov forcing)
    FM_FIELD = 2,  // fx, fy planes [ny][nx] in the arithmetic type
    FM_SC = 3      // Shan-Chen: F from the psi plane [ny][nx] of this step
};

// Threads per block of every step kernel.
constexpr int kBlock = 256;

// The resident kernel: one block of kResidentBlock threads keeps a small
// lattice and runs many steps in one launch.  Its step time grows with the
// lattice (one compute unit does all the work); on MI355X it beats graphed
// single-step launches up to about 512 groups of nodes (16 x 16: 1.7 against
// 3.0 us per step; 64 x 32 FP32: 3.5 against 4.2) and loses beyond (64 x 32
// FP64, 1024 groups: 4.9 against 4.0), hence the default limit.
constexpr int kResidentBlock = 1024;
constexpr int kResidentMaxGroups = 512;

// Spare bytes at the end of every population buffer: a step's vector loads
// may reach one element past the last run (its lane is discarded), and
// must stay inside the allocation.
constexpr int64_t kTailGuardBytes = 64;

// Row padding: each direction's row starts on a multiple of kRowAlign
// elements so that the vector stores of every storage type are naturally
// aligned.  A row wider than kRowLineMinNodes (one two-step tile) starts on
// a 128-byte line, so that a tile's piece of a row covers whole lines: a
// line written in part costs the memory a read of the rest.  Measured on
// MI355X, FP32, two steps per launch: a 3000^2 lattice 102 -> 136 GLUPS,
// the seeded 256-lattice Kolmogorov batch 113 -> 130, 1024 lattices of
// 100^2 89 -> 111.  Narrower lattices keep kRowAlign: one tile covers whole
// rows, which row blocks keep contiguous, and the padding would only grow
// the footprint (4096 lattices of 40^2 lost a third with 64-element rows).
constexpr int kRowAlign = 8;
constexpr int kLineBytes = 128;
constexpr int kRowLineMinNodes = 64;
inline int64_t row_pitch(int nx, int eb)
{
    int64_t a = kRowAlign;
    if (nx > kRowLineMinNodes && kLineBytes / eb > a) a = kLineBytes / eb;
    return ((int64_t)nx + a - 1) / a * a;
}

// Row blocks: R = 2^rshift consecutive lattice rows keep each direction's R
// runs together, so that narrow lattices still stream long contiguous
// pieces; R doubles until a block's run of one direction reaches
// kBlockRunBytes (or R would exceed the lattice height).  Measured on
// batches of small lattices (64^2 to 512^2, FP32): 16 KB runs beat single
// rows by 3-6 %; a 4096^2 FP32 lattice (16 KB rows) keeps R = 1.
constexpr int64_t kBlockRunBytes = 16384;

// Nodes across a strip of the tile walk (8 tiles of 64 columns, 16 of 32).
// Measured on FP64 4096^2 with 32 x 16 tiles: strips of 128, 256, 512 and
// 1024 nodes gave 48, 56, 81 and 81 GLUPS.
constexpr int kStripNodes = 512;

// Division of 0 <= n < 2^31 by a fixed d >= 1 as a multiply and a shift
// (Granlund and Montgomery's round-up method): with 2^(s-1) < d <= 2^s,
// m = ceil(2^(31+s) / d) is below 2^32 and m d - 2^(31+s) < d <= 2^s, so
// n m / 2^(31+s) exceeds n / d by less than 1/d and its floor is floor(n / d).
// With n and the divisor uniform, the kernel does it on the scalar unit.
struct FastDiv {
    uint32_t m;
    int32_t sh;
};
inline FastDiv fast_div(uint32_t d)
{
    int s = 0;
    while (s < 31 && (1u << s) < d) ++s;
    const uint64_t p = (uint64_t)1 << (31 + s);
    return FastDiv{(uint32_t)((p + d - 1) / d), 31 + s};
}

// The strip walk of one lattice's tiles with its divisions prepared on the
// host (strip_tile's arithmetic without integer divides in the kernel).
struct StripWalk {
    int32_t sw, tiles_y, full, in_full, w;  // strip width, tile rows, full strips, their tiles, last strip's width
    FastDiv by_strip, by_sw, by_w;          // by sw * tiles_y, sw and w
};
inline StripWalk strip_walk(int tiles_x, int tiles_y, int sw)
{
    StripWalk p;
    p.sw = sw;
    p.tiles_y = tiles_y;
    p.full = tiles_x / sw;
    p.in_full = p.full * sw * tiles_y;
    p.w = tiles_x - p.full * sw;
    p.by_strip = fast_div((uint32_t)(sw * tiles_y));
    p.by_sw = fast_div((uint32_t)sw);
    p.by_w = fast_div((uint32_t)(p.w > 0 ? p.w : 1));
    return p;
}

// Everything a kernel needs to step one lattice.  Passed by value to the
// single-lattice kernel and stored in a device array for batches.
struct LatDesc {
    void *buf[2];        // two buffers: ping-pong; in place: read buf[0], write buf[1]
                         // (the same buffer outside the batch autotuner)
    const void *force;   // FM_ROW: table[ny]; FM_FIELD: fx plane then fy plane
    int64_t dstride;     // elements between two directions' runs in a row block (R pitch)
    int64_t pitch;       // elements between two rows of one direction in a row block
    int64_t bstride;     // elements between two row blocks (9 R pitch)
    int32_t nx, ny;      // lattice size
    int32_t bc_y;        // 0 periodic, 1 half-way bounce-back
    int32_t storage;     // StorageKind
    int32_t force_mode;  // ForceMode
    int32_t scheme;      // SchemeKind
    int32_t parity;      // batch: buffer holding the state at sequence start
    int32_t steps;       // batch: steps of this lattice in the sequence
    int32_t tpr;         // groups of vec nodes along a row: ceil(nx / vec)
    int32_t vec;         // nodes per thread along x
    int32_t inplace;     // 0: two buffers (pull form); 1: one buffer, AA pattern
    int32_t rshift;      // log2 of the rows per row block
    int32_t per;         // batch: steps per launch (1, 2, 4 or 8; parity counts launches)
    int64_t tile0;       // batch: first tile of this lattice in its group
    int64_t ntiles;      // batch: tiles of this lattice
    StripWalk walk;      // batch, fused steps: the strip walk of its tiles in the group's shape
    double inv_tpr;      // 1 / tpr, for the tile decode
    double Fx, Fy;       // FM_CONST force density
    double sc_g, sc_psi0, sc_rho;  // FM_SC: G, psi0 and rho_ref of psi = psi0 exp(-rho_ref/rho)
    double sc_psic;                // FM_SC: psi(rho0); the psi plane holds psi - sc_psic
    double rho0;
    // Relaxation and force weights of the collision (set_rates).
    double nap, nam;       // -(sb + s2)/2, -(sb - s2)/2
    double ns2, ns3, ns4;  // -s2, -s3, -s4
    double h3t;            // (1 - s3/2) cs^2, or 0 (Sec. III A)
    double g1;             // s1/2 + 1 - s2/2 (Eq. 21)
    double h2;             // 1 - s2/2 (Eq. 21)
};

// The collision's constants for S = diag(s0, s1, s1, sb, s2, s2, s3, s3, s4)
// (Sec. II A) and a forcing scheme (0: Eq. 12, 1: Eq. 21, 2: Premnath et
// al.'s, Eqs. 17-19), in double precision.  The second-order central
// moments relax as a trace at sb and a deviator at s2, so the changes of
// k~20 and k~02 are nap c20 + nam c02 and nam c20 + nap c02 (c = departure
// from equilibrium).  The scheme of Sec. III A is Eq. (12) without the
// third-order force moments: the same kernel with h3t = 0.
inline void set_rates(LatDesc &d, double s1, double sb, double s2, double s3, double s4, int scheme)
{
    d.scheme = scheme == 1 ? SCH_GUO_LBL : SCH_CONSISTENT;
    d.nap = -0.5 * (sb + s2);
    d.nam = -0.5 * (sb - s2);
    d.ns2 = -s2;
    d.ns3 = -s3;
    d.ns4 = -s4;
    d.h3t = scheme == 2 ? 0.0 : (1.0 - 0.5 * s3) / 3.0;
    d.g1 = 0.5 * s1 + 1.0 - 0.5 * s2;
    d.h2 = 1.0 - 0.5 * s2;
}

// Tile shapes of the two-step kernels (columns x rows of nodes per block of
// kBlock threads, 4 nodes per thread in its second step): 64 x 16 or 32 x
// 32, for FP64 storage (whose LDS holds half as many nodes) 64 x 8 or 32 x
// 16 with 2 nodes per thread.
enum TileShape { kTile64x16 = 0, kTile32x32 = 1 };
inline int tile_w(int shape) { return shape == kTile32x32 ? 32 : 64; }
inline int tile_h(int shape, int storage)
{
    const int h = shape == kTile32x32 ? 32 : 16;
    return storage == ST_F64 ? h / 2 : h;
}

// Four fused steps per launch (clbm_sweep.h): a wave marches down the rows of
// a strip of 64 lanes x vec columns.
constexpr int kSweepSteps = 4;
struct SweepPlan {
    int32_t vec;     // columns per lane (1 or 2); 0: this lattice takes no sweeps
    int32_t strips;  // strips across the lattice
    int32_t rows;    // rows per chunk: chunk c is rows [c rows, (c + 1) rows)
    int32_t units;   // strips x chunks, one wave each
    int32_t groups;  // groups of vec columns along a row: ceil(nx / vec)
    int32_t halo;    // lanes at each end of a wave that are collided, not stored
};

// Columns per lane compiled: two need the registers, which an FP64 lattice
// with walls or a per-node force no longer has (it would spill 78 to 156 of
// them; 1501 x 703 with both 17.3 us per step, no faster than pairs).
constexpr int sweep_max_vec(int storage, int force_mode, int bc_y)
{
    return storage == ST_F64 && (force_mode == FM_FIELD || bc_y) ? 1 : 2;
}

// Microseconds of one launch under a plan, from what bounds it: the VALU issue
// of the busiest SIMD (a wave collides rows + K - 1 rows of each of K levels on
// average, 0.230 us per level and column of a lane in FP32, 0.262 in FP64; one
// wave per SIMD hides its latencies to 72 % of the issue rate, two to 92 %), or
// memory at 4.8 TB/s (3.3 with one wave per SIMD; each chunk reads 2 K rows and
// each strip 2 halo lanes beyond its own), plus 3 us of launch.  Within 10 % of
// what 1024^2, 2048^2 and 4096^2 lattices take (FP64 48, 154, 500 us; FP32 31, 95,
// 295).
inline double sweep_us(int64_t nodes, int eb, int simds, int vec, int halo, int rows, int64_t units)
{
    const int64_t n = (units + simds - 1) / simds;  // waves on the busiest SIMD
    const double eff = n == 1 ? 0.72 : (n == 2 ? 0.92 : 0.95);
    const double valu = kSweepSteps * (eb == 8 ? 0.262 : 0.230) * vec * n * (rows + kSweepSteps) / eff;
    const double state = 9.0 * nodes * eb;
    const double reads = 64.0 / (64 - 2 * halo) * (1.0 + 2.0 * kSweepSteps / rows);
    const double mem = state * (1.0 + reads) / (n == 1 ? 3.3e6 : 4.8e6);
    return (valu > mem ? valu : mem) + 3.0;
}

// The plan of a lattice: columns per lane and rows per chunk with the least
// sweep_us among those that fill the SIMDs 1 .. 8 times.
inline SweepPlan sweep_plan(int nx, int ny, int eb, int simds, int max_vec)
{
    SweepPlan best{};
    double best_us = 0.0;
    for (int vec = 1; vec <= max_vec; ++vec) {
        SweepPlan p{};
        p.vec = vec;
        p.groups = (nx + vec - 1) / vec;
        // Every level loses one column at each side; the last group of a
        // ragged row holds fewer than vec of them.
        p.halo = (kSweepSteps + vec - 1) / vec + (nx % vec ? 1 : 0);
        p.strips = (p.groups + 63 - 2 * p.halo) / (64 - 2 * p.halo);
        for (int n = 1; n <= 8; ++n) {
            int64_t chunks = (int64_t)n * simds / p.strips;
            if (chunks < 1) continue;
            if (chunks > ny) chunks = ny;
            p.rows = (int)((ny + chunks - 1) / chunks);
            const int64_t units = (int64_t)p.strips * ((ny + p.rows - 1) / p.rows);
            p.units = (int32_t)units;
            const double us = sweep_us((int64_t)nx * ny, eb, simds, vec, p.halo, p.rows, units);
            if (best.vec == 0 || us < best_us) {
                best = p;
                best_us = us;
            }
        }
    }
    return best;
}

// Several fused steps per launch in LDS (clbm_tile.h).  A block's region is W
// x H cells, its tile the K - 1 cells less at each side that its K-th step
// still has.
enum RegionShape {
    kRegion32x24 = 0,
    kRegion32x32 = 1,
    kRegion64x16 = 2,
    kRegion32x16 = 3,
    kRegion64x32 = 4,
    kRegion64x48 = 5,
    kRegionShapes = 6,
    // With the Shan-Chen force, whose steps need two nodes less at each side.
    kRegionSc32x24 = 6,
    kRegionSc64x32 = 7
};
constexpr int region_w(int shape)
{
    return shape == kRegion64x16 || shape == kRegion64x32 || shape == kRegion64x48 || shape == kRegionSc64x32 ? 64 : 32;
}
constexpr int region_h(int shape)
{
    switch (shape) {
    case kRegion32x24:
    case kRegionSc32x24: return 24;
    case kRegion32x32:
    case kRegion64x32:
    case kRegionSc64x32: return 32;
    case kRegion64x48: return 48;
    default: return 16;
    }
}
// 64 x 48 only in 16-bit storage, where three blocks of its 48 KB of LDS share a
// compute unit (two between walls or with a force field, whose kernels take 82 to
// 124 VGPRs against 65 to 79: tile_form) (FP32 one of 96 KB: 1024^2 7.5 against
// 6.8 us per step in 64 x 32; FP64 would need 192 KB).
constexpr bool region_compiled(int shape, int storage)
{
    return shape != kRegion64x48 || !(storage == ST_F64 || storage == ST_F32);
}
constexpr int region_steps(int shape) { return shape == kRegion32x24 || shape == kRegion32x32 ? 8 : 4; }
constexpr int region_tile_w(int shape) { return region_w(shape) - 2 * (region_steps(shape) - 1); }
constexpr int region_tile_h(int shape) { return region_h(shape) - 2 * (region_steps(shape) - 1); }
struct TilePlan {
    int32_t steps;    // most steps of one launch (K); 0: this lattice takes no tiles
    int32_t shape;    // RegionShape
    int32_t tiles_x;  // tiles across the lattice
    int32_t tiles;
};

// Microseconds of one launch of K steps: a fixed part (launch, first loads,
// last stores) and the tiles a compute unit takes one after another or side
// by side (bytes: one buffer of all the lattices).  Fitted on MI355X to flows
// on 64 x 32 ... 4096^2 lattices, within 12 % (us per launch at 200^2, 512^2,
// 2048^2): FP32 32 x 24 8.7, 28; 32 x 32 9.8, 25; 64 x 16 6.8, 9.8, 94;
// 32 x 16 5.6, 11.3, 111; 64 x 32 9.8, 10.8, 91.  FP64 10.4, 41; 12.0, 40;
// 8.2, 13.7, 168; 6.0, 15.8, 184; 13.9, 15.8, 194.  FP16-SR 10.0, 36; 11.5, 31;
// 8.1, 11.5, 106; 6.0, 12.7, 125; 13.2, 14.0, 97; 64 x 48 18.5, 19.2, 93.
// Those flows were periodic with a constant or row force; form is tile_form's
// factor of the lattices.
inline double tile_us(int shape, int storage, int64_t tiles, int64_t bytes, int cus, double form = 1.0)
{
    struct Fit { double fixed, per; };
    static const Fit fit[4][kRegionShapes] = {
        {{5.0, 5.8}, {3.7, 9.0}, {4.2, 4.6}, {3.4, 2.5}, {1.5, 15.0}, {}},       // FP64
        {{4.8, 3.8}, {4.7, 5.07}, {4.2, 2.7}, {3.9, 1.45}, {3.5, 6.7}, {}},      // FP32
        {{4.5, 4.2}, {4.7, 5.45}, {5.0, 2.8}, {3.9, 1.52}, {7.0, 6.05}, {11.5, 9.4}},  // 16-bit, to nearest
        {{5.0, 4.9}, {5.0, 6.5}, {5.0, 3.25}, {3.9, 1.79}, {7.0, 7.2}, {13.0, 10.8}},   // 16-bit, stochastic
    };
    const int64_t n = (tiles + cus - 1) / cus;
    const int t = storage == ST_F64 ? 0 : (storage == ST_F32 ? 1 : (storage == ST_F16 || storage == ST_BF16 ? 2 : 3));
    // Tiles of FP32 and FP64 take longer where the two buffers no longer fit the
    // 256 MB Infinity Cache.
    const double miss = 2 * bytes > (int64_t)256 << 20 ? (t == 0 ? 1.17 : (t == 1 ? 1.08 : 1.0)) : 1.0;
    return fit[t][shape].fixed + fit[t][shape].per * miss * form * n;
}

// What a lattice's steps carry beside the collision.
struct Form {
    bool field, walls;  // a force per node; walls in y
};

// Time of a tile's steps against a periodic lattice without a force field, in
// 16-bit storage: between walls the 64-wide regions take 22 to 34 registers more
// and one block less shares a compute unit; a field takes them 6 to 10 and its
// loads (us per launch at 4096^2 FP16, periodic, field, walls: 64 x 48 280, 314,
// 325; 64 x 32 277, 294, 335; 64 x 16 321, 334, 353; FP16-SR 64 x 48 318, 358,
// 372; 64 x 32 328, 333, 382).  In FP32 and FP64 all regions take 3 to 9 % more,
// and the choice is the same.
inline double tile_form(int shape, int storage, Form f)
{
    if (storage == ST_F64 || storage == ST_F32) return 1.0;
    const bool nearest = storage == ST_F16 || storage == ST_BF16;
    switch (shape) {
    case kRegion64x48: return f.walls ? 1.17 : (f.field ? 1.12 : 1.0);
    case kRegion64x32: return f.walls ? (nearest ? 1.21 : 1.15) : (f.field ? (nearest ? 1.06 : 1.02) : 1.0);
    case kRegion64x16: return f.walls ? 1.09 : (f.field ? 1.03 : 1.0);
    case kRegion32x16: return f.walls ? 1.03 : 1.0;
    default: return 1.0;
    }
}
// The same of a fused pair, whose field loads are not hidden by more steps
// (4096^2 FP16 153 -> 175, FP16-SR 170 -> 186; walls cost nothing).
inline double pair_form(int storage, Form f)
{
    if (storage == ST_F64 || storage == ST_F32 || !f.field) return 1.0;
    return storage == ST_F16 || storage == ST_BF16 ? 1.13 : 1.08;
}

// Microseconds of one launch of a fused pair on `tiles` tiles of 64 x 16
// nodes (64 x 8 in FP64), four and more of which share a compute unit.
inline double pair_us(int storage, int64_t tiles, int cus, double form = 1.0)
{
    const double per = storage == ST_F64 ? 3.2 : (storage == ST_F32 ? 3.35 : (storage == ST_F16 || storage == ST_BF16 ? 2.27 : 2.55));
    return 6.0 + per * form * tiles / cus;
}

// The plan with the least time per step, which goes to *us_per_step.
inline TilePlan tile_plan(int nx, int ny, int storage, int64_t bytes, int cus, double *us_per_step, Form form = Form{})
{
    TilePlan best{};
    for (int shape = 0; shape < kRegionShapes; ++shape) {
        if (!region_compiled(shape, storage)) continue;
        TilePlan p{};
        p.shape = shape;
        p.steps = region_steps(shape);
        const int tw = region_tile_w(shape), th = region_tile_h(shape);
        p.tiles_x = (nx + tw - 1) / tw;
        const int64_t tiles = (int64_t)p.tiles_x * ((ny + th - 1) / th);
        if (tiles > INT32_MAX) continue;
        p.tiles = (int32_t)tiles;
        const double us = tile_us(shape, storage, tiles, bytes, cus, tile_form(shape, storage, form)) / p.steps;
        if (best.steps == 0 || us < *us_per_step) {
            best = p;
            *us_per_step = us;
        }
    }
    return best;
}

// Whether the last one or two steps of a run go to the tile kernel like the
// launches before them, or to the one-step kernel and the pair kernel.  A tile
// launch of n steps takes about n / K of a full one, but stores pieces of lines
// (58 columns and fewer), which costs memory a read of each: beyond the Infinity
// Cache it never pays (us, tile launch against the other: FP64 1500^2 one step 66
// / 57, two 73 / 67; FP16 4096^2 140 / 110, 170 / 153).  Within it the tile
// kernel wins where it has work enough to cover its fixed part (FP64 1024^2 24 /
// 30, 28 / 33; FP32 1500^2 25 / 31, 30 / 39; FP16 1500^2 17 / 19; but 512^2 FP64
// 8.1 / 7.3, FP16 768^2 8.4 / 7.2), unless its tiles cover much more than the
// lattice, or than the pairs' tiles do (16 x 20000 FP32 9.0 / 6.0 for one step,
// 11.7 / 13.4 for two; 64 x 20003 17.7 / 17.9, 24.0 / 22.4; 16-bit in many rounds
// of 32 x 16 regions, FP16 64 x 20003 24.9 / 17.2 for two, 768^2 12.2 / 12.2);
// between walls 16-bit tiles run at a lower occupancy (FP16 2048^2 36 / 35, 52 /
// 47).  Tiles of one round are launch-bound: equal.  Three steps take one launch
// instead of two (0.4 to 1.0 of their time).
struct ShortRun {
    int32_t shape, storage;
    bool walls;
    int64_t tiles, pair_tiles, nodes, bytes;  // bytes: one buffer of all the lattices
};
inline bool tiles_take(int64_t left, const ShortRun &r, int cus)
{
    if (left >= 3 || r.tiles <= cus) return true;
    const int64_t mb = (int64_t)1 << 20, both = 2 * r.bytes;
    if (both > 256 * mb) return false;
    const double cells = (double)r.tiles * region_tile_w(r.shape) * region_tile_h(r.shape);
    const double pair_cells = (double)r.pair_tiles * tile_w(kTile64x16) * tile_h(kTile64x16, r.storage);
    const bool f64 = r.storage == ST_F64, narrow = !(f64 || r.storage == ST_F32);  // narrow: 16-bit
    const bool work = both >= (narrow ? 64 : 40) * mb;
    if (left == 1) {
        const double most = f64 ? 1.5 : (r.shape == kRegion32x16 ? 1.2 : 1.3);
        return work && !(narrow && r.walls) && cells <= most * (double)r.nodes;
    }
    double most = f64 ? (work ? 1.5 : 1.0) : 1.3;
    if (!f64 && r.shape == kRegion32x16) most = !narrow ? 1.2 : (r.tiles > 9 * cus ? 0.6 : 1.3);
    if (narrow && r.walls && both >= 32 * mb && most > 0.9) most = 0.9;
    return cells <= most * pair_cells;
}

// The plan of a Shan-Chen lattice: regions of 32 x 24 cells and four steps
// (tiles of 18 x 10) or of 64 x 32 and two (58 x 26), whichever takes less
// time per step.
inline TilePlan sc_tile_plan(int nx, int ny, int storage, int cus)
{
    TilePlan p[2];
    double us[2];
    for (int k = 0; k < 2; ++k) {
        const int steps = k == 0 ? 4 : 2, h = 2 * steps - 1;
        const int tw = (k == 0 ? 32 : 64) - 2 * h, th = (k == 0 ? 24 : 32) - 2 * h;
        p[k].steps = steps;
        p[k].shape = k == 0 ? kRegionSc32x24 : kRegionSc64x32;
        p[k].tiles_x = (nx + tw - 1) / tw;
        p[k].tiles = p[k].tiles_x * ((ny + th - 1) / th);
        const int n = (p[k].tiles + cus - 1) / cus;
        us[k] = (3.5 + (k == 0 ? 4.0 : 8.0) * (storage == ST_F64 ? 1.5 : 1.0) * n) / steps;
    }
    return us[1] < us[0] ? p[1] : p[0];
}

// Steps per graph replay of a lattice (0: launch by launch), from those asked
// for (-1: the default), the fused steps of a launch of the tile or sweep kernel
// (0: single steps or pairs) and the bytes of a buffer.  Launch by launch each
// single step or pair takes 0.3 to 0.7 us more than in a replay (in place FP32
// 512^2 6.1 / 5.4 us, 900^2 12.6 / 12.3, 2000 x 1200 31.5 / 31.1; 3000^2 equal),
// so they replay 64 steps by default up to 256 MB of traffic per step.  Launches
// of the tile and sweep kernels take longer than the host needs to queue them and
// run as fast without a capture (64 x 32 FP64, 512 steps: 0.60 ms either way); a
// replay of a few of them is slower (of two steps 4.3 ms), so one asked for
// serves from eight launches on.
constexpr int kGraphSteps = 64;
constexpr int64_t kGraphMaxTraffic = (int64_t)256 << 20;
constexpr int kGraphMinFused = 8;
inline int graph_steps(int asked, int fused, int64_t bytes)
{
    if (fused) return asked >= kGraphMinFused * fused ? asked : 0;
    if (asked >= 0) return asked;
    return 2 * bytes <= kGraphMaxTraffic ? kGraphSteps : 0;
}

// Lattice descriptors carried in one upload kernel's arguments.
constexpr int kUploadMax = 12;
struct UploadPayload {
    LatDesc d[kUploadMax];
};

// Tile geometry of one lattice for blocks of kBlock threads and vec nodes
// per thread: the lattice is ny rows of tpr groups of vec nodes, numbered
// row by row, and tile t is groups [t kBlock, (t + 1) kBlock) -- every lane
// of every tile but the last has a group, whatever the row length.  The
// groups cover the padded row (a multiple of kRowAlign, which vec divides),
// so the stores of each row fill its padding too: no cache line is left
// partly written, which would cost a read of the line from HBM.
inline void tile_geometry(int64_t pitch, int ny, int vec, int32_t *tpr, double *inv_tpr,
                          int64_t *ntiles)
{
    const int slots = (int)(pitch / vec);
    *tpr = slots;
    *inv_tpr = 1.0 / slots;
    *ntiles = ((int64_t)slots * ny + kBlock - 1) / kBlock;
}

// Step kernel of a lattice within its storage type: storage scheme, force
// mode and forcing scheme.
inline int kernel_key(const LatDesc &d) { return (d.inplace * 4 + d.force_mode) * 2 + d.scheme; }
constexpr int kKernelKeys = 16;

// Launchers (clbm_kernels.hip).  All return the hipError_t of the launch.
// One step of a lattice: src is the buffer (two buffers) or phase (in
// place) holding the state; lds bytes of unused LDS per block cap the
// blocks resident on a compute unit (0: no cap).
hipError_t launch_step(const LatDesc &d, int src, int vec, size_t lds, hipStream_t s);
// One time step of the lattices of one batch group (all of one storage
// type and one kernel key, tiles numbered consecutively through their tile0
// fields).
// tile_lat[t] is the lattice holding tile t of the group.
hipError_t launch_batch(const LatDesc *lats, const int32_t *tile_lat, int64_t ntiles, int storage,
                        int key, int vec, int grid, int substep, size_t lds, hipStream_t s);
// Fill tile_lat[0, ntiles) for lattices [l_lo, l_hi) of a group from their
// tile0 / ntiles fields.
hipError_t launch_tile_map(const LatDesc *lats, int l_lo, int l_hi, int64_t ntiles,
                           int32_t *tile_lat, hipStream_t s);
// nsteps steps of a small lattice (no Shan-Chen force) in one launch of one
// block; vec is the storage type's default nodes per thread.
hipError_t launch_resident(const LatDesc &d, int src, int nsteps, hipStream_t s);
// Two fused steps (temporal blocking) from buffer src into src ^ 1: two
// buffers, any storage type, any force but Shan-Chen (step2_supported).
bool step2_supported(const LatDesc &d);
hipError_t launch_step2(const LatDesc &d, int src, hipStream_t s);
// Four fused steps from buffer src into src ^ 1 under a plan of sweep_plan:
// FP32 or FP64 storage, otherwise as step2_supported.
hipError_t launch_sweep(const LatDesc &d, int src, const SweepPlan &p, hipStream_t s);
template <int ST>
hipError_t launch_sweep_st(const LatDesc &d, int src, const SweepPlan &p, hipStream_t s);
// n <= p.steps fused steps from buffer src into src ^ 1 under a plan of
// tile_plan: as step2_supported, buffers below 4 GB (32-bit byte offsets).
hipError_t launch_tile(const LatDesc &d, int src, int n, const TilePlan &p, hipStream_t s);
template <int ST>
hipError_t launch_tile_st(const LatDesc &d, int src, int n, const TilePlan &p, hipStream_t s);
// Substep `sub` of a batch group whose lattices step in LDS tiles of one
// region shape: each lattice with more than K sub steps left (K the shape's)
// takes min(K, what is left) of them.  walls: a lattice of the group has them.
hipError_t launch_batch_tile(int storage, const LatDesc *lats, const int32_t *tile_lat, int64_t ntiles, int key,
                             bool walls, int shape, int sub, hipStream_t s);
template <int ST>
hipError_t launch_batch_tile_st(const LatDesc *lats, const int32_t *tile_lat, int64_t ntiles, int key, bool walls,
                                int shape, int sub, hipStream_t s);
// Pair substep `pair` of a batch group whose lattices step in pairs: each
// lattice with at least 2 pair + 2 steps left takes two fused steps, one
// with 2 pair + 1 left takes its last single step.  small: every buffer of
// the group is below 4 GB; storage is the group's; shape the tile shape
// (kTile64x16 or kTile32x32 of clbm_step2.h, which numbered the lattices'
// tiles); grid 0 launches one block per tile, grid > 0 that many persistent
// blocks walking the tiles.
hipError_t launch_batch2(int storage, const LatDesc *lats, const int32_t *tile_lat, int64_t ntiles, int key,
                         bool small, int pair, int shape, int grid, hipStream_t s);
// The same per storage type, one translation unit each (clbm_step_*.hip).
template <int ST>
hipError_t launch_batch2_st(const LatDesc *lats, const int32_t *tile_lat, int64_t ntiles, int key,
                            bool small, int pair, int shape, int grid, hipStream_t s);
template <int ST>
hipError_t launch_step2_st(const LatDesc &d, int src, hipStream_t s);
template <int ST>
hipError_t launch_resident_st(const LatDesc &d, int src, int nsteps, hipStream_t s);
template <int ST>
hipError_t launch_step_st(const LatDesc &d, int src, int vec, size_t lds, hipStream_t s);
template <int ST>
hipError_t launch_batch_st(const LatDesc *lats, const int32_t *tile_lat, int64_t ntiles, int key,
                           int vec, int grid, int substep, size_t lds, hipStream_t s);
// Write n <= kUploadMax descriptors to lats[first..first+n) on the stream.
hipError_t launch_upload(LatDesc *lats, int first, int n, const UploadPayload &p, hipStream_t s);
hipError_t launch_batch_advance(LatDesc *lats, int count, int chunk, hipStream_t s);
hipError_t launch_init(const LatDesc &d, int dst, const double *rho, const double *ux,
                       const double *uy, hipStream_t s);
hipError_t launch_set_populations(const LatDesc &d, int dst, const double *f, hipStream_t s);
hipError_t launch_get_populations(const LatDesc &d, int src, double *f, hipStream_t s);
// Moments and, with partials, FP64 partial sums; returns the number of partial
// blocks.
hipError_t launch_moments(const LatDesc &d, int src, double *rho, double *ux, double *uy,
                          const double *ux_ref, const double *uy_ref, double *partials,
                          int *nblocks, hipStream_t s);
// out[c] = the fixed-order sum of component c over the partial blocks, plus
// base0 for c = 0.
hipError_t launch_reduce(const double *partials, int nblocks, int ncomp, double *out, hipStream_t s,
                         double base0 = 0.0);
hipError_t launch_force_table(const LatDesc &d, void *table, double A, double k, hipStream_t s);
hipError_t launch_force_field(const LatDesc &d, void *field, const double *fx, const double *fy,
                              hipStream_t s);
// Shan-Chen: psi = psi0 exp(-rho_ref / rho) per node into d.force, from the
// state in buffer src, or (rho != NULL) from a given density field, or
// (src < 0, rho == NULL) from the rest density.
hipError_t launch_psi(const LatDesc &d, int src, const double *rho, hipStream_t s);
// Partial blocks the moments kernel uses for a lattice of n nodes (at most
// kMomentsMaxBlocks, whatever n).
constexpr int kMomentsMaxBlocks = 1024;
int moments_blocks(int64_t n);

}  // namespace clbm

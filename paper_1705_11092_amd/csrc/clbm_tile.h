// clbm_tile.h -- up to K fused steps per launch in LDS (two-buffer, pull
// form), for lattices whose steps are otherwise bound by launches and
// latencies.  Included by the translation units of the storage types, after
// clbm_step.h.
//
// A block owns a tile and collides, in its first step, the tile and K - 1
// nodes around it (its region, RW x RH cells), pulling the state from the
// caches; each later step pulls from the block's LDS and is needed on one
// node less at each side, until the last collides the tile alone and writes
// it to the other buffer.  A thread keeps the cells of one column (every
// NT / RW-th row of it), so its slot 0 stays in a register, its force is read
// once, and its LDS addresses are one register and constants.  LDS holds the
// other 8 slots once, streamed in place, one barrier per step.
//
// What bounds it: small lattices the serial chain of a launch (pulls, a barrier
// and a collision per step), about 9 us for eight steps; larger ones VALU issue,
// for the cells collided beyond the tile (64 x 32 and four steps: 1.18 per cell
// stored, 64 x 48 1.15, 64 x 16 1.38) and the last, partly filled round of
// tiles.  Hence small regions of eight steps where launches count, and the
// tallest of 64 columns whose LDS still lets two blocks (FP32, FP64) or three
// (16-bit; two between walls, by their registers) share a compute unit where the
// work does.  Us per step, pairs ->
// tiles: 64 x 32 FP64 2.8 -> 1.17, 200^2 FP64 3.6 -> 1.3, 512^2 FP32 3.6 -> 2.5,
// 1024^2 FP32 9.7 -> 5.9, 1501 x 703 FP64 17.1 -> 10.4, 4096^2 FP16 73.3 -> 68.0,
// 2048^2 FP16-SR 23.9 -> 21.6.
//
// The region is the periodic plane around the tile, so a lattice smaller than
// the region simply repeats.  Every node update is the one-step kernel's, so
// the result is bitwise that of n one-step launches.
#pragma once

#include <type_traits>

#include "clbm_step.h"

namespace clbm {
namespace {

// v in [-n, ...) brought into [0, n).
__device__ __forceinline__ int wrap_any(int v, int n)
{
    if (v < 0) v += n;
    if (v < 0 || v >= n) {
        v %= n;
        if (v < 0) v += n;
    }
    return v;
}

// Element at byte offset off of a buffer below 4 GB: the loads and stores take
// the uniform base and the 32-bit offset as they are.
template <typename T>
__device__ __forceinline__ T load_at(const T *base, uint32_t off)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + (uint64_t)off);
}
template <typename T>
__device__ __forceinline__ void store_at(T *base, uint32_t off, T v)
{
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + (uint64_t)off) = v;
}
// base advanced by a row's (and slot's) byte offset.  In regions 64 cells wide
// a wave's cells share their row, the offset is uniform, and the scalar unit
// adds it; in narrower ones it joins the lane's offset.
template <bool UNIFORM, typename T>
__device__ __forceinline__ T *row_base_at(T *base, uint32_t row, uint32_t &off)
{
    if constexpr (UNIFORM) {
        using C = std::conditional_t<std::is_const_v<T>, const char, char>;
        return reinterpret_cast<T *>(reinterpret_cast<C *>(base) + (uint64_t)row);
    }
    off += row;
    return base;
}

// Keeps a loop-invariant value, and all that follows from it, from being formed
// ahead of the loop: the last step's store addresses, 9 per cell, would
// otherwise sit in registers through every step.
template <bool UNIFORM>
__device__ __forceinline__ void form_here(uint32_t &v)
{
    if constexpr (UNIFORM)
        asm volatile("" : "+s"(v));
    else
        asm volatile("" : "+v"(v));
}

template <int RW_, int RH_, int K_, int NT_>
struct Region {
    static constexpr int RW = RW_, RH = RH_, K = K_, NT = NT_;
    static constexpr int TW = RW - 2 * (K - 1), TH = RH - 2 * (K - 1);  // the tile
    static constexpr int RPP = NT / RW;                                 // rows per pass of the block
    static constexpr int M = RH / RPP;                                  // cells per thread
    // Waves per SIMD to leave room for: two blocks of 512 threads on a
    // compute unit (FP64 between walls would take 134 VGPRs, one block).
    static constexpr int WV = NT == 512 ? 4 : 1;
    static_assert(NT % RW == 0 && RH % RPP == 0, "whole rows per pass, whole passes");
};

// n <= K steps of the tile at (x0, y0) from buffer src into src ^ 1.
// WALL: the lattice may have walls (d.bc_y says).
template <int ST, int FM, int SCH, typename RG, bool WALL>
__device__ __forceinline__ void tile_steps(const LatDesc &d, int src, int x0, int y0, int n,
                                           typename Storage<ST>::T (&lds)[8][RG::RH][RG::RW])
{
    using S = Storage<ST>;
    using T = typename S::T;
    using R = typename S::R;
    constexpr int RW = RG::RW, RH = RG::RH, M = RG::M, H = RG::K - 1;
    // Cells loaded and collided together: more at once cost registers, and
    // with them the second block on the compute unit.
    constexpr int kStage = 2;
    const T *in = static_cast<const T *>(d.buf[src]);
    T *out = static_cast<T *>(d.buf[src ^ 1]);
    const Rates<R> rt = rates_of<R>(d);
    constexpr bool kU = RW % 64 == 0;  // a wave's cells lie in one row
    const int c = threadIdx.x % RW;
    const int rt0 = kU ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / RW) : (int)threadIdx.x / RW;
    const int we = d.nx - x0 < RG::TW ? d.nx - x0 : RG::TW;  // the tile's columns and rows in the lattice
    const int he = d.ny - y0 < RG::TH ? d.ny - y0 : RG::TH;

    const int x = wrap_any(x0 - H + c, d.nx);
    constexpr uint32_t kB = sizeof(T);
    const uint32_t cm = (uint32_t)(x == 0 ? d.nx - 1 : x - 1) * kB, c0 = (uint32_t)x * kB,
                   cp = (uint32_t)(x == d.nx - 1 ? 0 : x + 1) * kB;
    const uint32_t bs = (uint32_t)d.bstride * kB, pb = (uint32_t)d.pitch * kB, ds = (uint32_t)d.dstride * kB;
    auto row_off = [&](int y) {  // bytes
        return (uint32_t)(y >> d.rshift) * bs + (uint32_t)(y & ((1 << d.rshift) - 1)) * pb;
    };

    T keep[M];
    R Fx[M], Fy[M];
    uint32_t node[M];
    bool lo[M], hi[M], dead[M];

    // One cell after its collision, rounded: after the last step to the other
    // buffer, before that to LDS.  The region streams in place (the AA
    // pattern): odd steps read a cell's own slots and write its value of slot
    // i into its slot opp(i); even steps read slot opp(i) of cell x - e_i and
    // write slot i of cell x + e_i.  A location is read and written by one cell
    // in a step, so a step needs no second copy, and cells follow one another
    // in any order.
    auto finish = [&](int m, int r, const R (&g)[9], int l, bool odd) {
        T rv[9];
        if constexpr (S::kDither) {
            const uint32_t h = hash32(__float_as_uint(g[0]) ^ (node[m] * 0x9e3779b9u));
#pragma unroll
            for (int i = 0; i < 9; ++i) rv[i] = S::from_r_sr(g[i], sr_operand(h, i));
        } else {
#pragma unroll
            for (int i = 0; i < 8; i += 2) round_pair<ST>(g[i], g[i + 1], &rv[i]);
            rv[8] = S::from_r(g[8]);
        }
        if (l < n) {
            keep[m] = rv[0];
            T *p = &lds[0][r][c];
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                const int own = (opp_of(i) - 1) * RH * RW;
                int o = odd ? own : (i - 1) * RH * RW + ey_of(i) * RW + ex_of(i);
                // Beyond a wall: reflected into the cell's own reversed slot.
                if (WALL && !odd && ((ey_of(i) == -1 && lo[m]) || (ey_of(i) == 1 && hi[m]))) o = own;
                p[o] = rv[i];
            }
        } else {
            uint32_t ro = row_off(y0 + r - H);
            uint32_t co = (uint32_t)(x0 + c - H) * kB;
            form_here<kU>(ro);
            form_here<false>(co);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                uint32_t o = co;
                T *p = row_base_at<kU>(out, (uint32_t)i * ds + ro, o);
                store_at(p, o, rv[i]);
            }
        }
    };
    // Whether step l is needed at region row r and this thread's column: the
    // tile and n - l nodes around it.
    auto needed = [&](int r, int l) {
        const int e = n - l;
        return r >= H - e && r < H + he + e && c >= H - e && c < H + we + e;
    };

    // Step 1, from the state.
#pragma unroll
    for (int m0 = 0; m0 < M; m0 += kStage) {
        R ga[kStage][9];
#pragma unroll
        for (int m = m0; m < m0 + kStage && m < M; ++m) {
            const int r = rt0 + m * RG::RPP;
            int y = y0 - H + r;
            dead[m] = false;
            if (WALL && d.bc_y) {
                dead[m] = y < 0 || y >= d.ny;
                y = y < 0 ? 0 : (y >= d.ny ? d.ny - 1 : y);
            } else {
                y = wrap_any(y, d.ny);
            }
            lo[m] = WALL && d.bc_y && y == 0;
            hi[m] = WALL && d.bc_y && y == d.ny - 1;
            node[m] = (uint32_t)y * (uint32_t)d.nx + (uint32_t)x;
            if (!needed(r, 1) || dead[m]) continue;
            force_at<R, FM>(d, x, y, Fx[m], Fy[m]);
            const uint32_t r0 = row_off(y);
            const uint32_t rm = row_off(y == 0 ? d.ny - 1 : y - 1);
            const uint32_t rp = row_off(y == d.ny - 1 ? 0 : y + 1);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                uint32_t ro = (uint32_t)i * ds + (ey_of(i) == 0 ? r0 : (ey_of(i) == 1 ? rm : rp));
                uint32_t o = ex_of(i) == 0 ? c0 : (ex_of(i) == 1 ? cm : cp);
                if (WALL && ((ey_of(i) == 1 && lo[m]) || (ey_of(i) == -1 && hi[m]))) {
                    ro = (uint32_t)opp_of(i) * ds + r0;
                    o = c0;
                }
                const T *p = row_base_at<kU>(in, ro, o);
                ga[m - m0][i] = S::to_r(load_at(p, o));
            }
        }
#pragma unroll
        for (int m = m0; m < m0 + kStage && m < M; ++m) {
            const int r = rt0 + m * RG::RPP;
            if (!needed(r, 1) || dead[m]) continue;
            collide<R, SCH>(ga[m - m0], Fx[m], Fy[m], rt);
            finish(m, r, ga[m - m0], 1, true);
        }
        if (m0 + kStage < M) __builtin_amdgcn_sched_barrier(0);
    }
    auto step = [&](int l, auto odd_) {
        constexpr bool odd = decltype(odd_)::value;
        __syncthreads();
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int r = rt0 + m * RG::RPP;
            if (!needed(r, l) || dead[m]) continue;
            R g[9];
            g[0] = S::to_r(keep[m]);
            const T *p = &lds[0][r][c];
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                const int own = (i - 1) * RH * RW;
                int o = odd ? own : (opp_of(i) - 1) * RH * RW - ey_of(i) * RW - ex_of(i);
                if (WALL && !odd && ((ey_of(i) == 1 && lo[m]) || (ey_of(i) == -1 && hi[m]))) o = own;
                g[i] = S::to_r(p[o]);
            }
            collide<R, SCH>(g, Fx[m], Fy[m], rt);
            finish(m, r, g, l, odd);
            if (m % kStage == kStage - 1 && m + 1 < M) __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int l = 2; l <= n; l += 2) {
        step(l, std::false_type{});
        if (l + 1 <= n) step(l + 1, std::true_type{});
    }
}

// The same with the Shan-Chen force (periodic lattices).  A step's force
// needs psi of the neighbours' densities of that step, which are pulled from
// their neighbours in turn: a step is needed on two nodes less at each side
// than the one before.  A step pulls its cells and writes their psi to LDS,
// and after a barrier takes the force from there, collides and writes the
// slots, one copy of which is enough.  The 200^2 FP64 droplet takes 2.4 us per
// step, 9.0 with a psi pass and a step kernel of one launch each; the chain of
// barriers bounds it.
template <int RW_, int RH_, int K_, int NT_>
struct ScRegion {
    static constexpr int RW = RW_, RH = RH_, K = K_, NT = NT_, H = 2 * K - 1;
    static constexpr int TW = RW - 2 * H, TH = RH - 2 * H;
    static constexpr int RPP = NT / RW, M = RH / RPP;
    static_assert(NT % RW == 0 && RH % RPP == 0, "whole rows per pass, whole passes");
};
template <int ST, typename RG>
struct ScLds {
    typename Storage<ST>::T v[8][RG::RH][RG::RW];
    typename Storage<ST>::R psi[RG::RH][RG::RW];
};

template <int ST, int SCH, typename RG>
__device__ __forceinline__ void sc_tile_steps(const LatDesc &d, int src, int x0, int y0, int n, ScLds<ST, RG> &lds)
{
    using S = Storage<ST>;
    using T = typename S::T;
    using R = typename S::R;
    constexpr int RW = RG::RW, RH = RG::RH, M = RG::M, H = RG::H;
    const T *in = static_cast<const T *>(d.buf[src]);
    T *out = static_cast<T *>(d.buf[src ^ 1]);
    const Rates<R> rt = rates_of<R>(d);
    constexpr bool kU = RW % 64 == 0;  // a wave's cells lie in one row
    const int c = threadIdx.x % RW;
    const int rt0 = kU ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / RW) : (int)threadIdx.x / RW;
    const int we = d.nx - x0 < RG::TW ? d.nx - x0 : RG::TW;
    const int he = d.ny - y0 < RG::TH ? d.ny - y0 : RG::TH;
    const int x = wrap_any(x0 - H + c, d.nx);
    constexpr uint32_t kB = sizeof(T);
    const uint32_t cm = (uint32_t)(x == 0 ? d.nx - 1 : x - 1) * kB, c0 = (uint32_t)x * kB,
                   cp = (uint32_t)(x == d.nx - 1 ? 0 : x + 1) * kB;
    const uint32_t bs = (uint32_t)d.bstride * kB, pb = (uint32_t)d.pitch * kB, ds = (uint32_t)d.dstride * kB;
    auto row_off = [&](int y) {  // bytes
        return (uint32_t)(y >> d.rshift) * bs + (uint32_t)(y & ((1 << d.rshift) - 1)) * pb;
    };
    // Cells within e nodes of the tile.
    auto near = [&](int r, int e) { return r >= H - e && r < H + he + e && c >= H - e && c < H + we + e; };

    T keep[M];
    uint32_t node[M];
    R g[M][9];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int r = rt0 + m * RG::RPP;
        const int y = wrap_any(y0 - H + r, d.ny);
        node[m] = (uint32_t)y * (uint32_t)d.nx + (uint32_t)x;
        if (!near(r, 2 * n - 1)) continue;
        const uint32_t r0 = row_off(y), rm = row_off(y == 0 ? d.ny - 1 : y - 1),
                       rp = row_off(y == d.ny - 1 ? 0 : y + 1);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            uint32_t o = ex_of(i) == 0 ? c0 : (ex_of(i) == 1 ? cm : cp);
            const T *p = row_base_at<kU>(in, (uint32_t)i * ds + (ey_of(i) == 0 ? r0 : (ey_of(i) == 1 ? rm : rp)), o);
            g[m][i] = S::to_r(load_at(p, o));
        }
    }
    for (int l = 1; l <= n; ++l) {
        const int e = 2 * (n - l);  // this step's collisions reach e nodes beyond the tile
        if (l > 1) {
            __syncthreads();
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const int r = rt0 + m * RG::RPP;
                if (!near(r, e + 1)) continue;
                g[m][0] = S::to_r(keep[m]);
                const T *p = &lds.v[0][r][c];
#pragma unroll
                for (int i = 1; i < 9; ++i) g[m][i] = S::to_r(p[(i - 1) * RH * RW - ey_of(i) * RW - ex_of(i)]);
            }
        }
        // psi of the density, as the psi pass forms it.
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int r = rt0 + m * RG::RPP;
            if (!near(r, e + 1)) continue;
            double dr = 0.0;
#pragma unroll
            for (int i = 0; i < 9; ++i) dr += (double)g[m][i];
            lds.psi[r][c] = R(shan_chen_psi(d, d.rho0 + dr));
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int r = rt0 + m * RG::RPP;
            if (!near(r, e)) continue;
            R Fx, Fy;
            const R *q = &lds.psi[r][c];
            shan_chen_force<R>(d, q, q - 1, q + 1, q - RW, q - RW - 1, q - RW + 1, q + RW, q + RW - 1, q + RW + 1, Fx,
                               Fy);
            collide<R, SCH>(g[m], Fx, Fy, rt);
            T rv[9];
            if constexpr (S::kDither) {
                const uint32_t h = hash32(__float_as_uint(g[m][0]) ^ (node[m] * 0x9e3779b9u));
#pragma unroll
                for (int i = 0; i < 9; ++i) rv[i] = S::from_r_sr(g[m][i], sr_operand(h, i));
            } else {
#pragma unroll
                for (int i = 0; i < 8; i += 2) round_pair<ST>(g[m][i], g[m][i + 1], &rv[i]);
                rv[8] = S::from_r(g[m][8]);
            }
            if (l < n) {
                keep[m] = rv[0];
#pragma unroll
                for (int i = 1; i < 9; ++i) lds.v[i - 1][r][c] = rv[i];
            } else {
                uint32_t ro = row_off(y0 + r - H);
                uint32_t co = (uint32_t)(x0 + c - H) * kB;
                form_here<kU>(ro);
                form_here<false>(co);
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    uint32_t o = co;
                    T *p = row_base_at<kU>(out, (uint32_t)i * ds + ro, o);
                    store_at(p, o, rv[i]);
                }
            }
        }
    }
}

template <int ST, int SCH, typename RG>
__global__ __launch_bounds__(RG::NT) void k_sc_tile(LatDesc d, int src, int n, int tiles_x)
{
    __shared__ ScLds<ST, RG> lds;
    const int t = (int)xcd_order(blockIdx.x, gridDim.x);
    const int ty = t / tiles_x, tx = t - ty * tiles_x;
    sc_tile_steps<ST, SCH, RG>(d, src, tx * RG::TW, ty * RG::TH, n, lds);
}

template <int ST, typename RG>
using TileLds = typename Storage<ST>::T[8][RG::RH][RG::RW];

template <int ST, int FM, int SCH, typename RG, bool WALL>
__global__ __launch_bounds__(RG::NT) __attribute__((amdgpu_waves_per_eu(RG::WV))) void
k_tile(LatDesc d, int src, int n, int tiles_x)
{
    __shared__ TileLds<ST, RG> lds;
    const int t = (int)xcd_order(blockIdx.x, gridDim.x);
    const int ty = t / tiles_x, tx = t - ty * tiles_x;
    tile_steps<ST, FM, SCH, RG, WALL>(d, src, tx * RG::TW, ty * RG::TH, n, lds);
}

// Substep `sub` of a batch group: one block per tile (tiles numbered lattice
// by lattice, tile_lat naming each tile's lattice).  The buffer parity of a
// lattice counts launches.
template <int ST, int FM, int SCH, typename RG, bool WALL>
__global__ __launch_bounds__(RG::NT) __attribute__((amdgpu_waves_per_eu(RG::WV))) void
k_batch_tile(const LatDesc *__restrict__ lats, const int32_t *__restrict__ tile_lat, int64_t ntiles, int sub)
{
    __shared__ TileLds<ST, RG> lds;
    const int64_t t = xcd_order(blockIdx.x, ntiles);
    const LatDesc &d = lats[tile_lat[t]];
    const int left = d.steps - RG::K * sub;
    if (left <= 0) return;  // the whole block: one lattice per tile
    int tx, ty;
    strip_tile((int)(t - d.tile0), d.walk, tx, ty);
    tile_steps<ST, FM, SCH, RG, WALL>(d, (d.parity + sub) & 1, tx * RG::TW, ty * RG::TH, left < RG::K ? left : RG::K,
                                      lds);
}

// The regions by shape.
template <int ST, int SHAPE>
using RegionOf = std::conditional_t<
    SHAPE == kRegion32x24, Region<32, 24, 8, 768>,
    std::conditional_t<
        SHAPE == kRegion32x32, Region<32, 32, 8, 1024>,
        std::conditional_t<SHAPE == kRegion64x16, Region<64, 16, 4, 512>,
                           std::conditional_t<SHAPE == kRegion32x16, Region<32, 16, 4, 512>,
                                              std::conditional_t<SHAPE == kRegion64x32, Region<64, 32, 4, 512>,
                                                                 Region<64, 48, 4, 512>>>>>>;

}  // namespace

// n <= p.steps fused steps of one lattice from buffer src into buffer
// src ^ 1.
template <int ST, int SHAPE>
hipError_t tile_shape_launch(const LatDesc &d, int src, int n, const TilePlan &p, hipStream_t s)
{
    using RG = RegionOf<ST, SHAPE>;
    static_assert(RG::RW == region_w(SHAPE) && RG::RH == region_h(SHAPE) && RG::K == region_steps(SHAPE), "shape");
    const dim3 grid((unsigned)p.tiles);
    switch ((d.force_mode * 2 + d.scheme) * 2 + (d.bc_y ? 1 : 0)) {
#define CLBM_TL(FM, SCH, WALL)                                                            \
    case (FM * 2 + SCH) * 2 + WALL:                                                       \
        k_tile<ST, FM, SCH, RG, WALL><<<grid, RG::NT, 0, s>>>(d, src, n, p.tiles_x);      \
        break;
#define CLBM_TL2(FM, SCH) CLBM_TL(FM, SCH, 0) CLBM_TL(FM, SCH, 1)
        CLBM_TL2(FM_CONST, SCH_CONSISTENT)
        CLBM_TL2(FM_CONST, SCH_GUO_LBL)
        CLBM_TL2(FM_ROW, SCH_CONSISTENT)
        CLBM_TL2(FM_ROW, SCH_GUO_LBL)
        CLBM_TL2(FM_FIELD, SCH_CONSISTENT)
        CLBM_TL2(FM_FIELD, SCH_GUO_LBL)
#undef CLBM_TL2
#undef CLBM_TL
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int ST, typename RG>
hipError_t sc_tile_launch(const LatDesc &d, int src, int n, const TilePlan &p, hipStream_t s)
{
    const dim3 grid((unsigned)p.tiles);
    if (d.scheme == SCH_CONSISTENT)
        k_sc_tile<ST, SCH_CONSISTENT, RG><<<grid, RG::NT, 0, s>>>(d, src, n, p.tiles_x);
    else
        k_sc_tile<ST, SCH_GUO_LBL, RG><<<grid, RG::NT, 0, s>>>(d, src, n, p.tiles_x);
    return hipGetLastError();
}

template <int ST>
hipError_t launch_tile_st(const LatDesc &d, int src, int n, const TilePlan &p, hipStream_t s)
{
    switch (p.shape) {
    case kRegionSc32x24: return sc_tile_launch<ST, ScRegion<32, 24, 4, 768>>(d, src, n, p, s);
    case kRegionSc64x32: return sc_tile_launch<ST, ScRegion<64, 32, 2, 1024>>(d, src, n, p, s);
    case kRegion32x24: return tile_shape_launch<ST, kRegion32x24>(d, src, n, p, s);
    case kRegion32x32: return tile_shape_launch<ST, kRegion32x32>(d, src, n, p, s);
    case kRegion64x16: return tile_shape_launch<ST, kRegion64x16>(d, src, n, p, s);
    case kRegion32x16: return tile_shape_launch<ST, kRegion32x16>(d, src, n, p, s);
    case kRegion64x32: return tile_shape_launch<ST, kRegion64x32>(d, src, n, p, s);
    default:
        if constexpr (region_compiled(kRegion64x48, ST)) {
            if (p.shape == kRegion64x48) return tile_shape_launch<ST, kRegion64x48>(d, src, n, p, s);
        }
        return hipErrorInvalidValue;
    }
}

template <int ST, int SHAPE>
hipError_t batch_tile_shape_launch(const LatDesc *lats, const int32_t *tile_lat, int64_t ntiles, int key, bool walls,
                                   int sub, hipStream_t s)
{
    using RG = RegionOf<ST, SHAPE>;
    const dim3 grid((unsigned)ntiles);
    switch (key * 2 + (walls ? 1 : 0)) {
#define CLBM_TL(FM, SCH, WALL)                                                                             \
    case (FM * 2 + SCH) * 2 + WALL:                                                                        \
        k_batch_tile<ST, FM, SCH, RG, WALL><<<grid, RG::NT, 0, s>>>(lats, tile_lat, ntiles, sub);          \
        break;
#define CLBM_TL2(FM, SCH) CLBM_TL(FM, SCH, 0) CLBM_TL(FM, SCH, 1)
        CLBM_TL2(FM_CONST, SCH_CONSISTENT)
        CLBM_TL2(FM_CONST, SCH_GUO_LBL)
        CLBM_TL2(FM_ROW, SCH_CONSISTENT)
        CLBM_TL2(FM_ROW, SCH_GUO_LBL)
        CLBM_TL2(FM_FIELD, SCH_CONSISTENT)
        CLBM_TL2(FM_FIELD, SCH_GUO_LBL)
#undef CLBM_TL2
#undef CLBM_TL
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int ST>
hipError_t launch_batch_tile_st(const LatDesc *lats, const int32_t *tile_lat, int64_t ntiles, int key, bool walls,
                                int shape, int sub, hipStream_t s)
{
    switch (shape) {
    case kRegion32x24: return batch_tile_shape_launch<ST, kRegion32x24>(lats, tile_lat, ntiles, key, walls, sub, s);
    case kRegion32x32: return batch_tile_shape_launch<ST, kRegion32x32>(lats, tile_lat, ntiles, key, walls, sub, s);
    case kRegion64x16: return batch_tile_shape_launch<ST, kRegion64x16>(lats, tile_lat, ntiles, key, walls, sub, s);
    case kRegion32x16: return batch_tile_shape_launch<ST, kRegion32x16>(lats, tile_lat, ntiles, key, walls, sub, s);
    case kRegion64x32: return batch_tile_shape_launch<ST, kRegion64x32>(lats, tile_lat, ntiles, key, walls, sub, s);
    default:
        if constexpr (region_compiled(kRegion64x48, ST)) {
            if (shape == kRegion64x48)
                return batch_tile_shape_launch<ST, kRegion64x48>(lats, tile_lat, ntiles, key, walls, sub, s);
        }
        return hipErrorInvalidValue;
    }
}

}  // namespace clbm

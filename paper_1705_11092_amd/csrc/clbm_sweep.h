// clbm_sweep.h -- K fused steps per launch in registers (two-buffer, pull
// form).  Included by the translation units of the storage types, after
// clbm_step.h.
//
// A wave takes a strip of the lattice, 64 lanes of V consecutive columns,
// and marches down its rows.  In one iteration it collides one row of each
// of K time levels: level 1 (step n + 1) at row y, read from HBM, level 2 at
// row y - 1, ... level K at row y - K + 1, written to HBM.  A node of level
// l + 1 pulls (Eq. 10) from rows r - 1, r and r + 1 of level l: of these the
// row r + 1 was collided a moment ago by the same lanes, and of the other
// two only the slots still to be pulled are kept, 9 values per node and
// level, in registers.  Slots with e_x != 0 come from a neighbouring column:
// a register of the same lane, or, for the lane's first or last column, the
// neighbouring lane's, brought over by a wave shift (DPP).  There is no LDS,
// no barrier, and no wave depends on another.
//
// The strip's outer columns lose their neighbours, one column per level and
// side, so the outer `halo` lanes are only collided, not stored; likewise
// the rows above and below a wave's rows are collided again by the waves
// that own them.  Every node update is the one-step kernel's arithmetic on
// the same values, rounded to the storage type between the levels, so the
// result is bitwise that of K one-step launches.
//
// What bounds it: VALU issue in FP32 (4096^2: 148 instructions per update with
// the halo, 92 to 95 % of issue at the clock the chip holds, 2.16 to 2.19 GHz from
// card to card, 73 to 77 us per step against 106 in pairs); in FP64 its longer
// instructions and the latency of two waves per SIMD (122 to 133 against 197 us).
// Four levels: a fifth or sixth lost more to halo and registers than the state's
// traffic gives back.
#pragma once

#include <type_traits>

#include "clbm_step.h"

namespace clbm {
namespace {

// The value of the lane below (from_left) or above (from_right) in the wave
// (zero beyond its ends, in lanes whose result is not used).
template <typename R, int CTRL>
__device__ __forceinline__ R wave_shift(R v)
{
    if constexpr (sizeof(R) == 8) {
        int b[2];
        __builtin_memcpy(b, &v, 8);
        b[0] = __builtin_amdgcn_update_dpp(0, b[0], CTRL, 0xf, 0xf, true);
        b[1] = __builtin_amdgcn_update_dpp(0, b[1], CTRL, 0xf, 0xf, true);
        __builtin_memcpy(&v, b, 8);
    } else {
        int b;
        __builtin_memcpy(&b, &v, 4);
        b = __builtin_amdgcn_update_dpp(0, b, CTRL, 0xf, 0xf, true);
        __builtin_memcpy(&v, &b, 4);
    }
    return v;
}
template <typename R>
__device__ __forceinline__ R from_left(R v) { return wave_shift<R, 0x138>(v); }   // wave_shr:1
template <typename R>
__device__ __forceinline__ R from_right(R v) { return wave_shift<R, 0x130>(v); }  // wave_shl:1

// The seam of a row whose length is not a multiple of V: the last group has
// only r real columns, and column 0 follows its column r - 1.
struct Seam {
    int r;  // in the lane that holds the row's last group: its real columns
            // (less than V); otherwise 0
};

// Column by column the values of the column to the left (x - 1) or right
// (x + 1) of v.
template <bool SEAM, int V, typename R>
__device__ __forceinline__ void shift_right(const R (&v)[V], R (&o)[V], const Seam &s)
{
    R last = v[V - 1];
    if constexpr (SEAM) {
#pragma unroll
        for (int k = 0; k + 1 < V; ++k)
            if (s.r == k + 1) last = v[k];
    }
    o[0] = from_left(last);
#pragma unroll
    for (int k = 1; k < V; ++k) o[k] = v[k - 1];
}
template <bool SEAM, int V, typename R>
__device__ __forceinline__ void shift_left(const R (&v)[V], R (&o)[V], const Seam &s)
{
    const R next = from_right(v[0]);
#pragma unroll
    for (int k = 0; k + 1 < V; ++k) {
        o[k] = v[k + 1];
        if constexpr (SEAM) {
            if (s.r == k + 1) o[k] = next;
        }
    }
    o[V - 1] = next;
}
template <bool SEAM, int E, int V, typename R>
__device__ __forceinline__ void shift_x(const R (&v)[V], R (&o)[V], const Seam &s)
{
    if constexpr (E == 1)
        shift_right<SEAM, V, R>(v, o, s);
    else if constexpr (E == -1)
        shift_left<SEAM, V, R>(v, o, s);
    else {
#pragma unroll
        for (int k = 0; k < V; ++k) o[k] = v[k];
    }
}

// V nodes' values in the storage type, as the one-step kernel stores them.
template <int ST, int V>
__device__ __forceinline__ void round_nodes(const typename Storage<ST>::R (&g)[9][V], uint32_t node,
                                            Pack<typename Storage<ST>::T, V> (&q)[9])
{
    using S = Storage<ST>;
    if constexpr (S::kDither) {
        uint32_t h[V];
#pragma unroll
        for (int k = 0; k < V; ++k) h[k] = hash32(__float_as_uint(g[0][k]) ^ ((node + (uint32_t)k) * 0x9e3779b9u));
#pragma unroll
        for (int i = 0; i < 9; ++i) {
#pragma unroll
            for (int k = 0; k + 1 < V; k += 2) {
                const auto two = S::from_r_sr2(g[i][k], sr_operand(h[k], i), g[i][k + 1], sr_operand(h[k + 1], i));
                q[i].v[k] = two[0];
                q[i].v[k + 1] = two[1];
            }
            if constexpr (V % 2) q[i].v[V - 1] = S::from_r_sr(g[i][V - 1], sr_operand(h[V - 1], i));
        }
    } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
#pragma unroll
            for (int k = 0; k + 1 < V; k += 2) round_pair<ST>(g[i][k], g[i][k + 1], &q[i].v[k]);
            if constexpr (V % 2) q[i].v[V - 1] = S::from_r(g[i][V - 1]);
        }
    }
}

// What a level keeps of the row it collided last (mid, up1) and of the one
// before (up0) for the next level to pull: slots 0, 1, 3 and 2, 5, 6, already
// moved to the columns that pull them.
template <typename R, int V>
struct Held {
    R mid[3][V], up0[3][V], up1[3][V];
};

template <int ST, int FM, int SCH, int K, int V, bool WALL, bool SEAM>
__device__ __forceinline__ void sweep_strip(const LatDesc &d, int src, int base, bool store, int ya, int yb,
                                            const Seam &seam)
{
    using S = Storage<ST>;
    using T = typename S::T;
    using R = typename S::R;
    const T *in = static_cast<const T *>(d.buf[src]);
    T *out = static_cast<T *>(d.buf[src ^ 1]);
    const Rates<R> rt = rates_of<R>(d);
    const uint32_t off = (uint32_t)base * (uint32_t)sizeof(T);

    Held<R, V> h[K];
#pragma unroll
    for (int l = 0; l < K; ++l)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < V; ++k) h[l].mid[j][k] = h[l].up0[j][k] = h[l].up1[j][k] = R(0);

    // The state of step n that row y pulls, one aligned vector per slot.
    typedef T Row __attribute__((ext_vector_type(V)));
    Row raw[9];
    auto load_row = [&](int y) {
        const bool lo = WALL && y == 0, hi = WALL && y == d.ny - 1;
        const int64_t r0 = row_base(d, y);
        const int64_t rm = row_base(d, y == 0 ? d.ny - 1 : y - 1);
        const int64_t rp = row_base(d, y == d.ny - 1 ? 0 : y + 1);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            int64_t o = (int64_t)i * d.dstride + (ey_of(i) == 0 ? r0 : (ey_of(i) == 1 ? rm : rp));
            if (WALL && ey_of(i) == 1) o = lo ? (int64_t)opp_of(i) * d.dstride + r0 : o;
            if (WALL && ey_of(i) == -1) o = hi ? (int64_t)opp_of(i) * d.dstride + r0 : o;
            const char *p = reinterpret_cast<const char *>(in + o);
            raw[i] = *reinterpret_cast<const Row *>(p + (uint64_t)off);
        }
    };
    auto wrap = [&](int y) { return y < 0 ? y + d.ny : (y >= d.ny ? y - d.ny : y); };
    // The body force of row y (any row of the march: beyond a wall the
    // wall's, not used).  Memory waits are in issue order, so the forces of
    // levels 2 .. K of an iteration are loaded ahead of the next row's state,
    // and level 1's with that state; a row's force is the same for the whole
    // wave and comes by scalar loads.
    R F[K][2][V];
    auto load_force = [&](int l, int y) {
        if constexpr (FM == FM_CONST) {
#pragma unroll
            for (int k = 0; k < V; ++k) {
                F[l][0][k] = R(d.Fx);
                F[l][1][k] = R(d.Fy);
            }
        } else {
            y = WALL ? (y < 0 ? 0 : (y >= d.ny ? d.ny - 1 : y)) : wrap(y);
            if constexpr (FM == FM_ROW) {
                typedef const __attribute__((address_space(4))) R *Table;
                const R f = reinterpret_cast<Table>(reinterpret_cast<uint64_t>(d.force))[y];
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    F[l][0][k] = f;
                    F[l][1][k] = R(0);
                }
            } else if constexpr (SEAM) {
#pragma unroll
                for (int k = 0; k < V; ++k)
                    force_at<R, FM>(d, base + k < d.nx ? base + k : d.nx - 1, y, F[l][0][k], F[l][1][k]);
            } else {
                const R *f = static_cast<const R *>(d.force) + (int64_t)y * d.nx;
                const Pack<R, V> a = load_pack<R, V, false>(f + (uint32_t)base);
                const Pack<R, V> b = load_pack<R, V, false>(f + (int64_t)d.nx * d.ny + (uint32_t)base);
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    F[l][0][k] = a.v[k];
                    F[l][1][k] = b.v[k];
                }
            }
        }
    };

    const int first = ya - (K - 1), iters = (yb - ya) + 2 * K - 2;
    load_force(0, first);
    if (!WALL || first >= 0) load_row(WALL ? first : wrap(first));
    // Iteration t of the march.  STEADY: every level has its rows, none of
    // them next to a wall, and there is a next row to load; without the
    // conditions the levels schedule into one another and their values stay in
    // place.
    auto iterate = [&](int t, auto steady_) {
        constexpr bool STEADY = decltype(steady_)::value, EDGE = WALL && !STEADY;
        const int y1 = first + t;  // level 1's row
        R p[9][V];                 // the last collided level's row
        auto update = [&](int y, R (&g)[9][V], const R (&f)[2][V], bool last) {
            // The collision and the rounding of row y.
#pragma unroll
            for (int k = 0; k < V; ++k) {
                R n[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) n[i] = g[i][k];
                collide<R, SCH>(n, f[0][k], f[1][k], rt);
#pragma unroll
                for (int i = 0; i < 9; ++i) g[i][k] = n[i];
            }
            Pack<T, V> s[9];
            round_nodes<ST, V>(g, (uint32_t)y * (uint32_t)d.nx + (uint32_t)base, s);
            if (last) {
                if constexpr (SEAM) {
#pragma unroll
                    for (int i = 0; i < 9; ++i)
#pragma unroll
                        for (int k = 1; k < V; ++k)
                            if (base + k >= d.nx) s[i].v[k] = s[i].v[k - 1];
                }
                if (store) {
                    const int64_t r0 = row_base(d, y);
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        char *o = reinterpret_cast<char *>(out + (int64_t)i * d.dstride + r0);
                        store_pack<T, V, true>(reinterpret_cast<T *>(o + (uint64_t)off), s[i]);
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < 9; ++i)
#pragma unroll
                    for (int k = 0; k < V; ++k) p[i][k] = S::to_r(s[i].v[k]);
            }
        };

#pragma unroll
        for (int l = 1; l < K; ++l) load_force(l, y1 - l);
        const bool on1 = !EDGE || (y1 >= 0 && y1 < d.ny);
        if (on1) {
            const int y = WALL ? y1 : wrap(y1);
            R g[9][V];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                R v[V];
#pragma unroll
                for (int k = 0; k < V; ++k) v[k] = S::to_r(raw[i][k]);
                if (ex_of(i) == 1)
                    shift_x<SEAM, 1, V, R>(v, g[i], seam);
                else if (ex_of(i) == -1)
                    shift_x<SEAM, -1, V, R>(v, g[i], seam);
                else
                    shift_x<SEAM, 0, V, R>(v, g[i], seam);
                if (EDGE && ((ey_of(i) == 1 && y == 0) || (ey_of(i) == -1 && y == d.ny - 1))) {
#pragma unroll
                    for (int k = 0; k < V; ++k) g[i][k] = v[k];
                }
            }
            update(y, g, F[0], K == 1);
        }
        // The next row's loads, in flight while the other levels collide.
        if (STEADY || t + 1 < iters) {
            const int yn = y1 + 1;
            load_force(0, yn);
            if (!WALL || (yn >= 0 && yn < d.ny)) load_row(WALL ? yn : wrap(yn));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int l = 1; l < K; ++l) {
            // Level l + 1 at row yl from level l, whose row yl + 1 is in p.
            const int yl = y1 - l;
            const bool have = STEADY || (t >= 2 * (l - 1) && (!WALL || (yl + 1 >= 0 && yl + 1 < d.ny)));
            const bool go = STEADY || (t >= 2 * l && (!WALL || (yl >= 0 && yl < d.ny)));
            Held<R, V> &c = h[l];
            R g[9][V];
#pragma unroll
            for (int k = 0; k < V; ++k) {
                g[2][k] = c.up0[0][k];
                g[5][k] = c.up0[1][k];
                g[6][k] = c.up0[2][k];
                g[0][k] = c.mid[0][k];
                g[1][k] = c.mid[1][k];
                g[3][k] = c.mid[2][k];
                if (EDGE) {
                    // The row beyond the upper wall: the node's own reversed
                    // slots, kept unshifted in up1.
                    g[4][k] = c.up1[0][k];
                    g[7][k] = c.up1[1][k];
                    g[8][k] = c.up1[2][k];
                }
            }
            if (have) {
#pragma unroll
                for (int k = 0; k < V; ++k) g[4][k] = p[4][k];
                shift_x<SEAM, -1, V, R>(p[7], g[7], seam);
                shift_x<SEAM, 1, V, R>(p[8], g[8], seam);
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int k = 0; k < V; ++k) c.up0[j][k] = c.up1[j][k];
#pragma unroll
                for (int k = 0; k < V; ++k) c.mid[0][k] = p[0][k];
                shift_x<SEAM, 1, V, R>(p[1], c.mid[1], seam);
                shift_x<SEAM, -1, V, R>(p[3], c.mid[2], seam);
#pragma unroll
                for (int k = 0; k < V; ++k) c.up1[0][k] = p[2][k];
                shift_x<SEAM, 1, V, R>(p[5], c.up1[1], seam);
                shift_x<SEAM, -1, V, R>(p[6], c.up1[2], seam);
                if (EDGE && yl + 1 == 0) {
#pragma unroll
                    for (int k = 0; k < V; ++k) {
                        c.up0[0][k] = p[4][k];
                        c.up0[1][k] = p[7][k];
                        c.up0[2][k] = p[8][k];
                    }
                }
                if (EDGE && yl + 1 == d.ny - 1) {
#pragma unroll
                    for (int k = 0; k < V; ++k) {
                        c.up1[0][k] = p[2][k];
                        c.up1[1][k] = p[5][k];
                        c.up1[2][k] = p[6][k];
                    }
                }
            }
            if (go) update(WALL ? yl : wrap(yl), g, F[l], l == K - 1);
        }
    };
    int t = 0;
    if constexpr (sizeof(R) == 4) {
        // The steady part: after every level has started, and with walls
        // while level 1 stays below the upper one and level K above the lower
        // one.  129 VALU instructions per update collided (1030 for the 8 of an
        // iteration with two columns) against 135 (66 of the 1080 moves) with the
        // conditions, 201 VGPRs against 171.  In FP64 it would spill 450 registers.
        int t1 = 2 * (K - 1), t2 = iters - 1;
        if (WALL) {
            t1 = t1 > K - first ? t1 : K - first;
            t2 = t2 < d.ny - 2 - first ? t2 : d.ny - 2 - first;
        }
        for (; t < t1 && t < iters; ++t) iterate(t, std::false_type{});
        for (; t < t2; ++t) iterate(t, std::true_type{});
    }
    for (; t < iters; ++t) iterate(t, std::false_type{});
}

// Waves per SIMD the compiler must leave room for: 2 with two columns per
// lane (FP32 182-210 VGPRs; FP64 256), 3 with one (FP32 94-128, FP64 141-166),
// but 2 in FP64 with a per-node force (157-176), which would spill.
template <int ST, int FM, int V>
constexpr int sweep_waves() { return V == 1 && !(ST == ST_F64 && FM == FM_FIELD) ? 3 : 2; }

template <int ST, int FM, int SCH, int K, int V, bool WALL>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sweep_waves<ST, FM, V>()))) void
k_sweep(LatDesc d, int src, SweepPlan p)
{
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int u = (int)xcd_order(blockIdx.x, gridDim.x) * (kBlock / 64) + w;
    if (u >= p.units) return;
    const int chunk = u / p.strips, strip = u - chunk * p.strips;
    const int lane = threadIdx.x & 63;
    const int ya = chunk * p.rows, yb = ya + p.rows < d.ny ? ya + p.rows : d.ny;
    const int q = strip * (64 - 2 * p.halo) + lane - p.halo;  // group, counted around the periodic row
    const bool store = lane >= p.halo && lane < 64 - p.halo && q < p.groups;
    int qw = q < 0 ? q + p.groups : q;
    if (qw >= p.groups) qw %= p.groups;
    const int r = d.nx - (p.groups - 1) * V;
    const Seam seam{qw == p.groups - 1 && r != V ? r : 0};
    if (__any(seam.r))
        sweep_strip<ST, FM, SCH, K, V, WALL, true>(d, src, qw * V, store, ya, yb, seam);
    else
        sweep_strip<ST, FM, SCH, K, V, WALL, false>(d, src, qw * V, store, ya, yb, seam);
}

}  // namespace

// Four fused steps of one lattice from buffer src into buffer src ^ 1, under
// the plan sweep_plan made for it.
template <int ST>
hipError_t launch_sweep_st(const LatDesc &d, int src, const SweepPlan &p, hipStream_t s)
{
    const dim3 grid((unsigned)((p.units + kBlock / 64 - 1) / (kBlock / 64))), block(kBlock);
    switch ((d.force_mode * 2 + d.scheme) * 2 + (d.bc_y ? 1 : 0)) {
#define CLBM_SW(FM, SCH, WALL)                                                    \
    case (FM * 2 + SCH) * 2 + WALL:                                               \
        if constexpr (sweep_max_vec(ST, FM, WALL) == 2) {                         \
            if (p.vec == 2) {                                                     \
                k_sweep<ST, FM, SCH, kSweepSteps, 2, WALL><<<grid, block, 0, s>>>(d, src, p); \
                break;                                                            \
            }                                                                     \
        }                                                                         \
        if (p.vec != 1) return hipErrorInvalidValue;                              \
        k_sweep<ST, FM, SCH, kSweepSteps, 1, WALL><<<grid, block, 0, s>>>(d, src, p); \
        break;
#define CLBM_SW2(FM, SCH) CLBM_SW(FM, SCH, 0) CLBM_SW(FM, SCH, 1)
        CLBM_SW2(FM_CONST, SCH_CONSISTENT)
        CLBM_SW2(FM_CONST, SCH_GUO_LBL)
        CLBM_SW2(FM_ROW, SCH_CONSISTENT)
        CLBM_SW2(FM_ROW, SCH_GUO_LBL)
        CLBM_SW2(FM_FIELD, SCH_CONSISTENT)
        CLBM_SW2(FM_FIELD, SCH_GUO_LBL)
#undef CLBM_SW2
#undef CLBM_SW
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace clbm

// Two-dimensional extension of the scheme: u_t = u_xx + u_yy on the unit
// square.  The paper states that the group explicit method extends to two
// dimensions without giving formulas; here every level m applies the
// one-dimensional level m of Section 2 (two-point groups, Eq. (3)/(4), a
// point alone beside a wall by Eq. (1)/(2)) along every row with
// r_x = tau/h_x^2, then along every column with r_y = tau/h_y^2 (first-order
// splitting; each line is paired by the level's global index exactly as a
// single rod is).  Walls are constant in time.
//
// Each direction is taken as ge_level.h takes a rod: in FP64 in two stages, an
// explicit one over the other parity's pairs, then the 2x2 solve of its own, 3
// instructions a point; in FP32 as an increment from second differences, 5
// instructions and one rounding of u.  (FP32 in two stages was faster,
// 4096 x 4096 points 0.49 ms for 96 levels, but its error against 64 bits was
// 1.4 times this form's at the median over 40 grids: 1.8e-7 against 1.3e-7.)
//
// A workgroup of 8 waves holds a window of 128 columns by 8 R rows in
// registers: lane l of a wave columns 2l and 2l + 1 of its R rows.  A level's
// x part takes its neighbours by DPP moves; its y part works on the lane's own
// rows, and the rows at a wave's ends meet their neighbours in LDS, one row
// each way and one barrier a level.  The halo of D + 1 points a side (the
// invalid region entering from an open edge grows by one point per level after
// the first, in each direction by itself) is shared by 8 R rows, so a launch
// can fuse many levels, and two or more workgroups are resident per compute
// unit, one loading or storing while another computes.
//
// A window that would reach past a wall is moved to end there, so a wall is
// the fill of a first or last lane or the neighbour row of a first or last
// wave, with cs for k; a window that starts at an odd column or row pairs that
// direction the other way round.  Only a grid smaller than a window has wall
// nodes inside one: those lanes and rows are set to the wall's value at each
// stage.  Every point gets the same operations whatever the window, its rows
// and the levels per launch, so none of them changes a bit.
//
// Measured, 96 levels: 4096 x 4096 points FP64 0.98 ms (1.76 when a wave held
// its tile alone, two columns by 36 rows a lane and four levels per launch),
// FP32 0.68 (1.07); 196 x 578 FP64 71 us (416), FP32 71 (349).  VALU issue (6 instructions a
// point and level, 11 lane moves to 16 of them) and the halo's recompute bind
// large grids, one window's level latency small ones.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "ge_2d.h"
#include "ge_kernels.h"
#include "ge_level.h"

namespace ge {
namespace {

using dev::Par;
using dev::for_levels;
using dev::kWave;

constexpr int kCols = 2 * kWave;      // columns of a window
constexpr int kNW = 8;                // waves of a window

template <typename T> struct Dir {    // one direction's constants (Coef, ge_level.h)
    T r, k, c1, c2, cs;
};

template <typename T> struct Block2dArgs {
    const T *in;
    T *out;
    int nx, ny, tx, ntiles;           // tiles per row of tiles, tiles
    int cx, cy, halo, nlev;           // core columns and rows, halo, levels
    int64_t level0;
    Dir<T> x, y;
    T gw, ge, gs, gn;
};

// Two columns: in LDS, and in memory (any element's alignment).
template <typename T> struct Pair2;
template <> struct Pair2<float> {
    typedef float type __attribute__((ext_vector_type(2)));
    typedef float mem __attribute__((ext_vector_type(2), aligned(4)));
};
template <> struct Pair2<double> {
    typedef double type __attribute__((ext_vector_type(2)));
    typedef double mem __attribute__((ext_vector_type(2), aligned(8)));
};

// What a window holds of the walls: kOpen no x wall, kEnds an x wall at its
// first or last column; a y wall at its first or last row costs nothing and
// is not told apart.  kInside: the grid ends inside the window.
enum Walls2d : int { kOpen, kEnds, kInside };

// FP64 meets its neighbours with one row a side, FP32 with two.
template <typename T> constexpr bool kTwoStage = sizeof(T) == 8;
template <typename T> constexpr int kEdge = kTwoStage<T> ? 1 : 2;
template <typename T> constexpr int kRowsAtOnce = 4;

// The factors of a point: of the solve's difference (FP64: f), or of its own
// second difference and of its partner's (FP32: f, g).
template <typename T> struct Factor {
    T f, g;
};
template <typename T> __device__ __forceinline__ Factor<T> paired(const Dir<T> &c)
{
    if constexpr (kTwoStage<T>) return Factor<T>{c.k, T(0)};
    else return Factor<T>{c.c1, c.c2};
}
template <typename T> __device__ __forceinline__ Factor<T> alone(const Dir<T> &c)
{
    return Factor<T>{c.cs, T(0)};
}
template <typename T> __device__ __forceinline__ Factor<T> pick(bool is_alone, const Dir<T> &c)
{
    const Factor<T> p = paired(c), l = alone(c);
    return Factor<T>{is_alone ? l.f : p.f, is_alone ? l.g : p.g};
}
// FP32: a point's new value
// (rounded before it is added, see ge_level.h)
template <typename T> __device__ __forceinline__ T step(T u, T D, T Dq, Factor<T> k)
{
    return u + dev::fmaT(k.g, Dq, k.f * D);
}

// One lane's view of the x walls.
template <typename T> struct XWalls {
    T gw, ge;              // their values
    Factor<T> l, r;        // P = 1: the factors of the lane's first / last column
    Factor<T> in;          // P = 0: those of its first column
    bool a_wall, b_wall;   // kInside: the column is the east wall's node or past it
};

// The x part of one row.
template <typename T, int P, int KIND>
__device__ __forceinline__ void x_part(T &a, T &b, const XWalls<T> &x, const Dir<T> &c)
{
    using dev::fmaT;
    constexpr bool OPEN = KIND == kOpen;
    auto set_wall = [&](T &p, T &q) {
        if constexpr (KIND == kInside) {
            p = x.a_wall ? x.ge : p;
            q = x.b_wall ? x.ge : q;
        }
    };
    const Factor<T> in = KIND == kInside ? x.in : paired(c), pr = paired(c);
    set_wall(a, b);
    if constexpr (kTwoStage<T>) {
        T va, vb;
        if constexpr (P == 0) {
            va = fmaT(-c.r, a - dev::edge_left<OPEN>(x.gw, b), a);
            vb = fmaT(c.r, dev::edge_right<OPEN>(x.ge, a) - b, b);
            set_wall(va, vb);
            const T w = vb - va;
            a = fmaT(in.f, w, va);
            b = fmaT(-pr.f, w, vb);
        } else {
            const T d = b - a;
            va = fmaT(c.r, d, a);
            vb = fmaT(-c.r, d, b);
            set_wall(va, vb);
            a = fmaT(-x.l.f, va - dev::edge_left<OPEN>(x.gw, vb), va);
            b = fmaT(x.r.f, dev::edge_right<OPEN>(x.ge, va) - vb, vb);
        }
    } else {
        const T dm = a - dev::edge_left<OPEN>(x.gw, b), d0 = b - a;
        const T dp = dev::edge_right<OPEN>(x.ge, a) - b;
        const T Da = d0 - dm, Db = dp - d0;
        if constexpr (P == 0) {
            a = step(a, Da, Db, in);
            b = step(b, Db, Da, pr);
        } else {
            // beside a wall the partner's factor is 0
            a = step(a, Da, dev::edge_left<OPEN>(T(0), Db), x.l);
            b = step(b, Db, dev::edge_right<OPEN>(T(0), Da), x.r);
        }
    }
}

// The y part of one column's R rows.  lo, hi: the rows before and after them,
// nearest first (FP64: old values at P = 0, the explicit stage's at P = 1;
// FP32: old values).  klo, khi: the factors of the first and last row at
// P = 1; kf(q): those of a pair's lower row q inside the wave.
template <typename T, int R, int P>
__device__ __forceinline__ void y_explicit(T (&u)[R], T lo, T hi, const Dir<T> &c)
{
    using dev::fmaT;
    if constexpr (P == 0) {
        u[0] = fmaT(-c.r, u[0] - lo, u[0]);
#pragma unroll
        for (int q = 1; q + 1 < R; q += 2) {
            const T d = u[q + 1] - u[q];
            u[q] = fmaT(c.r, d, u[q]);
            u[q + 1] = fmaT(-c.r, d, u[q + 1]);
        }
        u[R - 1] = fmaT(c.r, hi - u[R - 1], u[R - 1]);
    } else {
#pragma unroll
        for (int q = 0; q < R; q += 2) {
            const T d = u[q + 1] - u[q];
            u[q] = fmaT(c.r, d, u[q]);
            u[q + 1] = fmaT(-c.r, d, u[q + 1]);
        }
    }
}
template <typename T, int R, int P, typename K>
__device__ __forceinline__ void y_solve(T (&v)[R], T lo, T hi, const Dir<T> &c, Factor<T> klo,
                                        Factor<T> khi, K &&kf)
{
    using dev::fmaT;
    if constexpr (P == 0) {
#pragma unroll
        for (int q = 0; q < R; q += 2) {
            const T w = v[q + 1] - v[q];
            v[q] = fmaT(kf(q).f, w, v[q]);
            v[q + 1] = fmaT(-c.k, w, v[q + 1]);
        }
    } else {
        v[0] = fmaT(-klo.f, v[0] - lo, v[0]);
#pragma unroll
        for (int q = 1; q + 1 < R; q += 2) {
            const T w = v[q + 1] - v[q];
            v[q] = fmaT(kf(q).f, w, v[q]);
            v[q + 1] = fmaT(-c.k, w, v[q + 1]);
        }
        v[R - 1] = fmaT(khi.f, hi - v[R - 1], v[R - 1]);
    }
}
template <typename T, int R, int P, typename K>
__device__ __forceinline__ void y_increment(T (&u)[R], const T (&lo)[2], const T (&hi)[2],
                                            const Dir<T> &c, Factor<T> klo, Factor<T> khi, K &&kf)
{
    const Factor<T> pr = paired(c);
    if constexpr (P == 0) {
        T dprev = u[0] - lo[0];
#pragma unroll
        for (int q = 0; q < R; q += 2) {
            const T d0 = u[q + 1] - u[q];
            const T d1 = (q + 2 < R ? u[q + 2] : hi[0]) - u[q + 1];
            const T Da = d0 - dprev, Db = d1 - d0;
            u[q] = step(u[q], Da, Db, kf(q));
            u[q + 1] = step(u[q + 1], Db, Da, pr);
            dprev = d1;
        }
    } else {
        const T dm = u[0] - lo[0], d0 = u[1] - u[0];
        const T dk = u[R - 1] - u[R - 2], dr = hi[0] - u[R - 1];
        const T Dm = dm - (lo[0] - lo[1]), Dp = (hi[1] - hi[0]) - dr;
        const T first = step(u[0], d0 - dm, Dm, klo), last = step(u[R - 1], dr - dk, Dp, khi);
        T dprev = d0;
#pragma unroll
        for (int q = 1; q + 1 < R; q += 2) {
            const T da = u[q + 1] - u[q], db = u[q + 2] - u[q + 1];
            const T Da = da - dprev, Db = db - da;
            u[q] = step(u[q], Da, Db, kf(q));
            u[q + 1] = step(u[q + 1], Db, Da, pr);
            dprev = db;
        }
        u[0] = first;
        u[R - 1] = last;
    }
}

// The levels of one wave (ODD: the window's row and column parities differ).
template <typename T, int R, int NW, int KIND, bool ODD, typename X>
__device__ __forceinline__ void wave_levels(const Block2dArgs<T> &a, int x0, int y0, int w,
                                            T (&ua)[R], T (&ub)[R], X *xch)
{
    constexpr int E = kEdge<T>;
    const int lane = threadIdx.x & (kWave - 1);
    const int ia = x0 + 2 * lane, row0 = y0 + w * R;
    XWalls<T> xw;
    xw.gw = a.gw;
    xw.ge = a.ge;
    xw.l = pick(KIND != kOpen && ia == 0, a.x);
    xw.r = pick(KIND != kOpen && ia + 2 == a.nx, a.x);
    xw.in = pick(KIND == kInside && ia + 1 == a.nx, a.x);
    xw.a_wall = ia >= a.nx;
    xw.b_wall = ia + 1 >= a.nx;
    const bool south = row0 == 0, north = y0 + NW * R == a.ny && w == NW - 1;
    const Factor<T> klo = pick(south, a.y), khi = pick(row0 + R == a.ny, a.y);
    auto kf = [&](int q) { return pick(KIND == kInside && row0 + q + 1 == a.ny, a.y); };
    // the north wall's row, and those past it, when they are the wave's
    auto set_wall = [&]() {
        if constexpr (KIND == kInside) {
#pragma unroll
            for (int q = 0; q < R; ++q)
                if (row0 + q >= a.ny) ua[q] = ub[q] = a.gn;
        }
    };
    // xch: [2 slots][waves][first, last rows][E][lanes] column pairs
    auto slot = [&](int s, int wave, int end, int i) {
        return xch + (((s * NW + wave) * 2 + end) * E + i) * kWave;
    };
    for_levels(a.level0 + (x0 & 1), a.nlev, [&](auto par, int lev) {
        constexpr int PX = decltype(par)::value, PY = ODD ? 1 - PX : PX;
        const int s = lev & 1;
        T loa[E], lob[E], hia[E], hib[E];
        auto put = [&]() {
#pragma unroll
            for (int i = 0; i < E; ++i) {
                slot(s, w, 0, i)[lane] = X{ua[i], ub[i]};
                slot(s, w, 1, i)[lane] = X{ua[R - 1 - i], ub[R - 1 - i]};
            }
        };
        auto take = [&]() {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < E; ++i) {
                X lo = slot(s, w > 0 ? w - 1 : 0, 1, i)[lane];
                X hi = slot(s, w < NW - 1 ? w + 1 : NW - 1, 0, i)[lane];
                if (south) lo = X{a.gs, a.gs};
                if (north) hi = X{a.gn, a.gn};
                loa[i] = lo.x;
                lob[i] = lo.y;
                hia[i] = hi.x;
                hib[i] = hi.y;
            }
        };
        // the rows at the wave's ends first, so that they are on their way
        // while the others take their x part
#pragma unroll
        for (int i = 0; i < E; ++i) {
            x_part<T, PX, KIND>(ua[i], ub[i], xw, a.x);
            x_part<T, PX, KIND>(ua[R - 1 - i], ub[R - 1 - i], xw, a.x);
        }
        constexpr bool EARLY = KIND != kInside && (PY == 0 || !kTwoStage<T>);
        if constexpr (EARLY) put();
#pragma unroll
        for (int q = E; q < R - E; ++q) {
            x_part<T, PX, KIND>(ua[q], ub[q], xw, a.x);
            // a few rows in flight at a time: left alone, the scheduler takes
            // all rows' moves first and runs out of registers
            if (q % kRowsAtOnce<T> == kRowsAtOnce<T> - 1) __builtin_amdgcn_sched_barrier(0);
        }
        set_wall();
        if constexpr (!kTwoStage<T>) {
            if constexpr (!EARLY) put();
            take();
            y_increment<T, R, PY>(ua, loa, hia, a.y, klo, khi, kf);
            y_increment<T, R, PY>(ub, lob, hib, a.y, klo, khi, kf);
        } else if constexpr (PY == 0) {
            if constexpr (!EARLY) put();
            take();
            y_explicit<T, R, 0>(ua, loa[0], hia[0], a.y);
            y_explicit<T, R, 0>(ub, lob[0], hib[0], a.y);
            __builtin_amdgcn_sched_barrier(0);
            set_wall();
            y_solve<T, R, 0>(ua, T(0), T(0), a.y, klo, khi, kf);
            y_solve<T, R, 0>(ub, T(0), T(0), a.y, klo, khi, kf);
            __builtin_amdgcn_sched_barrier(0);
        } else {
            y_explicit<T, R, 1>(ua, T(0), T(0), a.y);
            y_explicit<T, R, 1>(ub, T(0), T(0), a.y);
            set_wall();
            put();
            take();
            y_solve<T, R, 1>(ua, loa[0], hia[0], a.y, klo, khi, kf);
            y_solve<T, R, 1>(ub, lob[0], hib[0], a.y, klo, khi, kf);
        }
    });
}

// Two workgroups of 8 waves are to be resident: at most 128 registers.
// INSIDE: the grid is smaller than a window (a kernel of its own: its wall
// tests would cost the others registers).
template <typename T, int R, int NW, bool INSIDE>
__global__ __launch_bounds__(NW *kWave, 4) void block2d_kernel(Block2dArgs<T> a)
{
    using X = typename Pair2<T>::type;
    using M = typename Pair2<T>::mem;
    __shared__ __attribute__((aligned(16))) unsigned char lds[2 * NW * 2 * kEdge<T> * kWave * 2 * sizeof(T)];
    X *xch = reinterpret_cast<X *>(lds);
    const int t = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);   // XCD-aware
    if (t >= a.ntiles)
        return;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int cx0 = (t % a.tx) * a.cx, cy0 = (t / a.tx) * a.cy;
    const int x0 = max(0, min(cx0 - a.halo, a.nx - kCols));
    const int y0 = max(0, min(cy0 - a.halo, a.ny - NW * R));
    const int row0 = y0 + w * R, ia = x0 + 2 * lane;
    T ua[R], ub[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
        // wave-uniform row address, so that it stays in scalar registers
        const T *row = a.in + (int64_t)(row0 + q) * a.nx + x0;
        if constexpr (INSIDE) {
            ua[q] = row0 + q < a.ny && ia < a.nx ? row[2 * lane] : T(0);
            ub[q] = row0 + q < a.ny && ia + 1 < a.nx ? row[2 * lane + 1] : T(0);
        } else {
            const M v = *reinterpret_cast<const M *>(row + 2 * lane);
            ua[q] = v.x;
            ub[q] = v.y;
        }
    }
    // single registers from here on: as the halves of the loads' tuples they
    // would be copied for each of the paths below, past the 128 registers
#pragma unroll
    for (int q = 0; q < R; ++q) asm("" : "+v"(ua[q]), "+v"(ub[q]));
    const bool ends = x0 == 0 || x0 + kCols == a.nx, odd = ((x0 ^ y0) & 1) != 0;
    if constexpr (INSIDE) {
        if (odd) wave_levels<T, R, NW, kInside, true>(a, x0, y0, w, ua, ub, xch);
        else wave_levels<T, R, NW, kInside, false>(a, x0, y0, w, ua, ub, xch);
    } else if (ends) {
        if (odd) wave_levels<T, R, NW, kEnds, true>(a, x0, y0, w, ua, ub, xch);
        else wave_levels<T, R, NW, kEnds, false>(a, x0, y0, w, ua, ub, xch);
    } else {
        if (odd) wave_levels<T, R, NW, kOpen, true>(a, x0, y0, w, ua, ub, xch);
        else wave_levels<T, R, NW, kOpen, false>(a, x0, y0, w, ua, ub, xch);
    }
    const int cx1 = min(cx0 + a.cx, a.nx), cy1 = min(cy0 + a.cy, a.ny);
    const bool has_a = ia >= cx0 && ia < cx1, has_b = ia + 1 >= cx0 && ia + 1 < cx1;
#pragma unroll
    for (int q = 0; q < R; ++q) {
        if (row0 + q < cy0 || row0 + q >= cy1) continue;   // wave-uniform
        T *o = a.out + (int64_t)(row0 + q) * a.nx + x0 + 2 * lane;
        if (has_a && has_b) *reinterpret_cast<M *>(o) = M{ua[q], ub[q]};
        else if (has_a) o[0] = ua[q];
        else if (has_b) o[1] = ub[q];
    }
}

template <typename T> Dir<T> dir(double r)
{
    return Dir<T>{(T)r, (T)(r / (1.0 + 2.0 * r)), (T)((r + r * r) / (1.0 + 2.0 * r)),
                  (T)(r * r / (1.0 + 2.0 * r)), (T)(r / (1.0 + r))};
}

// The launches of a call whose launches take at most `depth` levels (an even
// number leaves the result in u; the levels are spread evenly over them), and
// the halo of the longest.
struct Launches {
    int64_t n;
    int levels, halo;
};
Launches launches_of(int64_t nsteps, int depth)
{
    Launches l;
    l.n = (nsteps + depth - 1) / depth;
    if ((l.n & 1) && nsteps > l.n) ++l.n;
    l.levels = (int)((nsteps + l.n - 1) / l.n);
    l.halo = (l.levels + 2) / 2 * 2;
    return l;
}

// Rows per wave and levels per launch: the pair with the least estimated time
// of the call, in us.  One window per compute unit takes `one` for a level,
// many at once `many` each; half of the grid's traffic at 5.8 TB/s (a grid of
// 4096 x 4096 FP64 and its copy just exceed the 256 MB cache) is not hidden,
// and a launch costs 2.4 us.  Fitted to 96 levels of 196 x 578 to 4096 x 4096
// points and within 25% of all of them: small grids want few rows (196 x 578
// FP64 4 rows, 10 levels per launch 78 us, 8 rows at best 95), larger ones
// more rows and fewer levels (4096 x 4096 FP64 8 rows, 6 or 8 levels 1.00 ms,
// 12 levels 1.16; 2048 x 2048 FP32 16 rows 0.23 ms, 8 rows 0.27).  FP64 holds at
// most 8 rows a lane: 16 spill at two workgroups per unit (1.10 ms at best).
// A launch has the halo of the call's own levels, so a call of one level (8192
// x 1024 FP64) recomputes 1.10 points a point and not the 1.72 of eight levels.
struct Shape {
    int rows;
    double one64, many64, one32, many32;
};
constexpr Shape kShapes[] = {{4, 0.53, 0.53, 0.41, 0.41}, {8, 0.88, 0.70, 0.72, 0.50},
                             {16, 0.0, 0.0, 1.1, 0.75}};
constexpr int kDepths[] = {1, 2, 4, 6, 8, 10, 12, 16, 20, 24};
constexpr double kUnits = 256.0, kBytesPerUs = 5.8e6, kLaunchUs = 2.4;

struct Choice {
    int rows;
    Launches l;
};

Choice choose(const Grid2dArgs &g, bool f64)
{
    Choice best{4, launches_of(g.nsteps, 4)};
    double best_us = 1e300;
    for (const Shape &s : kShapes) {
        const double one = f64 ? s.one64 : s.one32, many = f64 ? s.many64 : s.many32;
        const int rows = kNW * s.rows;
        if (one == 0.0 || (s.rows > 4 && g.ny < rows)) continue;
        for (int d : kDepths) {
            if (g.depth != 0 && d != g.depth) continue;
            const Launches l = launches_of(g.nsteps, d);
            if (2 * l.halo >= rows) continue;
            const double cx = kCols - 2 * l.halo, cy = rows - 2 * l.halo;
            const double tiles = std::ceil(g.nx / cx) * std::ceil(g.ny / cy);
            const double mem = 2.0 * g.nx * g.ny * (f64 ? 8 : 4) / kBytesPerUs;
            const double level = std::max(one, many * std::ceil(tiles / kUnits));
            // an odd number of launches is followed by a copy
            const double t = l.n * (level * l.levels + 0.5 * mem + kLaunchUs) +
                             (l.n & 1) * (mem + kLaunchUs);
            if (t < best_us) {
                best_us = t;
                best = Choice{s.rows, l};
            }
        }
    }
    return best;
}

template <typename T, int R>
hipError_t run(const Grid2dArgs &g, const Choice &c, hipStream_t stream)
{
    Block2dArgs<T> a{};
    a.nx = (int)g.nx;
    a.ny = (int)g.ny;
    a.halo = c.l.halo;
    a.cx = kCols - 2 * c.l.halo;
    a.cy = kNW * R - 2 * c.l.halo;
    const int64_t tx = (g.nx + a.cx - 1) / a.cx, ty = (g.ny + a.cy - 1) / a.cy;
    if (tx * ty > 0x7ffffff0LL) return hipErrorInvalidValue;
    a.tx = (int)tx;
    a.ntiles = (int)(tx * ty);
    a.x = dir<T>(g.rx);
    a.y = dir<T>(g.ry);
    a.gw = (T)g.gw;
    a.ge = (T)g.ge;
    a.gs = (T)g.gs;
    a.gn = (T)g.gn;
    T *bufs[2] = {static_cast<T *>(g.u), static_cast<T *>(g.work)};
    const int64_t launches = c.l.n;
    int64_t done = 0;
    const dim3 grid((unsigned)(((int64_t)a.ntiles + 7) / 8 * 8));
    for (int64_t i = 0; i < launches; ++i) {
        a.in = bufs[i & 1];
        a.out = bufs[(i + 1) & 1];
        a.level0 = g.step0 + done;
        a.nlev = (int)(g.nsteps / launches + (i < g.nsteps % launches ? 1 : 0));
        if (g.nx < kCols || g.ny < kNW * R)
            hipLaunchKernelGGL((block2d_kernel<T, R, kNW, true>), grid, dim3(kNW * kWave), 0, stream, a);
        else
            hipLaunchKernelGGL((block2d_kernel<T, R, kNW, false>), grid, dim3(kNW * kWave), 0, stream, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        done += a.nlev;
    }
    if (launches & 1)
        return hipMemcpyAsync(g.u, g.work, (size_t)(g.nx * g.ny) * sizeof(T),
                              hipMemcpyDeviceToDevice, stream);
    return hipSuccess;
}

}  // namespace

hipError_t launch_2d(int prec, const Grid2dArgs &g, hipStream_t stream)
{
    // indices inside a launch are 32-bit: rows and columns below 2^31
    if (g.nx < 1 || g.ny < 1 || g.nx > 0x7fffff00LL || g.ny > 0x7fffff00LL ||
        (g.depth != 0 && g.depth != 1 && g.depth != 2 && g.depth != 4) ||
        (prec != kFP64 && prec != kFP32))
        return hipErrorInvalidValue;
    const Choice c = choose(g, prec == kFP64);
    if (prec == kFP64)
        return c.rows == 4 ? run<double, 4>(g, c, stream) : run<double, 8>(g, c, stream);
    return c.rows == 4   ? run<float, 4>(g, c, stream)
           : c.rows == 8 ? run<float, 8>(g, c, stream)
                         : run<float, 16>(g, c, stream);
}

}  // namespace ge

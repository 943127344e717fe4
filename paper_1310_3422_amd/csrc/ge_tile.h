// One window of the tiled GE sweep (Section 2, two-point groups), shared by
// the single-rod kernels (ge_sweep_kernels.h) and the multi-pass tasks of the
// batch kernel (ge_batch.hip).
//
// A window of W = NW*64*K consecutive points starts at ws; thread `tid`
// (0 .. NW*64-1 of the threads sweeping it) holds points ws + tid*K ..
// ws + tid*K + K-1 in registers, the window advances a.nlev levels there
// (ge_level.h) and the core of tile t, [t*core, t*core + core), is stored.
// Edge values cross waves through LDS with one barrier per level (NW > 1);
// a single-wave window (NW = 1) has no barrier, so waves of one workgroup
// may sweep different windows.
#pragma once

#include "ge_kernels.h"
#include "ge_level.h"

namespace ge {
namespace dev {

// What bounds a window (FP64 and FP32).
//   kOpen  : both ends are open window edges (halo points);
//   kEnds  : it starts at the left wall (ws = 0), ends at the right one
//            (ws + W = n), or both, so a wall enters as the fill value of the
//            first or last lane and costs nothing inside the levels: a tile
//            reaching the right wall is moved left to end there;
//   kInside: the rod is shorter than the window, the right wall node lies at
//            a run-time element (a branch tree per access).
enum WindowKind : int { kOpen = 0, kEnds = 1, kInside = 2 };

// Start of tile t's window.
template <int64_t W>
__device__ __forceinline__ int64_t window_start(const TileArgs &a, int64_t t)
{
    return t == 0 ? 0 : min(t * a.core - a.halo, a.n - W);
}

// The lane's points of the window starting at ws, or its source profile.
template <typename T, int K, int KIND>
__device__ __forceinline__ void load_window(const T *__restrict__ p, int64_t g0, int64_t n,
                                            T (&v)[K])
{
    if constexpr (KIND == kInside) load_lane_guarded<T, K>(p + g0, g0, n, v);
    else load_lane<T, K>(p + g0, v);
}

// The wall value each level reads, 64 levels at a time: a level of the
// window's parity 0 reads g(t_m), one of parity 1 (a lone point) g(t_{m+1}).
// Lane l holds level base + l's, so a level takes its value with a lane read
// and waits for no load.  At parity 1 the value is NaN when g(t_m) is
// infinite or NaN: the levels read one wall value in two, and an unusable one
// between them is to show in the result as well.
template <typename T> struct WallFeed {
    T v;
    // levels base .. base+63 of a launch of nlev levels whose first has
    // window parity p0; g: g(t_m) of the launch's levels, or null: constant c
    __device__ __forceinline__ void fill(const double *g, double c, int base, int nlev, int p0)
    {
        double x = c;
        if (g) {
            const int lev = min(base + (int)(threadIdx.x & (kWave - 1)), nlev - 1);
            const double g0 = g[lev];
            x = ((lev + p0) & 1) == 0 ? g0 : __builtin_fma(0.0, g0, g[lev + 1]);
        }
        v = (T)x;
    }
    __device__ __forceinline__ T at(int lev) const
    {
        if constexpr (sizeof(T) == 8) {
            const long long b = __double_as_longlong(v);
            const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lev & (kWave - 1));
            const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lev & (kWave - 1));
            return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
        } else {
            return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lev & (kWave - 1)));
        }
    }
};

// Advance the loaded window of tile t (start ws) by the launch's levels and
// store its core: FP64 or FP32.
template <typename T, int K, int NW, bool SRC, int KIND>
__device__ __forceinline__ void sweep_plain(const TileArgs &a, int tid, int64_t t, int64_t ws,
                                            T (&u)[K], const T (&b)[K])
{
    constexpr int W = NW * kWave * K;
    constexpr bool WALL = KIND != kOpen, OPEN = KIND == kOpen && NW == 1;
    const int lane = tid & (kWave - 1);
    // the wave index is uniform across the wave: let the compiler keep
    // everything derived from it in scalar registers
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t n = a.n;
    const int64_t core_lo = t * a.core;
    const int64_t core_hi = min(core_lo + a.core, n);
    const int64_t g0 = ws + (int64_t)tid * K;       // global index of my first point
    T *out = static_cast<T *>(a.out);

    // FP64 meets its neighbours with one value a side, FP32 with two
    constexpr bool TWO_STAGE = sizeof(T) == 8;
    constexpr int E = TWO_STAGE ? 1 : 2;
    __shared__ T xs[2][NW][2 * E];

    // wall geometry (uniform over the window)
    const bool left = WALL && ws == 0;
    const bool right = KIND == kEnds && ws + W == n;
    const int qR = KIND == kInside ? (int)n : 0;   // right wall node's place in the window
    const int kR = qR % K, lR = qR / K;
    const int qS = qR - 1;                         // the point beside it
    const int kS = KIND == kInside ? qS % K : K - 1, lS = KIND == kInside ? qS / K : NW * kWave - 1;
    const bool own_L = WALL && a.flux && left && core_lo == 0;
    const bool own_R = WALL && a.flux && (right || KIND == kInside) && core_hi == n;
    double acc = 0.0, accR = 0.0;
    if (own_L) acc = a.flux[0];
    if (own_R) accR = a.flux[1];

    const Coef<T> cf = lane_coef(Coef<T>{(T)a.r, (T)a.k, (T)a.c1, (T)a.c2, (T)a.cs});
    const bool lane_l = left && tid == 0, lane_r = right && tid == NW * kWave - 1;
    const T kl = lane_l ? cf.cs : cf.k, kr = lane_r ? cf.cs : cf.k;
    const T cl = lane_l ? cf.cs : cf.c1, cr = lane_r ? cf.cs : cf.c1;
    const T pl = lane_l ? T(0) : cf.c2, pr = lane_r ? T(0) : cf.c2;
    const bool flux = WALL && a.flux != nullptr;   // uniform
    WallFeed<T> wl, wr;
    const int par0 = (int)((a.level0 + ws) & 1);   // the first level's parity in the window
    double an = SRC ? a.src_a[0] : 0.0;            // each loaded a level ahead of its use

    // FP32: the source weights of both parities, formed once per launch
    constexpr int KB = SRC && !TWO_STAGE ? K : 1;
    T B0[KB], B1[KB];
    if constexpr (SRC && !TWO_STAGE) {
        T bl = from_left(T(0), b[K - 1]), br = from_right(T(0), b[0]);
        if constexpr (NW > 1) {
            if (lane == 0) xs[0][w][0] = b[0];
            if (lane == kWave - 1) xs[0][w][1] = b[K - 1];
            __syncthreads();
            if (lane == 0 && w > 0) bl = xs[0][w - 1][1];
            if (lane == kWave - 1 && w < NW - 1) br = xs[0][w + 1][0];
            __syncthreads();
        }
        const T e1 = (T)a.e1, e2 = (T)a.e2, es = (T)a.es;
        increment_source<T, K, 0>(b, bl, br, e1, e2, e1, e1, B0);
        increment_source<T, K, 1>(b, bl, br, e1, e2, lane_l ? es : e1, lane_r ? es : e1, B1);
    }

    // values entering the wave at its edges: from the neighbouring waves
    // through LDS, a wall value, or (at an open window edge) anything
    auto exchange = [&](int slot, T gl, T gr, T (&xl)[E], T (&xr)[E]) {
        if constexpr (NW > 1) {
#pragma unroll
            for (int i = 0; i < E; ++i) {
                if (lane == 0) xs[slot][w][i] = u[i];
                if (lane == kWave - 1) xs[slot][w][E + i] = u[K - 1 - i];
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < E; ++i) {
                xl[i] = xs[slot][w > 0 ? w - 1 : 0][E + i];
                xr[i] = xs[slot][w < NW - 1 ? w + 1 : NW - 1][i];
            }
        }
        if constexpr (WALL) {
#pragma unroll
            for (int i = 0; i < E; ++i) {
                if (left && w == 0) xl[i] = gl;
                if (right && w == NW - 1) xr[i] = gr;
            }
        }
    };

    // a window starting at an odd point pairs its points the other way round
    for_levels(a.level0 + (ws & 1), a.nlev, [&](auto par, int lev) {
        constexpr int P = decltype(par)::value;
        T gl = T(0), gr = T(0);
        if constexpr (WALL) {
            if ((lev & (kWave - 1)) == 0) {
                wl.fill(a.gl_t, a.gl0, lev, a.nlev, par0);
                // a wall node inside the window is read by the levels at
                // which the point beside it is not alone
                wr.fill(a.gr_t, a.gr0, lev, a.nlev, KIND == kInside ? par0 + (int)n : par0);
            }
            gl = wl.at(lev);
            gr = wr.at(lev);
        }
        const bool single = KIND == kInside && (((int)n - 1 + P) & 1) == 0;
        T xl[E] = {}, xr[E] = {};
        T lone = T(0);
        if constexpr (TWO_STAGE) {
            if (KIND == kInside && !single) put_at<T, K>(u, kR, tid == lR, gr);
            if constexpr (P == 0) exchange(lev & 1, gl, gr, xl, xr);
            explicit_stage<T, K, P, OPEN, OPEN>(u, xl[0], xr[0], cf);
            if constexpr (SRC) source_stage<T, K>(u, b, (T)(a.tau * an));
            if constexpr (P == 1) exchange(lev & 1, gl, gr, xl, xr);
            if (KIND == kInside && single)
                lone = lone_point(get_at<T, K>(u, kS, T(0)), gr, cf.cs);
            solve_stage<T, K, P, OPEN, OPEN>(u, xl[0], xr[0], cf, kl, kr);
        } else {
            if constexpr (KIND == kInside) put_at<T, K>(u, kR, tid == lR, gr);
            exchange(lev & 1, gl, gr, xl, xr);
            auto level = [&](const T (&B)[K]) {
                if (KIND == kInside && single)
                    lone = lone_increment<T, K, SRC>(u, b, (T)an, kS, xl[0], gr, cf.cs, (T)a.es);
                increment_level<T, K, SRC, P, OPEN, OPEN>(u, B, (T)an, xl[0], xl[E - 1], xr[0], xr[E - 1],
                                                    cf, cl, pl, cr, pr);
            };
            // An open window without a source takes the same operations from
            // pair_level, of which a SIMD issues 1.18 in 4 cycles, two waves at
            // once, against 1.04 of increment_level (2^24 points, 2000 levels
            // 3.86 ms against 4.47; 5e7 points, 192 levels 1.07 against 1.26;
            // 4096 rods 11.0 against 11.8).  The instructions are the same; half
            // of increment_level's results here fall into one of the four
            // register banks, where pair_level's are spread evenly.
            if constexpr (!SRC && OPEN) {
                const PairCoef<T> pc{cf.c1, cf.c2, cf.cs, T(0), T(0), T(0)};
                FluxTap none{false, 0.0, 0.0, 0.0, 0.0};
                T e[K];
                pair_level<T, K, 0, false, P, true, false>(
                    u, e, b, T(0), T(0), xl[0], xl[E - 1], xr[0], xr[E - 1], T(0), T(0), T(0), T(0),
                    pc, T(0), WallLevel<T>{false, T(0)}, none);
            } else if constexpr (!SRC) level(b);
            else if constexpr (P == 0) level(B0);
            else level(B1);
        }
        if (KIND == kInside && single) put_at<T, K>(u, kS, tid == lS, lone);
        if constexpr (SRC) an = a.src_a[lev + 1 < a.nlev ? lev + 1 : lev];
        if (WALL && flux) {
            // wall first differences at the new level, accumulated in FP64
            if (own_L && tid == 0)
                acc = acc + a.tau * ((double)u[0] - (a.gl_t ? a.gl_t[lev + 1] : a.gl0)) / a.h;
            if (own_R) {
                const T v = KIND == kInside ? get_at<T, K>(u, kS, T(0)) : u[K - 1];
                if (tid == lS)
                    accR = accR + a.tau * ((double)v - (a.gr_t ? a.gr_t[lev + 1] : a.gr0)) / a.h;
            }
        }
    });

    if (own_L && tid == 0) a.flux[0] = acc;
    if (own_R && tid == lS) a.flux[1] = accR;

    T fin = T(0);
    if constexpr (WALL) store_lane_guarded<T, K>(out + g0, g0, core_lo, core_hi, u, fin);
    else store_lane_chunks<T, K>(out + g0, g0, core_lo, core_hi, u, fin);
    raise_if_nonfinite(a.status, fin);
}

template <typename T, int K, int NW, bool SRC, int KIND>
__device__ __forceinline__ void run_plain(const TileArgs &a, int tid, int64_t t, int64_t ws)
{
    T u[K], b[K];
    const int64_t g0 = ws + (int64_t)tid * K;
    load_window<T, K, KIND>(static_cast<const T *>(a.in), g0, a.n, u);
    if constexpr (SRC) load_window<T, K, KIND>(static_cast<const T *>(a.src_b), g0, a.n, b);
    sweep_plain<T, K, NW, SRC, KIND>(a, tid, t, ws, u, b);
}

// ---- the compensated pair --------------------------------------------------
// The lane's points of the window starting at ws, their compensation and
// source profile; guarded at a wall.
template <typename T, int K, bool SRC, bool WALL>
__device__ __forceinline__ void load_pair(const TileArgs &a, int tid, int64_t ws, T (&s)[K],
                                          T (&e)[K], T (&b)[K])
{
    const int64_t g0 = ws + (int64_t)tid * K;
    const T *in_s = static_cast<const T *>(a.in);
    const T *in_e = in_s + a.estride;
    const T *srcb = static_cast<const T *>(a.src_b);
    if constexpr (WALL) {
        load_lane_guarded<T, K>(in_s + g0, g0, a.n, s);
        load_lane_guarded<T, K>(in_e + g0, g0, a.n, e);
        if constexpr (SRC) load_lane_guarded<T, K>(srcb + g0, g0, a.n, b);
    } else {
        load_lane<T, K>(in_s + g0, s);
        load_lane<T, K>(in_e + g0, e);
        if constexpr (SRC) load_lane<T, K>(srcb + g0, b);
    }
}

// Advance the loaded window of tile t (start ws) by the launch's levels and
// store its core.
template <typename T, int K, int NW, bool SRC, bool WALL>
__device__ __forceinline__ void sweep_pair(const TileArgs &a, int tid, int64_t t, int64_t ws,
                                           T (&s)[K], T (&e)[K], const T (&b)[K])
{
    constexpr int W = NW * kWave * K;
    const int lane = tid & (kWave - 1);
    // the wave index is uniform across the wave: let the compiler keep
    // everything derived from it in scalar registers
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t n = a.n;
    const int64_t core_lo = t * a.core;
    const int64_t core_hi = min(core_lo + a.core, n);
    const int64_t g0 = ws + (int64_t)tid * K;       // global index of my first point

    T *out_s = static_cast<T *>(a.out);
    T *out_e = out_s + a.estride_out;

    __shared__ T xs[2][NW][4];
    __shared__ T xe[2][NW][4];
    __shared__ T xb[NW][2];

    // source profile of the neighbours' edge points (fixed for the launch)
    T bl = T(0), br = T(0);
    if constexpr (SRC) {
        bl = from_left(T(0), b[K - 1]);
        br = from_right(T(0), b[0]);
        if constexpr (NW > 1) {
            if (lane == 0) xb[w][0] = b[0];
            if (lane == kWave - 1) xb[w][1] = b[K - 1];
            __syncthreads();
            if (lane == 0 && w > 0) bl = xb[w - 1][1];
            if (lane == kWave - 1 && w < NW - 1) br = xb[w + 1][0];
        }
    }

    // wall geometry (uniform over the workgroup)
    const bool left_wall = WALL && (ws == 0);
    const int64_t qR = n - ws;                     // window position of the right wall node
    const bool ghost_in = WALL && (qR < W);
    const bool ghost_edge = WALL && (qR == W);
    const int kR = (int)(ghost_in ? (qR % K) : 0);
    const int lR = (int)(ghost_in ? (qR / K) : -1);          // thread holding it
    const int64_t qS = qR - 1;                     // window position of point n-1
    const bool has_S = WALL && (qS >= 0) && (qS < W);
    const int kS = (int)(has_S ? (qS % K) : 0);
    const int lS = (int)(has_S ? (qS / K) : -1);
    const bool flux_on = WALL && (a.flux != nullptr);
    const bool own_L = flux_on && left_wall && core_lo == 0;
    const bool own_R = flux_on && has_S && (n - 1 >= core_lo) && (n - 1 < core_hi);
    double accL = 0.0, accR = 0.0;
    if (own_L) accL = a.flux[0];
    if (own_R) accR = a.flux[1];

    const PairCoef<T> cf = lane_coef(PairCoef<T>{(T)a.c1, (T)a.c2, (T)a.cs, (T)a.e1, (T)a.e2, (T)a.es});
    FluxTap ft{own_L && tid == 0, accL, a.tau, a.h, 0.0};

    // Interior tiles with a source form each point's source weight for both
    // parities once (source_weights); wall tiles keep the profile for the
    // lone points' formulas.  The same bits either way.
    constexpr bool COMB = SRC && !WALL;
    T B0[COMB ? K : 1], B1[COMB ? K : 1];
    if constexpr (COMB) {
        source_weights<T, K, 0>(b, bl, br, cf, B0);
        source_weights<T, K, 1>(b, bl, br, cf, B1);
    }

    for_levels(a.level0, a.nlev, [&](auto par, int lev) {
        constexpr int p = decltype(par)::value;
        double glo = a.gl0, gln = a.gl0, gro = a.gr0, grn = a.gr0;
        if constexpr (WALL) {
            if (a.gl_t) { glo = a.gl_t[lev]; gln = a.gl_t[lev + 1]; }
            if (a.gr_t) { gro = a.gr_t[lev]; grn = a.gr_t[lev + 1]; }
            if (ghost_in) {
                T gh, gl_;
                split_wall<T, true>(gro, gh, gl_);
                put_at<T, K>(s, kR, tid == lR, gh);
                put_at<T, K>(e, kR, tid == lR, gl_);
            }
        }

        // Values entering the wave at its edges: from the neighbouring waves
        // through LDS, or (at an open window edge) anything -- those points
        // lie in the halo.  They ride in as the DPP fill of lanes 0 and 63.
        T xl = T(0), xl2 = T(0), xr = T(0), xr2 = T(0);
        T yl = T(0), yl2 = T(0), yr = T(0), yr2 = T(0);
        if constexpr (NW > 1) {
            const int pb = lev & 1;
            if (lane == 0) { xs[pb][w][0] = s[0]; xs[pb][w][1] = s[1]; }
            if (lane == kWave - 1) { xs[pb][w][2] = s[K - 2]; xs[pb][w][3] = s[K - 1]; }
            {
                if (lane == 0) { xe[pb][w][0] = e[0]; xe[pb][w][1] = e[1]; }
                if (lane == kWave - 1) { xe[pb][w][2] = e[K - 2]; xe[pb][w][3] = e[K - 1]; }
            }
            __syncthreads();
            const int wl = w > 0 ? w - 1 : 0, wr = w < NW - 1 ? w + 1 : NW - 1;
            xl = xs[pb][wl][3]; xr = xs[pb][wr][0];
            xl2 = xs[pb][wl][2]; xr2 = xs[pb][wr][1];
            {
                yl = xe[pb][wl][3]; yr = xe[pb][wr][0];
                yl2 = xe[pb][wl][2]; yr2 = xe[pb][wr][1];
            }
        }
        WallLevel<T> wlv{false, T(0)};
        T gr_hi = T(0), gr_lo = T(0), dgr = T(0);
        bool singR = false;
        if constexpr (WALL) {
            if (left_wall && w == 0) {
                T gh, glw;
                split_wall<T, true>(glo, gh, glw);
                xl = gh;
                yl = glw;
            }
            if (ghost_edge && w == NW - 1) {
                T gh, glw;
                split_wall<T, true>(gro, gh, glw);
                xr = gh;
                yr = glw;
            }
            wlv.dgl = (T)(gln - glo);
            wlv.isL = left_wall && (p == 1) && (tid == 0);
            ft.gln = gln;
            split_wall<T, true>(gro, gr_hi, gr_lo);
            dgr = (T)(grn - gro);
            singR = has_S && (((n - 1 + p) & 1) == 0);
        }
        const T an = SRC ? (T)a.src_a[lev] : T(0);
        Lone<T> lone{T(0), T(0)};
        if (WALL && singR)
            lone = right_lone<T, K, SRC>(s, e, b, kS, xl, yl, gr_hi, gr_lo, dgr, cf, an);
        if constexpr (COMB) {
            if constexpr (p == 0)
                pair_level<T, K, 2, WALL, p, NW == 1 && !WALL>(s, e, B0, bl, br, xl, xl2, xr,
                                                                   xr2, yl, yl2, yr, yr2, cf, an,
                                                                   wlv, ft);
            else
                pair_level<T, K, 2, WALL, p, NW == 1 && !WALL>(s, e, B1, bl, br, xl, xl2, xr,
                                                                   xr2, yl, yl2, yr, yr2, cf, an,
                                                                   wlv, ft);
        } else {
            pair_level<T, K, SRC ? 1 : 0, WALL, p, NW == 1 && !WALL>(
                s, e, b, bl, br, xl, xl2, xr, xr2, yl, yl2, yr, yr2, cf, an, wlv, ft);
        }
        if (WALL && singR) {
            put_at<T, K>(s, kS, tid == lS, lone.s);
            put_at<T, K>(e, kS, tid == lS, lone.e);
        }
        if (WALL && own_R) {
            // wall first difference at the new level, accumulated in FP64
            const double v = (double)get_at<T, K>(s, kS, T(0)) +
                             (double)get_at<T, K>(e, kS, T(0));
            if (tid == lS) accR = accR + a.tau * (v - grn) / a.h;
        }
    });
    accL = ft.accL;

    if (own_L && tid == 0) a.flux[0] = accL;
    if (own_R && tid == lS) a.flux[1] = accR;

    T fin = T(0);
    if constexpr (WALL) {
        store_lane_guarded<T, K>(out_s + g0, g0, core_lo, core_hi, s, fin);
        store_lane_guarded<T, K>(out_e + g0, g0, core_lo, core_hi, e, fin);
    } else {
        store_lane_chunks<T, K>(out_s + g0, g0, core_lo, core_hi, s, fin);
        store_lane_chunks<T, K>(out_e + g0, g0, core_lo, core_hi, e, fin);
    }
    raise_if_nonfinite(a.status, fin);
}

template <typename T, int K, int NW, bool SRC, bool WALL>
__device__ __forceinline__ void run_pair(const TileArgs &a, int tid, int64_t t, int64_t ws)
{
    T s[K], e[K], b[K];
    load_pair<T, K, SRC, WALL>(a, tid, ws, s, e, b);
    sweep_pair<T, K, NW, SRC, WALL>(a, tid, t, ws, s, e, b);
}

// Tile t's window, whichever kind it is (n >= W for FP64 and FP32).
template <typename T, int K, int NW, bool COMP, bool SRC>
__device__ __forceinline__ void run_tile(const TileArgs &a, int tid, int64_t t)
{
    constexpr int64_t W = NW * kWave * K;
    if constexpr (COMP) {
        const int64_t ws = t == 0 ? 0 : t * a.core - a.halo;
        if (ws == 0 || ws + W >= a.n) run_pair<T, K, NW, SRC, true>(a, tid, t, ws);
        else run_pair<T, K, NW, SRC, false>(a, tid, t, ws);
    } else {
        const int64_t ws = window_start<W>(a, t);
        if (t == 0 || ws + W == a.n) run_plain<T, K, NW, SRC, kEnds>(a, tid, t, ws);
        else run_plain<T, K, NW, SRC, kOpen>(a, tid, t, ws);
    }
}

}  // namespace dev
}  // namespace ge

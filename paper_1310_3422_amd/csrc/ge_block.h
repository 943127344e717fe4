// A window of overlapping waves, shared by the single-rod kernel (ge_block.hip)
// and the batch kernels (ge_batch_windows.hip).
//
// The waves of a window overlap by 2 h points (h = kBlockOverlap) and advance
// h - 1 levels on their own, each with open edges, before they refresh what
// has gone stale through LDS (one barrier).  A wave's window starts at any
// point: the last one ends where the workgroup's does, and a wave that starts
// at an odd point pairs its points the other way round.  A wall is the fill of
// a first or last lane.  Every point gets the operations it gets everywhere
// (ge_level.h): the same bits.
#pragma once

#include "ge_kernels.h"
#include "ge_level.h"
#include "ge_tile.h"

namespace ge {
namespace dev {

// What a workgroup's window and its waves are.
struct BlockShape {
    int64_t core_lo, core_hi;   // points stored
    int64_t lo, hi;             // points held
    int waves;                  // waves that hold them
};

template <int K>
__device__ __forceinline__ BlockShape block_shape(const TileArgs &a, int64_t t)
{
    constexpr int W = kWave * K, STEP = W - 2 * kBlockOverlap;
    BlockShape s;
    s.core_lo = t * a.core;
    s.core_hi = min(s.core_lo + a.core, a.n);
    s.hi = min(s.core_hi + a.halo, a.n);
    s.lo = s.core_lo > a.halo ? s.core_lo - a.halo : 0;
    if (s.hi - s.lo < W) s.lo = s.hi - W;           // a short last core (n >= W)
    if (s.lo < 0) {
        s.lo = 0;
        s.hi = W;
    }
    const int len = (int)(s.hi - s.lo);
    s.waves = len <= W ? 1 : 1 + (len - W + STEP - 1) / STEP;
    return s;
}

// One wave of a window: points p0 .. p0 + 64 K - 1, of which it owns
// [own_lo, own_hi) (its neighbours take theirs of the rest from it).  LEFT,
// RIGHT: that edge is a wall, else an open one.
template <typename T, int K, bool SRC, bool LEFT, bool RIGHT>
__device__ __forceinline__ void block_wave(const TileArgs &a, const BlockShape &sh, int64_t p0,
                                           int64_t own_lo, int64_t own_hi, T *buf, int stride)
{
    constexpr bool TWO_STAGE = sizeof(T) == 8;
    constexpr int W = kWave * K, H = kBlockOverlap;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t g0 = p0 + lane * K;
    T u[K], b[K];
    load_lane<T, K>(static_cast<const T *>(a.in) + g0, u);
    if constexpr (SRC) load_lane<T, K>(static_cast<const T *>(a.src_b) + g0, b);

    const bool lane_l = LEFT && lane == 0, lane_r = RIGHT && lane == kWave - 1;
    const bool flux = (LEFT || RIGHT) && a.flux != nullptr;    // uniform
    const bool own_L = lane_l && a.flux && sh.core_lo == 0;
    const bool own_R = lane_r && a.flux && sh.core_hi == a.n;
    double acc_l = own_L ? a.flux[0] : 0.0, acc_r = own_R ? a.flux[1] : 0.0;
    const Coef<T> cf = lane_coef(Coef<T>{(T)a.r, (T)a.k, (T)a.c1, (T)a.c2, (T)a.cs});
    const T kl = lane_l ? cf.cs : cf.k, kr = lane_r ? cf.cs : cf.k;
    const T cl = lane_l ? cf.cs : cf.c1, cr = lane_r ? cf.cs : cf.c1;
    const T pl = lane_l ? T(0) : cf.c2, pr = lane_r ? T(0) : cf.c2;
    WallFeed<T> wl, wr;
    const int par0 = (int)((a.level0 + p0) & 1);   // the first level's parity in the window
    double an = SRC ? a.src_a[0] : 0.0;
    constexpr int KB = SRC && !TWO_STAGE ? K : 1;
    T B0[KB], B1[KB];
    if constexpr (SRC && !TWO_STAGE) {
        const T bl = from_left(T(0), b[K - 1]), br = from_right(T(0), b[0]);
        const T e1 = (T)a.e1, e2 = (T)a.e2, es = (T)a.es;
        increment_source<T, K, 0>(b, bl, br, e1, e2, e1, e1, B0);
        increment_source<T, K, 1>(b, bl, br, e1, e2, lane_l ? es : e1, lane_r ? es : e1, B1);
    }

    int done = 0;
    for (int blk = 0;; ++blk) {
        const int nb = min(a.nlev - done, H - 1);
        if constexpr (LEFT) wl.fill(a.gl_t, a.gl0, done, a.nlev, par0);
        if constexpr (RIGHT) wr.fill(a.gr_t, a.gr0, done, a.nlev, par0);
        for_levels(par0 + done, nb, [&](auto par, int lev) {
            constexpr int P = decltype(par)::value;
            T gl = T(0), gr = T(0);
            if constexpr (LEFT) gl = wl.at(lev);
            if constexpr (RIGHT) gr = wr.at(lev);
            if constexpr (TWO_STAGE) {
                explicit_stage<T, K, P, !LEFT, !RIGHT>(u, gl, gr, cf);
                if constexpr (SRC) source_stage<T, K>(u, b, (T)(a.tau * an));
                solve_stage<T, K, P, !LEFT, !RIGHT>(u, gl, gr, cf, kl, kr);
            } else if constexpr (!SRC) {
                increment_level<T, K, false, P, !LEFT, !RIGHT>(u, u, T(0), gl, gl, gr, gr, cf, cl,
                                                               pl, cr, pr);
            } else if constexpr (P == 0) {
                increment_level<T, K, true, P, !LEFT, !RIGHT>(u, B0, (T)an, gl, gl, gr, gr, cf, cl,
                                                              pl, cr, pr);
            } else {
                increment_level<T, K, true, P, !LEFT, !RIGHT>(u, B1, (T)an, gl, gl, gr, gr, cf, cl,
                                                              pl, cr, pr);
            }
            if constexpr (SRC) an = a.src_a[min(done + lev + 1, a.nlev - 1)];
            if (flux) {
                // wall first differences at the new level, accumulated in FP64
                const int m = done + lev + 1;
                if (own_L) acc_l = acc_l + a.tau * ((double)u[0] - (a.gl_t ? a.gl_t[m] : a.gl0)) / a.h;
                if (own_R)
                    acc_r = acc_r + a.tau * ((double)u[K - 1] - (a.gr_t ? a.gr_t[m] : a.gr0)) / a.h;
            }
        });
        done += nb;
        if (done >= a.nlev)
            break;
        // every wave puts down what it owns and takes its edges' points from
        // their owners; the buffers alternate, so one barrier is enough
        T *x = buf + (blk & 1) * stride;
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (g0 + j >= own_lo && g0 + j < own_hi) x[g0 + j - sh.lo] = u[j];
        __syncthreads();
        if (lane * K < H || (lane + 1) * K > W - H) {
#pragma unroll
            for (int j = 0; j < K; ++j) u[j] = x[g0 + j - sh.lo];
        }
    }
    if (own_L) a.flux[0] = acc_l;
    if (own_R) a.flux[1] = acc_r;

    // a rod in one window is advanced in place: every load has to be in
    // before any store (a call of few levels passes no other barrier)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    T fin = T(0);
    store_lane_guarded<T, K>(static_cast<T *>(a.out) + g0, g0, max(own_lo, sh.core_lo),
                             min(own_hi, sh.core_hi), u, fin);
    raise_if_nonfinite(a.status, fin);
}

// A value of a given lane, in every lane.
__device__ __forceinline__ double value_of_lane(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The same for the compensated pair: s and e, each with its own half of the
// buffers.  The walls' FP64 values between two refreshes are held one a lane.
template <int K, bool SRC, bool LEFT, bool RIGHT>
__device__ __forceinline__ void block_wave_pair(const TileArgs &a, const BlockShape &sh,
                                                int64_t p0, int64_t own_lo, int64_t own_hi,
                                                float *buf, int stride)
{
    using T = float;
    constexpr bool WALL = LEFT || RIGHT;
    constexpr int W = kWave * K, H = kBlockOverlap;
    static_assert(H <= kWave, "a refresh's wall values fit one register");
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t g0 = p0 + lane * K;
    const T *in = static_cast<const T *>(a.in);
    T *out = static_cast<T *>(a.out);
    T s[K], e[K], b[K];
    load_lane<T, K>(in + g0, s);
    load_lane<T, K>(in + a.estride + g0, e);
    if constexpr (SRC) load_lane<T, K>(static_cast<const T *>(a.src_b) + g0, b);
    T bl = T(0), br = T(0);
    if constexpr (SRC) {
        bl = from_left(T(0), b[K - 1]);
        br = from_right(T(0), b[0]);
    }
    const bool lane_l = LEFT && lane == 0, lane_r = RIGHT && lane == kWave - 1;
    const bool own_L = lane_l && a.flux && sh.core_lo == 0;
    const bool own_R = lane_r && a.flux && sh.core_hi == a.n;
    double acc_r = own_R ? a.flux[1] : 0.0;
    FluxTap ft{own_L, own_L ? a.flux[0] : 0.0, a.tau, a.h, 0.0};
    const PairCoef<T> cf =
        lane_coef(PairCoef<T>{(T)a.c1, (T)a.c2, (T)a.cs, (T)a.e1, (T)a.e2, (T)a.es});
    const int par0 = (int)((a.level0 + p0) & 1);   // the first level's parity in the window
    double an = SRC ? a.src_a[0] : 0.0;

    int done = 0;
    for (int blk = 0;; ++blk) {
        const int nb = min(a.nlev - done, H - 1);
        double wl = a.gl0, wr = a.gr0;             // lane l: level done + l
        if (LEFT && a.gl_t) wl = a.gl_t[min(done + lane, a.nlev)];
        if (RIGHT && a.gr_t) wr = a.gr_t[min(done + lane, a.nlev)];
        for_levels(par0 + done, nb, [&](auto par, int lev) {
            constexpr int P = decltype(par)::value;
            T xl = T(0), yl = T(0), xr = T(0), yr = T(0), dgr = T(0);
            double grn = 0.0;
            WallLevel<T> wlv{false, T(0)};
            if constexpr (LEFT) {
                const double glo = value_of_lane(wl, lev), gln = value_of_lane(wl, lev + 1);
                split_wall<T, true>(glo, xl, yl);
                wlv.dgl = (T)(gln - glo);
                wlv.isL = P == 1 && lane_l;
                ft.gln = gln;
            }
            if constexpr (RIGHT) {
                const double gro = value_of_lane(wr, lev);
                grn = value_of_lane(wr, lev + 1);
                split_wall<T, true>(gro, xr, yr);
                dgr = (T)(grn - gro);
            }
            // the window ends at the wall: its last point is alone at parity 1
            Lone<T> lone{T(0), T(0)};
            if constexpr (RIGHT && P == 1)
                lone = right_lone<T, K, SRC>(s, e, b, K - 1, T(0), T(0), xr, yr, dgr, cf, (T)an);
            pair_level<T, K, SRC ? 1 : 0, WALL, P, !WALL>(s, e, b, bl, br, xl, T(0), xr, T(0), yl,
                                                          T(0), yr, T(0), cf, (T)an, wlv, ft);
            if constexpr (RIGHT && P == 1) {
                s[K - 1] = lane_r ? lone.s : s[K - 1];
                e[K - 1] = lane_r ? lone.e : e[K - 1];
            }
            if constexpr (SRC) an = a.src_a[min(done + lev + 1, a.nlev - 1)];
            if (RIGHT && own_R)
                acc_r = acc_r + a.tau * (((double)s[K - 1] + (double)e[K - 1]) - grn) / a.h;
        });
        done += nb;
        if (done >= a.nlev)
            break;
        T *x = buf + (blk & 1) * 2 * stride;
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (g0 + j >= own_lo && g0 + j < own_hi) {
                x[g0 + j - sh.lo] = s[j];
                x[stride + g0 + j - sh.lo] = e[j];
            }
        __syncthreads();
        if (lane * K < H || (lane + 1) * K > W - H) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                s[j] = x[g0 + j - sh.lo];
                e[j] = x[stride + g0 + j - sh.lo];
            }
        }
    }
    if (own_L) a.flux[0] = ft.accL;
    if (own_R) a.flux[1] = acc_r;

    // every load in before any store, as in block_wave
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    T fin = T(0);
    const int64_t lo = max(own_lo, sh.core_lo), hi = min(own_hi, sh.core_hi);
    store_lane_guarded<T, K>(out + g0, g0, lo, hi, s, fin);
    store_lane_guarded<T, K>(out + a.estride_out + g0, g0, lo, hi, e, fin);
    raise_if_nonfinite(a.status, fin);
}

// The whole workgroup: window t of the rod, advanced a.nlev levels.  buf: two
// buffers of `stride` values (for the pair twice that), at least the window's
// points each.
template <typename T, int K, bool SRC, bool PAIR = false>
__device__ __forceinline__ void block_window(const TileArgs &a, int64_t t, T *buf, int stride)
{
    constexpr int W = kWave * K, STEP = W - 2 * kBlockOverlap;
    const BlockShape sh = block_shape<K>(a, t);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    if (w >= sh.waves) {
        // a wave without points passes the others' barriers: one per refresh
        // and the one before the stores
        for (int done = kBlockOverlap - 1; done < a.nlev; done += kBlockOverlap - 1) __syncthreads();
        __syncthreads();
        return;
    }
    const int64_t last = sh.hi - W;                    // start of the last wave
    const bool is_last = w == sh.waves - 1;
    const int64_t p0 = is_last ? last : sh.lo + (int64_t)w * STEP;
    const int64_t next = w + 2 >= sh.waves ? last : p0 + STEP;
    const int64_t own_lo = w == 0 ? sh.lo : p0 + kBlockOverlap;
    const int64_t own_hi = is_last ? sh.hi : next + kBlockOverlap;
    const bool left = p0 == 0, right = p0 + W == a.n;
    if constexpr (PAIR) {
        if (left && right) block_wave_pair<K, SRC, true, true>(a, sh, p0, own_lo, own_hi, buf, stride);
        else if (left) block_wave_pair<K, SRC, true, false>(a, sh, p0, own_lo, own_hi, buf, stride);
        else if (right) block_wave_pair<K, SRC, false, true>(a, sh, p0, own_lo, own_hi, buf, stride);
        else block_wave_pair<K, SRC, false, false>(a, sh, p0, own_lo, own_hi, buf, stride);
        return;
    }
    if (left && right) block_wave<T, K, SRC, true, true>(a, sh, p0, own_lo, own_hi, buf, stride);
    else if (left) block_wave<T, K, SRC, true, false>(a, sh, p0, own_lo, own_hi, buf, stride);
    else if (right) block_wave<T, K, SRC, false, true>(a, sh, p0, own_lo, own_hi, buf, stride);
    else block_wave<T, K, SRC, false, false>(a, sh, p0, own_lo, own_hi, buf, stride);
}

}  // namespace dev
}  // namespace ge

// One level of the GE sweep on a register tile, shared by the single-rod
// tile kernel (ge_sweep_kernels.h) and the persistent batch kernel (ge_batch.hip).
//
// Scheme (Section 2, two-point groups): at level m with p = m mod 2 the
// points are coupled as (0,1),(2,3),... (0-based) when p = 0 and
// (1,2),(3,4),... when p = 1.
//
// FP64 evaluates a level in the two stages that Eq. (3)/(4) are the solution
// of: an explicit one over the other parity's pairs, then the 2x2 solve of
// this parity's pairs (i left of q):
//     v_i = u_i - r (u_i - u_{i-1}),   v_q = u_q + r (u_{q+1} - u_q),
//     w = v_q - v_i,   u_i' = v_i + k w,   u_q' = v_q - k w,   k = r/(1+2r).
// Both stages work on pairs, so a difference serves two points: 3 VALU
// instructions a point (a subtraction per pair and an FMA per point, twice)
// where second differences take 4.  Two roundings of u per level, as
// fma(c2, D_q, fma(c1, D_i, u)) has: against extended precision, r from 1/4 to
// 64, the error is 0.3 to 1.06 of that form's, at most 0.1 from r = 300 on.  The
// exception is r = 1 (k = 1/3, where second differences happen to round well)
// over long runs of short rods: 1.6 times at 1024 points and 1000 levels, 2.5
// at 300 points (1e-16 against 4e-16 at the worst).  A point
// alone beside a wall (scheme A, Eq. (1), or B, Eq. (2)) is a pair with the
// wall node, the wall's old value in the explicit stage and its new one in
// the second, and cs = r/(1+r) for k.  A source f = a(t) b(x) adds
// tau a(t_m + tau/2) b_i to v_i.
//
// FP32 rounds u once per level, so it forms the increment from second
// differences, D_i = u_{i-1} - 2u_i + u_{i+1} = d_i - d_{i-1} from first
// differences d_i = u_{i+1} - u_i (exact for smooth data, so the increment
// carries a relative rounding error), rounds it and adds it:
//     u_i' = u_i + (c1 D_i + c2 D_q),   c1 = (r+r^2)/(1+2r), c2 = r^2/(1+2r),
// with q the partner of i: 5 instructions a point.  The increment's own
// rounding is needed: where c1, c2 are dyadic or thirds the exact increment often
// lies half a unit of u from its neighbours, and one folded into the addition,
// fma(c1, fma(cs, D_q, D_i), u) at 4 instructions, breaks every such tie the
// way that the rounding of cs points.  Against extended precision that form's
// error was 3.8 times this one's at r = 1 (300 points, 2000 levels), 1.4 to 1.9
// times at r = 1/2 and 1.6 at r = 1/4.  Two stages would take 3 instructions,
// but their roundings part from this form's by up to 4e-5 of u where
// increments fall below half a unit of u (30000 points, r = 0.3, 6000
// levels).  A point alone beside a wall is u_i' = u_i + cs D_i, cs = r/(1+r),
// with the wall's new value in D_i.  A source adds a(t_m + tau/2) (e1 b_i +
// e2 b_q) to the increment of a pair member and a(t_m + tau/2) es b_i to a lone
// point's, e1 = tau(1+r)/(1+2r), e2 = tau r/(1+2r), es = tau/(1+r).
//
// The compensated FP32 pair (s, e), value s + e:
//     u_i' = u_i + c1 D_i + c2 D_q,   c1 = (r+r^2)/(1+2r), c2 = r^2/(1+2r),
// where q is i's partner, and u_i' = u_i + cs (D_i + g(t_{m+1}) - g(t_m)) for
// a point alone beside a wall, D_i with the wall value at t_m.  A source adds
// a(t_m + tau/2) (e1 b_i + e2 b_q) to a pair member and a(t_m + tau/2) es b_i
// to a lone point.  D comes from the s and e first differences' differences,
// summed at the end, and the increment is added with Kahan's compensated sum.
//
// Layout: each lane holds K consecutive points in registers; neighbour
// values cross lanes by DPP wave shifts, and the lanes at a wave's edges
// receive theirs as the DPP fill value.
//
// Determinism: every point, in every kernel and tile, halo or core, is
// advanced by the same expression sequence with explicit fma() and no
// contraction (-ffp-contract=off), so results do not depend on the tiling,
// the levels per launch, the grid, or whether a rod runs alone or in a batch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ge_kernels.h"

namespace ge {
namespace dev {

constexpr int kWave = 64;

// ---- cross-lane moves ------------------------------------------------------
// DPP wave shifts by one lane; the lane with no source (lane 0 for a shift
// right, lane 63 for a shift left) receives `fill`.
__device__ __forceinline__ int shr1_i(int fill, int v)
{
    return __builtin_amdgcn_update_dpp(fill, v, 0x138, 0xF, 0xF, false);  // wave_shr:1
}
__device__ __forceinline__ int shl1_i(int fill, int v)
{
    return __builtin_amdgcn_update_dpp(fill, v, 0x130, 0xF, 0xF, false);  // wave_shl:1
}
// value held by lane l-1 (lane 0: fill)
__device__ __forceinline__ float from_left(float fill, float v)
{
    return __int_as_float(shr1_i(__float_as_int(fill), __float_as_int(v)));
}
// value held by lane l+1 (lane 63: fill)
__device__ __forceinline__ float from_right(float fill, float v)
{
    return __int_as_float(shl1_i(__float_as_int(fill), __float_as_int(v)));
}
__device__ __forceinline__ double from_left(double fill, double v)
{
    const long long b = __double_as_longlong(v), f = __double_as_longlong(fill);
    const int lo = shr1_i((int)(f & 0xffffffffll), (int)(b & 0xffffffffll));
    const int hi = shr1_i((int)(f >> 32), (int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double from_right(double fill, double v)
{
    const long long b = __double_as_longlong(v), f = __double_as_longlong(fill);
    const int lo = shl1_i((int)(f & 0xffffffffll), (int)(b & 0xffffffffll));
    const int hi = shl1_i((int)(f >> 32), (int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// The same shifts where the lane without a source may receive any value (a
// wave whose edges are open window edges: those points lie in the halo).
// bound_ctrl makes that lane read zero, so no fill operand has to be set up.
__device__ __forceinline__ int shr1z_i(int v) { return __builtin_amdgcn_mov_dpp(v, 0x138, 0xF, 0xF, true); }
__device__ __forceinline__ int shl1z_i(int v) { return __builtin_amdgcn_mov_dpp(v, 0x130, 0xF, 0xF, true); }
__device__ __forceinline__ float from_left_open(float v)
{
    return __int_as_float(shr1z_i(__float_as_int(v)));
}
__device__ __forceinline__ float from_right_open(float v)
{
    return __int_as_float(shl1z_i(__float_as_int(v)));
}
__device__ __forceinline__ double from_left_open(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = shr1z_i((int)(b & 0xffffffffll)), hi = shr1z_i((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double from_right_open(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = shl1z_i((int)(b & 0xffffffffll)), hi = shl1z_i((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// edge value from the left / right neighbour lane, with the fill used only
// when the wave's edge is not open
template <bool OPEN, typename T>
__device__ __forceinline__ T edge_left(T fill, T v)
{
    if constexpr (OPEN) return from_left_open(v);
    else return from_left(fill, v);
}
template <bool OPEN, typename T>
__device__ __forceinline__ T edge_right(T fill, T v)
{
    if constexpr (OPEN) return from_right_open(v);
    else return from_right(fill, v);
}

__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Raise a status word (StatusWord, ge_kernels.h): host-mapped memory of the
// plan, written with a plain system-scope store, so no read-modify-write
// crosses the bus.
__device__ __forceinline__ void raise_status(int *status, int word)
{
    __hip_atomic_store(status + word, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The stored values are tested as they are stored: acc + v * 0 over them
// stays 0 while they are finite and becomes NaN once one is NaN or infinite
// (one FMA per value, no compare).  Values a lane holds but does not store
// (halo points, points past a wall) are not tested: past a wall they are
// not part of the problem and may grow without bound.
template <typename T>
__device__ __forceinline__ void finite_acc(T &acc, T v)
{
    acc = fmaT(v, T(0), acc);
}

// Raise kStatusNonfinite if some lane's stored values were not all finite;
// at most one store per wave.  Called by every lane of the wave.
template <typename T>
__device__ __forceinline__ void raise_if_nonfinite(int *status, T acc)
{
    if (!status) return;
    const uint64_t m = __ballot(!__builtin_isfinite(acc));
    if (m != 0 && (threadIdx.x & (kWave - 1)) == (unsigned)__builtin_ctzll(m))
        raise_status(status, kStatusNonfinite);
}

// ---- 16-byte vector access to a lane's K contiguous values ----------------
// type: at a 16-byte boundary.  any: at the element's alignment, for a window
// that ends at a wall and may start at any element (a vector type, whose parts
// the compiler keeps in one tuple of registers: where it is not needed, it costs
// registers).
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef double double2_any __attribute__((ext_vector_type(2), aligned(8)));
template <typename T> struct V16;
template <> struct V16<float> {
    using type = float4;
    using any = float4_any;
    static constexpr int E = 4;
};
template <> struct V16<double> {
    using type = double2;
    using any = double2_any;
    static constexpr int E = 2;
};

template <typename T, int K>
__device__ __forceinline__ void load_lane(const T *__restrict__ p, T (&v)[K])
{
    using V = typename V16<T>::any;
    constexpr int E = V16<T>::E;
    constexpr int C = K / E;                      // whole chunks, then single values
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const V x = reinterpret_cast<const V *>(p)[c];
#pragma unroll
        for (int i = 0; i < E; ++i) v[c * E + i] = x[i];
    }
#pragma unroll
    for (int j = C * E; j < K; ++j) v[j] = p[j];
}

template <typename T, int K>
__device__ __forceinline__ void load_lane_guarded(const T *__restrict__ p, int64_t g0,
                                                  int64_t n, T (&v)[K])
{
    using V = typename V16<T>::type;
    constexpr int E = V16<T>::E;
    const V *q = reinterpret_cast<const V *>(p);
#pragma unroll
    for (int c = 0; c < K / E; ++c) {
        if (g0 + (c + 1) * E <= n) {
            const V x = q[c];
            if constexpr (E == 4) {
                v[4 * c] = x.x; v[4 * c + 1] = x.y; v[4 * c + 2] = x.z; v[4 * c + 3] = x.w;
            } else {
                v[2 * c] = x.x; v[2 * c + 1] = x.y;
            }
        } else {
#pragma unroll
            for (int i = 0; i < E; ++i)
                v[c * E + i] = (g0 + c * E + i < n) ? p[c * E + i] : T(0);
        }
    }
}

// Store the values whose global index lies in [lo, hi).  lo and hi are
// multiples of the chunk width on the fast path.
template <typename T, int K>
__device__ __forceinline__ void store_lane_chunks(T *__restrict__ p, int64_t g0, int64_t lo,
                                                  int64_t hi, const T (&v)[K], T &fin)
{
    using V = typename V16<T>::type;
    constexpr int E = V16<T>::E;
    V *q = reinterpret_cast<V *>(p);
#pragma unroll
    for (int c = 0; c < K / E; ++c) {
        const int64_t g = g0 + c * E;
        if (g >= lo && g < hi) {
#pragma unroll
            for (int i = 0; i < E; ++i) finite_acc(fin, v[c * E + i]);
            V x;
            if constexpr (E == 4) {
                x.x = v[4 * c]; x.y = v[4 * c + 1]; x.z = v[4 * c + 2]; x.w = v[4 * c + 3];
            } else {
                x.x = v[2 * c]; x.y = v[2 * c + 1];
            }
            q[c] = x;
        }
    }
}

// Store the values whose global index lies in [lo, hi), any lo and hi: whole
// 16-byte chunks where they lie inside, single values where one straddles.
template <typename T, int K>
__device__ __forceinline__ void store_lane_guarded(T *__restrict__ p, int64_t g0, int64_t lo,
                                                   int64_t hi, const T (&v)[K], T &fin)
{
    using V = typename V16<T>::any;
    constexpr int E = V16<T>::E;
#pragma unroll
    for (int c = 0; c < K; c += E) {
        if (c + E <= K && g0 + c >= lo && g0 + c + E <= hi) {
            V x;
#pragma unroll
            for (int i = 0; i < E; ++i) {
                finite_acc(fin, v[c + i]);
                x[i] = v[c + i];
            }
            *reinterpret_cast<V *>(p + c) = x;
        } else {
#pragma unroll
            for (int i = 0; i < E; ++i)
                if (c + i < K && g0 + c + i >= lo && g0 + c + i < hi) {
                    finite_acc(fin, v[c + i]);
                    p[c + i] = v[c + i];
                }
        }
    }
}

// Store the values whose global index lies in [lo, n), lo a multiple of the
// chunk width: whole 16-byte chunks where they lie below n, single values in the
// chunk that straddles n.
template <typename T, int K>
__device__ __forceinline__ void store_lane_range(T *__restrict__ p, int64_t g0, int64_t lo,
                                                 int64_t n, const T (&v)[K], T &fin)
{
    using V = typename V16<T>::type;
    constexpr int E = V16<T>::E;
    V *q = reinterpret_cast<V *>(p);
#pragma unroll
    for (int c = 0; c < K / E; ++c) {
        if (g0 + c * E < lo)
            continue;
        if (g0 + (c + 1) * E <= n) {
#pragma unroll
            for (int i = 0; i < E; ++i) finite_acc(fin, v[c * E + i]);
            V x;
            if constexpr (E == 4) {
                x.x = v[4 * c]; x.y = v[4 * c + 1]; x.z = v[4 * c + 2]; x.w = v[4 * c + 3];
            } else {
                x.x = v[2 * c]; x.y = v[2 * c + 1];
            }
            q[c] = x;
        } else {
#pragma unroll
            for (int i = 0; i < E; ++i)
                if (g0 + c * E + i < n) {
                    finite_acc(fin, v[c * E + i]);
                    p[c * E + i] = v[c * E + i];
                }
        }
    }
}

// Store the values whose global index is below n: whole 16-byte chunks
// where they lie below n, single values in the chunk that straddles n.
template <typename T, int K>
__device__ __forceinline__ void store_lane_upto(T *__restrict__ p, int64_t g0, int64_t n,
                                                const T (&v)[K], T &fin)
{
    using V = typename V16<T>::type;
    constexpr int E = V16<T>::E;
    V *q = reinterpret_cast<V *>(p);
#pragma unroll
    for (int c = 0; c < K / E; ++c) {
        if (g0 + (c + 1) * E <= n) {
#pragma unroll
            for (int i = 0; i < E; ++i) finite_acc(fin, v[c * E + i]);
            V x;
            if constexpr (E == 4) {
                x.x = v[4 * c]; x.y = v[4 * c + 1]; x.z = v[4 * c + 2]; x.w = v[4 * c + 3];
            } else {
                x.x = v[2 * c]; x.y = v[2 * c + 1];
            }
            q[c] = x;
        } else {
#pragma unroll
            for (int i = 0; i < E; ++i)
                if (g0 + c * E + i < n) {
                    finite_acc(fin, v[c * E + i]);
                    p[c * E + i] = v[c * E + i];
                }
        }
    }
}

// Access to element k of a lane's register tile for a wave-uniform k, as a
// switch: one scalar branch tree and a single move per call.  (An equality
// chain over the tile would be folded into one dynamically indexed access,
// which for tiles above 32 registers goes through scratch memory.)
#define GE_CASES8(b) GE_C(b + 0) GE_C(b + 1) GE_C(b + 2) GE_C(b + 3) \
    GE_C(b + 4) GE_C(b + 5) GE_C(b + 6) GE_C(b + 7)
#define GE_CASES64 GE_CASES8(0) GE_CASES8(8) GE_CASES8(16) GE_CASES8(24) \
    GE_CASES8(32) GE_CASES8(40) GE_CASES8(48) GE_CASES8(56)

// v[k] = x in the lanes where `pred` holds (k outside [0, K): no change).
template <typename T, int K>
__device__ __forceinline__ void put_at(T (&v)[K], int k, bool pred, T x)
{
    static_assert(K <= 64, "tiles are at most 64 values per lane");
    switch (k) {
#define GE_C(i) \
    case i: \
        if constexpr ((i) < K) v[i] = pred ? x : v[i]; \
        break;
        GE_CASES64
#undef GE_C
    default: break;
    }
}

// v[k] (k outside [0, K): `otherwise`).
template <typename T, int K>
__device__ __forceinline__ T get_at(const T (&v)[K], int k, T otherwise)
{
    T r = otherwise;
    switch (k) {
#define GE_C(i) \
    case i: \
        if constexpr ((i) < K) r = v[i]; \
        break;
        GE_CASES64
#undef GE_C
    default: break;
    }
    return r;
}


// Wall value split for the state type: (hi, lo) with hi + lo ~ g.
template <typename T, bool COMP>
__device__ __forceinline__ void split_wall(double g, T &hi, T &lo)
{
    hi = (T)g;
    lo = COMP ? (T)(g - (double)hi) : T(0);
}

// Constants of the scheme in the state's type.
template <typename T> struct Coef {
    T r, k;     // r, r/(1+2r): FP64
    T c1, c2;   // (r+r^2)/(1+2r), r^2/(1+2r): FP32
    T cs;       // r/(1+r)
};

// The coefficients as the level loop reads them.  For FP32 they are moved
// to vector registers once: measured on MI355X, chains of FP32 VALU
// instructions with a scalar-register operand issued at half the rate of
// the same chains with vector-register operands only (no packed forms in
// either).  FP64 instructions issue at one rate either way.
template <typename T>
__device__ __forceinline__ Coef<T> lane_coef(Coef<T> c)
{
    if constexpr (sizeof(T) == 4) asm("" : "+v"(c.c1), "+v"(c.c2), "+v"(c.cs));
    return c;
}

// Constants of the compensated pair's form.
template <typename T> struct PairCoef {
    T c1, c2, cs;   // (r+r^2)/(1+2r), r^2/(1+2r), r/(1+r)
    T e1, e2, es;   // tau(1+r)/(1+2r), tau r/(1+2r), tau/(1+r)
};
template <typename T>
__device__ __forceinline__ PairCoef<T> lane_coef(PairCoef<T> c)
{
    asm("" : "+v"(c.c1), "+v"(c.c2), "+v"(c.cs), "+v"(c.e1), "+v"(c.e2), "+v"(c.es));
    return c;
}

// ---- the two stages of a level (FP64) ---------------------------------------
// The lane's K points (K even) in place.  Parity P couples (2q, 2q+1) inside
// the lane when P = 0 and across lanes when P = 1; the explicit stage runs
// over the other parity's pairs.  xl, xr: the values left of lane 0 and right
// of lane 63 (OL, OR: that side is an open window edge and takes no value).
template <typename T, int K, int P, bool OL, bool OR>
__device__ __forceinline__ void explicit_stage(T (&u)[K], T xl, T xr, const Coef<T> &c)
{
    if constexpr (P == 0) {
        const T ul = edge_left<OL>(xl, u[K - 1]), ur = edge_right<OR>(xr, u[0]);
        u[0] = fmaT(-c.r, u[0] - ul, u[0]);
#pragma unroll
        for (int j = 1; j + 1 < K; j += 2) {
            const T d = u[j + 1] - u[j];
            u[j] = fmaT(c.r, d, u[j]);
            u[j + 1] = fmaT(-c.r, d, u[j + 1]);
        }
        u[K - 1] = fmaT(c.r, ur - u[K - 1], u[K - 1]);
    } else {
#pragma unroll
        for (int j = 0; j < K; j += 2) {
            const T d = u[j + 1] - u[j];
            u[j] = fmaT(c.r, d, u[j]);
            u[j + 1] = fmaT(-c.r, d, u[j + 1]);
        }
    }
}

// kl, kr: the coefficient of the lane's first and last point at P = 1 (k, or
// cs in the lane whose point stands alone beside a wall).
template <typename T, int K, int P, bool OL, bool OR>
__device__ __forceinline__ void solve_stage(T (&v)[K], T xl, T xr, const Coef<T> &c, T kl, T kr)
{
    if constexpr (P == 0) {
#pragma unroll
        for (int j = 0; j < K; j += 2) {
            const T w = v[j + 1] - v[j];
            v[j] = fmaT(c.k, w, v[j]);
            v[j + 1] = fmaT(-c.k, w, v[j + 1]);
        }
    } else {
        const T vl = edge_left<OL>(xl, v[K - 1]), vr = edge_right<OR>(xr, v[0]);
        v[0] = fmaT(-kl, v[0] - vl, v[0]);
#pragma unroll
        for (int j = 1; j + 1 < K; j += 2) {
            const T w = v[j + 1] - v[j];
            v[j] = fmaT(c.k, w, v[j]);
            v[j + 1] = fmaT(-c.k, w, v[j + 1]);
        }
        v[K - 1] = fmaT(kr, vr - v[K - 1], v[K - 1]);
    }
}

// The source term ta b of every point, ta = tau a(t_m + tau/2).
template <typename T, int K>
__device__ __forceinline__ void source_stage(T (&v)[K], const T (&b)[K], T ta)
{
#pragma unroll
    for (int j = 0; j < K; ++j) v[j] = fmaT(ta, b[j], v[j]);
}

// A point alone beside a wall (a wall node at a run-time position): its new
// value from its v and the wall's new value, as solve_stage forms it.
template <typename T>
__device__ __forceinline__ T lone_point(T v, T g, T cs)
{
    return fmaT(cs, g - v, v);
}

// ---- the increment form (FP32) ---------------------------------------------
// The source weights of the lane's points at parity P, e1 b_i + e2 b_q, q the
// partner of i (neighbouring lanes' points through bl = b_{-1}, br = b_K: 0 at a
// wall, whose lone point has no partner).  el, er: e1 of the lane's first and
// last point at P = 1, es in the lane whose point stands alone beside a wall.
template <typename T, int K, int P>
__device__ __forceinline__ void increment_source(const T (&b)[K], T bl, T br, T e1, T e2, T el,
                                                 T er, T (&B)[K])
{
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const int q = ((j + P) & 1) == 0 ? j + 1 : j - 1;
        B[j] = fmaT(q < 0 ? el : q == K ? er : e1, b[j], e2 * (q < 0 ? bl : q == K ? br : b[q]));
    }
}

// One level of parity P of the lane's K points.  xl, xl2, xr, xr2: u_{-1},
// u_{-2}, u_K, u_{K+1} for lanes 0 / 63 (unused on an open side).  Beside a wall xl
// (xr) is its old value at P = 0 and its new one at P = 1, xl2 (xr2) any
// finite value, and cl, pl (cr, pr), the factors of the lane's first (last)
// point at P = 1, are cs and 0 in place of c1 and c2.
template <typename T, int K, bool SRC, int P, bool OL, bool OR>
__device__ __forceinline__ void increment_level(T (&u)[K], const T (&B)[K], T an, T xl, T xl2, T xr,
                                                T xr2, const Coef<T> &c, T cl, T pl, T cr, T pr)
{
    const T ul = edge_left<OL>(xl, u[K - 1]), ur = edge_right<OR>(xr, u[0]);
    // u_j from the factors f, g of its own and its partner's second difference
    auto upd = [&](int j, T D, T Dq, T f, T g) {
        T inc = fmaT(f, D, g * Dq);
        if constexpr (SRC) inc = fmaT(an, B[j], inc);
        u[j] = u[j] + inc;
    };
    if constexpr (P == 0) {
        T dprev = u[0] - ul;
#pragma unroll
        for (int j = 0; j < K; j += 2) {
            const T d0 = u[j + 1] - u[j];
            const T d1 = (j + 2 < K ? u[j + 2] : ur) - u[j + 1];
            const T Da = d0 - dprev, Db = d1 - d0;
            upd(j, Da, Db, c.c1, c.c2);
            upd(j + 1, Db, Da, c.c1, c.c2);
            dprev = d1;
        }
    } else {
        // pairs (-1,0), (1,2), ..., (K-1,K): the partners' second differences
        // of the lane's edge points come from the lanes beside
        const T dm = u[0] - ul, d0 = u[1] - u[0];
        const T dk = u[K - 1] - u[K - 2], dr = ur - u[K - 1];
        const T D0 = d0 - dm, DK = dr - dk;
        T fl = T(0), fr = T(0);
        if constexpr (!OL) fl = dm - (xl - xl2);
        if constexpr (!OR) fr = (xr2 - xr) - dr;
        const T Dl = edge_left<OL>(fl, DK), Dr = edge_right<OR>(fr, D0);
        T dprev = d0;
#pragma unroll
        for (int j = 1; j + 1 < K; j += 2) {
            const T da = u[j + 1] - u[j], db = u[j + 2] - u[j + 1];
            const T Da = da - dprev, Db = db - da;
            if (j == 1) upd(0, D0, Dl, cl, pl);
            upd(j, Da, Db, c.c1, c.c2);
            upd(j + 1, Db, Da, c.c1, c.c2);
            dprev = db;
        }
        if constexpr (K == 2) upd(0, D0, Dl, cl, pl);
        upd(K - 1, DK, Dr, cr, pr);
    }
}

// The point alone beside a right wall node at a run-time position: element
// kS of its lane, u_{n-2} before it (xl: the fill of lane 0); g: the wall's
// new value; b: the source profile.
template <typename T, int K, bool SRC>
__device__ __forceinline__ T lone_increment(const T (&u)[K], const T (&b)[K], T an, int kS, T xl,
                                            T g, T cs, T es)
{
    const T ul = from_left(xl, u[K - 1]);
    const T u1 = get_at<T, K>(u, kS, T(0)), u0 = get_at<T, K>(u, kS - 1, ul);
    T inc = cs * ((g - u1) - (u1 - u0));
    if constexpr (SRC) inc = fmaT(an, es * get_at<T, K>(b, kS, T(0)), inc);
    return u1 + inc;
}

// ---- the compensated pair (COMP), and FP32 in the persistent batch form and in
// open windows without a source ----
// A first difference of two points given as (s, e).  The s and e parts stay
// apart: for smooth data the s differences (and their differences) are
// exact, and summing the s and e second differences only at the end keeps D
// accurate to the precision of the pair.
template <typename T, bool COMP> struct Dif { T s; };
template <typename T> struct Dif<T, true> { T s, e; };

template <bool COMP = true, typename T>
__device__ __forceinline__ Dif<T, COMP> dif(T s1, T e1, T s0, T e0)
{
    if constexpr (COMP) return Dif<T, COMP>{s1 - s0, e1 - e0};
    else return Dif<T, COMP>{s1 - s0};
}

// second difference D = db - da from consecutive first differences
template <typename T, bool COMP>
__device__ __forceinline__ T sd(Dif<T, COMP> da, Dif<T, COMP> db)
{
    if constexpr (COMP) return (db.s - da.s) + (db.e - da.e);
    else return db.s - da.s;
}

// What a level needs to know about the left wall, seen from one lane (the
// right wall, at a data-dependent element, is handled by right_lone /
// put_at around the level).
template <typename T> struct WallLevel {
    bool isL;       // this lane's point 0 is the lone point at the left wall now
    T dgl;          // g_L(t_{m+1}) - g_L(t_m)
};

// Optional FP64 wall-flux accumulation at the left wall (first difference
// tau (u_1 - g_L)/h at every new level); the right wall's is taken by the
// caller after the level.
struct FluxTap {
    bool left;             // this lane owns the left accumulation
    double accL;
    double tau, h, gln;
};

// The source weight of every point of the lane at parity P,
// B_i = e1 b_i + e2 b_q with q the partner of i (neighbouring lanes' points
// through bl = b_{-1}, br = b_K), formed by the same expression the
// per-level update uses; a launch's profile is fixed, so these are formed
// once per launch and each level adds a(t) B_i with one FMA.
template <typename T, int K, int P>
__device__ __forceinline__ void source_weights(const T (&b)[K], T bl, T br, const PairCoef<T> &c,
                                               T (&B)[K])
{
    if constexpr (P == 0) {
#pragma unroll
        for (int q = 0; q < K / 2; ++q) {
            B[2 * q] = fmaT(c.e1, b[2 * q], c.e2 * b[2 * q + 1]);
            B[2 * q + 1] = fmaT(c.e1, b[2 * q + 1], c.e2 * b[2 * q]);
        }
    } else {
        B[0] = fmaT(c.e1, b[0], c.e2 * bl);
#pragma unroll
        for (int q = 1; q < K / 2; ++q) {
            const int j = 2 * q - 1;
            B[j] = fmaT(c.e1, b[j], c.e2 * b[j + 1]);
            B[j + 1] = fmaT(c.e1, b[j + 1], c.e2 * b[j]);
        }
        B[K - 1] = fmaT(c.e1, b[K - 1], c.e2 * br);
    }
}

// Advance the K points of every lane by one level of parity P (known at
// compile time: a runtime parity would merge the two groupings' results for
// every point each level and cost the register file).
//   s, e : the lane's points (e is the compensation; not read without COMP)
//   b    : SRC = 1: the lane's source profile, bl, br: profile of u_{-1}
//          and u_K; SRC = 2: the weights of this parity (source_weights)
//   xl, xl2, xr, xr2 : u_{-1}, u_{-2}, u_K, u_{K+1} for lanes 0 / 63 (DPP
//          fill from the neighbouring waves, a wall value, or anything at
//          an open window edge); yl.. the same for e
// WALL instantiations apply the lone-point formulas and the flux tap; every
// other point of every instantiation evaluates the same expressions.  OPEN:
// both edges of the wave are open window edges, so the fills are not used.
// Without COMP a point gets the operations that increment_level gives it.
template <typename T, int K, int SRC, bool WALL, int P, bool OPEN = false, bool COMP = true>
__device__ __forceinline__ void pair_level(T (&s)[K], T (&e)[K], const T (&b)[K], T bl, T br,
                                           T xl, T xl2, T xr, T xr2, T yl, T yl2, T yr, T yr2,
                                           const PairCoef<T> &c, T an, const WallLevel<T> &wl,
                                           FluxTap &ft)
{
    static_assert(!(WALL && SRC == 2), "wall tiles take the source from the profile");
    const T c1 = c.c1, c2 = c.c2, cs = c.cs, e1 = c.e1, e2 = c.e2, es = c.es;
    // u_{-1} and u_K: neighbour lanes' edge points
    const T sl = edge_left<OPEN>(xl, s[K - 1]), sr = edge_right<OPEN>(xr, s[0]);
    T el = T(0), er = T(0);
    if constexpr (COMP) {
        el = edge_left<OPEN>(yl, e[K - 1]);
        er = edge_right<OPEN>(yr, e[0]);
    }
    auto dif = [](T s1, T e1_, T s0, T e0) { return ::ge::dev::dif<COMP>(s1, e1_, s0, e0); };

    // advance point j from D_self and D_partner (bp: partner's profile)
    auto upd = [&](int j, T Ds, T Dp, T bp) {
        T inc = fmaT(c1, Ds, c2 * Dp);
        if constexpr (SRC == 1) inc = fmaT(an, fmaT(e1, b[j], e2 * bp), inc);
        if constexpr (SRC == 2) inc = fmaT(an, b[j], inc);
        if constexpr (WALL) {
            if (j == 0) {
                T alt = cs * (Ds + wl.dgl);
                if constexpr (SRC) alt = fmaT(an, es * b[j], alt);
                inc = wl.isL ? alt : inc;
            }
        }
        if constexpr (COMP) {
            // Kahan: the pair absorbs the increment, e keeps what s lost
            const T y = inc + e[j];
            const T tt = s[j] + y;
            e[j] = y - (tt - s[j]);
            s[j] = tt;
        } else {
            s[j] = s[j] + inc;
        }
        if constexpr (WALL) {
            // wall first differences at the new level, accumulated in FP64
            if (ft.left && j == 0) {
                const double v = (double)s[j] + (COMP ? (double)e[j] : 0.0);
                ft.accL = ft.accL + ft.tau * (v - ft.gln) / ft.h;
            }
        }
    };

    if constexpr (P == 0) {
        // pairs (2q, 2q+1) inside the lane
        auto dprev = dif(s[0], e[0], sl, el);                       // d_{-1}
#pragma unroll
        for (int q = 0; q < K / 2; ++q) {
            const int j = 2 * q;
            const auto d0 = dif(s[j + 1], e[j + 1], s[j], e[j]);    // d_j
            const auto d1 = (j + 2 < K) ? dif(s[j + 2], e[j + 2], s[j + 1], e[j + 1])
                                        : dif(sr, er, s[j + 1], e[j + 1]);
            const T Da = sd(dprev, d0), Db = sd(d0, d1);
            upd(j, Da, Db, b[j + 1]);
            upd(j + 1, Db, Da, b[j]);
            dprev = d1;
        }
    } else {
        // pairs (-1,0), (1,2), ..., (K-1,K): the lane's edge points pair
        // with the neighbouring lanes' edge points, so u_{-2} and u_{K+1}
        // are needed too
        const T sl2 = edge_left<OPEN>(xl2, s[K - 2]), sr2 = edge_right<OPEN>(xr2, s[1]);
        T el2 = T(0), er2 = T(0);
        if constexpr (COMP) {
            el2 = edge_left<OPEN>(yl2, e[K - 2]);
            er2 = edge_right<OPEN>(yr2, e[1]);
        }
        const auto dm2 = dif(sl, el, sl2, el2);                     // d_{-2}
        const auto dm1 = dif(s[0], e[0], sl, el);                   // d_{-1}
        const auto d0 = dif(s[1], e[1], s[0], e[0]);                // d_0
        const auto dK1 = dif(sr, er, s[K - 1], e[K - 1]);           // d_{K-1}
        const auto dK = dif(sr2, er2, sr, er);                      // d_K
        const auto dK2 = dif(s[K - 1], e[K - 1], s[K - 2], e[K - 2]);  // d_{K-2}
        upd(0, sd(dm1, d0), sd(dm2, dm1), bl);
        auto dprev = d0;
#pragma unroll
        for (int q = 1; q < K / 2; ++q) {
            const int j = 2 * q - 1;
            const auto da = dif(s[j + 1], e[j + 1], s[j], e[j]);   // d_j
            const auto db = dif(s[j + 2], e[j + 2], s[j + 1], e[j + 1]);  // d_{j+1}
            const T Da = sd(dprev, da), Db = sd(da, db);
            upd(j, Da, Db, b[j + 1]);
            upd(j + 1, Db, Da, b[j]);
            dprev = db;
        }
        upd(K - 1, sd(dK2, dK1), sd(dK1, dK), br);
    }
}

// The lone point n-1 beside the right wall (scheme B, Eq. (2), in the
// second-difference form): its new value from the level's old values.  It
// sits at element kS of lane lS; u_{n-2} is element kS-1, or for kS = 0 the
// last element of the lane to the left (xl/yl: that lane's fill value for
// lane 0).  g_hi/g_lo: the wall value at t_m as state values; dgr:
// g_R(t_{m+1}) - g_R(t_m).  The arithmetic is the per-point update's.
template <typename T> struct Lone { T s, e; };

template <typename T, int K, bool SRC, bool COMP = true>
__device__ __forceinline__ Lone<T> right_lone(const T (&s)[K], const T (&e)[K], const T (&b)[K],
                                              int kS, T xl, T yl, T g_hi, T g_lo, T dgr,
                                              const PairCoef<T> &c, T an)
{
    const T sl = from_left(xl, s[K - 1]);
    const T el = COMP ? from_left(yl, e[K - 1]) : T(0);
    const T u1 = get_at<T, K>(s, kS, T(0));
    const T e1 = COMP ? get_at<T, K>(e, kS, T(0)) : T(0);
    const T u0 = get_at<T, K>(s, kS - 1, sl);
    const T e0 = COMP ? get_at<T, K>(e, kS - 1, el) : T(0);
    const T Ds = sd(dif<COMP>(u1, e1, u0, e0), dif<COMP>(g_hi, g_lo, u1, e1));
    T inc = c.cs * (Ds + dgr);
    if constexpr (SRC) inc = fmaT(an, c.es * get_at<T, K>(b, kS, T(0)), inc);
    if constexpr (!COMP) return Lone<T>{u1 + inc, T(0)};
    const T y = inc + e1;
    const T tt = u1 + y;
    return Lone<T>{tt, y - (tt - u1)};
}

// Run levels level0 .. level0+nlev-1 as f(parity, lev) with the parity a
// compile-time constant: an odd first level alone, then even/odd pairs, then
// a last even level if one is left.
template <int V> struct Par { static constexpr int value = V; };

template <typename F>
__device__ __forceinline__ void for_levels(int64_t level0, int nlev, F &&f)
{
    int lev = 0;
    if ((level0 & 1) && nlev > 0) {
        f(Par<1>{}, 0);
        lev = 1;
    }
    for (; lev + 1 < nlev; lev += 2) {
        f(Par<0>{}, lev);
        f(Par<1>{}, lev + 1);
    }
    if (lev < nlev)
        f(Par<0>{}, lev);
}

}  // namespace dev
}  // namespace ge

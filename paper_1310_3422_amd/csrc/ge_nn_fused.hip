// The surrogate's 64-level jump with all six layers fused: one workgroup
// takes a tile of points of one rod from u to u_next, keeping every
// activation in LDS, so HBM sees only u (read) and u_next (written) -- the
// layer-by-layer path writes and re-reads 128 bytes per point per layer.
//
// A layer of tap spacing d reads its input 2d rows either side, so a tile of
// P points is computed from rows up to kFHalo = 64 beyond each side; a layer
// is computed only where the layers after it (twice the sum of their
// spacings) will read it, and only inside the rod: rows outside it hold
// zeros from the start, which is the zero padding of the layer-by-layer
// path.  The arithmetic (the features, the MFMA accumulation order, the
// epilogues and the jump) is the same expression sequence as the
// layer-by-layer kernels, so both paths give the same bits.
//
// Blocks of 64 rows are dealt to two teams of four waves; a wave of a team
// takes 16 of the 64 output channels, holds its quarter of the layer's
// weights in registers (10 fragments) and loads the next layer's a whole
// layer ahead.  The 16 positions of a matrix instruction need not be
// neighbours: tile t of a block is the rows S + d t, S = {4 d i + j, j < d}, so
// that tile t's tap k is tile t + k - 2, and eight fragments serve the
// block's four tiles of five taps (20 without).  The new values stay in
// registers until every wave has read its inputs and then go to LDS in place.
//
// What bounds it is issue on the SIMDs: a GELU with its bias, residual and
// conversion takes 8.5 vector instructions and two transcendentals of twice
// the time, and the matrix instructions' time adds to theirs: leaving the one
// or the other out (each measured alone) saves what it costs, whether the
// two are interleaved instruction by instruction, in groups, or left to the
// two waves of a SIMD.  So the rows count (a tile of up to 864 points where
// 512 were taken: 1.14 computed per point against 1.25), and no wave waits
// for weights (with 32 channels a wave, which has no registers for the next
// layer's, the same time at 4096 points and 500 rods, 8% more at 64 rods of
// 2048 points).  4096 points, 1024 rods: 1251 -> 1090 us; 512 points, 64
// rods 46 -> 30; 4096 points, one rod
// 45 -> 24; where 512-point tiles filled the chip exactly once or twice, 1-4%
// slower (3072 points, 80 rods: 96.5 -> 100).
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "ge_nn.h"
#include "ge_nn_dev.h"

namespace ge {
namespace nn {
namespace {

using namespace dev;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kFHalo = 64;                 // rows beyond each side (2 x sum of spacings at most)
constexpr int kFPad = 2 * kMaxDil;         // LDS rows beyond the computed rows on each side
constexpr int kFTeams = 2;                 // teams of four waves
constexpr int kFThreads = 4 * kFTeams * 64;
constexpr int kFB = 4;                     // 16-row tiles per block
constexpr int kFBlock = 16 * kFB;          // rows per block
constexpr int kFMine = 8;                  // blocks per team at most
constexpr int kFMaxRows = kFBlock * kFTeams * kFMine;
constexpr int kFRows = kFMaxRows + 2 * kFPad;
// Points per workgroup at most.  A layer's blocks end at most 63 rows past
// those that it needs, reach rows beyond the tile, and read 2d further, where
// reach + 2d <= kFHalo: P + 2 kFHalo + 63 <= kFMaxRows + kFPad.
constexpr int kFMaxP = kFMaxRows + kFPad - 2 * kFHalo - kFBlock;
constexpr int kFFrags = kFB + kTaps - 1;   // fragments that serve a block
constexpr int kFCU = 256;
constexpr int kFFixed = 4;                 // a workgroup's fixed cost, in blocks (measured)

// LDS row i holds position w0 - kFHalo - kFPad + i; computed row q is LDS
// row q + kFPad.  A row is 64 channels in eight 16-byte chunks, permuted by
// XOR with three bits of the row chosen so that the rows of a fragment lie
// in different banks for every spacing: a fragment's rows differ in row bits
// (0,1,2,3) for d = 16, (0,1,2,5), (0,1,4,5), (0,3,4,5), (2,3,4,5) for d = 1;
// the first three of each set (and the first two with the sum of the third
// and fourth, the hardware's other grouping of lanes) map to independent
// values.  Bits from 6 on do not enter, so a block further is a constant
// further.
__device__ __forceinline__ int chunk_at(int row, int chunk)
{
    const int f = (row ^ ((row >> 2) & 2) ^ ((row >> 4 & 1) * 5)) & 7;
    return row * 64 + ((chunk ^ f) * 8);
}

template <int I, int N, typename F>
__device__ __forceinline__ void unroll_steps(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unroll_steps<I + 1, N>(f);
    }
}

// A wave's weights of one layer in registers, the A operand of the
// transposed product (each lane ends with four output channels of one
// position).  Row m is output channel c0 + 8 (m / 4) + m % 4, so that a lane's
// channels lie in the chunk that it reads of the layer's input.  The last
// layer has its 16 rows in their own order.
template <int KC>
struct WeightFrags {
    bf16x8 v[kTaps][KC];
    __device__ __forceinline__ void load(const void *wt, int cout, int row, int lane)
    {
        const bf16 *p = static_cast<const bf16 *>(wt) + row * (32 * KC) + 8 * (lane >> 4);
#pragma unroll
        for (int k = 0; k < kTaps; ++k)
#pragma unroll
            for (int c = 0; c < KC; ++c)
                v[k][c] = *reinterpret_cast<const bf16x8 *>(&p[k * cout * (32 * KC) + 32 * c]);
        // keep the loads here, ahead of the work that hides them
        __builtin_amdgcn_sched_barrier(0);
    }
};

// What a layer computes: `count` blocks from row `lo` on (computed rows)
struct Blocks {
    int lo, count;
};

// The lane's row of tile 0 within a block, for spacing d (a power of two)
__device__ __forceinline__ int lane_row(int r16, int d)
{
    const int s = __builtin_ctz(d);
    return ((r16 >> s) << (s + 2)) | (r16 & (d - 1));
}

// A wave's place in the workgroup
struct Place {
    int lane, team, quarter;
    int c0;      // the lane's first output channel: four from there
};

// The LDS places of the lane's chunk (of the first 32 channels) of the
// fragments of the team's first block: tiles t0 - 2 and on
template <int N>
__device__ __forceinline__ void fragment_places(const Place &pl, int d, int lo, int t0,
                                                int (&at)[N])
{
    const int row = lo + kFBlock * pl.team + lane_row(pl.lane & 15, d) + kFPad;
#pragma unroll
    for (int f = 0; f < N; ++f) at[f] = chunk_at(row + (t0 + f - 2) * d, pl.lane >> 4);
}

// ... and of the lane's four channels in the block's tiles
__device__ __forceinline__ void own_places(const Place &pl, int d, int lo, int (&at)[kFB])
{
    const int row = lo + kFBlock * pl.team + lane_row(pl.lane & 15, d) + kFPad;
#pragma unroll
    for (int t = 0; t < kFB; ++t) at[t] = chunk_at(row + t * d, pl.c0 / 8) + pl.c0 % 8;
}

// half of a team's blocks further
template <int N>
__device__ __forceinline__ void advance(int (&at)[N])
{
#pragma unroll
    for (int f = 0; f < N; ++f) {
        at[f] += kFTeams * (kFMine / 2) * kFBlock * 64;
        asm("" : "+v"(at[f]));
    }
}

__device__ __forceinline__ bf16x8 chunk_of(const bf16 *act, int at, int c, int blocks)
{
    // the chunk of the other 32 channels lies 4 chunks away, by XOR
    return *reinterpret_cast<const bf16x8 *>(&act[(at ^ (32 * c)) + blocks * kFBlock * 64]);
}

// gelu() of two values, in turn: a transcendental's result may not be used by
// the next instruction, so each has the other's in between
__device__ __forceinline__ void gelu_two(float z0, float z1, float &h0, float &h1)
{
    const float p0 = z0 * fmaf(z0 * z0, kGeluE2, kGeluE0);
    const float p1 = z1 * fmaf(z1 * z1, kGeluE2, kGeluE0);
    const float e0 = __builtin_amdgcn_exp2f(p0);
    const float e1 = __builtin_amdgcn_exp2f(p1);
    __builtin_amdgcn_sched_barrier(0);
    const float s0 = 1.0f + e0, s1 = 1.0f + e1;
    __builtin_amdgcn_sched_barrier(0);
    const float r0 = __builtin_amdgcn_rcpf(s0);
    const float r1 = __builtin_amdgcn_rcpf(s1);
    __builtin_amdgcn_sched_barrier(0);
    h0 = z0 * r0;
    h1 = z1 * r1;
}

// A GELU layer for the team's blocks: matrix work (taps outer, channel
// chunks inner, the order of conv_kernel), bias, GELU and the residual
// (layers 2..5), into registers as four bfloat16 channels per lane and tile.
template <int KC, bool RES>
__device__ __forceinline__ void gelu_layer(const bf16 *act, const WeightFrags<KC> &w,
                                           const float *bias, int d, const Place &pl, Blocks need,
                                           bf16x4 (&out)[kFMine][kFB])
{
    const f32x4 bl = *reinterpret_cast<const f32x4 *>(&bias[pl.c0]);
    int at[kFFrags], old[kFB];
    fragment_places(pl, d, need.lo, 0, at);
    if constexpr (RES) own_places(pl, d, need.lo, old);
#pragma unroll
    for (int i = 0; i < kFMine; ++i) {
        if (i == kFMine / 2) {
            // the rest lies beyond the reach of an LDS instruction's offset
            advance(at);
            if constexpr (RES) advance(old);
        }
        if (pl.team + kFTeams * i < need.count) {
            constexpr int kHalf = kFMine / 2;
            bf16x8 fr[kFFrags][KC];
            bf16x4 own[kFB];
            f32x4 acc[kFB], h;
            auto fetch = [&](int f) {
#pragma unroll
                for (int c = 0; c < KC; ++c) fr[f][c] = chunk_of(act, at[f], c, kFTeams * (i % kHalf));
            };
            // two values of tile t's epilogue: channels 2 Q, 2 Q + 1
            auto piece = [&](auto tt, auto qq) {
                constexpr int t = decltype(tt)::value, Q = decltype(qq)::value;
                float h0, h1;
                gelu_two(acc[t][2 * Q] + bl[2 * Q], acc[t][2 * Q + 1] + bl[2 * Q + 1], h0,
                         h1);
                if constexpr (RES) {
                    h0 += bf2f(own[t][2 * Q]);
                    h1 += bf2f(own[t][2 * Q + 1]);
                }
                h[2 * Q] = h0;
                h[2 * Q + 1] = h1;
                if constexpr (Q == 1) {
                    // two values per conversion instruction (round to nearest even)
                    out[i][t] = __builtin_convertvector(h, bf16x4);
                    // here, and not where it is stored
                    asm volatile("" : "+v"(out[i][t]));
                }
            };
#pragma unroll
            for (int f = 0; f <= kTaps; ++f) fetch(f);
            __builtin_amdgcn_sched_barrier(0);
            // two tiles at a time: consecutive matrix instructions do not
            // wait for each other
            unroll_steps<0, kFB / 2>([&](auto tt) {
                constexpr int t = 2 * decltype(tt)::value;
                acc[t] = acc[t + 1] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (t + 2 < kFB) {
                    fetch(t + kTaps + 1);
                    fetch(t + kTaps + 2);
                }
                if constexpr (RES)
#pragma unroll
                    for (int x = t; x < t + 2; ++x)
                        own[x] = *reinterpret_cast<const bf16x4 *>(
                            &act[old[x] + kFTeams * (i % kHalf) * kFBlock * 64]);
                unroll_steps<0, kTaps>([&](auto kk) {
                    constexpr int k = decltype(kk)::value;
#pragma unroll
                    for (int c = 0; c < KC; ++c)
#pragma unroll
                        for (int x = t; x < t + 2; ++x)
                            acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                w.v[k][c], fr[x + k][c], acc[x], 0, 0, 0);
                    if constexpr (t > 0 && k < 4)
                        piece(std::integral_constant<int, t - 2 + k / 2>{},
                              std::integral_constant<int, k % 2>{});
                });
            });
            unroll_steps<0, 4>([&](auto qq) {
                constexpr int q = decltype(qq)::value;
                piece(std::integral_constant<int, kFB - 2 + q / 2>{},
                      std::integral_constant<int, q % 2>{});
            });
        }
    }
}

// The layer's values in place; rows outside the rod [in_lo, in_hi), in
// computed rows, are zero
__device__ __forceinline__ void store_layer(bf16 *act, const bf16x4 (&out)[kFMine][kFB], int d,
                                            const Place &pl, Blocks need, int in_lo, int in_hi)
{
    const int row0 = need.lo + kFBlock * pl.team + lane_row(pl.lane & 15, d);
    int at[kFB];
    own_places(pl, d, need.lo, at);
    const bf16 z = f2bf(0.f);
    const bf16x4 zero{z, z, z, z};
#pragma unroll
    for (int i = 0; i < kFMine; ++i) {
        if (i == kFMine / 2) advance(at);
        const int block = pl.team + kFTeams * i;
        if (block < need.count) {
            // wave-uniform: only the blocks at a rod's ends test
            const int q0 = need.lo + kFBlock * block;
            const bool inside = q0 >= in_lo && q0 + kFBlock <= in_hi;
#pragma unroll
            for (int t = 0; t < kFB; ++t) {
                bf16x4 *place =
                    reinterpret_cast<bf16x4 *>(
                        &act[at[t] + kFTeams * (i % (kFMine / 2)) * kFBlock * 64]);
                if (inside) {
                    *place = out[i][t];
                } else {
                    const int q = row0 + t * d + kFBlock * kFTeams * i;
                    *place = q >= in_lo && q < in_hi ? out[i][t] : zero;
                }
            }
        }
    }
}

// P <= kFMaxP points per workgroup
__global__ __launch_bounds__(kFThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void jump_fused_kernel(FusedArgs a, int P)
{
    __shared__ __attribute__((aligned(16))) bf16 act[kFRows * 64];
    __shared__ __attribute__((aligned(16))) float bias[6][64];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = blockIdx.y;
    const int W = a.width;
    const int w0 = blockIdx.x * P;
    const int64_t base = (int64_t)b * W;
    const float *ub = a.u + base;
    const float sc = a.scale[b];
    const float rb = a.r[b];
    const float rn = (rb - 1.25f) / 0.75f;
    // quarters 0, 1 take channels 8 g .. + 3 and 8 g + 4 .. + 7 of the first
    // 32, quarters 2, 3 of the other 32
    const int quarter = wv & 3, qc = 32 * (quarter >> 1) + 4 * (quarter & 1);
    const Place pl{lane, wv >> 2, quarter, qc + 8 * (lane >> 4)};
    const int wrow = qc + 8 * ((lane & 15) >> 2) + (lane & 3);
    // the rod, in computed rows
    const int in_lo = kFHalo - w0, in_hi = kFHalo + W - w0;

    WeightFrags<1> w1;
    w1.load(a.w[0], 64, wrow, lane);
    WeightFrags<2> w;
    w.load(a.w[1], 64, wrow, lane);
    // features (channels 0, 1 of layer 1's 32) of every LDS row; rows outside
    // the rod are zero in all 64.  All of a thread's points are asked for
    // before any is used.
    constexpr int kMy = (kFRows + kFThreads - 1) / kFThreads;
    const int rows = P + 2 * kFHalo + 2 * kFPad, x0 = w0 - kFHalo - kFPad;
    float um[kMy], uc[kMy], up[kMy];
#pragma unroll
    for (int j = 0; j < kMy; ++j) {
        const int i = tid + j * kFThreads, x = x0 + i;
        const bool in = i < rows && x >= 0 && x < W;
        um[j] = in && x > 0 ? ub[x - 1] : 0.f;
        uc[j] = in ? ub[x] : 0.f;
        up[j] = in && x < W - 1 ? ub[x + 1] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < kMy; ++j) {
        const int i = tid + j * kFThreads, x = x0 + i;
        if (i >= rows) break;
        const bool in = x >= 0 && x < W;
        const float d = (um[j] - uc[j]) + (up[j] - uc[j]);
        const float f0 = in ? d / sc : 0.f, f1 = in ? rn : 0.f;
        const uint32_t lo = (uint32_t)__builtin_bit_cast(uint16_t, f2bf(f0)) |
                            ((uint32_t)__builtin_bit_cast(uint16_t, f2bf(f1)) << 16);
        *reinterpret_cast<uint4 *>(&act[chunk_at(i, 0)]) = make_uint4(lo, 0, 0, 0);
#pragma unroll
        for (int c = 1; c < 8; ++c)
            if (c < 4 || !in)
                *reinterpret_cast<uint4 *>(&act[chunk_at(i, c)]) = make_uint4(0, 0, 0, 0);
    }
    for (int i = tid; i < 6 * 64; i += kFThreads) {
        const int l = i / 64, c = i % 64;
        bias[l][c] = (l < 5 || c < 16) ? a.bias[l][c] : 0.f;
    }
    __syncthreads();

    // the blocks with rows that the layers after this one read (h rows
    // beyond the tile) inside the rod
    auto need = [&](int h) {
        const int lo = kFHalo - h > in_lo ? kFHalo - h : in_lo;
        const int hi = kFHalo + P + h < in_hi ? kFHalo + P + h : in_hi;
        return Blocks{lo, (hi - lo + kFBlock - 1) / kFBlock};
    };
    int reach = 0;
#pragma unroll
    for (int l = 1; l < 6; ++l) reach += 2 * a.dil[l];

    bf16x4 out[kFMine][kFB];
    {
        const Blocks n = need(reach);
        gelu_layer<1, false>(act, w1, bias[0], a.dil[0], pl, n, out);
        __syncthreads();   // every wave has read its inputs
        store_layer(act, out, a.dil[0], pl, n, in_lo, in_hi);
        __syncthreads();
    }
#pragma unroll 1
    for (int l = 1; l < 5; ++l) {
        // the next layer's weights, a whole layer ahead (layer 6 has 16 rows)
        WeightFrags<2> next;
        next.load(a.w[l + 1], l < 4 ? 64 : 16, l < 4 ? wrow : lane & 15, lane);
        reach -= 2 * a.dil[l];
        const Blocks n = need(reach);
        gelu_layer<2, true>(act, w, bias[l], a.dil[l], pl, n, out);
        __syncthreads();
        store_layer(act, out, a.dil[l], pl, n, in_lo, in_hi);
        w = next;
        __syncthreads();
    }
    // layer 6 (64 -> 1, padded to 16 outputs) and the jump: wave q of a team
    // takes tile q of its blocks
    const Blocks n = need(0);
    const int d = a.dil[5];
    int at[kTaps];
    fragment_places(pl, d, n.lo, quarter, at);
    const float b0 = bias[5][0];
    const float amp = 64.0f * rb * sc;
#pragma unroll
    for (int i = 0; i < kFMine; ++i) {
        const int block = pl.team + kFTeams * i;
        if (block >= n.count) break;
        const int q = n.lo + kFBlock * block + lane_row(lane & 15, d) + quarter * d;
        const int p = q - kFHalo;                   // point within the tile
        const int x = w0 + p;
        const bool mine = lane < 16 && p >= 0 && p < P && x < W;
        const float uo = mine ? ub[x] : 0.f;
        f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kTaps; ++k)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    w.v[k][c], chunk_of(act, at[k], c, kFTeams * i), acc, 0, 0, 0);
        // channel 0 of the position
        if (mine) a.u_next[base + x] = uo + amp * (acc[0] + b0);
    }
}

// Per-rod scale: RMS of the rod's second differences (zero walls).
__global__ __launch_bounds__(256) void rod_scale_kernel(const float *u, int W, float *scale)
{
    const int b = blockIdx.x, tid = threadIdx.x;
    const float *ub = u + (int64_t)b * W;
    __shared__ float red[256];
    float ss = 0.f;
    // kAhead of a thread's points asked for before any is used: the few rods
    // of a small batch leave nothing else to hide the loads behind
    constexpr int kAhead = 8;
    for (int i0 = tid; i0 < W; i0 += 256 * kAhead) {
        float um[kAhead], uc[kAhead], up[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const int i = i0 + 256 * j;
            um[j] = i > 0 && i < W ? ub[i - 1] : 0.f;
            uc[j] = i < W ? ub[i] : 0.f;
            up[j] = i < W - 1 ? ub[i + 1] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            if (i0 + 256 * j >= W) break;
            const float d = (um[j] - uc[j]) + (up[j] - uc[j]);
            ss += d * d;
        }
    }
    red[tid] = ss;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) red[tid] += red[tid + s];
        __syncthreads();
    }
    if (tid == 0) scale[b] = sqrtf(red[0] / W) + 1e-30f;
}

}  // namespace

hipError_t launch_rod_scale(const float *u, int W, int batch, float *scale, hipStream_t s)
{
    hipLaunchKernelGGL(rod_scale_kernel, dim3(batch), dim3(256), 0, s, u, W, scale);
    return hipGetLastError();
}

hipError_t launch_jump_fused(const FusedArgs &a, int batch, hipStream_t s)
{
    int reach = 0;
    for (int l = 0; l < 6; ++l) {
        if (a.dil[l] < 1 || a.dil[l] > kMaxDil || 16 % a.dil[l] != 0) return hipErrorInvalidValue;
        reach += 2 * a.dil[l];
    }
    if (reach > kFHalo) return hipErrorInvalidValue;   // the tile would not stay valid
    hipError_t e = launch_rod_scale(a.u, a.width, batch, a.scale, s);
    if (e != hipSuccess) return e;
    // Points per workgroup: the fewest rounds of workgroups over the chip
    // (one fits a CU) times what a round costs, its blocks of rows and a share
    // that no size reduces (features, weights, barriers).
    int64_t best = 0;
    int P = 0;
    for (int64_t most = kFMaxP; most > 0; most -= kFBlock) {
        const int64_t tiles = (a.width + most - 1) / most;
        // P + 4 rows of layer 5 (two each side) in whole blocks, if that fits
        const int even = (int)((a.width + tiles - 1) / tiles);
        const int whole = (even + 4 + kFBlock - 1) / kFBlock * kFBlock - 4;
        const int p = whole <= most ? whole : even;
        const int64_t wgs = batch * ((a.width + (int64_t)p - 1) / p);
        const int64_t blocks = (p + 2 * kFHalo + kFBlock - 1) / kFBlock;
        const int64_t cost = (wgs + kFCU - 1) / kFCU * (blocks + kFFixed);
        if (P == 0 || cost < best) {
            best = cost;
            P = p;
        }
    }
    const dim3 grid((a.width + P - 1) / P, batch);
    hipLaunchKernelGGL(jump_fused_kernel, grid, dim3(kFThreads), 0, s, a, P);
    return hipGetLastError();
}

}  // namespace nn
}  // namespace ge

// Weight and bias gradients of the surrogate's layers:
//   dW[k][o][i] = sum_{b,w} g[b][w][o] x[b][w + (k - 2) d][i],  db[o] = sum g[b][w][o].
//
// The GEMM runs with M = output channels, N = input channels and K =
// positions, so both operands have to be read down the channels-last rows.
// The rows go to LDS as they lie in memory (16-byte copies, no transposition)
// and the fragments come from ds_read_b64_tr_b16, which hands each lane four
// rows of one channel; a tap is a shift by whole rows, so one copy of x serves
// all five.  A workgroup of 8 waves takes two 128-position segments at a
// time, four waves each: wave q holds the 16 input channels (layers 2..6) or
// output channels (layer 1) number q for every tap, so the taps share the g
// fragments, 18 LDS reads for 20 MFMAs, and the reads fit beside the matrix
// work.  The next segments' rows are loaded into registers during the
// current ones' MFMAs.  Channels that are padding (layer 1 has 2 inputs,
// layer 6 one output) are left out: 16 of them are computed.
//
// Every workgroup owns a fixed range of segments and writes its sums;
// wgrad_reduce_kernel adds them in a fixed order, so training is
// deterministic.
//
// Measured at 64 rods x 4096 points: the six layers' products and sums take
// 157 us in place of 1640 us (tiles transposed element by element, one copy
// of x per tap; sums by one thread per element).
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ge_nn.h"
#include "ge_nn_dev.h"

namespace ge {
namespace nn {
namespace {

using namespace dev;

typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int kSeg = kWgradSegment;            // positions per segment
constexpr int kXRows = kSeg + 4 * kMaxDil;     // rows of x a segment reads, at most
constexpr int kHalf = 256;                     // threads per segment (4 waves)

// Eight consecutive rows r0 .. r0+7 (r0 = row + 8 (lane / 16)) of channel
// col + lane % 16, from rows of PITCH bf16 in LDS: the K fragment of one
// 16-channel operand.  Lane l of a group of 16 addresses four channels of row
// l / 4 and receives channel l of rows 0..3.
template <int PITCH>
__device__ __forceinline__ bf16x8 column_fragment(const bf16 *lds, int row, int col, int lane)
{
    const int r16 = lane & 15, g4 = lane >> 4;
    const bf16 *p = lds + (row + 8 * g4 + (r16 >> 2)) * PITCH + col + 4 * (r16 & 3);
    typedef __attribute__((address_space(3))) s16x4 *lp;
    union { s16x4 s[2]; bf16x8 v; } u;
    u.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)p);
    u.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + 4 * PITCH));
    return u.v;
}

// XC, GC: channels of a row of x and g in memory; NI, MO: input and output
// channels computed (64, or the first 16).
template <int XC, int GC, int NI, int MO>
__global__ __launch_bounds__(2 * kHalf) void wgrad_kernel(WgradArgs a)
{
    static_assert(NI == 64 || MO == 64, "one operand spans the four waves");
    constexpr int MT = NI == 64 ? MO / 16 : 1;     // output-channel tiles per wave
    constexpr int XP = NI + 8, GP = MO + 8;        // LDS pitch (bf16)
    constexpr int XQ = NI / 8, GQ = MO / 8;        // 16-byte chunks per row
    constexpr int XN = (kXRows * XQ + kHalf - 1) / kHalf, GN = (kSeg * GQ + kHalf - 1) / kHalf;
    constexpr int kTile = kXRows * XP + kSeg * GP; // one segment's LDS (bf16)
    constexpr int kAcc = kTaps * MT * 256 * 4;     // one half's sums (floats)
    constexpr int kLds = 2 * kTile * 2 > kAcc * 4 ? 2 * kTile * 2 : kAcc * 4;
    __shared__ __attribute__((aligned(16))) unsigned char lds[kLds];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wv >> 2, q = wv & 3, ht = tid & (kHalf - 1);
    bf16 *xs = reinterpret_cast<bf16 *>(lds) + half * kTile;
    bf16 *gs = xs + kXRows * XP;

    const int W = a.width, d = a.dil;
    const int per_rod = W / kSeg;
    const int64_t nseg = (int64_t)a.batch * per_rod;
    const int64_t s_lo = nseg * blockIdx.x / gridDim.x;
    const int64_t s_hi = nseg * (blockIdx.x + 1) / gridDim.x;
    const int rows = kSeg + 4 * d;

    f32x4 acc[kTaps][MT];
#pragma unroll
    for (int k = 0; k < kTaps; ++k)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[k][m] = f32x4{0.f, 0.f, 0.f, 0.f};
    float db[8] = {};                              // the thread's eight channels of g

    uint4 xv[XN], gv[GN];
    const uint4 zero = make_uint4(0, 0, 0, 0);
    auto fetch = [&](int64_t sg) {
        const bool on = sg < s_hi;
        const int64_t b = on ? sg / per_rod : 0;
        const int p0 = on ? (int)(sg % per_rod) * kSeg : 0;
        const bf16 *x = static_cast<const bf16 *>(a.x) + b * W * XC;
        const bf16 *g = static_cast<const bf16 *>(a.g) + b * W * GC;
#pragma unroll
        for (int j = 0; j < GN; ++j) {
            const int i = ht + j * kHalf;
            gv[j] = zero;
            if (on && i < kSeg * GQ)
                gv[j] = *reinterpret_cast<const uint4 *>(&g[(int64_t)(p0 + i / GQ) * GC + (i % GQ) * 8]);
        }
#pragma unroll
        for (int j = 0; j < XN; ++j) {
            const int i = ht + j * kHalf, w = p0 - 2 * d + i / XQ;
            xv[j] = zero;
            if (on && i < rows * XQ && w >= 0 && w < W)
                xv[j] = *reinterpret_cast<const uint4 *>(&x[(int64_t)w * XC + (i % XQ) * 8]);
        }
    };

    fetch(s_lo + half);
    for (int64_t sg = s_lo; sg < s_hi; sg += 2) {
        __syncthreads();                           // the previous segments are no longer read
#pragma unroll
        for (int j = 0; j < GN; ++j) {
            const int i = ht + j * kHalf;
            if (i < kSeg * GQ)
                *reinterpret_cast<uint4 *>(&gs[(i / GQ) * GP + (i % GQ) * 8]) = gv[j];
            // every chunk of the thread is the same eight channels (GQ divides kHalf)
            const bf16x8 v = __builtin_bit_cast(bf16x8, gv[j]);
#pragma unroll
            for (int c = 0; c < 8; ++c) db[c] += bf2f(v[c]);
        }
#pragma unroll
        for (int j = 0; j < XN; ++j) {
            const int i = ht + j * kHalf;
            if (i < rows * XQ)
                *reinterpret_cast<uint4 *>(&xs[(i / XQ) * XP + (i % XQ) * 8]) = xv[j];
        }
        __syncthreads();
        fetch(sg + 2 + half);
#pragma unroll
        for (int ks = 0; ks < kSeg / 32; ++ks) {
            bf16x8 gf[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m)
                gf[m] = column_fragment<GP>(gs, 32 * ks, NI == 64 ? 16 * m : 16 * q, lane);
#pragma unroll
            for (int k = 0; k < kTaps; ++k) {
                const bf16x8 xf =
                    column_fragment<XP>(xs + k * d * XP, 32 * ks, NI == 64 ? 16 * q : 0, lane);
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    acc[k][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gf[m], xf, acc[k][m], 0, 0, 0);
            }
        }
    }

    // the second half's sums join the first's
    __syncthreads();
    f32x4 *sums = reinterpret_cast<f32x4 *>(lds);
    if (half == 1) {
#pragma unroll
        for (int k = 0; k < kTaps; ++k)
#pragma unroll
            for (int m = 0; m < MT; ++m) sums[(k * MT + m) * kHalf + ht] = acc[k][m];
    }
    __syncthreads();
    float *part = a.part + (int64_t)blockIdx.x * (kTaps * MO * NI + MO);
    if (half == 0) {
        const int r16 = lane & 15, g4 = lane >> 4;
#pragma unroll
        for (int k = 0; k < kTaps; ++k)
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const f32x4 v = acc[k][m] + sums[(k * MT + m) * kHalf + ht];
                const int o0 = (NI == 64 ? 16 * m : 16 * q) + 4 * g4, i = (NI == 64 ? 16 * q : 0) + r16;
#pragma unroll
                for (int j = 0; j < 4; ++j) part[(k * MO + o0 + j) * NI + i] = v[j];
            }
    }
    __syncthreads();
    float *dbs = reinterpret_cast<float *>(lds);
#pragma unroll
    for (int c = 0; c < 8; ++c) dbs[tid * 8 + c] = db[c];
    __syncthreads();
    if (tid < MO) {
        // channel tid: threads of chunk tid / 8, in thread order
        float s = 0.f;
        for (int t = tid / 8; t < 2 * kHalf; t += GQ) s += dbs[t * 8 + tid % 8];
        part[kTaps * MO * NI + tid] = s;
    }
}

// The workgroups' sums into the flat, unpadded gradient dw[(k*co + o)*ci + i]
// then db[o] of each layer: four threads an element, each adding a quarter of
// the workgroups in order, the quarters added in order.
constexpr int kRedElems = 64;
__global__ __launch_bounds__(4 * kRedElems) void wgrad_reduce_kernel(WgradReduceArgs a)
{
    __shared__ float quarter[4][kRedElems];
    int l = 0;
    while (l + 1 < a.layers && (int)blockIdx.x >= a.l[l + 1].block0) ++l;
    const WgradReduceLayer &L = a.l[l];
    const int e = ((int)blockIdx.x - L.block0) * kRedElems + (threadIdx.x & (kRedElems - 1));
    const int qt = threadIdx.x / kRedElems;
    const int nw = kTaps * L.co * L.ci;
    float s = 0.f;
    if (e < nw + L.co) {
        const int k = e / (L.co * L.ci), o = e / L.ci % L.co, i = e % L.ci;
        const int src = e < nw ? (k * L.mo + o) * L.ni + i : kTaps * L.mo * L.ni + (e - nw);
        const int64_t stride = kTaps * L.mo * L.ni + L.mo;
        const int lo = a.nblocks * qt / 4, hi = a.nblocks * (qt + 1) / 4;
        const float *p = L.part + src;
#pragma unroll 8
        for (int b = lo; b < hi; ++b) s += p[b * stride];
    }
    quarter[qt][threadIdx.x & (kRedElems - 1)] = s;
    __syncthreads();
    if (qt == 0 && e < nw + L.co)
        L.grad[e] = ((s + quarter[1][threadIdx.x]) + quarter[2][threadIdx.x]) + quarter[3][threadIdx.x];
}

}  // namespace

int wgrad_blocks(int width, int batch)
{
    // one workgroup per compute unit, each with at least one pair of segments
    const int64_t pairs = ((int64_t)batch * (width / kWgradSegment) + 1) / 2;
    return (int)(pairs < kMaxWgradBlocks ? pairs : kMaxWgradBlocks);
}

int wgrad_computed(int channels) { return channels <= 16 ? 16 : 64; }

int64_t wgrad_part_floats(int ci, int co)
{
    const int ni = wgrad_computed(ci), mo = wgrad_computed(co);
    return (int64_t)kTaps * mo * ni + mo;
}

hipError_t launch_wgrad(int ci, int co, const WgradArgs &a, int blocks, hipStream_t s)
{
    if (a.dil < 1 || a.dil > kMaxDil || a.width % kWgradSegment != 0) return hipErrorInvalidValue;
    const dim3 grid(blocks), threads(2 * kHalf);
    if (ci == 64 && co == 64)
        hipLaunchKernelGGL((wgrad_kernel<64, 64, 64, 64>), grid, threads, 0, s, a);
    else if (ci <= 16 && co == 64)
        hipLaunchKernelGGL((wgrad_kernel<32, 64, 16, 64>), grid, threads, 0, s, a);
    else if (ci == 64 && co <= 16)
        hipLaunchKernelGGL((wgrad_kernel<64, 32, 64, 16>), grid, threads, 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const WgradReduce *r, int layers, int nblocks, hipStream_t s)
{
    if (layers < 1 || layers > 6) return hipErrorInvalidValue;
    WgradReduceArgs a{};
    a.layers = layers;
    a.nblocks = nblocks;
    int blocks = 0;
    for (int l = 0; l < layers; ++l) {
        const int n = kTaps * r[l].co * r[l].ci + r[l].co;
        a.l[l] = WgradReduceLayer{r[l].part, r[l].grad, r[l].ci, r[l].co, wgrad_computed(r[l].ci),
                                  wgrad_computed(r[l].co), blocks};
        blocks += (n + kRedElems - 1) / kRedElems;
    }
    hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(blocks), dim3(4 * kRedElems), 0, s, a);
    return hipGetLastError();
}

}  // namespace nn
}  // namespace ge

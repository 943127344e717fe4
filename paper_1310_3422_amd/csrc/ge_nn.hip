// Kernels of the learned 64-level propagator (the surrogate): a 1D
// convolutional network over the points of a rod, channels last
// (x[b][w][c], bfloat16 storage, FP32 accumulation on the matrix cores).
//
//   layer 1 : pre1 = conv(x, W1) + b1,          h1 = gelu(pre1)         (2 -> 64)
//   layer l : pre_l = conv(h_{l-1}, W_l) + b_l, h_l = h_{l-1} + gelu(pre_l)  (l=2..5)
//   layer 6 : out = conv(h5, W6) + b6                                     (64 -> 1)
//   conv(x, W)[b, w, o] = sum_{k<5} sum_i W[k, o, i] x[b, w + k - 2, i], zero padding.
//
// Channel counts are padded to the matrix-core tiles: the 2 input features
// to 32 channels, the single output to 16.  Every convolution -- forward,
// input gradient (a convolution with the taps reversed and the weight
// transposed) -- runs in conv_kernel as an implicit GEMM on
// v_mfma_f32_16x16x32_bf16: A = activations (positions x input channels),
// B = weights (input x output channels), K = 5 taps x input channels.  The
// weight gradients are in ge_nn_wgrad.hip.
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ge_nn.h"
#include "ge_nn_dev.h"

namespace ge {
namespace nn {
namespace {

using namespace dev;

constexpr int kMT = 128;          // positions per workgroup tile
constexpr int kThreads = 256;     // 4 waves, 32 positions each
constexpr int kConvGroups = 512;

// ---------------------------------------------------------------------------
// Convolution as an implicit GEMM.
//   x   : [B][W][CIN] bf16 input, read at offsets (k - 2) d from each output
//   wt  : [5][COUT][CIN] bf16 weights (B operand layout: output channel rows)
//   bias: [COUT] fp32 (may be null)
// Epilogues (EPI):
//   kEpiGelu    : pre = acc + bias -> pre_out (bf16), act_out = gelu(pre)
//   kEpiGeluRes : as kEpiGelu with act_out = x + gelu(pre) (CIN == COUT)
//   kEpiOut     : out_f32[b][w] = acc + bias (channel 0)
//   kEpiBwd     : (no bias) gh = acc (+ res_in) -> gh_out (bf16, optional);
//                 gp_out = bf16(gh) * gelu'(pre_in) (bf16)
//   kEpiF32     : out_f32[b][w][o] = acc + bias, every channel, unrounded
//                 (the per-layer probe that checks the products)
// LDS rows are padded by 16 bytes so that 16 lanes reading 16 bytes from 16
// consecutive rows hit distinct banks.
//
// Memory binds a layer (the forward pass reads 128 bytes a point and writes
// 256, the backward reads 384 and writes 256), so a workgroup stays for many
// tiles: the weights go to LDS once, the next tile's rows are loaded into
// registers during the current one's products, and so are the epilogue's
// operands.  The weights' rows are dealt to the matrix rows so that a lane ends
// with twice eight consecutive channels of a position (matrix row 4 g + j of
// tile 2 h + s is channel 32 h + 8 g + 4 s + j), so every access of the
// epilogue is 16 bytes and four lanes make 64 contiguous.  No sum changes its
// order.  Measured at 64 rods x 4096 points: a hidden layer 27.5 us forward (53
// with a workgroup per tile and 8-byte accesses), 41 backward (67): 3.7 and 4.1
// TB/s of the 4.7 a large copy reaches.
template <int CIN, int COUT, int EPI>
__global__ __launch_bounds__(kThreads, 2) void conv_kernel(ConvArgs a)
{
    constexpr int XS = CIN + 8;                 // padded row (bf16 elements)
    constexpr int NT = COUT / 16;               // output channel tiles
    constexpr int KC = CIN / 32;                // 32-channel K chunks per tap
    constexpr int CPR = CIN / 8;                // 16-byte chunks per row
    constexpr int ROWS = kMT + 4 * kMaxDil;     // rows of a tile, at most
    constexpr int XN = (ROWS * CPR + kThreads - 1) / kThreads;
    __shared__ __attribute__((aligned(16))) bf16 xs[ROWS * XS];
    __shared__ __attribute__((aligned(16))) bf16 ws[kTaps * COUT * XS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g4 = lane >> 4;
    const int W = a.width, d = a.dil;
    const int per_rod = W / kMT, ntiles = per_rod * a.batch;
    const int rows = kMT + 4 * d;

    // weight row of channel c: matrix row 4 (c / 8 % 4) + c % 4 of tile 2 (c / 32) + c / 4 % 2
    const bf16 *wt = static_cast<const bf16 *>(a.w);
    for (int i = tid; i < kTaps * COUT * CPR; i += kThreads) {
        const int row = i / CPR, ch = (i % CPR) * 8, k = row / COUT, c = row % COUT;
        const int to = COUT == 64 ? 16 * (2 * (c >> 5) + ((c >> 2) & 1)) + 4 * ((c >> 3) & 3) + (c & 3) : c;
        copy16(&ws[(k * COUT + to) * XS + ch], &wt[row * CIN + ch]);
    }
    // first channel of the lane's four in tile n
    auto channel = [&](int n) { return COUT == 64 ? 32 * (n >> 1) + 8 * g4 + 4 * (n & 1) : 4 * g4; };
    float bl[NT][4];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int j = 0; j < 4; ++j) bl[n][j] = a.bias ? a.bias[channel(n) + j] : 0.f;

    // input rows w0-2d .. w0+kMT+2d-1 of a tile (zero outside the rod)
    uint4 xv[XN];
    auto fetch = [&](int tile) {
        const int b = tile / per_rod, w0 = (tile - b * per_rod) * kMT;
        const bf16 *x = static_cast<const bf16 *>(a.x) + (int64_t)b * W * CIN;
#pragma unroll
        for (int j = 0; j < XN; ++j) {
            const int i = tid + j * kThreads, w = w0 - 2 * d + i / CPR;
            xv[j] = make_uint4(0, 0, 0, 0);
            if (tile < ntiles && i < rows * CPR && w >= 0 && w < W)
                xv[j] = *reinterpret_cast<const uint4 *>(&x[(int64_t)w * CIN + (i % CPR) * 8]);
        }
    };

    fetch(blockIdx.x);
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        __syncthreads();                        // the previous tile is no longer read
#pragma unroll
        for (int j = 0; j < XN; ++j) {
            const int i = tid + j * kThreads;
            if (i < rows * CPR)
                *reinterpret_cast<uint4 *>(&xs[(i / CPR) * XS + (i % CPR) * 8]) = xv[j];
        }
        __syncthreads();
        fetch(tile + (int)gridDim.x);

        // position pl of the tile, element o of its output row
        const int64_t rowbase = (int64_t)tile * kMT;
        auto place = [&](int m) { return 32 * wv + 16 * m + r16; };
        auto element = [&](int m, int n) { return (rowbase + place(m)) * COUT + channel(n); };
        // the backward epilogue's operands, loaded ahead of the products
        constexpr int NH = EPI == kEpiBwd ? NT / 2 : 0;
        bf16x8 pre[2][NH ? NH : 1], res[2][NH ? NH : 1];
        if constexpr (EPI == kEpiBwd) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int h = 0; h < NH; ++h) {
                    const int64_t o = element(m, 2 * h);
                    pre[m][h] = *reinterpret_cast<const bf16x8 *>(&static_cast<const bf16 *>(a.pre_in)[o]);
                    if (a.res_in)
                        res[m][h] =
                            *reinterpret_cast<const bf16x8 *>(&static_cast<const bf16 *>(a.res_in)[o]);
                }
        }

        f32x4 acc[2][NT];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < kTaps; ++k) {
#pragma unroll
            for (int c = 0; c < KC; ++c) {
                bf16x8 af[2], bfr[NT];
#pragma unroll
                for (int m = 0; m < 2; ++m)
                    af[m] = *reinterpret_cast<const bf16x8 *>(
                        &xs[(32 * wv + 16 * m + r16 + k * d) * XS + 32 * c + 8 * g4]);
#pragma unroll
                for (int n = 0; n < NT; ++n)
                    bfr[n] = *reinterpret_cast<const bf16x8 *>(
                        &ws[(k * COUT + 16 * n + r16) * XS + 32 * c + 8 * g4]);
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int n = 0; n < NT; ++n)
                        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[n], af[m], acc[m][n],
                                                                           0, 0, 0);
            }
        }

        // epilogue: the product is taken transposed (weights as the A operand),
        // so a lane holds four consecutive channels of one position per tile
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int pl = place(m);
            if constexpr (EPI == kEpiOut) {
                if (channel(0) == 0) a.out_f32[rowbase + pl] = acc[m][0][0] + bl[0][0];
            } else if constexpr (EPI == kEpiF32) {
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    float4 v;
                    v.x = a.bias ? acc[m][n][0] + bl[n][0] : acc[m][n][0];
                    v.y = a.bias ? acc[m][n][1] + bl[n][1] : acc[m][n][1];
                    v.z = a.bias ? acc[m][n][2] + bl[n][2] : acc[m][n][2];
                    v.w = a.bias ? acc[m][n][3] + bl[n][3] : acc[m][n][3];
                    *reinterpret_cast<float4 *>(&a.out_f32[element(m, n)]) = v;
                }
            } else {
#pragma unroll
                for (int h = 0; h < NT / 2; ++h) {
                    const int64_t o = element(m, 2 * h);
                    bf16x8 one, two;
                    bf16x8 xres;
                    if constexpr (EPI == kEpiGeluRes)
                        xres = *reinterpret_cast<const bf16x8 *>(&xs[(pl + 2 * d) * XS + channel(2 * h)]);
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int n = 2 * h + j / 4;
                        float v = acc[m][n][j % 4];
                        if constexpr (EPI == kEpiBwd) {
                            if (a.res_in) v += bf2f(res[m][h][j]);
                            one[j] = f2bf(v);
                            two[j] = f2bf(bf2f(one[j]) * gelu_grad(bf2f(pre[m][h][j])));
                        } else {
                            v += bl[n][j % 4];
                            one[j] = f2bf(v);
                            float act = gelu(v);
                            if constexpr (EPI == kEpiGeluRes) act += bf2f(xres[j]);
                            two[j] = f2bf(act);
                        }
                    }
                    bf16 *p1 = static_cast<bf16 *>(EPI == kEpiBwd ? a.gh_out : a.pre_out);
                    bf16 *p2 = static_cast<bf16 *>(EPI == kEpiBwd ? a.gp_out : a.act_out);
                    if (p1) *reinterpret_cast<bf16x8 *>(&p1[o]) = one;
                    *reinterpret_cast<bf16x8 *>(&p2[o]) = two;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Features of one rod: the second difference D_i = u_{i-1} - 2u_i + u_{i+1}
// (zero walls) scaled by its RMS s (rod_scale_kernel), and the mesh ratio
// mapped to [-1, 1] over [0.5, 2]; other channels zero.  One thread a point,
// its 64-byte row in four stores.
__global__ __launch_bounds__(256) void features_kernel(const float *u, const float *r, int W,
                                                       int64_t M, bf16 *x, const float *scale)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= M) return;
    const int b = (int)(p / W), i = (int)(p - (int64_t)b * W);
    const float *ub = u + (int64_t)b * W;
    const float um = i > 0 ? ub[i - 1] : 0.f, up = i < W - 1 ? ub[i + 1] : 0.f;
    const float d = (um - ub[i]) + (up - ub[i]);
    const float rn = (r[b] - 1.25f) / 0.75f;
    const uint32_t lo = (uint32_t)__builtin_bit_cast(uint16_t, f2bf(d / scale[b])) |
                        ((uint32_t)__builtin_bit_cast(uint16_t, f2bf(rn)) << 16);
    uint4 *row = reinterpret_cast<uint4 *>(x + p * 32);
    row[0] = make_uint4(lo, 0, 0, 0);
    row[1] = row[2] = row[3] = make_uint4(0, 0, 0, 0);
}

// Loss on the normalised increment t = (u64 - u) / (64 r s), and its
// gradient 2 (out - t) / M into channel 0 of a 32-channel bf16 tensor.
// Per-block partial sums of the squared error go to part (reduced in order).
__global__ __launch_bounds__(256) void loss_kernel(const float *out, const float *u,
                                                   const float *u64, const float *r,
                                                   const float *scale, int W, int64_t M,
                                                   bf16 *g, float *part)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    __shared__ float red[256];
    float e2 = 0.f;
    if (i < M) {
        const int64_t b = i / W;
        const float t = (u64[i] - u[i]) / (64.0f * r[b] * scale[b]);
        const float d = out[i] - t;
        e2 = d * d;
        uint4 *gr = reinterpret_cast<uint4 *>(g + i * 32);
        gr[0] = make_uint4(__builtin_bit_cast(uint16_t, f2bf(2.0f * d / (float)M)), 0, 0, 0);
        gr[1] = gr[2] = gr[3] = make_uint4(0, 0, 0, 0);
    }
    red[threadIdx.x] = e2;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// The partial sums added in a fixed order: each of 256 threads adds every
// 256th, then a tree over the threads.
__global__ __launch_bounds__(256) void sum_parts_kernel(const float *part, int n, float scale,
                                                        float *out)
{
    __shared__ float red[256];
    const int tid = threadIdx.x;
    float s = 0.f;
    for (int i = tid; i < n; i += 256) s += part[i];
    red[tid] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (tid < k) red[tid] += red[tid + k];
        __syncthreads();
    }
    if (tid == 0) out[0] = red[0] * scale;
}

// u_next = u + 64 r s out (the jump), optionally to a separate buffer
__global__ void jump_kernel(const float *u, const float *out, const float *r,
                            const float *scale, int W, int64_t M, float *u_next)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    const int64_t b = i / W;
    u_next[i] = u[i] + 64.0f * r[b] * scale[b] * out[i];
}

// Widening and narrowing copies between the network's FP32 state and the
// FP64 state of the GE sweep.
__global__ void widen_kernel(const float *u, double *d, int64_t M)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < M) d[i] = (double)u[i];
}
__global__ void narrow_kernel(const double *d, float *u, int64_t M)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < M) u[i] = (float)d[i];
}

// Re-check of one jump, one workgroup per rod: rel-L2 distance of the
// network's result a (FP32) from the GE result b (FP64), in FP64.  A rod is
// flagged when the distance exceeds tol or is not a number; the per-rod
// counters of accepted and rejected windows are advanced.
__global__ __launch_bounds__(256) void recheck_kernel(const float *a, const double *b, int W,
                                                      double tol, int *flag, double *err,
                                                      int *acc, int *fb)
{
    const int rod = blockIdx.x, tid = threadIdx.x;
    const float *ar = a + (int64_t)rod * W;
    const double *br = b + (int64_t)rod * W;
    __shared__ double rd[256], rn[256];
    double d2 = 0.0, n2 = 0.0;
    for (int i = tid; i < W; i += 256) {
        const double d = (double)ar[i] - br[i];
        d2 += d * d;
        n2 += br[i] * br[i];
    }
    rd[tid] = d2;
    rn[tid] = n2;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) {
            rd[tid] += rd[tid + s];
            rn[tid] += rn[tid + s];
        }
        __syncthreads();
    }
    if (tid == 0) {
        const double rel = rn[0] > 0.0 ? sqrt(rd[0] / rn[0]) : (rd[0] > 0.0 ? INFINITY : 0.0);
        const int f = !(rel <= tol);
        flag[rod] = f;
        if (err) err[rod] = rel;
        if (acc) acc[rod] += 1 - f;
        if (fb) fb[rod] += f;
    }
}

// Number of flagged rods, summed in order by one thread.
__global__ void count_kernel(const int *flag, int n, int *out)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        int c = 0;
        for (int i = 0; i < n; ++i) c += flag[i];
        out[0] = c;
    }
}

// u = flagged ? saved : network result, rod by rod.
__global__ void select_kernel(float *u, const float *unn, const float *save, const int *flag,
                              int W, int64_t M)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    u[i] = flag[i / W] ? save[i] : unn[i];
}

// Flagged rods take the GE result.
__global__ void take_ge_kernel(float *u, const double *ge, const int *flag, int W, int64_t M)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M) return;
    if (flag[i / W]) u[i] = (float)ge[i];
}

// Adam on the FP32 master parameters.
__global__ void adam_kernel(float *p, const float *g, float *m, float *v, int64_t n, float lr,
                            float b1, float b2, float eps, float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// Master weights of one layer (FP32 [5][co][ci]) -> padded bf16 copies:
// forward B layout wf[k][o][i] (o < cop, i < cip) and input-gradient layout
// wd[k][i][o] = W[4 - k][o][i] (i < cip as output, o < cop_in as input).
__global__ void pack_kernel(const float *wm, const float *bm, int ci, int co, int cip, int cop,
                            int cod, bf16 *wf, float *bf, bf16 *wd)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nf = (int64_t)kTaps * cop * cip;
    if (idx < nf) {
        const int k = (int)(idx / (cop * cip)), rem = (int)(idx % (cop * cip));
        const int o = rem / cip, i = rem % cip;
        wf[idx] = f2bf((o < co && i < ci) ? wm[(k * co + o) * ci + i] : 0.f);
    }
    if (wd) {
        const int64_t nd = (int64_t)kTaps * cip * cod;
        if (idx < nd) {
            const int k = (int)(idx / (cip * cod)), rem = (int)(idx % (cip * cod));
            const int i = rem / cod, o = rem % cod;
            wd[idx] = f2bf((o < co && i < ci) ? wm[((kTaps - 1 - k) * co + o) * ci + i] : 0.f);
        }
    }
    if (idx < cop) bf[idx] = idx < co ? bm[idx] : 0.f;
}

}  // namespace

hipError_t launch_conv(int cin, int cout, int epi, ConvArgs a, int batch, hipStream_t s)
{
    a.batch = batch;
    if (a.dil < 1 || a.dil > kMaxDil || a.width % kMT != 0) return hipErrorInvalidValue;
    // two workgroups per compute unit (their LDS), each for several tiles
    const int64_t tiles = (int64_t)(a.width / kMT) * batch;
    const dim3 grid((unsigned)(tiles < kConvGroups ? tiles : kConvGroups));
#define GE_CONV(CI, CO, E) \
    if (cin == CI && cout == CO && epi == E) { \
        hipLaunchKernelGGL((conv_kernel<CI, CO, E>), grid, dim3(kThreads), 0, s, a); \
        return hipGetLastError(); \
    }
    GE_CONV(32, 64, kEpiGelu)
    GE_CONV(64, 64, kEpiGeluRes)
    GE_CONV(64, 16, kEpiOut)
    GE_CONV(32, 64, kEpiBwd)
    GE_CONV(64, 64, kEpiBwd)
    GE_CONV(32, 64, kEpiF32)
    GE_CONV(64, 64, kEpiF32)
    GE_CONV(64, 16, kEpiF32)
#undef GE_CONV
    return hipErrorInvalidValue;
}

hipError_t launch_features(const float *u, const float *r, int W, int batch, void *x,
                           float *scale, hipStream_t s)
{
    hipError_t e = launch_rod_scale(u, W, batch, scale, s);
    if (e != hipSuccess) return e;
    const int64_t M = (int64_t)W * batch;
    hipLaunchKernelGGL(features_kernel, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, s, u, r, W,
                       M, static_cast<bf16 *>(x), scale);
    return hipGetLastError();
}

hipError_t launch_loss(const float *out, const float *u, const float *u64, const float *r,
                       const float *scale, int W, int batch, void *g, float *part,
                       float *loss, hipStream_t s)
{
    const int64_t M = (int64_t)W * batch;
    const int nb = (int)((M + 255) / 256);
    hipLaunchKernelGGL(loss_kernel, dim3(nb), dim3(256), 0, s, out, u, u64, r, scale, W, M,
                       static_cast<bf16 *>(g), part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !loss) return e;
    hipLaunchKernelGGL(sum_parts_kernel, dim3(1), dim3(256), 0, s, part, nb, 1.0f / (float)M, loss);
    return hipGetLastError();
}

int loss_blocks(int W, int batch) { return (int)(((int64_t)W * batch + 255) / 256); }

hipError_t launch_jump(const float *u, const float *out, const float *r, const float *scale,
                       int W, int batch, float *u_next, hipStream_t s)
{
    const int64_t M = (int64_t)W * batch;
    hipLaunchKernelGGL(jump_kernel, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, s, u, out,
                       r, scale, W, M, u_next);
    return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, int64_t n, float lr,
                       float b1, float b2, float eps, int step, hipStream_t s)
{
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, g, m,
                       v, n, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_pack(const float *wm, const float *bm, int ci, int co, int cip, int cop,
                       int cod, void *wf, float *bf, void *wd, hipStream_t s)
{
    const int64_t n = (int64_t)kTaps * (cop > cod ? cop : cod) * cip + cop;
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, wm, bm,
                       ci, co, cip, cop, cod, static_cast<bf16 *>(wf), bf,
                       static_cast<bf16 *>(wd));
    return hipGetLastError();
}

namespace {
inline dim3 grid_for(int64_t M) { return dim3((unsigned)((M + 255) / 256)); }
}  // namespace

hipError_t launch_widen(const float *u, double *d, int64_t M, hipStream_t s)
{
    hipLaunchKernelGGL(widen_kernel, grid_for(M), dim3(256), 0, s, u, d, M);
    return hipGetLastError();
}

hipError_t launch_narrow(const double *d, float *u, int64_t M, hipStream_t s)
{
    hipLaunchKernelGGL(narrow_kernel, grid_for(M), dim3(256), 0, s, d, u, M);
    return hipGetLastError();
}

hipError_t launch_recheck(const float *a, const double *b, int W, int batch, double tol, int *flag,
                          double *err, int *acc, int *fb, int *count, hipStream_t s)
{
    hipLaunchKernelGGL(recheck_kernel, dim3(batch), dim3(256), 0, s, a, b, W, tol, flag, err, acc,
                       fb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(count_kernel, dim3(1), dim3(64), 0, s, flag, batch, count);
    return hipGetLastError();
}

hipError_t launch_select(float *u, const float *unn, const float *save, const int *flag, int W,
                         int batch, hipStream_t s)
{
    const int64_t M = (int64_t)W * batch;
    hipLaunchKernelGGL(select_kernel, grid_for(M), dim3(256), 0, s, u, unn, save, flag, W, M);
    return hipGetLastError();
}

hipError_t launch_take_ge(float *u, const double *ge, const int *flag, int W, int batch,
                          hipStream_t s)
{
    const int64_t M = (int64_t)W * batch;
    hipLaunchKernelGGL(take_ge_kernel, grid_for(M), dim3(256), 0, s, u, ge, flag, W, M);
    return hipGetLastError();
}

}  // namespace nn
}  // namespace ge

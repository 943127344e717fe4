// A batch of rods in windows: every rod is split into as many
// workgroups or waves as it is worth, so no compute unit waits for another's
// long rod and no rod's waves wait at the barriers of a stranger's.  (In the
// persistent form of ge_batch.hip a rod is one workgroup's: 149 FP32 rods of up
// to 50256 points took 3.3 us a level, the time of the longest alone, and 583
// rods of 215 points, 16 to a workgroup, kept 37 of 256 units busy.)
//
//   * rods of fewer than 256 points: one wave each;
//   * rods of up to one block window (4464 points): a workgroup of four
//     overlapping waves (ge_block.h) each, all levels in one launch, in place;
//   * longer rods: windows with halos in passes of several levels, ping-ponging
//     between u and the workspace, an even number of passes; block windows
//     with hundreds of levels per pass while they leave units idle, else
//     single-wave windows (ge_tile.h).
//
// The last runs beside the others, on a stream of the plan.  Every point
// gets the operations ge_step_n gives it: the same bits.
//
// Measured: 4096 FP32 rods of 256 to 65536 points, 2000 levels, 11.0 ms (8.7e12
// updates/s; VALU issue binds, 5 instructions a point and the halos' recompute;
// 12.6 in the persistent form); 1024 FP64 rods of 4096 points, 64 levels, 40 us
// (120); the 149 rods above, 41 levels, 50 us (135); 768 FP32 rods of 1565
// points, 715 levels, 138 us (1074).  The compensated pair: 4096 rods of 256
// to 65536 points, 200 levels, 3.22 ms (3.46); 300 of 1000 to 4000, 300
// levels, 185 us (1043); 51 of 535 to 16585, 26 levels, 70 us (199).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ge_batch.h"
#include "ge_block.h"
#include "ge_kernels.h"
#include "ge_level.h"
#include "ge_tile.h"

namespace ge {
namespace {

using namespace dev;

constexpr int kPerGroup = 4;        // waves per workgroup of the single-wave kernels

// One rod's sweep: level0 and nlev of the launch, from in to out.
__device__ __forceinline__ TileArgs rod_args(const BatchWinArgs &a, const BatchRod &rd,
                                             const void *in, void *out)
{
    TileArgs ta{};
    ta.in = in;
    ta.out = out;
    ta.n = rd.n;
    ta.level0 = a.level0;
    ta.nlev = a.nlev;
    ta.r = rd.r;
    ta.k = rd.k;
    ta.cs = rd.cs;
    ta.c1 = rd.c1;
    ta.c2 = rd.c2;
    ta.gl0 = rd.gl;
    ta.gr0 = rd.gr;
    ta.h = 1.0;
    ta.status = a.status;
    ta.estride = in == out || !(a.pass & 1) ? a.estride : a.estride2;
    ta.estride_out = in == out || (a.pass & 1) ? a.estride : a.estride2;
    return ta;
}

// This workgroup's (wave's) entry: consecutive ones go to the same XCD.
__device__ __forceinline__ int xcd_order(int waves)
{
    const int b = (int)(blockIdx.x % 8) * (int)(gridDim.x / 8) + (int)(blockIdx.x / 8);
    return b * waves + (waves > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) : 0);
}

template <typename T, bool PAIR>
__global__ __launch_bounds__(kPerGroup *kWave) void tiny_kernel(BatchWinArgs a)
{
    const int i = xcd_order(kPerGroup);
    if (i >= a.count)
        return;
    const BatchRod rd = a.rods[a.list[i].rod];
    T *u = static_cast<T *>(a.u) + rd.off;
    TileArgs ta = rod_args(a, rd, u, u);
    ta.core = rd.n;
    ta.ntiles = 1;
    if constexpr (PAIR) run_pair<T, 4, 1, false, true>(ta, threadIdx.x & (kWave - 1), 0, 0);
    else run_plain<T, 4, 1, false, kInside>(ta, threadIdx.x & (kWave - 1), 0, 0);
}

// Windows of four overlapping waves: whole rods in place (a.core = 0), or
// windows of a pass.  Narrow (up to 8 points a lane) and wide ones are kernels
// of their own: the wide ones' registers and LDS would halve the others'
// workgroups per unit.
template <typename T, bool WIDE, bool PAIR>
__global__ __launch_bounds__(kBatchBlockWaves *kWave) void block_windows_kernel(BatchWinArgs a)
{
    constexpr int CAP = block_capacity(WIDE ? 18 : kBatchNarrowK, kBatchBlockWaves);
    __shared__ T buf[(PAIR ? 4 : 2) * CAP];
    const int i = xcd_order(1);
    if (i >= a.count)
        return;
    const BatchWindow w = a.list[i];
    const BatchRod rd = a.rods[w.rod];
    T *u = static_cast<T *>(a.u) + rd.off, *u2 = static_cast<T *>(a.u2) + w.woff;
    TileArgs ta = a.core == 0 ? rod_args(a, rd, u, u)
                              : rod_args(a, rd, (a.pass & 1) ? u2 : u, (a.pass & 1) ? u : u2);
    ta.core = a.core == 0 ? rd.n : a.core;
    ta.halo = a.core == 0 ? 0 : a.halo;
    ta.ntiles = (rd.n + ta.core - 1) / ta.core;
    if constexpr (WIDE) {
        if (w.k == 12) block_window<T, 12, false, PAIR>(ta, w.tile, buf, CAP);
        else if (w.k == 18) block_window<T, 18, false, PAIR>(ta, w.tile, buf, CAP);
    } else {
        if (w.k == 4) block_window<T, 4, false, PAIR>(ta, w.tile, buf, CAP);
        else if (w.k == 6) block_window<T, 6, false, PAIR>(ta, w.tile, buf, CAP);
        else if (w.k == 8) block_window<T, 8, false, PAIR>(ta, w.tile, buf, CAP);
    }
}

template <typename T, int K, bool PAIR>
__global__ __launch_bounds__(kPerGroup *kWave) void wave_windows_kernel(BatchWinArgs a)
{
    const int i = xcd_order(kPerGroup);
    if (i >= a.count)
        return;
    const BatchWindow w = a.list[i];
    const BatchRod rd = a.rods[w.rod];
    T *u = static_cast<T *>(a.u) + rd.off, *u2 = static_cast<T *>(a.u2) + w.woff;
    TileArgs ta = rod_args(a, rd, (a.pass & 1) ? u2 : u, (a.pass & 1) ? u : u2);
    ta.core = a.core;
    ta.halo = a.halo;
    ta.ntiles = (rd.n + ta.core - 1) / ta.core;
    run_tile<T, K, 1, PAIR, false>(ta, threadIdx.x & (kWave - 1), w.tile);
}

template <typename T, bool PAIR>
hipError_t launch(BatchWinKind kind, int k, const BatchWinArgs &a, hipStream_t stream)
{
    const int per = kind == kWinBlock ? 1 : kPerGroup;
    const unsigned groups = (unsigned)((a.count + per - 1) / per);
    const dim3 grid((groups + 7) / 8 * 8), waves(kPerGroup * kWave);
    if (kind == kWinTiny)
        hipLaunchKernelGGL((tiny_kernel<T, PAIR>), grid, waves, 0, stream, a);
    else if (kind == kWinBlock && k <= kBatchNarrowK)
        hipLaunchKernelGGL((block_windows_kernel<T, false, PAIR>), grid, dim3(kBatchBlockWaves * kWave), 0,
                           stream, a);
    else if (kind == kWinBlock)
        hipLaunchKernelGGL((block_windows_kernel<T, true, PAIR>), grid, dim3(kBatchBlockWaves * kWave), 0,
                           stream, a);
    else if (k == 16)
        hipLaunchKernelGGL((wave_windows_kernel<T, 16, PAIR>), grid, waves, 0, stream, a);
    else if (k == 32 && !PAIR)
        hipLaunchKernelGGL((wave_windows_kernel<T, PAIR ? 16 : 32, PAIR>), grid, waves, 0, stream, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace

hipError_t launch_batch_windows(int prec, BatchWinKind kind, int k, const BatchWinArgs &a,
                                hipStream_t stream)
{
    if (a.count < 1) return hipSuccess;
    if (prec == kFP64) return launch<double, false>(kind, k, a, stream);
    if (prec == kFP32) return launch<float, false>(kind, k, a, stream);
    if (prec == kFP32C) return launch<float, true>(kind, k, a, stream);
    return hipErrorInvalidValue;
}

}  // namespace ge

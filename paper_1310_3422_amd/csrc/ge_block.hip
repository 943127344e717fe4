// Rods too short to fill the chip with tiles: windows of several
// waves that advance hundreds of levels per launch.
//
// Such a rod leaves most compute units idle, and a call's time is the number
// of launches times their fixed cost plus the levels times the latency of
// one.  So a workgroup of NW waves takes a window wide enough for a halo of
// hundreds of points a side -- recomputing it costs nothing while units are
// idle -- and keeps a level short: the waves of a window overlap by 2 h points
// (h = kBlockOverlap) and advance h - 1 levels on their own, each with open
// edges, before they refresh what has gone stale through LDS (one barrier).
// A rod that fits one window takes all its levels in one launch, in place.
//
// A wave's window starts at any point: the last one ends where the
// workgroup's does, and a wave that starts at an odd point pairs its points
// the other way round.  A wall is the fill of a first or last lane.  Every
// point gets the operations it gets everywhere (ge_level.h): the same bits.
//
// Bound by the latency and issue of one wave's level (4 points a lane, FP64:
// 13 FP64 instructions and 4 lane moves, 0.087 us with its share of the
// refresh).  960 levels of 800 points: 84 us, in one window of 32 points a
// lane before 489; of 60000 points 92 us, in tiles before 171 (4 points a
// lane, 48 levels per launch) and 285 (32 points).  The pair's level is four
// times the instructions: 0.18 us; 960 levels of 800 points 174 us (669 in one
// window of tiles), of 131071 196 (533).
#include "ge_block.h"
#include "ge_kernels.h"

namespace ge {
namespace {

using namespace dev;

template <typename T, int K, int NW, bool SRC, bool PAIR>
__global__ __launch_bounds__(NW *kWave) void block_kernel(TileArgs a)
{
    constexpr int CAP = block_capacity(K, NW);
    __shared__ T buf[(PAIR ? 4 : 2) * CAP];
    // consecutive windows go to the same XCD, as in tile_kernel
    const int64_t t = (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (t < a.ntiles)
        block_window<T, K, SRC, PAIR>(a, t, buf, CAP);
}

template <typename T, int K, int NW, bool PAIR>
hipError_t launch(bool src, const TileArgs &a, hipStream_t stream)
{
    const dim3 grid((unsigned)((a.ntiles + 7) / 8 * 8)), threads(NW * kWave);
    if (src) hipLaunchKernelGGL((block_kernel<T, K, NW, true, PAIR>), grid, threads, 0, stream, a);
    else hipLaunchKernelGGL((block_kernel<T, K, NW, false, PAIR>), grid, threads, 0, stream, a);
    return hipGetLastError();
}

template <typename T, bool PAIR>
hipError_t launch_t(int k, int nw, bool src, const TileArgs &a, hipStream_t stream)
{
#define GE_B(KK, N) \
    if (k == KK && nw == N) return launch<T, KK, N, PAIR>(src, a, stream)
    GE_B(4, 4);
    GE_B(6, 4);
    GE_B(8, 4);
    GE_B(10, 4);
    GE_B(8, 8);
#undef GE_B
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_block(int prec, int k, int nw, bool src, const TileArgs &a, hipStream_t stream)
{
    // every window fits its waves, and holds at least one wave's points
    if (a.n < (int64_t)kWave * k || a.core < 1 ||
        (a.ntiles > 1 && a.core + 2 * (int64_t)a.halo > block_capacity(k, nw)) ||
        (a.ntiles == 1 && a.n > block_capacity(k, nw)) ||
        (a.ntiles > 1 && (a.in == a.out || a.halo < a.nlev + 1)))
        return hipErrorInvalidValue;
    if (prec == kFP64) return launch_t<double, false>(k, nw, src, a, stream);
    if (prec == kFP32) return launch_t<float, false>(k, nw, src, a, stream);
    if (prec == kFP32C) return launch_t<float, true>(k, nw, src, a, stream);
    return hipErrorInvalidValue;
}

}  // namespace ge

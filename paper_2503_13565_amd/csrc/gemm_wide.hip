// MXFP4 weights in the block kernel of gemm_wide.h: row-major, tile-major, and row-major with any K % 32 == 0.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

constexpr Cost kCosts[] = {
    {1, 1, 8, 1, 1, 4.509f, 0.038f, 0.747f, 0.068f},
    {1, 1, 8, 1, 2, 4.480f, 0.081f, 0.551f, 0.119f},
    {1, 1, 8, 1, 3, 4.556f, 0.112f, 0.470f, 0.181f},
    {1, 2, 4, 1, 1, 4.061f, 0.092f, 0.223f, 0.115f},
    {1, 2, 4, 1, 2, 4.308f, 0.140f, 0.238f, 0.210f},
    {1, 2, 4, 1, 3, 4.350f, 0.229f, 1.507f, 0.268f},
    {1, 4, 2, 1, 1, 4.040f, 0.161f, 0.185f, 0.179f},
    {1, 4, 2, 1, 2, 4.103f, 0.286f, 0.466f, 0.308f},
    {1, 4, 2, 1, 3, 4.420f, 0.517f, 0.846f, 0.297f},
    {1, 1, 8, 2, 3, 5.723f, 0.173f, 2.857f, 0.204f},
    {1, 2, 4, 2, 1, 4.501f, 0.146f, 0.733f, 0.145f},
    {1, 2, 4, 2, 2, 4.643f, 0.198f, 0.760f, 0.225f},
    {1, 2, 4, 2, 3, 5.668f, 0.264f, 2.385f, 0.311f},
    {1, 2, 4, 2, 4, 5.399f, 0.389f, 2.964f, 0.380f},
    {1, 4, 2, 2, 1, 4.215f, 0.226f, 0.547f, 0.213f},
    {1, 4, 2, 2, 2, 4.659f, 0.410f, 1.045f, 0.353f},
    {1, 4, 2, 2, 3, 5.774f, 0.558f, 3.035f, 0.468f},
    {1, 4, 2, 2, 4, 6.199f, 0.715f, 3.685f, 0.454f},
    {1, 8, 1, 2, 2, 4.013f, 0.807f, 2.124f, 0.480f},
    {1, 2, 4, 3, 3, 5.825f, 0.317f, 3.639f, 0.426f},
    {1, 4, 2, 3, 1, 4.631f, 0.318f, 0.971f, 0.224f},
    {1, 4, 2, 3, 2, 5.257f, 0.431f, 3.466f, 0.518f},
    {1, 4, 2, 3, 3, 7.025f, 0.643f, 5.014f, 0.565f},
    {1, 2, 4, 4, 3, 6.550f, 0.431f, 4.432f, 0.431f},
    {1, 4, 2, 4, 2, 5.104f, 0.546f, 3.955f, 0.452f},
    {1, 4, 2, 4, 3, 7.130f, 0.668f, 4.921f, 0.637f},
    {1, 8, 1, 4, 1, 4.073f, 0.621f, 1.305f, 0.500f},
    {1, 8, 1, 4, 2, 6.249f, 1.031f, 5.105f, 0.841f},
    {1, 8, 1, 6, 2, 9.337f, 1.136f, 7.388f, 1.129f},
    {1, 8, 1, 6, 3, 12.12f, 1.520f, 10.37f, 1.933f},
    {1, 8, 1, 8, 2, 11.95f, 1.524f, 10.22f, 1.239f},
    {1, 8, 1, 8, 3, 10.88f, 2.061f, 12.51f, 1.498f},
    {2, 4, 1, 4, 3, 7.673f, 1.316f, 7.349f, 1.250f},
};

constexpr auto kLaunch = launches<kMx, kCosts>(), kLaunchTiled = launches<kMxTiled, kCosts>(), kLaunchRagged = launches<kMxRagged, kCosts>();

}  // namespace

bool gemm_wide_can_run(const GemmArgs& a, const DeviceInfo& dev)
{
    if (a.k % 32 != 0 || a.m < 1 || a.ldx > (1 << 21))              // a block's activation rows behind one 32-bit offset
        return false;
    if (dev.lds_bytes < 160 * 1024)
        return false;
    return a.part_val == nullptr || (a.n + 127) / 128 <= a.parts;   // (a column of partial winners per 128 weight rows)
}

hipError_t launch_gemm_wide(const GemmArgs& a, const DeviceInfo& dev, int* parts_used, hipStream_t stream, bool tiled,
                            const Epilogue* epi)
{
    if (!gemm_wide_can_run(a, dev) || (tiled && a.k % 128 != 0))
        return hipErrorInvalidValue;
    Args w{a.x, a.q, a.s, a.n, a.k, a.m, (int)a.ldx, 0, 0, 0, 0, block_out(a, epi)};
    const int c = pick_shape<kCosts, 4>(a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return (tiled ? kLaunchTiled : a.k % 128 != 0 ? kLaunchRagged : kLaunch)[c](w, dev, stream);
}

}  // namespace mxfp4

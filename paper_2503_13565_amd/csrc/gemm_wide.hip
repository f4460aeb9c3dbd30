// MXFP4 weights in the block kernel of gemm_wide.h: row-major, tile-major, and row-major with any K % 32 == 0.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

constexpr Cost kCosts[] = {
    {1, 1, 8, 1, 1, 3.724f, 0.062f, 0.883f, 0.059f},
    {1, 1, 8, 1, 2, 3.948f, 0.079f, 0.931f, 0.089f},
    {1, 1, 8, 1, 3, 4.205f, 0.097f, 1.050f, 0.122f},
    {1, 2, 4, 1, 1, 3.459f, 0.090f, 0.386f, 0.078f},
    {1, 2, 4, 1, 2, 3.644f, 0.131f, 0.535f, 0.136f},
    {1, 2, 4, 1, 3, 4.023f, 0.189f, 2.250f, 0.181f},
    {1, 4, 2, 1, 1, 3.370f, 0.157f, 0.414f, 0.110f},
    {1, 4, 2, 1, 2, 3.747f, 0.254f, 0.879f, 0.177f},
    {1, 2, 4, 2, 2, 4.234f, 0.178f, 1.074f, 0.164f},
    {1, 2, 4, 2, 3, 4.761f, 0.228f, 2.994f, 0.210f},
    {1, 2, 4, 2, 4, 5.022f, 0.300f, 3.412f, 0.287f},
    {1, 4, 2, 2, 1, 3.673f, 0.218f, 0.703f, 0.151f},
    {1, 4, 2, 2, 2, 4.190f, 0.327f, 1.291f, 0.260f},
    {1, 4, 2, 2, 3, 5.069f, 0.428f, 3.034f, 0.422f},
    {1, 8, 1, 2, 2, 4.412f, 0.648f, 1.956f, 0.464f},
    {1, 2, 4, 3, 3, 5.448f, 0.304f, 3.990f, 0.307f},
    {1, 4, 2, 3, 1, 4.257f, 0.290f, 1.007f, 0.215f},
    {1, 4, 2, 3, 2, 4.798f, 0.422f, 2.933f, 0.393f},
    {1, 4, 2, 3, 3, 6.242f, 0.537f, 4.725f, 0.528f},
    {1, 2, 4, 4, 3, 6.690f, 0.391f, 4.652f, 0.405f},
    {1, 4, 2, 4, 2, 5.218f, 0.429f, 3.278f, 0.428f},
    {1, 4, 2, 4, 3, 6.762f, 0.586f, 4.044f, 0.634f},
    {1, 8, 1, 4, 1, 4.124f, 0.586f, 1.650f, 0.412f},
    {1, 8, 1, 4, 2, 6.822f, 0.837f, 5.039f, 0.785f},
    {1, 8, 1, 6, 2, 8.877f, 1.034f, 5.601f, 1.103f},
    {2, 4, 1, 4, 3, 9.003f, 1.219f, 6.400f, 1.175f},
    {1, 8, 1, 8, 2, 11.10f, 1.346f, 9.165f, 1.309f},
    {1, 8, 1, 8, 3, 12.85f, 1.957f, 8.726f, 2.422f},
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
    const int c = pick_shape(kCosts, std::size(kCosts), a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF, 4, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return (tiled ? kLaunchTiled : a.k % 128 != 0 ? kLaunchRagged : kLaunch)[c](w, dev, stream);
}

}  // namespace mxfp4

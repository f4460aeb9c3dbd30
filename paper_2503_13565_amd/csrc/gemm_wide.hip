// MXFP4 weights in the block kernel of gemm_wide.h: row-major, tile-major, and row-major with any K % 32 == 0.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts[] = {
    {1, 1, 8, 1, 1, 4.29f, 0.060f, 1.20f, 0.047f},
    {1, 1, 8, 1, 2, 4.71f, 0.070f, 1.46f, 0.078f},
    {1, 1, 8, 1, 3, 5.05f, 0.107f, 1.73f, 0.099f},
    {1, 1, 8, 1, 4, 5.04f, 0.145f, 1.82f, 0.125f},
    {1, 1, 8, 1, 6, 5.46f, 0.224f, 4.12f, 0.185f},
    {1, 1, 8, 1, 8, 6.23f, 0.282f, 4.93f, 0.248f},
    {1, 1, 8, 2, 1, 5.18f, 0.101f, 3.47f, 0.101f},
    {1, 1, 8, 2, 2, 5.56f, 0.145f, 3.83f, 0.134f},
    {1, 1, 8, 2, 3, 5.98f, 0.182f, 4.27f, 0.164f},
    {1, 1, 8, 2, 4, 6.22f, 0.219f, 4.80f, 0.192f},
    {1, 1, 8, 2, 6, 7.51f, 0.290f, 6.36f, 0.240f},
    {1, 2, 4, 4, 1, 4.28f, 0.332f, 2.83f, 0.297f},
    {1, 2, 4, 4, 2, 5.42f, 0.378f, 4.55f, 0.310f},
    {1, 2, 4, 4, 3, 6.60f, 0.465f, 5.28f, 0.416f},
    {2, 2, 2, 4, 2, 7.37f, 0.685f, 5.26f, 0.647f},
    {2, 2, 2, 4, 3, 9.18f, 0.845f, 5.97f, 0.860f},
    {2, 4, 1, 4, 2, 8.47f, 0.990f, 0.57f, 1.088f},
    {2, 4, 1, 4, 3, 11.68f, 1.322f, 5.43f, 1.589f},
    {1, 8, 1, 8, 2, 13.11f, 1.649f, 10.94f, 1.719f},
    {1, 8, 1, 8, 3, 17.49f, 2.228f, 15.91f, 2.251f},
    {1, 4, 2, 4, 1, 4.52f, 0.447f, 1.79f, 0.317f},
    {1, 4, 2, 4, 2, 6.33f, 0.526f, 2.02f, 0.463f},
    {1, 4, 2, 4, 3, 8.68f, 0.704f, 4.44f, 0.877f},
};

#define MXFP4_WIDE(...)                                                                             \
    {launch_block<kMx, __VA_ARGS__>, launch_block<kMxTiled, __VA_ARGS__>, launch_block<kMxRagged, __VA_ARGS__>}
hipError_t (*const kLaunch[][3])(const Args&, const DeviceInfo&, hipStream_t) = {
    MXFP4_WIDE(1, 1, 8, 1, 1),
    MXFP4_WIDE(1, 1, 8, 1, 2),
    MXFP4_WIDE(1, 1, 8, 1, 3),
    MXFP4_WIDE(1, 1, 8, 1, 4),
    MXFP4_WIDE(1, 1, 8, 1, 6),
    MXFP4_WIDE(1, 1, 8, 1, 8),
    MXFP4_WIDE(1, 1, 8, 2, 1),
    MXFP4_WIDE(1, 1, 8, 2, 2),
    MXFP4_WIDE(1, 1, 8, 2, 3),
    MXFP4_WIDE(1, 1, 8, 2, 4),
    MXFP4_WIDE(1, 1, 8, 2, 6),
    MXFP4_WIDE(1, 2, 4, 4, 1),
    MXFP4_WIDE(1, 2, 4, 4, 2),
    MXFP4_WIDE(1, 2, 4, 4, 3),
    MXFP4_WIDE(2, 2, 2, 4, 2),
    MXFP4_WIDE(2, 2, 2, 4, 3),
    MXFP4_WIDE(2, 4, 1, 4, 2),
    MXFP4_WIDE(2, 4, 1, 4, 3),
    MXFP4_WIDE(1, 8, 1, 8, 2),
    MXFP4_WIDE(1, 8, 1, 8, 3),
    MXFP4_WIDE(1, 4, 2, 4, 1),
    MXFP4_WIDE(1, 4, 2, 4, 2),
    MXFP4_WIDE(1, 4, 2, 4, 3),
};
#undef MXFP4_WIDE
constexpr int kShapes = sizeof kCosts / sizeof kCosts[0];
static_assert(kShapes == sizeof kLaunch / sizeof kLaunch[0], "one cost per shape");

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
    Args w{a.x, a.q, a.s, a.n, a.k, a.m, (int)a.ldx, 0, 0, 0, block_out(a, epi)};
    const int c = pick_shape(kCosts, kShapes, a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return kLaunch[c][tiled ? 1 : a.k % 128 != 0 ? 2 : 0](w, dev, stream);
}

}  // namespace mxfp4

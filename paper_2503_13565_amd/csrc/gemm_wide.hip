// MXFP4 weights in the block kernel of gemm_wide.h: row-major, tile-major, and row-major with any K % 32 == 0.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts[] = {
    {1, 1, 8, 1, 1, 4.23f, 0.055f, 1.16f, 0.049f},
    {1, 1, 8, 1, 2, 4.51f, 0.075f, 1.40f, 0.073f},
    {1, 1, 8, 1, 3, 4.66f, 0.112f, 1.62f, 0.096f},
    {1, 1, 8, 1, 4, 4.67f, 0.155f, 1.73f, 0.123f},
    {1, 1, 8, 1, 6, 5.29f, 0.211f, 3.88f, 0.179f},
    {1, 1, 8, 1, 8, 5.86f, 0.276f, 4.65f, 0.240f},
    {1, 1, 8, 2, 1, 5.10f, 0.099f, 3.34f, 0.103f},
    {1, 1, 8, 2, 2, 5.59f, 0.129f, 3.95f, 0.108f},
    {1, 1, 8, 2, 3, 5.68f, 0.175f, 4.01f, 0.155f},
    {1, 1, 8, 2, 4, 6.05f, 0.192f, 4.71f, 0.156f},
    {1, 1, 8, 2, 6, 7.21f, 0.287f, 5.86f, 0.240f},
    {1, 2, 4, 4, 1, 4.45f, 0.304f, 2.94f, 0.259f},
    {1, 2, 4, 4, 2, 5.60f, 0.346f, 4.50f, 0.296f},
    {1, 2, 4, 4, 3, 6.92f, 0.426f, 5.63f, 0.365f},
    {2, 2, 2, 4, 2, 7.68f, 0.609f, 5.36f, 0.601f},
    {2, 2, 2, 4, 3, 9.76f, 0.749f, 7.03f, 0.718f},
    {2, 4, 1, 4, 2, 9.24f, 0.924f, 0.75f, 0.972f},
    {2, 4, 1, 4, 3, 11.60f, 1.275f, 5.75f, 1.423f},
    {1, 8, 1, 8, 2, 14.14f, 1.536f, 10.05f, 1.691f},
    {1, 8, 1, 8, 3, 17.04f, 2.171f, 14.60f, 2.183f},
    {1, 4, 2, 4, 1, 4.45f, 0.401f, 1.63f, 0.305f},
    {1, 4, 2, 4, 2, 6.68f, 0.500f, 2.07f, 0.422f},
    {1, 4, 2, 4, 3, 8.60f, 0.643f, 4.77f, 0.792f},
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

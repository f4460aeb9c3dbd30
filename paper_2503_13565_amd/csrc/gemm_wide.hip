// MXFP4 weights in the block kernel of gemm_wide.h: row-major, tile-major, and row-major with any K % 32 == 0.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts[] = {
    {1, 1, 8, 1, 1, 3.46f, 0.068f, 0.92f, 0.051f},
    {1, 1, 8, 1, 2, 3.83f, 0.089f, 1.10f, 0.079f},
    {1, 1, 8, 1, 3, 4.19f, 0.117f, 1.39f, 0.103f},
    {1, 1, 8, 1, 4, 4.44f, 0.144f, 1.71f, 0.127f},
    {1, 1, 8, 1, 6, 5.12f, 0.198f, 3.73f, 0.189f},
    {1, 2, 4, 1, 1, 2.92f, 0.100f, 0.28f, 0.088f},
    {1, 2, 4, 1, 2, 3.15f, 0.159f, 0.63f, 0.138f},
    {1, 2, 4, 1, 3, 3.44f, 0.218f, 1.06f, 0.191f},
    {1, 4, 2, 1, 1, 2.73f, 0.185f, 0.30f, 0.139f},
    {1, 4, 2, 1, 2, 2.90f, 0.300f, 0.55f, 0.265f},
    {1, 4, 2, 1, 3, 3.26f, 0.423f, 0.82f, 0.379f},
    {1, 1, 8, 2, 3, 5.54f, 0.151f, 3.95f, 0.142f},
    {1, 2, 4, 2, 1, 3.23f, 0.142f, 0.70f, 0.120f},
    {1, 2, 4, 2, 2, 3.68f, 0.196f, 1.08f, 0.172f},
    {1, 2, 4, 2, 3, 4.20f, 0.258f, 1.47f, 0.228f},
    {1, 2, 4, 2, 4, 4.64f, 0.311f, 3.14f, 0.304f},
    {1, 4, 2, 2, 1, 3.20f, 0.220f, 0.49f, 0.188f},
    {1, 4, 2, 2, 2, 3.61f, 0.329f, 0.97f, 0.306f},
    {1, 4, 2, 2, 3, 4.61f, 0.451f, 0.98f, 0.452f},
    {1, 4, 2, 2, 4, 5.03f, 0.574f, 2.87f, 0.615f},
    {1, 8, 1, 2, 2, 4.08f, 0.653f, 0.37f, 0.681f},
    {1, 2, 4, 3, 3, 5.43f, 0.298f, 3.67f, 0.312f},
    {1, 4, 2, 3, 1, 3.35f, 0.272f, 0.72f, 0.243f},
    {1, 4, 2, 3, 2, 4.89f, 0.381f, 0.80f, 0.395f},
    {1, 4, 2, 3, 3, 5.92f, 0.535f, 2.68f, 0.605f},
    {1, 2, 4, 4, 2, 4.71f, 0.289f, 3.35f, 0.271f},
    {1, 2, 4, 4, 3, 5.79f, 0.358f, 4.14f, 0.371f},
    {1, 4, 2, 4, 1, 3.44f, 0.327f, 0.99f, 0.296f},
    {1, 8, 1, 4, 1, 4.63f, 0.552f, 0.62f, 0.534f},
    {1, 4, 2, 4, 2, 5.59f, 0.452f, 2.59f, 0.488f},
    {1, 4, 2, 4, 3, 5.84f, 0.655f, 3.00f, 0.697f},
    {1, 8, 1, 4, 2, 6.37f, 0.863f, 0.55f, 0.964f},
    {1, 8, 1, 6, 2, 8.95f, 1.145f, 2.96f, 1.343f},
    {1, 8, 1, 6, 3, 11.31f, 1.690f, 7.65f, 1.784f},
    {2, 4, 1, 4, 2, 7.33f, 0.903f, 0.35f, 1.004f},
    {2, 4, 1, 4, 3, 8.79f, 1.244f, 2.56f, 1.413f},
    {2, 2, 2, 4, 3, 7.10f, 0.688f, 3.33f, 0.775f},
    {1, 8, 1, 8, 2, 9.90f, 1.478f, 5.53f, 1.669f},
    {1, 8, 1, 8, 3, 12.04f, 2.153f, 7.99f, 2.292f},
};

#define MXFP4_WIDE(...)                                                                             \
    {launch_block<kMx, __VA_ARGS__>, launch_block<kMxTiled, __VA_ARGS__>, launch_block<kMxRagged, __VA_ARGS__>}
hipError_t (*const kLaunch[][3])(const Args&, const DeviceInfo&, hipStream_t) = {
    MXFP4_WIDE(1, 1, 8, 1, 1),
    MXFP4_WIDE(1, 1, 8, 1, 2),
    MXFP4_WIDE(1, 1, 8, 1, 3),
    MXFP4_WIDE(1, 1, 8, 1, 4),
    MXFP4_WIDE(1, 1, 8, 1, 6),
    MXFP4_WIDE(1, 2, 4, 1, 1),
    MXFP4_WIDE(1, 2, 4, 1, 2),
    MXFP4_WIDE(1, 2, 4, 1, 3),
    MXFP4_WIDE(1, 4, 2, 1, 1),
    MXFP4_WIDE(1, 4, 2, 1, 2),
    MXFP4_WIDE(1, 4, 2, 1, 3),
    MXFP4_WIDE(1, 1, 8, 2, 3),
    MXFP4_WIDE(1, 2, 4, 2, 1),
    MXFP4_WIDE(1, 2, 4, 2, 2),
    MXFP4_WIDE(1, 2, 4, 2, 3),
    MXFP4_WIDE(1, 2, 4, 2, 4),
    MXFP4_WIDE(1, 4, 2, 2, 1),
    MXFP4_WIDE(1, 4, 2, 2, 2),
    MXFP4_WIDE(1, 4, 2, 2, 3),
    MXFP4_WIDE(1, 4, 2, 2, 4),
    MXFP4_WIDE(1, 8, 1, 2, 2),
    MXFP4_WIDE(1, 2, 4, 3, 3),
    MXFP4_WIDE(1, 4, 2, 3, 1),
    MXFP4_WIDE(1, 4, 2, 3, 2),
    MXFP4_WIDE(1, 4, 2, 3, 3),
    MXFP4_WIDE(1, 2, 4, 4, 2),
    MXFP4_WIDE(1, 2, 4, 4, 3),
    MXFP4_WIDE(1, 4, 2, 4, 1),
    MXFP4_WIDE(1, 8, 1, 4, 1),
    MXFP4_WIDE(1, 4, 2, 4, 2),
    MXFP4_WIDE(1, 4, 2, 4, 3),
    MXFP4_WIDE(1, 8, 1, 4, 2),
    MXFP4_WIDE(1, 8, 1, 6, 2),
    MXFP4_WIDE(1, 8, 1, 6, 3),
    MXFP4_WIDE(2, 4, 1, 4, 2),
    MXFP4_WIDE(2, 4, 1, 4, 3),
    MXFP4_WIDE(2, 2, 2, 4, 3),
    MXFP4_WIDE(1, 8, 1, 8, 2),
    MXFP4_WIDE(1, 8, 1, 8, 3),
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
    Args w{a.x, a.q, a.s, a.n, a.k, a.m, (int)a.ldx, 0, 0, 0, 0, block_out(a, epi)};
    const int c = pick_shape(kCosts, kShapes, a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF, 4, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return kLaunch[c][tiled ? 1 : a.k % 128 != 0 ? 2 : 0](w, dev, stream);
}

}  // namespace mxfp4

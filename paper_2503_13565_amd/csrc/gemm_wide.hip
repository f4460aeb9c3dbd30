// MXFP4 weights in the block kernel of gemm_wide.h: row-major, tile-major, and row-major with any K % 32 == 0.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts[] = {
    {1, 1, 8, 1, 1, 3.622f, 0.058f, 0.686f, 0.058f},
    {1, 1, 8, 1, 2, 3.841f, 0.077f, 0.785f, 0.090f},
    {1, 1, 8, 1, 3, 3.946f, 0.113f, 0.966f, 0.119f},
    {1, 2, 4, 1, 1, 3.510f, 0.100f, 0.362f, 0.079f},
    {1, 2, 4, 1, 2, 3.827f, 0.137f, 0.594f, 0.134f},
    {1, 2, 4, 1, 3, 3.980f, 0.194f, 1.082f, 0.149f},
    {1, 4, 2, 1, 1, 3.386f, 0.174f, 0.478f, 0.113f},
    {1, 4, 2, 1, 2, 3.641f, 0.251f, 0.778f, 0.163f},
    {1, 1, 8, 2, 3, 4.658f, 0.156f, 3.111f, 0.161f},
    {1, 2, 4, 2, 2, 4.246f, 0.183f, 1.079f, 0.166f},
    {1, 2, 4, 2, 3, 4.785f, 0.239f, 3.122f, 0.221f},
    {1, 4, 2, 2, 1, 3.644f, 0.217f, 0.685f, 0.152f},
    {1, 4, 2, 2, 2, 4.146f, 0.323f, 1.194f, 0.242f},
    {1, 4, 2, 2, 3, 5.014f, 0.429f, 3.059f, 0.425f},
    {1, 8, 1, 2, 2, 4.324f, 0.616f, 1.823f, 0.444f},
    {1, 2, 4, 3, 3, 6.123f, 0.313f, 4.433f, 0.310f},
    {1, 4, 2, 3, 1, 4.140f, 0.280f, 0.978f, 0.202f},
    {1, 4, 2, 3, 2, 4.752f, 0.395f, 2.816f, 0.383f},
    {1, 4, 2, 3, 3, 5.950f, 0.516f, 4.163f, 0.507f},
    {1, 2, 4, 4, 3, 6.346f, 0.368f, 4.390f, 0.393f},
    {1, 4, 2, 4, 2, 5.225f, 0.433f, 3.313f, 0.450f},
    {1, 4, 2, 4, 3, 6.753f, 0.585f, 4.280f, 0.638f},
    {1, 8, 1, 4, 1, 4.147f, 0.606f, 1.668f, 0.414f},
    {1, 8, 1, 4, 2, 6.889f, 0.863f, 5.098f, 0.832f},
    {1, 8, 1, 6, 2, 9.250f, 1.074f, 5.661f, 1.178f},
    {2, 4, 1, 4, 3, 9.174f, 1.204f, 6.128f, 1.224f},
    {1, 8, 1, 8, 2, 11.32f, 1.383f, 8.953f, 1.413f},
    {1, 8, 1, 8, 3, 12.40f, 2.021f, 9.467f, 2.519f},
};

#define MXFP4_WIDE(...)                                                                             \
    {launch_block<kMx, __VA_ARGS__>, launch_block<kMxTiled, __VA_ARGS__>, launch_block<kMxRagged, __VA_ARGS__>}
hipError_t (*const kLaunch[][3])(const Args&, const DeviceInfo&, hipStream_t) = {
    MXFP4_WIDE(1, 1, 8, 1, 1),
    MXFP4_WIDE(1, 1, 8, 1, 2),
    MXFP4_WIDE(1, 1, 8, 1, 3),
    MXFP4_WIDE(1, 2, 4, 1, 1),
    MXFP4_WIDE(1, 2, 4, 1, 2),
    MXFP4_WIDE(1, 2, 4, 1, 3),
    MXFP4_WIDE(1, 4, 2, 1, 1),
    MXFP4_WIDE(1, 4, 2, 1, 2),
    MXFP4_WIDE(1, 1, 8, 2, 3),
    MXFP4_WIDE(1, 2, 4, 2, 2),
    MXFP4_WIDE(1, 2, 4, 2, 3),
    MXFP4_WIDE(1, 4, 2, 2, 1),
    MXFP4_WIDE(1, 4, 2, 2, 2),
    MXFP4_WIDE(1, 4, 2, 2, 3),
    MXFP4_WIDE(1, 8, 1, 2, 2),
    MXFP4_WIDE(1, 2, 4, 3, 3),
    MXFP4_WIDE(1, 4, 2, 3, 1),
    MXFP4_WIDE(1, 4, 2, 3, 2),
    MXFP4_WIDE(1, 4, 2, 3, 3),
    MXFP4_WIDE(1, 2, 4, 4, 3),
    MXFP4_WIDE(1, 4, 2, 4, 2),
    MXFP4_WIDE(1, 4, 2, 4, 3),
    MXFP4_WIDE(1, 8, 1, 4, 1),
    MXFP4_WIDE(1, 8, 1, 4, 2),
    MXFP4_WIDE(1, 8, 1, 6, 2),
    MXFP4_WIDE(2, 4, 1, 4, 3),
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

// The other draft formats in the block kernel of gemm_wide.h (K % 128 == 0): E4M3, E5M2, E2M3, E3M2 and the
// ternary codes.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts8[] = {
    {1, 1, 8, 1, 1, 3.52f, 0.081f, 0.664f, 0.104f},
    {1, 2, 4, 1, 1, 3.20f, 0.142f, 0.f, 0.194f},
    {1, 4, 2, 1, 1, 2.92f, 0.284f, 0.f, 0.322f},
    {1, 4, 2, 1, 2, 2.67f, 0.583f, 0.f, 0.566f},
    {1, 1, 8, 2, 1, 4.48f, 0.117f, 2.94f, 0.124f},
    {1, 2, 4, 2, 1, 3.45f, 0.181f, 0.164f, 0.228f},
    {1, 4, 2, 2, 1, 3.17f, 0.316f, 0.268f, 0.358f},
    {1, 4, 2, 2, 2, 3.13f, 0.653f, 0.826f, 0.556f},
    {1, 4, 2, 3, 1, 3.67f, 0.345f, 0.416f, 0.389f},
    {1, 4, 2, 3, 2, 3.60f, 0.686f, 0.540f, 0.616f},
    {1, 2, 4, 4, 1, 4.42f, 0.255f, 1.95f, 0.322f},
    {1, 4, 2, 4, 1, 3.74f, 0.420f, 0.f, 0.456f},
    {1, 4, 2, 4, 2, 3.60f, 0.756f, 2.26f, 0.734f},
    {1, 8, 1, 4, 1, 2.50f, 0.819f, 0.192f, 0.682f},
    {1, 8, 1, 4, 2, 4.06f, 1.30f, 3.54f, 1.35f},
    {1, 8, 1, 8, 2, 7.16f, 1.68f, 8.49f, 1.82f},
};
#define MXFP4_WIDE(...) {launch_block<kE4m3, __VA_ARGS__>, launch_block<kE5m2, __VA_ARGS__>}
hipError_t (*const kLaunch8[][2])(const Args&, const DeviceInfo&, hipStream_t) = {
    MXFP4_WIDE(1, 1, 8, 1, 1),
    MXFP4_WIDE(1, 2, 4, 1, 1),
    MXFP4_WIDE(1, 4, 2, 1, 1),
    MXFP4_WIDE(1, 4, 2, 1, 2),
    MXFP4_WIDE(1, 1, 8, 2, 1),
    MXFP4_WIDE(1, 2, 4, 2, 1),
    MXFP4_WIDE(1, 4, 2, 2, 1),
    MXFP4_WIDE(1, 4, 2, 2, 2),
    MXFP4_WIDE(1, 4, 2, 3, 1),
    MXFP4_WIDE(1, 4, 2, 3, 2),
    MXFP4_WIDE(1, 2, 4, 4, 1),
    MXFP4_WIDE(1, 4, 2, 4, 1),
    MXFP4_WIDE(1, 4, 2, 4, 2),
    MXFP4_WIDE(1, 8, 1, 4, 1),
    MXFP4_WIDE(1, 8, 1, 4, 2),
    MXFP4_WIDE(1, 8, 1, 8, 2),
};
#undef MXFP4_WIDE
static_assert(sizeof kCosts8 / sizeof kCosts8[0] == sizeof kLaunch8 / sizeof kLaunch8[0], "one cost per shape");

const Cost kCosts6[] = {
    {1, 1, 8, 1, 1, 3.64f, 0.068f, 0.764f, 0.095f},
    {1, 2, 4, 1, 1, 3.37f, 0.108f, 0.f, 0.165f},
    {1, 2, 4, 1, 2, 3.42f, 0.212f, 0.f, 0.319f},
    {1, 4, 2, 1, 1, 3.10f, 0.225f, 0.f, 0.294f},
    {1, 4, 2, 1, 2, 2.76f, 0.476f, 0.f, 0.582f},
    {1, 2, 4, 2, 1, 3.53f, 0.168f, 0.593f, 0.187f},
    {1, 4, 2, 2, 1, 3.27f, 0.278f, 0.208f, 0.346f},
    {1, 4, 2, 2, 2, 3.48f, 0.510f, 0.983f, 0.553f},
    {1, 4, 2, 3, 1, 3.68f, 0.323f, 0.726f, 0.346f},
    {1, 4, 2, 3, 2, 4.36f, 0.596f, 2.16f, 0.569f},
    {1, 2, 4, 4, 1, 4.61f, 0.243f, 1.92f, 0.311f},
    {1, 4, 2, 4, 1, 3.84f, 0.372f, 0.798f, 0.408f},
    {1, 8, 1, 4, 1, 3.79f, 0.675f, 1.10f, 0.679f},
    {1, 8, 1, 4, 2, 4.63f, 1.22f, 1.70f, 1.56f},
    {1, 8, 1, 8, 2, 9.77f, 1.65f, 7.25f, 1.91f},
};
#define MXFP4_WIDE(...) {launch_block<kE2m3, __VA_ARGS__>, launch_block<kE3m2, __VA_ARGS__>}
hipError_t (*const kLaunch6[][2])(const Args&, const DeviceInfo&, hipStream_t) = {
    MXFP4_WIDE(1, 1, 8, 1, 1),
    MXFP4_WIDE(1, 2, 4, 1, 1),
    MXFP4_WIDE(1, 2, 4, 1, 2),
    MXFP4_WIDE(1, 4, 2, 1, 1),
    MXFP4_WIDE(1, 4, 2, 1, 2),
    MXFP4_WIDE(1, 2, 4, 2, 1),
    MXFP4_WIDE(1, 4, 2, 2, 1),
    MXFP4_WIDE(1, 4, 2, 2, 2),
    MXFP4_WIDE(1, 4, 2, 3, 1),
    MXFP4_WIDE(1, 4, 2, 3, 2),
    MXFP4_WIDE(1, 2, 4, 4, 1),
    MXFP4_WIDE(1, 4, 2, 4, 1),
    MXFP4_WIDE(1, 8, 1, 4, 1),
    MXFP4_WIDE(1, 8, 1, 4, 2),
    MXFP4_WIDE(1, 8, 1, 8, 2),
};
#undef MXFP4_WIDE
static_assert(sizeof kCosts6 / sizeof kCosts6[0] == sizeof kLaunch6 / sizeof kLaunch6[0], "one cost per shape");

const Cost kCosts2[] = {
    {1, 1, 8, 1, 1, 3.63f, 0.064f, 0.902f, 0.054f},
    {1, 1, 8, 1, 2, 3.82f, 0.094f, 1.24f, 0.078f},
    {1, 1, 8, 1, 4, 4.43f, 0.160f, 1.80f, 0.137f},
    {1, 2, 4, 1, 1, 3.37f, 0.117f, 0.432f, 0.075f},
    {1, 2, 4, 1, 2, 3.69f, 0.178f, 0.738f, 0.126f},
    {1, 4, 2, 1, 1, 3.25f, 0.213f, 0.540f, 0.128f},
    {1, 4, 2, 1, 2, 3.63f, 0.333f, 0.525f, 0.277f},
    {1, 2, 4, 2, 1, 3.66f, 0.151f, 0.774f, 0.118f},
    {1, 2, 4, 2, 2, 4.11f, 0.221f, 1.18f, 0.177f},
    {1, 4, 2, 2, 1, 3.40f, 0.274f, 0.756f, 0.170f},
    {1, 4, 2, 2, 2, 4.03f, 0.408f, 1.27f, 0.306f},
    {1, 4, 2, 3, 1, 3.71f, 0.333f, 0.916f, 0.227f},
    {1, 4, 2, 3, 2, 4.52f, 0.469f, 1.81f, 0.387f},
    {1, 2, 4, 4, 2, 5.17f, 0.328f, 3.28f, 0.329f},
    {1, 4, 2, 4, 1, 3.86f, 0.372f, 1.36f, 0.279f},
    {1, 4, 2, 4, 2, 5.61f, 0.509f, 3.21f, 0.557f},
    {1, 8, 1, 4, 1, 4.26f, 0.642f, 1.23f, 0.531f},
    {1, 8, 1, 4, 2, 6.83f, 1.00f, 0.580f, 0.946f},
    {1, 8, 1, 8, 2, 11.01f, 1.60f, 5.68f, 1.71f},
};
#define MXFP4_WIDE(...) {launch_block<kT2, __VA_ARGS__>}
hipError_t (*const kLaunch2[][1])(const Args&, const DeviceInfo&, hipStream_t) = {
    MXFP4_WIDE(1, 1, 8, 1, 1),
    MXFP4_WIDE(1, 1, 8, 1, 2),
    MXFP4_WIDE(1, 1, 8, 1, 4),
    MXFP4_WIDE(1, 2, 4, 1, 1),
    MXFP4_WIDE(1, 2, 4, 1, 2),
    MXFP4_WIDE(1, 4, 2, 1, 1),
    MXFP4_WIDE(1, 4, 2, 1, 2),
    MXFP4_WIDE(1, 2, 4, 2, 1),
    MXFP4_WIDE(1, 2, 4, 2, 2),
    MXFP4_WIDE(1, 4, 2, 2, 1),
    MXFP4_WIDE(1, 4, 2, 2, 2),
    MXFP4_WIDE(1, 4, 2, 3, 1),
    MXFP4_WIDE(1, 4, 2, 3, 2),
    MXFP4_WIDE(1, 2, 4, 4, 2),
    MXFP4_WIDE(1, 4, 2, 4, 1),
    MXFP4_WIDE(1, 4, 2, 4, 2),
    MXFP4_WIDE(1, 8, 1, 4, 1),
    MXFP4_WIDE(1, 8, 1, 4, 2),
    MXFP4_WIDE(1, 8, 1, 8, 2),
};
#undef MXFP4_WIDE
static_assert(sizeof kCosts2 / sizeof kCosts2[0] == sizeof kLaunch2 / sizeof kLaunch2[0], "one cost per shape");

}  // namespace

bool gemm_wide_fmt_can_run(const GemmArgs& a, const DeviceInfo& dev)
{
    return a.k % 128 == 0 && gemm_wide_can_run(a, dev) && (reinterpret_cast<uintptr_t>(a.s) & 3) == 0 &&
           (reinterpret_cast<uintptr_t>(a.q) & 15) == 0 && (a.part_val == nullptr || (a.n + 63) / 64 <= a.parts);
}

hipError_t launch_gemm_wide_fmt(int code, const GemmArgs& a, const DeviceInfo& dev, int* parts_used, hipStream_t stream)
{
    if (!gemm_wide_fmt_can_run(a, dev))
        return hipErrorInvalidValue;
    const int kind = code == 8 ? 0 : code == 24 ? 1 : code == 6 ? 2 : code == 22 ? 3 : code == 2 ? 4 : -1;
    if (kind < 0)
        return hipErrorInvalidValue;
    Args w{a.x, a.q, a.s, a.n, a.k, a.m, (int)a.ldx, 0, 0, 0, 0, block_out(a, nullptr)};
    const Cost* costs = kind < 2 ? kCosts8 : kind < 4 ? kCosts6 : kCosts2;
    const size_t bytes = kind < 2 ? sizeof kCosts8 : kind < 4 ? sizeof kCosts6 : sizeof kCosts2;
    const int c = pick_shape(costs, (int)(bytes / sizeof costs[0]), a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF,
                             kind < 2 ? 8 : kind < 4 ? 6 : 2, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return (kind < 2 ? kLaunch8[c][kind] : kind < 4 ? kLaunch6[c][kind - 2] : kLaunch2[c][0])(w, dev, stream);
}

}  // namespace mxfp4

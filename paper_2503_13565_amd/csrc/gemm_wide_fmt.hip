// The other draft formats in the block kernel of gemm_wide.h (K % 128 == 0): E4M3, E5M2, E2M3, E3M2 and the
// ternary codes.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts8[] = {
    {1, 1, 8, 1, 1, 3.509f, 0.081f, 0.581f, 0.108f},
    {1, 2, 4, 1, 1, 3.322f, 0.139f, 0.f, 0.198f},
    {1, 4, 2, 1, 1, 3.185f, 0.264f, 0.182f, 0.336f},
    {1, 4, 2, 1, 2, 3.126f, 0.520f, 0.652f, 0.432f},
    {1, 1, 8, 2, 1, 4.293f, 0.122f, 2.731f, 0.128f},
    {1, 2, 4, 2, 1, 3.669f, 0.185f, 0.574f, 0.221f},
    {1, 4, 2, 2, 1, 3.321f, 0.304f, 0.409f, 0.339f},
    {1, 4, 2, 2, 2, 3.546f, 0.622f, 1.128f, 0.463f},
    {1, 4, 2, 3, 1, 3.785f, 0.353f, 0.631f, 0.358f},
    {1, 4, 2, 3, 2, 4.234f, 0.640f, 2.298f, 0.577f},
    {1, 2, 4, 4, 1, 4.716f, 0.276f, 2.966f, 0.302f},
    {1, 4, 2, 4, 1, 4.227f, 0.427f, 1.002f, 0.411f},
    {1, 4, 2, 4, 2, 4.551f, 0.659f, 3.207f, 0.607f},
    {1, 8, 1, 4, 1, 4.073f, 0.678f, 1.394f, 0.597f},
    {1, 8, 1, 4, 2, 5.530f, 1.265f, 4.935f, 1.075f},
    {1, 8, 1, 8, 2, 10.39f, 1.487f, 7.528f, 1.611f},
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
    {1, 1, 8, 1, 1, 3.806f, 0.072f, 0.723f, 0.093f},
    {1, 2, 4, 1, 1, 3.416f, 0.116f, 0.f, 0.160f},
    {1, 2, 4, 1, 2, 3.426f, 0.206f, 0.f, 0.283f},
    {1, 4, 2, 1, 1, 3.254f, 0.224f, 0.212f, 0.224f},
    {1, 4, 2, 1, 2, 3.206f, 0.418f, 0.913f, 0.307f},
    {1, 1, 8, 2, 1, 4.446f, 0.118f, 2.857f, 0.121f},
    {1, 2, 4, 2, 1, 3.754f, 0.156f, 0.547f, 0.180f},
    {1, 4, 2, 2, 1, 3.445f, 0.270f, 0.420f, 0.261f},
    {1, 4, 2, 2, 2, 3.745f, 0.529f, 0.882f, 0.374f},
    {1, 4, 2, 3, 1, 3.956f, 0.331f, 0.839f, 0.295f},
    {1, 4, 2, 3, 2, 4.294f, 0.539f, 2.276f, 0.508f},
    {1, 2, 4, 4, 1, 4.419f, 0.244f, 2.794f, 0.252f},
    {1, 4, 2, 4, 1, 3.900f, 0.373f, 1.094f, 0.322f},
    {1, 4, 2, 4, 2, 4.507f, 0.608f, 3.006f, 0.568f},
    {1, 8, 1, 4, 1, 4.186f, 0.652f, 1.435f, 0.551f},
    {1, 8, 1, 4, 2, 5.960f, 1.163f, 5.081f, 1.119f},
    {1, 8, 1, 8, 2, 8.990f, 1.600f, 5.428f, 1.698f},
};
#define MXFP4_WIDE(...) {launch_block<kE2m3, __VA_ARGS__>, launch_block<kE3m2, __VA_ARGS__>}
hipError_t (*const kLaunch6[][2])(const Args&, const DeviceInfo&, hipStream_t) = {
    MXFP4_WIDE(1, 1, 8, 1, 1),
    MXFP4_WIDE(1, 2, 4, 1, 1),
    MXFP4_WIDE(1, 2, 4, 1, 2),
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
static_assert(sizeof kCosts6 / sizeof kCosts6[0] == sizeof kLaunch6 / sizeof kLaunch6[0], "one cost per shape");

const Cost kCosts2[] = {
    {1, 1, 8, 1, 1, 3.652f, 0.065f, 0.757f, 0.055f},
    {1, 1, 8, 1, 2, 3.807f, 0.097f, 0.848f, 0.085f},
    {1, 2, 4, 1, 1, 3.538f, 0.122f, 0.447f, 0.082f},
    {1, 2, 4, 1, 2, 3.768f, 0.174f, 0.800f, 0.126f},
    {1, 4, 2, 1, 1, 3.405f, 0.229f, 0.569f, 0.136f},
    {1, 4, 2, 1, 2, 3.735f, 0.361f, 0.934f, 0.235f},
    {1, 1, 8, 2, 2, 4.722f, 0.145f, 3.242f, 0.135f},
    {1, 2, 4, 2, 1, 3.833f, 0.165f, 0.954f, 0.110f},
    {1, 2, 4, 2, 2, 4.255f, 0.233f, 1.416f, 0.161f},
    {1, 4, 2, 2, 1, 3.610f, 0.281f, 0.762f, 0.165f},
    {1, 4, 2, 2, 2, 4.214f, 0.410f, 1.422f, 0.287f},
    {1, 4, 2, 3, 1, 4.010f, 0.324f, 1.060f, 0.222f},
    {1, 4, 2, 3, 2, 4.944f, 0.475f, 1.896f, 0.341f},
    {1, 2, 4, 4, 2, 6.097f, 0.331f, 3.870f, 0.329f},
    {1, 4, 2, 4, 1, 4.368f, 0.380f, 1.407f, 0.281f},
    {1, 4, 2, 4, 2, 5.323f, 0.510f, 3.631f, 0.498f},
    {1, 8, 1, 4, 1, 4.324f, 0.667f, 1.617f, 0.464f},
    {1, 8, 1, 4, 2, 6.954f, 0.987f, 4.795f, 0.988f},
    {1, 8, 1, 8, 2, 10.50f, 1.487f, 6.196f, 1.604f},
};
#define MXFP4_WIDE(...) {launch_block<kT2, __VA_ARGS__>}
hipError_t (*const kLaunch2[][1])(const Args&, const DeviceInfo&, hipStream_t) = {
    MXFP4_WIDE(1, 1, 8, 1, 1),
    MXFP4_WIDE(1, 1, 8, 1, 2),
    MXFP4_WIDE(1, 2, 4, 1, 1),
    MXFP4_WIDE(1, 2, 4, 1, 2),
    MXFP4_WIDE(1, 4, 2, 1, 1),
    MXFP4_WIDE(1, 4, 2, 1, 2),
    MXFP4_WIDE(1, 1, 8, 2, 2),
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

// The other draft formats in the block kernel of gemm_wide.h (K % 128 == 0): E4M3, E5M2, E2M3, E3M2 and the
// ternary codes.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts8[] = {
    {1, 1, 8, 1, 1, 4.51f, 0.072f, 1.44f, 0.071f},
    {1, 1, 8, 1, 2, 4.98f, 0.123f, 1.56f, 0.131f},
    {1, 1, 8, 1, 4, 5.80f, 0.237f, 3.29f, 0.222f},
    {1, 1, 8, 2, 1, 5.54f, 0.109f, 3.54f, 0.122f},
    {1, 1, 8, 2, 2, 5.96f, 0.184f, 4.14f, 0.180f},
    {1, 1, 8, 2, 4, 7.42f, 0.288f, 6.07f, 0.248f},
    {1, 2, 4, 4, 1, 4.62f, 0.364f, 3.01f, 0.326f},
    {1, 2, 4, 4, 2, 5.96f, 0.461f, 4.57f, 0.425f},
    {1, 4, 2, 4, 1, 4.89f, 0.483f, 1.47f, 0.371f},
    {1, 4, 2, 4, 2, 7.08f, 0.676f, 0.f, 0.841f},
    {2, 4, 1, 4, 2, 8.92f, 1.214f, 3.20f, 1.509f},
    {1, 8, 1, 8, 2, 13.60f, 1.746f, 9.74f, 1.965f},
};
const Cost kCosts6[] = {
    {1, 1, 8, 1, 1, 4.52f, 0.064f, 1.23f, 0.070f},
    {1, 1, 8, 1, 2, 5.02f, 0.118f, 1.50f, 0.130f},
    {1, 1, 8, 1, 4, 5.74f, 0.246f, 4.03f, 0.236f},
    {1, 1, 8, 2, 1, 5.52f, 0.113f, 3.51f, 0.130f},
    {1, 1, 8, 2, 2, 6.32f, 0.162f, 4.22f, 0.186f},
    {1, 1, 8, 2, 4, 7.36f, 0.303f, 5.92f, 0.266f},
    {1, 2, 4, 4, 1, 4.63f, 0.372f, 2.91f, 0.352f},
    {1, 2, 4, 4, 2, 6.07f, 0.472f, 4.70f, 0.423f},
    {1, 4, 2, 4, 1, 4.75f, 0.515f, 1.72f, 0.371f},
    {1, 4, 2, 4, 2, 6.47f, 0.724f, 4.79f, 0.681f},
    {2, 4, 1, 4, 2, 8.40f, 1.351f, 3.77f, 1.529f},
    {1, 8, 1, 8, 2, 14.05f, 1.843f, 7.03f, 2.234f},
};
const Cost kCosts2[] = {
    {1, 1, 8, 1, 1, 4.35f, 0.061f, 1.11f, 0.053f},
    {1, 1, 8, 1, 2, 4.81f, 0.094f, 1.50f, 0.077f},
    {1, 1, 8, 1, 4, 5.46f, 0.165f, 2.10f, 0.150f},
    {1, 1, 8, 2, 1, 5.43f, 0.101f, 3.50f, 0.106f},
    {1, 1, 8, 2, 2, 6.04f, 0.139f, 3.92f, 0.154f},
    {1, 1, 8, 2, 4, 6.95f, 0.224f, 4.79f, 0.240f},
    {1, 2, 4, 4, 1, 4.57f, 0.337f, 2.99f, 0.298f},
    {1, 2, 4, 4, 2, 5.80f, 0.402f, 4.33f, 0.351f},
    {1, 4, 2, 4, 1, 4.73f, 0.460f, 1.34f, 0.352f},
    {1, 4, 2, 4, 2, 6.88f, 0.610f, 2.32f, 0.485f},
    {2, 4, 1, 4, 2, 9.05f, 1.137f, 1.12f, 1.093f},
    {1, 8, 1, 8, 2, 14.92f, 1.663f, 8.29f, 1.821f},
};

#define MXFP4_WIDE(...)                                                                                             \
    {launch_block<kE4m3, __VA_ARGS__>, launch_block<kE5m2, __VA_ARGS__>, launch_block<kE2m3, __VA_ARGS__>,            \
     launch_block<kE3m2, __VA_ARGS__>, launch_block<kT2, __VA_ARGS__>}
hipError_t (*const kLaunch[][5])(const Args&, const DeviceInfo&, hipStream_t) = {
    MXFP4_WIDE(1, 1, 8, 1, 1),
    MXFP4_WIDE(1, 1, 8, 1, 2),
    MXFP4_WIDE(1, 1, 8, 1, 4),
    MXFP4_WIDE(1, 1, 8, 2, 1),
    MXFP4_WIDE(1, 1, 8, 2, 2),
    MXFP4_WIDE(1, 1, 8, 2, 4),
    MXFP4_WIDE(1, 2, 4, 4, 1),
    MXFP4_WIDE(1, 2, 4, 4, 2),
    MXFP4_WIDE(1, 4, 2, 4, 1),
    MXFP4_WIDE(1, 4, 2, 4, 2),
    MXFP4_WIDE(2, 4, 1, 4, 2),
    MXFP4_WIDE(1, 8, 1, 8, 2),
};
#undef MXFP4_WIDE
constexpr int kShapes = sizeof kCosts8 / sizeof kCosts8[0];
static_assert(kShapes == sizeof kLaunch / sizeof kLaunch[0], "one cost per shape");

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
    Args w{a.x, a.q, a.s, a.n, a.k, a.m, (int)a.ldx, 0, 0, 0, block_out(a, nullptr)};
    const int c = pick_shape(kind < 2 ? kCosts8 : kind < 4 ? kCosts6 : kCosts2, kShapes, a.m, a.n, a.k, dev.cus,
                             a.part_val ? a.parts : 0x7FFFFFFF, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return kLaunch[c][kind](w, dev, stream);
}

}  // namespace mxfp4

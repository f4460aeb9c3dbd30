// Unquantised BF16 weights in the block kernel of gemm_wide.h (any K % 8 == 0).
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts[] = {
    {1, 1, 8, 1, 1, 3.780f, 0.142f, 0.573f, 0.199f},
    {1, 2, 4, 1, 1, 3.296f, 0.260f, 0.f, 0.370f},
    {1, 4, 2, 1, 1, 3.324f, 0.520f, 0.176f, 0.657f},
    {1, 4, 2, 1, 2, 2.938f, 1.046f, 1.549f, 0.816f},
    {1, 1, 8, 2, 1, 4.155f, 0.185f, 2.585f, 0.203f},
    {1, 2, 4, 2, 1, 3.402f, 0.292f, 0.628f, 0.360f},
    {1, 4, 2, 2, 1, 3.349f, 0.531f, 0.350f, 0.636f},
    {1, 4, 2, 2, 2, 3.464f, 1.060f, 2.887f, 0.857f},
    {1, 4, 2, 3, 1, 3.626f, 0.573f, 0.815f, 0.588f},
    {1, 4, 2, 3, 2, 4.446f, 1.069f, 3.219f, 1.005f},
    {1, 2, 4, 4, 1, 4.317f, 0.396f, 2.696f, 0.428f},
    {1, 4, 2, 4, 1, 3.946f, 0.615f, 1.062f, 0.615f},
    {1, 4, 2, 4, 2, 4.794f, 1.082f, 3.729f, 1.075f},
    {1, 8, 1, 4, 1, 4.210f, 1.080f, 1.242f, 1.019f},
    {1, 8, 1, 4, 2, 6.305f, 1.961f, 4.235f, 1.883f},
    {1, 8, 1, 8, 2, 9.855f, 2.460f, 6.286f, 2.506f},
};

#define MXFP4_WIDE(...) launch_block<kBf16, __VA_ARGS__>
hipError_t (*const kLaunch[])(const Args&, const DeviceInfo&, hipStream_t) = {
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
constexpr int kShapes = sizeof kCosts / sizeof kCosts[0];
static_assert(kShapes == sizeof kLaunch / sizeof kLaunch[0], "one cost per shape");

}  // namespace

bool gemm_wide_bf16_can_run(const Bf16Args& a, const DeviceInfo& dev)
{
    if (a.k % 8 != 0 || a.m < 1 || a.ldx > (1 << 21) || a.ldw > 0x3FFFFFFF || dev.lds_bytes < 160 * 1024)
        return false;
    if (((int64_t)(a.n - 1) * a.ldw + a.k) * 2 > kOob)
        return false;
    return a.part_val == nullptr || (a.n + 63) / 64 <= a.parts;
}

hipError_t launch_gemm_wide_bf16(const Bf16Args& a, const DeviceInfo& dev, int* parts_used, hipStream_t stream)
{
    if (!gemm_wide_bf16_can_run(a, dev))
        return hipErrorInvalidValue;
    Args w{a.x, reinterpret_cast<const uint8_t*>(a.w), nullptr, a.n, a.k, a.m, (int)a.ldx, (int)a.ldw, 0, 0, 0,
           BlockOut{a.y, a.ldy, a.part_val, a.part_idx, nullptr, nullptr, a.n, a.m, a.parts, 0, 0}};
    const int c = pick_shape(kCosts, kShapes, a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF, 16, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return kLaunch[c](w, dev, stream);
}

}  // namespace mxfp4

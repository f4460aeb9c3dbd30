// Unquantised BF16 weights in the block kernel of gemm_wide.h (any K % 8 == 0).
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts[] = {
    {1, 1, 8, 1, 1, 3.45f, 0.135f, 0.663f, 0.177f},
    {1, 2, 4, 1, 1, 3.05f, 0.257f, 0.552f, 0.307f},
    {1, 4, 2, 1, 1, 2.64f, 0.541f, 1.11f, 0.476f},
    {1, 4, 2, 1, 2, 3.53f, 0.981f, 0.692f, 0.962f},
    {1, 1, 8, 2, 1, 4.18f, 0.175f, 2.43f, 0.209f},
    {1, 2, 4, 2, 1, 3.14f, 0.307f, 0.717f, 0.336f},
    {1, 4, 2, 2, 1, 2.91f, 0.567f, 1.14f, 0.515f},
    {1, 4, 2, 2, 2, 4.04f, 1.01f, 1.79f, 1.02f},
    {1, 4, 2, 3, 1, 3.35f, 0.587f, 0.722f, 0.606f},
    {1, 4, 2, 3, 2, 4.47f, 1.06f, 1.97f, 1.14f},
    {1, 2, 4, 4, 1, 4.04f, 0.395f, 1.63f, 0.438f},
    {1, 4, 2, 4, 1, 3.57f, 0.631f, 0.781f, 0.636f},
    {1, 8, 1, 4, 1, 4.02f, 1.08f, 0.884f, 1.12f},
    {1, 8, 1, 4, 2, 5.77f, 1.99f, 4.28f, 2.13f},
    {1, 8, 1, 8, 2, 9.26f, 2.38f, 9.86f, 2.34f},
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

// Unquantised BF16 weights in the block kernel of gemm_wide.h (any K % 8 == 0).
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

const Cost kCosts[] = {
    {1, 1, 8, 1, 1, 4.46f, 0.113f, 1.37f, 0.124f},
    {1, 1, 8, 1, 2, 5.27f, 0.228f, 2.39f, 0.209f},
    {1, 1, 8, 1, 4, 7.30f, 0.417f, 5.55f, 0.427f},
    {1, 1, 8, 2, 1, 5.65f, 0.147f, 3.59f, 0.161f},
    {1, 1, 8, 2, 2, 6.94f, 0.256f, 5.42f, 0.230f},
    {1, 1, 8, 2, 4, 8.58f, 0.472f, 6.54f, 0.515f},
    {1, 2, 4, 4, 1, 4.88f, 0.409f, 3.63f, 0.363f},
    {1, 2, 4, 4, 2, 6.27f, 0.618f, 4.04f, 0.684f},
    {1, 4, 2, 4, 1, 4.57f, 0.594f, 0.77f, 0.647f},
    {1, 4, 2, 4, 2, 7.79f, 0.987f, 2.73f, 1.275f},
    {2, 4, 1, 4, 2, 9.68f, 1.937f, 3.04f, 2.291f},
    {1, 8, 1, 8, 2, 12.47f, 2.422f, 13.42f, 2.361f},
};

#define MXFP4_WIDE(...) launch_block<kBf16, __VA_ARGS__>
hipError_t (*const kLaunch[])(const Args&, const DeviceInfo&, hipStream_t) = {
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
    Args w{a.x, reinterpret_cast<const uint8_t*>(a.w), nullptr, a.n, a.k, a.m, (int)a.ldx, (int)a.ldw, 0, 0,
           BlockOut{a.y, a.ldy, a.part_val, a.part_idx, nullptr, nullptr, a.n, a.m, a.parts, 0, 0}};
    const int c = pick_shape(kCosts, kShapes, a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return kLaunch[c](w, dev, stream);
}

}  // namespace mxfp4

// Unquantised BF16 weights in the block kernel of gemm_wide.h (any K % 8 == 0).
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

constexpr Cost kCosts[] = {
    {1, 1, 8, 1, 1, 3.685f, 0.146f, 0.354f, 0.209f},
    {1, 2, 4, 1, 1, 3.667f, 0.267f, 0.263f, 0.400f},
    {1, 4, 2, 1, 1, 3.895f, 0.532f, 0.341f, 0.671f},
    {1, 4, 2, 1, 2, 3.947f, 1.087f, 0.848f, 1.462f},
    {1, 1, 8, 2, 1, 4.711f, 0.189f, 2.284f, 0.222f},
    {1, 2, 4, 2, 1, 4.709f, 0.294f, 0.488f, 0.411f},
    {1, 4, 2, 2, 1, 3.750f, 0.605f, 0.608f, 0.659f},
    {1, 4, 2, 2, 2, 4.623f, 1.131f, 2.094f, 1.258f},
    {1, 4, 2, 3, 1, 4.145f, 0.602f, 1.143f, 0.641f},
    {1, 4, 2, 3, 2, 4.737f, 1.131f, 2.982f, 1.232f},
    {1, 2, 4, 4, 1, 5.172f, 0.386f, 2.825f, 0.418f},
    {1, 4, 2, 4, 1, 4.191f, 0.634f, 1.198f, 0.666f},
    {1, 4, 2, 4, 2, 5.115f, 1.182f, 3.670f, 1.136f},
    {1, 8, 1, 4, 1, 3.984f, 1.050f, 1.644f, 1.081f},
    {1, 8, 1, 4, 2, 6.368f, 2.068f, 5.338f, 2.093f},
    {1, 8, 1, 8, 2, 9.822f, 2.675f, 11.51f, 2.267f},
};

constexpr auto kLaunch = launches<kBf16, kCosts>();

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
    const int c = pick_shape<kCosts, 16>(a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return kLaunch[c](w, dev, stream);
}

}  // namespace mxfp4

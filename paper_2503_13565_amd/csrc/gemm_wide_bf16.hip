// Unquantised BF16 weights in the block kernel of gemm_wide.h (any K % 8 == 0).
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

constexpr Cost kCosts[] = {
    {1, 1, 8, 1, 1, 3.341f, 0.138f, 0.497f, 0.196f},
    {1, 2, 4, 1, 1, 3.187f, 0.250f, 0.f, 0.361f},
    {1, 4, 2, 1, 1, 3.209f, 0.501f, 0.203f, 0.631f},
    {1, 4, 2, 1, 2, 2.594f, 1.011f, 1.528f, 0.794f},
    {1, 1, 8, 2, 1, 3.994f, 0.176f, 2.514f, 0.196f},
    {1, 2, 4, 2, 1, 3.422f, 0.294f, 0.623f, 0.361f},
    {1, 4, 2, 2, 1, 3.360f, 0.533f, 0.345f, 0.636f},
    {1, 4, 2, 2, 2, 3.541f, 1.050f, 2.797f, 0.867f},
    {1, 4, 2, 3, 1, 3.645f, 0.576f, 0.838f, 0.590f},
    {1, 4, 2, 3, 2, 4.413f, 1.069f, 3.155f, 1.010f},
    {1, 2, 4, 4, 1, 4.212f, 0.389f, 2.693f, 0.416f},
    {1, 4, 2, 4, 1, 3.914f, 0.682f, 1.088f, 0.617f},
    {1, 4, 2, 4, 2, 4.770f, 1.086f, 3.754f, 1.074f},
    {1, 8, 1, 4, 1, 4.237f, 1.081f, 1.268f, 1.024f},
    {1, 8, 1, 4, 2, 6.103f, 2.006f, 4.303f, 1.929f},
    {1, 8, 1, 8, 2, 9.309f, 2.480f, 6.431f, 2.503f},
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
    const int c = pick_shape(kCosts, std::size(kCosts), a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF, 16, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    return kLaunch[c](w, dev, stream);
}

}  // namespace mxfp4

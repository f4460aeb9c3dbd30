// The other draft formats in the block kernel of gemm_wide.h (K % 128 == 0): E4M3, E5M2, E2M3, E3M2 and the
// ternary codes.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

constexpr Cost kCosts8[] = {
    {1, 1, 8, 1, 1, 3.509f, 0.082f, 0.606f, 0.109f},
    {1, 2, 4, 1, 1, 3.503f, 0.132f, 0.f, 0.208f},
    {1, 4, 2, 1, 1, 3.130f, 0.260f, 0.217f, 0.360f},
    {1, 4, 2, 1, 2, 3.316f, 0.558f, 0.724f, 0.459f},
    {1, 1, 8, 2, 1, 4.468f, 0.115f, 2.588f, 0.122f},
    {1, 2, 4, 2, 1, 3.609f, 0.182f, 0.596f, 0.216f},
    {1, 4, 2, 2, 1, 3.406f, 0.310f, 0.424f, 0.345f},
    {1, 4, 2, 2, 2, 3.629f, 0.560f, 1.118f, 0.464f},
    {1, 4, 2, 3, 1, 3.730f, 0.346f, 0.614f, 0.349f},
    {1, 4, 2, 3, 2, 4.328f, 0.600f, 2.334f, 0.618f},
    {1, 2, 4, 4, 1, 4.841f, 0.271f, 2.916f, 0.296f},
    {1, 4, 2, 4, 1, 3.876f, 0.430f, 0.989f, 0.415f},
    {1, 4, 2, 4, 2, 4.871f, 0.658f, 3.342f, 0.619f},
    {1, 8, 1, 4, 1, 4.135f, 0.678f, 1.336f, 0.613f},
    {1, 8, 1, 4, 2, 5.680f, 1.250f, 4.844f, 1.080f},
    {1, 8, 1, 8, 2, 10.67f, 1.570f, 7.428f, 1.646f},
};
constexpr auto kLaunchE4m3 = launches<kE4m3, kCosts8>(), kLaunchE5m2 = launches<kE5m2, kCosts8>();

constexpr Cost kCosts6[] = {
    {1, 1, 8, 1, 1, 3.854f, 0.073f, 0.728f, 0.094f},
    {1, 2, 4, 1, 1, 3.426f, 0.116f, 0.f, 0.160f},
    {1, 2, 4, 1, 2, 3.828f, 0.199f, 0.f, 0.283f},
    {1, 4, 2, 1, 1, 3.256f, 0.226f, 0.264f, 0.215f},
    {1, 4, 2, 1, 2, 3.348f, 0.439f, 0.999f, 0.315f},
    {1, 1, 8, 2, 1, 4.469f, 0.117f, 2.857f, 0.121f},
    {1, 2, 4, 2, 1, 3.765f, 0.158f, 0.571f, 0.180f},
    {1, 4, 2, 2, 1, 3.472f, 0.267f, 0.424f, 0.262f},
    {1, 4, 2, 2, 2, 3.832f, 0.529f, 0.810f, 0.385f},
    {1, 4, 2, 3, 1, 4.021f, 0.334f, 0.847f, 0.295f},
    {1, 4, 2, 3, 2, 4.646f, 0.537f, 2.144f, 0.514f},
    {1, 2, 4, 4, 1, 4.303f, 0.248f, 2.904f, 0.258f},
    {1, 4, 2, 4, 1, 4.035f, 0.397f, 1.145f, 0.353f},
    {1, 4, 2, 4, 2, 5.005f, 0.616f, 3.021f, 0.518f},
    {1, 8, 1, 4, 1, 4.170f, 0.657f, 1.407f, 0.533f},
    {1, 8, 1, 4, 2, 6.538f, 1.119f, 4.837f, 0.973f},
    {1, 8, 1, 8, 2, 9.933f, 1.600f, 6.196f, 1.840f},
};
constexpr auto kLaunchE2m3 = launches<kE2m3, kCosts6>(), kLaunchE3m2 = launches<kE3m2, kCosts6>();

constexpr Cost kCosts2[] = {
    {1, 1, 8, 1, 1, 3.666f, 0.065f, 0.796f, 0.054f},
    {1, 1, 8, 1, 2, 3.943f, 0.098f, 1.084f, 0.082f},
    {1, 2, 4, 1, 1, 3.480f, 0.115f, 0.389f, 0.078f},
    {1, 2, 4, 1, 2, 3.663f, 0.176f, 0.863f, 0.138f},
    {1, 4, 2, 1, 1, 3.355f, 0.211f, 0.488f, 0.128f},
    {1, 4, 2, 1, 2, 3.570f, 0.344f, 0.868f, 0.247f},
    {1, 2, 4, 2, 1, 3.653f, 0.152f, 0.863f, 0.121f},
    {1, 2, 4, 2, 2, 4.383f, 0.221f, 1.336f, 0.167f},
    {1, 4, 2, 2, 1, 3.635f, 0.278f, 0.759f, 0.166f},
    {1, 4, 2, 2, 2, 4.241f, 0.408f, 1.407f, 0.289f},
    {1, 4, 2, 3, 1, 3.816f, 0.325f, 1.052f, 0.221f},
    {1, 4, 2, 3, 2, 5.182f, 0.477f, 1.819f, 0.337f},
    {1, 2, 4, 4, 2, 5.925f, 0.318f, 3.849f, 0.324f},
    {1, 4, 2, 4, 1, 4.318f, 0.373f, 1.350f, 0.276f},
    {1, 4, 2, 4, 2, 5.455f, 0.523f, 3.705f, 0.504f},
    {1, 8, 1, 4, 1, 4.416f, 0.662f, 1.429f, 0.483f},
    {1, 8, 1, 4, 2, 6.932f, 0.982f, 4.741f, 0.984f},
    {1, 8, 1, 8, 2, 10.81f, 1.485f, 6.768f, 1.621f},
};
constexpr auto kLaunchT2 = launches<kT2, kCosts2>();

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
    const size_t count = kind < 2 ? std::size(kCosts8) : kind < 4 ? std::size(kCosts6) : std::size(kCosts2);
    const int c = pick_shape(costs, count, a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF,
                             kind < 2 ? 8 : kind < 4 ? 6 : 2, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    const Launch* const launch[] = {kLaunchE4m3.data(), kLaunchE5m2.data(), kLaunchE2m3.data(), kLaunchE3m2.data(), kLaunchT2.data()};
    return launch[kind][c](w, dev, stream);
}

}  // namespace mxfp4

// The other draft formats in the block kernel of gemm_wide.h (K % 128 == 0): E4M3, E5M2, E2M3, E3M2 and the
// ternary codes.
#include "gemm_wide.h"

namespace mxfp4 {

namespace {

using namespace wide;

constexpr Cost kCosts8[] = {
    {1, 1, 8, 1, 1, 3.509f, 0.082f, 0.606f, 0.102f},
    {1, 2, 4, 1, 1, 3.621f, 0.132f, 0.f, 0.208f},
    {1, 4, 2, 1, 1, 3.130f, 0.260f, 0.211f, 0.353f},
    {1, 4, 2, 1, 2, 3.593f, 0.551f, 0.724f, 0.459f},
    {1, 1, 8, 2, 1, 6.056f, 0.119f, 2.588f, 0.122f},
    {1, 2, 4, 2, 1, 3.609f, 0.182f, 0.596f, 0.216f},
    {1, 4, 2, 2, 1, 3.508f, 0.343f, 0.424f, 0.345f},
    {1, 4, 2, 2, 2, 4.131f, 0.560f, 1.118f, 0.464f},
    {1, 4, 2, 3, 1, 3.512f, 0.404f, 1.013f, 0.416f},
    {1, 4, 2, 3, 2, 4.241f, 0.612f, 1.767f, 0.623f},
    {1, 2, 4, 4, 1, 4.841f, 0.285f, 2.916f, 0.296f},
    {1, 4, 2, 4, 1, 3.876f, 0.430f, 0.989f, 0.407f},
    {1, 4, 2, 4, 2, 4.678f, 0.618f, 3.342f, 0.619f},
    {1, 8, 1, 4, 1, 3.804f, 0.678f, 1.323f, 0.613f},
    {1, 8, 1, 4, 2, 5.405f, 1.250f, 4.562f, 1.081f},
    {1, 8, 1, 8, 2, 10.58f, 1.503f, 7.428f, 1.356f},
};
constexpr auto kLaunchE4m3 = launches<kE4m3, kCosts8>(), kLaunchE5m2 = launches<kE5m2, kCosts8>();

constexpr Cost kCosts6[] = {
    {1, 1, 8, 1, 1, 4.692f, 0.036f, 0.578f, 0.103f},
    {1, 2, 4, 1, 1, 4.035f, 0.114f, 0.002f, 0.179f},
    {1, 2, 4, 1, 2, 4.075f, 0.214f, 0.091f, 0.295f},
    {1, 4, 2, 1, 1, 3.939f, 0.217f, 0.075f, 0.299f},
    {1, 4, 2, 1, 2, 3.865f, 0.486f, 0.396f, 0.530f},
    {1, 1, 8, 2, 1, 4.962f, 0.121f, 2.689f, 0.130f},
    {1, 2, 4, 2, 1, 4.282f, 0.189f, 0.503f, 0.208f},
    {1, 4, 2, 2, 1, 4.163f, 0.303f, 0.295f, 0.333f},
    {1, 4, 2, 2, 2, 4.535f, 0.591f, 0.977f, 0.449f},
    {1, 4, 2, 3, 1, 4.245f, 0.310f, 0.848f, 0.375f},
    {1, 4, 2, 3, 2, 4.544f, 0.633f, 3.744f, 0.528f},
    {1, 2, 4, 4, 1, 4.691f, 0.284f, 3.009f, 0.278f},
    {1, 4, 2, 4, 1, 4.767f, 0.424f, 1.145f, 0.391f},
    {1, 4, 2, 4, 2, 5.100f, 0.718f, 3.740f, 0.605f},
    {1, 8, 1, 4, 1, 4.097f, 0.783f, 1.104f, 0.622f},
    {1, 8, 1, 4, 2, 5.320f, 1.393f, 4.533f, 1.113f},
    {1, 8, 1, 8, 2, 10.22f, 1.806f, 7.852f, 1.758f},
};
constexpr auto kLaunchE2m3 = launches<kE2m3, kCosts6>(), kLaunchE3m2 = launches<kE3m2, kCosts6>();

constexpr Cost kCosts2[] = {
    {1, 1, 8, 1, 1, 3.666f, 0.065f, 0.796f, 0.054f},
    {1, 1, 8, 1, 2, 3.943f, 0.098f, 1.084f, 0.078f},
    {1, 2, 4, 1, 1, 3.480f, 0.117f, 0.496f, 0.078f},
    {1, 2, 4, 1, 2, 3.663f, 0.178f, 0.863f, 0.134f},
    {1, 4, 2, 1, 1, 3.251f, 0.220f, 0.586f, 0.128f},
    {1, 4, 2, 1, 2, 3.515f, 0.351f, 0.868f, 0.251f},
    {1, 2, 4, 2, 1, 3.653f, 0.152f, 0.863f, 0.121f},
    {1, 2, 4, 2, 2, 4.383f, 0.230f, 1.336f, 0.167f},
    {1, 4, 2, 2, 1, 3.635f, 0.278f, 0.835f, 0.177f},
    {1, 4, 2, 2, 2, 4.241f, 0.408f, 1.407f, 0.289f},
    {1, 4, 2, 3, 1, 3.713f, 0.307f, 1.285f, 0.221f},
    {1, 4, 2, 3, 2, 4.882f, 0.411f, 1.769f, 0.329f},
    {1, 2, 4, 4, 2, 4.932f, 0.318f, 3.849f, 0.324f},
    {1, 4, 2, 4, 1, 4.318f, 0.355f, 1.377f, 0.319f},
    {1, 4, 2, 4, 2, 5.310f, 0.492f, 3.705f, 0.504f},
    {1, 8, 1, 4, 1, 3.718f, 0.662f, 1.038f, 0.468f},
    {1, 8, 1, 4, 2, 6.932f, 0.982f, 5.225f, 0.844f},
    {1, 8, 1, 8, 2, 9.837f, 1.296f, 7.270f, 1.385f},
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
    const int cols = a.part_val ? a.parts : 0x7FFFFFFF;
    const int c = kind < 2   ? pick_shape<kCosts8, 8>(a.m, a.n, a.k, dev.cus, cols, &w)
                  : kind < 4 ? pick_shape<kCosts6, 6>(a.m, a.n, a.k, dev.cus, cols, &w)
                             : pick_shape<kCosts2, 2>(a.m, a.n, a.k, dev.cus, cols, &w);
    if (c < 0)
        return hipErrorInvalidValue;
    if (parts_used)
        *parts_used = w.tiles_n;
    const Launch* const launch[] = {kLaunchE4m3.data(), kLaunchE5m2.data(), kLaunchE2m3.data(), kLaunchE3m2.data(), kLaunchT2.data()};
    return launch[kind][c](w, dev, stream);
}

}  // namespace mxfp4

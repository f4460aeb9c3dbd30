// One and two activation rows on MXFP4 weights with K <= 2048 (arXiv 2503.13565, section 3.4.3, Eq. 2): what is left of the
// decode step where the weight rows are shorter than a step of the decode kernel in gemv_reg.hip.
//
// That kernel gives a wave pairs of steps of 2048 elements of one weight row and deals rows to resident waves: at K = 512
// three quarters of a step's lanes and every second step are empty, and 28000 rows took 8.9 us whatever K was (7 trips per
// wave, each a round trip to memory and a row's way through the lanes).  Here a wave takes P to 4 P rows at once, P = 4, 2 or
// 1 of them side by side in its lanes (K <= 512, 1024, 2048), and there are as many waves as that needs: every wave of a product is
// one round trip.  Its activations (at most 4 KB a row) come straight from memory, without LDS and without a barrier.
//   - One load brings the scale bytes of all rows (lane l: dword l % (16 / P) of row l / (16 / P)); a row's dword
//     reaches its lanes with one ds_bpermute, as in gemv_reg.hip.
//   - A row's sum takes the same operations in the same order as there (blocks of the missing lanes and steps are zeros, which a sum
//     that starts from +0 does not feel), so the results have the same bits.
// Bound by the launch, one round trip and, from some MB on, the stream.  Measured, us per launch with three sets of weights in rotation,
// gemv_reg.hip -> here: one row 4096 x 512 3.50 -> 2.12, 4096 x 2048 3.54 -> 2.89, 28000 x 512 8.7 -> 3.3, 28000 x 1024
// 8.9 -> 4.5, 28000 x 2048 9.2 -> 6.9 (30 MB: 4.4 TB/s), 57344 x 2048 15.7 -> 11.0 (5.7 TB/s); 8192 x 512 with residual 5.05 -> 2.9; two
// rows with the pick and its second launch 16000 x 1024 12.2 -> 8.4.
#include "common.h"
#include "kernels.h"
#include "../../include/mxfp4.h"

namespace mxfp4 {

namespace {

constexpr int kWaves = 4;               // per workgroup
constexpr int kNowhere = 0x7FFFFFF0;    // lane offset past any descriptor: the load returns zero

struct ShortArgs {
    const uint16_t* x;
    const uint8_t* q;
    const uint8_t* s;
    void* out;              // y (BF16 [MT, N]), or for the pick the partial winners: float [MT, parts], int32 [MT, parts]
    int n, k, ldx, ldy;
    int parts;              // > 0: the pick
    int blocks;
};

// MT activation rows, P weight rows side by side in a wave's lanes, R times P of them at once.
template <int MT, int P, int R, class Epi>
__device__ __forceinline__ void gemv_short_body(const ShortArgs& a, const Epi& epi)
{
    constexpr bool kEpi = !__is_same(Epi, NoEpilogue);
    constexpr int kLanes = 64 / P, kRows = R * P, kDwords = 16 / P;
    static_assert(R == 1 || R == 2 || R == 4, "the scale dwords of all rows in one load");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = a.n, nblk = a.k >> 5, row_bytes = nblk * kBlockBytes;
    const int blk = lane % kLanes, p = lane / kLanes;           // this lane's block, and which of the rows side by side
    const bool in_k = blk < nblk;

    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.q), 0, n * row_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.s), 0, n * nblk, 0x00020000);
    u32x4_t xv[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const __amdgpu_buffer_rsrc_t rx =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(a.x + (int64_t)m * a.ldx), 0, a.k * 2, 0x00020000);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            xv[m][j] = __builtin_amdgcn_raw_buffer_load_b128(rx, in_k ? blk * 64 : kNowhere, j * 16, 0);
    }

    bool gated = false;
    if constexpr (kEpi)
        gated = epi.act == MXFP4_ACT_SWIGLU;
    const int sum_at = (lane % P * kLanes + lane / P % R) * 4;  // lane o < kRows gets the sums of the group's row o from there
    float best_val[MT];
    int best_idx[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        best_val[m] = -INFINITY;
        best_idx[m] = 0x7FFFFFFF;
    }

    const int groups = (n + kRows - 1) / kRows;
    for (int g = blockIdx.x * kWaves + wave; g < groups; g += a.blocks * kWaves) {
        const int row0 = g * kRows;
        u32x4_t w[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int first = row0 + r * P;
            const bool live = in_k && first + p < n;
            w[r] = __builtin_amdgcn_raw_buffer_load_b128(rq, live ? p * row_bytes + blk * kBlockBytes : kNowhere,
                                                         first < n ? first * row_bytes : 0, 2);
        }
        const int s_row = lane / kDwords, s_at = lane % kDwords * 4;
        const uint32_t sw = __builtin_amdgcn_raw_buffer_load_b32(
            rs, s_at < nblk && s_row < kRows && row0 + s_row < n ? s_row * nblk + s_at : kNowhere, row0 * nblk, 0);
        const int row = row0 + lane;
        const bool own = lane < kRows && row < n;
        float bias = 0.f, residual[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m)
            residual[m] = 0.f;
        if constexpr (kEpi) {
            if (epi.bias && own)
                bias = bf16_bits_to_f32(epi.bias[row]);
            if (epi.residual && own)
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    residual[m] = bf16_bits_to_f32(epi.residual[(int64_t)m * epi.ldr + (gated ? row >> 1 : row)]);
        }
        float sum[MT][R];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < R; ++r)
                sum[m][r] = 0.f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // (the convert reads the exponent field of its scale operand only)
            const uint32_t dw = (uint32_t)__builtin_amdgcn_ds_bpermute(((r * P + p) * kDwords + (blk >> 2)) * 4, (int)sw);
            const float sc = in_k ? __uint_as_float((dw << ((3 - (blk & 3)) * 8)) >> 1) : 1.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t qd = w[r][j];
                const bf16x2_t w0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, sc, 0);
                const bf16x2_t w1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, sc, 1);
                const bf16x2_t w2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, sc, 2);
                const bf16x2_t w3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, sc, 3);
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    const uint32_t x0 = xv[m][j][0], x1 = xv[m][j][1], x2 = xv[m][j][2], x3 = xv[m][j][3];
                    float c = sum[m][r];
                    c = __builtin_amdgcn_fdot2_f32_bf16(w0, __builtin_bit_cast(bf16x2_t, x0), c, false);
                    c = __builtin_amdgcn_fdot2_f32_bf16(w1, __builtin_bit_cast(bf16x2_t, x1), c, false);
                    c = __builtin_amdgcn_fdot2_f32_bf16(w2, __builtin_bit_cast(bf16x2_t, x2), c, false);
                    c = __builtin_amdgcn_fdot2_f32_bf16(w3, __builtin_bit_cast(bf16x2_t, x3), c, false);
                    sum[m][r] = c;
                }
            }
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            // wave_sum's order, as far as the lanes of a row go
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float v = sum[m][r];
                v += dpp_f32<0xB1>(v);
                v += dpp_f32<0x4E>(v);
                v += dpp_f32<0x141>(v);
                v += dpp_f32<0x140>(v);
                if (P <= 2)
                    v += __shfl_xor(v, 16);
                if (P == 1)
                    v += __shfl_xor(v, 32);
                sum[m][r] = v;
            }
            float v = sum[m][0];                                // lane i of a row's lanes has row i's
#pragma unroll
            for (int r = 1; r < R; ++r) {
                float other = sum[m][r];
                asm("" : "+v"(other));                          // (a select of array elements becomes indexed memory)
                v = lane % R == r ? other : v;
            }
            v = __int_as_float(__builtin_amdgcn_ds_bpermute(sum_at, __float_as_int(v)));
            if constexpr (!kEpi) {
                if (a.parts > 0) {
                    if (own && v > best_val[m]) {               // (a lane's rows ascend)
                        best_val[m] = v;
                        best_idx[m] = row;
                    }
                } else if (own) {
                    static_cast<uint16_t*>(a.out)[(int64_t)m * a.ldy + row] = f32_to_bf16_rne(v);
                }
            } else {
                v += bias;
                const float up = __shfl_down(v, 1);             // rows (2 i, 2 i + 1) are (gate, up) pairs
                if (gated)
                    v = silu_gate(v, up);
                if (own && !(gated && (lane & 1)))
                    static_cast<uint16_t*>(a.out)[(int64_t)m * a.ldy + (gated ? row >> 1 : row)] = f32_to_bf16_rne(v + residual[m]);
            }
        }
    }
    if constexpr (!kEpi) {
        if (a.parts > 0) {
            __shared__ float wv[MT][kWaves];
            __shared__ int wi[MT][kWaves];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
#pragma unroll
                for (int off = 1; off < kRows; off <<= 1) {
                    const float v = __shfl_xor(best_val[m], off);
                    const int i = __shfl_xor(best_idx[m], off);
                    if (v > best_val[m] || (v == best_val[m] && i < best_idx[m])) {
                        best_val[m] = v;
                        best_idx[m] = i;
                    }
                }
                if (lane == 0) {
                    wv[m][wave] = best_val[m];
                    wi[m][wave] = best_idx[m];
                }
            }
            __syncthreads();
            if (tid < MT) {
                float bv = wv[tid][0];
                int bi = wi[tid][0];
                for (int w = 1; w < kWaves; ++w)
                    if (wv[tid][w] > bv || (wv[tid][w] == bv && wi[tid][w] < bi)) {
                        bv = wv[tid][w];
                        bi = wi[tid][w];
                    }
                float* part_val = static_cast<float*>(a.out);
                part_val[tid * a.parts + blockIdx.x] = bv;
                reinterpret_cast<int32_t*>(part_val + MT * a.parts)[tid * a.parts + blockIdx.x] = bi;
            }
        }
    }
}

// (plain scalars, so that they arrive in registers when a wave starts; the operands behind the product do not)
template <int MT, int P, int R>
__global__ __launch_bounds__(kWaves * 64) void gemv_short_kernel(const uint16_t* x, const uint8_t* q, const uint8_t* s, void* out, int n,
                                                                 int k, int ldx, int ldy, int parts, int blocks)
{
    gemv_short_body<MT, P, R>(ShortArgs{x, q, s, out, n, k, ldx, ldy, parts, blocks}, NoEpilogue{});
}
template <int MT, int P, int R>
__global__ __launch_bounds__(kWaves * 64) void gemv_short_fused_kernel(const uint16_t* x, const uint8_t* q, const uint8_t* s, void* out,
                                                                       int n, int k, int ldx, int ldy, int blocks, Epilogue epi)
{
    gemv_short_body<MT, P, R>(ShortArgs{x, q, s, out, n, k, ldx, ldy, 0, blocks}, epi);
}

template <int MT, int P, int R>
hipError_t launch_one(const GemmArgs& a, const DeviceInfo& dev, int* parts_used, hipStream_t stream, const Epilogue* epi)
{
    const int groups = (a.n + R * P - 1) / (R * P), all = (groups + kWaves - 1) / kWaves;
    const int blocks = a.part_val ? min(all, min(a.parts, dev.cus * 8)) : all;
    if (parts_used)
        *parts_used = blocks;
    if (epi)
        hipLaunchKernelGGL((gemv_short_fused_kernel<MT, P, R>), dim3(blocks), dim3(kWaves * 64), 0, stream, a.x, a.q, a.s, a.y, a.n,
                           a.k, (int)a.ldx, (int)a.ldy, blocks, *epi);
    else
        hipLaunchKernelGGL((gemv_short_kernel<MT, P, R>), dim3(blocks), dim3(kWaves * 64), 0, stream, a.x, a.q, a.s,
                           a.part_val ? static_cast<void*>(a.part_val) : static_cast<void*>(a.y), a.n, a.k, (int)a.ldx, (int)a.ldy,
                           a.part_val ? a.parts : 0, blocks);
    return hipGetLastError();
}

template <int MT, int P>
hipError_t launch_p(const GemmArgs& a, int r, const DeviceInfo& dev, int* parts_used, hipStream_t stream, const Epilogue* epi)
{
    return r == 1   ? launch_one<MT, P, 1>(a, dev, parts_used, stream, epi)
           : r == 2 ? launch_one<MT, P, 2>(a, dev, parts_used, stream, epi)
                    : launch_one<MT, P, 4>(a, dev, parts_used, stream, epi);
}

// How many times P rows a wave takes: one while that is few waves, then two, then four.  One row, us with one, two, four: 4096 x 512
// 2.12, 2.23, 2.51, 28000 x 512 3.71, 3.29, 3.48, 8192 x 2048 4.15, 3.63, 3.94, 28000 x 2048 9.37, 7.09, 6.98; two rows: 2048 x 512
// 2.30, 2.32, 2.60, 8192 x 512 2.77, 2.59, 2.85, 8192 x 2048 5.94, 4.26, 4.20, 28000 x 1024 with the pick 12.9, 12.8, 10.6.
template <int MT>
hipError_t launch_rows(const GemmArgs& a, const DeviceInfo& dev, int* parts_used, hipStream_t stream, const Epilogue* epi)
{
    const int p = a.k <= 512 ? 4 : a.k <= 1024 ? 2 : 1, waves = a.n / p, unit = dev.cus;
    const bool gated = epi && epi->act == MXFP4_ACT_SWIGLU;      // a wave has whole pairs of rows
    const int r = waves <= (MT == 1 ? 10 : 5) * unit && !(gated && p == 1) ? 1 : waves <= (MT == 1 ? 56 : 24) * unit ? 2 : 4;
    return p == 4   ? launch_p<MT, 4>(a, r, dev, parts_used, stream, epi)
           : p == 2 ? launch_p<MT, 2>(a, r, dev, parts_used, stream, epi)
                    : launch_p<MT, 1>(a, r, dev, parts_used, stream, epi);
}

}  // namespace

// K <= 2048: every wave has one step of a row.  With two and three steps (K to 6144) the same kernel was 0.93 to 1.2 of
// gemv_reg.hip's, by the box (8192 x 3072 4.5 to 4.8 us, 4.6 there).
bool gemv_short_can_run(const GemmArgs& a, const DeviceInfo& dev) { return a.m <= 2 && a.k <= 2048 && gemv_reg_can_run(a, dev); }

hipError_t launch_gemv_short(const GemmArgs& a, const DeviceInfo& dev, int* parts_used, hipStream_t stream, const Epilogue* epi)
{
    if (!gemv_short_can_run(a, dev))
        return hipErrorInvalidValue;
    return a.m == 2 ? launch_rows<2>(a, dev, parts_used, stream, epi) : launch_rows<1>(a, dev, parts_used, stream, epi);
}

}  // namespace mxfp4

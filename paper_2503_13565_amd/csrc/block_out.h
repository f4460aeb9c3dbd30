// What the block kernel (gemm_wide.h) does with a finished 16 x 16 fragment of sums: BF16 store,
// bias / gate / residual behind the product, or the row's best value for the fused pick.
#pragma once

#include "common.h"
#include "kernels.h"
#include "../../include/mxfp4.h"

namespace mxfp4 {

struct BlockOut {
    uint16_t* y;
    int64_t ldy;
    float* part_val;                    // pick: [M, parts], one partial winner per row and block column
    int32_t* part_idx;
    const uint16_t* bias;
    const uint16_t* residual;
    int n, m, parts, ldr, act;
};

inline BlockOut block_out(const GemmArgs& a, const Epilogue* epi)
{
    return {a.y,      a.ldy, a.part_val, a.part_idx, epi ? epi->bias : nullptr, epi ? epi->residual : nullptr, a.n, a.m,
            a.parts, epi ? epi->ldr : 0, epi ? epi->act : MXFP4_ACT_NONE};
}

// Lane (li, lg) holds the sums of weight rows col .. col + 3 for activation row `row`.  Pick: the best of
// the fragment's 16 weight rows goes to *slot (one per activation row, written by lanes 0 .. 15).
__device__ __forceinline__ void emit_fragment(const BlockOut& a, const f32x4_t sum, int row, int col, float2* slot)
{
    const int n = a.n, m = a.m;
    if (a.part_val != nullptr) {
        float best = -INFINITY;
        int idx = 0x7FFFFFFF;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (col + r < n && sum[r] > best) {                     // rows ascend: lowest index wins ties
                best = sum[r];
                idx = col + r;
            }
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {
            const float v = __shfl_xor(best, off);
            const int o = __shfl_xor(idx, off);
            if (v > best || (v == best && o < idx)) {
                best = v;
                idx = o;
            }
        }
        if ((threadIdx.x & 63) < 16)
            *slot = make_float2(best, __int_as_float(idx));
        return;
    }
    if (row >= m || col >= n)
        return;
    float z[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        z[r] = sum[r] + (a.bias && col + r < n ? bf16_bits_to_f32(a.bias[col + r]) : 0.f);
    uint16_t* y = a.y + (int64_t)row * a.ldy;
    const uint16_t* res = a.residual ? a.residual + (int64_t)row * a.ldr : nullptr;
    const bool gated = a.act == MXFP4_ACT_SWIGLU;
    if (gated) {                                                    // rows (0, 1) and (2, 3) are (gate, up) pairs
#pragma unroll
        for (int c = 0; c < 2; ++c)
            if (col + 2 * c < n)
                y[(col >> 1) + c] = f32_to_bf16_rne(silu_gate(z[2 * c], z[2 * c + 1]) +
                                                    (res ? bf16_bits_to_f32(res[(col >> 1) + c]) : 0.f));
        return;
    }
    uint16_t o[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
        o[r] = f32_to_bf16_rne(z[r] + (res && col + r < n ? bf16_bits_to_f32(res[col + r]) : 0.f));
    if ((a.ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(a.y) & 7) == 0 && col + 4 <= n) {
        *reinterpret_cast<uint2*>(y + col) = make_uint2(o[0] | (uint32_t)o[1] << 16, o[2] | (uint32_t)o[3] << 16);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (col + r < n)
                y[col + r] = o[r];
    }
}

// Pick: the block's winner of one activation row out of its `count` fragments (columns ascend).
__device__ __forceinline__ void publish_winner(const BlockOut& a, const float2* slots, int count, int row, int part)
{
    float best = -INFINITY;
    int idx = 0x7FFFFFFF;
    for (int e = 0; e < count; ++e) {
        const float2 c = slots[e];
        if (c.x > best) {
            best = c.x;
            idx = __float_as_int(c.y);
        }
    }
    a.part_val[(int64_t)row * a.parts + part] = best;
    a.part_idx[(int64_t)row * a.parts + part] = idx;
}

// Workgroups go to the eight dies round robin: a die takes a run of neighbouring blocks, the blocks of one
// weight strip next to each other, so that the strip comes from the die's L2 after the first.
__device__ __forceinline__ int block_on_die(int total, int block)
{
    const int die = block & 7, per = total >> 3, more = total & 7;
    return die * per + (die < more ? die : more) + (block >> 3);
}

}  // namespace mxfp4

// What the block kernel (gemm_wide.h) does with the finished sums of a block: BF16 store, bias / gate / residual behind
// the product, or the row's best value for the fused pick.
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

// `N` neighbouring 16-bit values at any even address (global accesses need no more than the element's alignment).
template <int N>
struct Packed {
    typedef __attribute__((ext_vector_type(N / 2))) unsigned int type;
    typedef type anywhere __attribute__((aligned(2)));
};
template <int N>
__device__ __forceinline__ void load_bf16(const uint16_t* from, int count, float* to)
{
    if (count >= N) {
        const typename Packed<N>::type v = *reinterpret_cast<const typename Packed<N>::anywhere*>(from);
#pragma unroll
        for (int i = 0; i < N; ++i)
            to[i] = bf16_bits_to_f32(v[i >> 1] >> (16 * (i & 1)) & 0xFFFFu);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i)
            to[i] = i < count ? bf16_bits_to_f32(from[i]) : 0.f;
    }
}
template <int N>
__device__ __forceinline__ void store_bf16(uint16_t* to, int count, const float* v)
{
    if (count >= N) {
        typename Packed<N>::type o;
#pragma unroll
        for (int i = 0; i < N; i += 2)
            o[i >> 1] = f32_to_bf16_rne(v[i]) | (uint32_t)f32_to_bf16_rne(v[i + 1]) << 16;
        *reinterpret_cast<typename Packed<N>::anywhere*>(to) = o;
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (i < count)
                to[i] = f32_to_bf16_rne(v[i]);
    }
}

// `N` neighbouring sums of activation row `row`, from weight row `col` on (a multiple of N): bias, gate, residual, store.
template <int N>
__device__ __forceinline__ void emit_sums(const BlockOut& a, const float (&sums)[N], int row, int col)
{
    if (row >= a.m || col >= a.n)
        return;
    float z[N], add[N] = {};
#pragma unroll
    for (int i = 0; i < N; ++i)
        z[i] = sums[i];
    if (a.bias) {
        float b[N];
        load_bf16<N>(a.bias + col, a.n - col, b);
#pragma unroll
        for (int i = 0; i < N; ++i)
            z[i] += b[i];
    }
    uint16_t* y = a.y + (int64_t)row * a.ldy;
    const uint16_t* res = a.residual ? a.residual + (int64_t)row * a.ldr : nullptr;
    if (a.act == MXFP4_ACT_SWIGLU) {                                    // rows (2 i, 2 i + 1) are (gate, up) pairs
        const int left = (a.n - col + 1) >> 1;
        if (res)
            load_bf16<N / 2>(res + (col >> 1), left, add);
#pragma unroll
        for (int i = 0; i < N / 2; ++i)
            z[i] = silu_gate(z[2 * i], z[2 * i + 1]) + add[i];
        store_bf16<N / 2>(y + (col >> 1), left, z);
    } else {
        if (res)
            load_bf16<N>(res + col, a.n - col, add);
#pragma unroll
        for (int i = 0; i < N; ++i)
            z[i] += add[i];
        store_bf16<N>(y + col, a.n - col, z);
    }
}

// Rows of finished sums in the LDS, kStride floats from row to row; row r is activation row row_of(r), its first sum weight
// row n0.
template <int kRows, int kCols, int kStride, class RowOf>
__device__ __forceinline__ void emit_rows(const BlockOut& a, const float* tile, int n0, RowOf row_of)
{
    constexpr int kChunks = kCols / 8;
#pragma unroll 1
    for (int e = threadIdx.x; e < kRows * kChunks; e += 512) {
        const f32x4_t* at = reinterpret_cast<const f32x4_t*>(tile + e / kChunks * kStride + e % kChunks * 8);
        const f32x4_t low = at[0], high = at[1];
        const float sums[8] = {low[0], low[1], low[2], low[3], high[0], high[1], high[2], high[3]};
        emit_sums(a, sums, row_of(e / kChunks), n0 + e % kChunks * 8);
    }
}

// Pick: the best of every such row, by sixteen threads, to column `part` of the partial winners.
template <int kRows, int kCols, int kStride, class RowOf>
__device__ __forceinline__ void pick_rows(const BlockOut& a, const float* tile, int n0, int part, RowOf row_of)
{
    for (int r = threadIdx.x >> 4; r < kRows; r += 512 / 16) {
        float best = -INFINITY;
        int idx = 0x7FFFFFFF;
        for (int c = threadIdx.x & 15; c < kCols; c += 16) {            // columns ascend: lowest index wins ties
            const float v = tile[r * kStride + c];
            if (n0 + c < a.n && v > best) {
                best = v;
                idx = n0 + c;
            }
        }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const float v = __shfl_xor(best, off);
            const int o = __shfl_xor(idx, off);
            if (v > best || (v == best && o < idx)) {
                best = v;
                idx = o;
            }
        }
        const int row = row_of(r);
        if ((threadIdx.x & 15) == 0 && row < a.m) {
            a.part_val[(int64_t)row * a.parts + part] = best;
            a.part_idx[(int64_t)row * a.parts + part] = idx;
        }
    }
}

// Workgroups go to the eight dies round robin: a die takes a run of neighbouring blocks, the blocks of one
// weight strip next to each other, so that the strip comes from the die's L2 after the first.
__device__ __forceinline__ int block_on_die(int total, int block)
{
    const int die = block & 7, per = total >> 3, more = total & 7;
    return die * per + (die < more ? die : more) + (block >> 3);
}

}  // namespace mxfp4

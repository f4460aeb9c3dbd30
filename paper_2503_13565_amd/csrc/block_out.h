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
            o[i >> 1] = f32_to_bf16_rne2(v[i], v[i + 1]);
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

// Four neighbouring values of the bias, from weight row `col` on (rows past the last one: the last one's again, not stored).
__device__ __forceinline__ f32x4_t bias_of(const BlockOut& a, int col)
{
    f32x4_t b;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        b[i] = bf16_bits_to_f32(a.bias[min(col + i, a.n - 1)]);
    return b;
}

// Whether 16 bytes of `p`'s rows lie on 16-byte boundaries, from a multiple of eight columns on.
__device__ __forceinline__ bool rows_aligned(const uint16_t* p, int64_t ld)
{
    return ((reinterpret_cast<uintptr_t>(p) >> 1 | (uint64_t)ld) & 7) == 0;
}

// kN floats of a row in the LDS from column `at` on.  Where that is no multiple of four, or not inside the row's kCols columns (what
// lies outside is not used): whole 16-byte reads, shifted into place.
template <int kN, int kCols>
__device__ __forceinline__ void row_floats(const float* row, int at, bool aligned, float* to)
{
    f32x4_t v[kN / 4 + 1];
    if (aligned) {
#pragma unroll
        for (int i = 0; i < kN / 4; ++i)
            v[i] = *reinterpret_cast<const f32x4_t*>(row + at + 4 * i);
    } else {
#pragma unroll
        for (int i = 0; i <= kN / 4; ++i)
            v[i] = *reinterpret_cast<const f32x4_t*>(row + min(max((at & ~3) + 4 * i, 0), kCols - 4));
#pragma unroll
        for (int i = 0; i < kN / 4; ++i) {                              // (shuffles: selects of elements became indexed memory)
            const f32x4_t next = v[i + 1];
            const f32x4_t one = __builtin_shufflevector(v[i], next, 1, 2, 3, 4), two = __builtin_shufflevector(v[i], next, 2, 3, 4, 5),
                          three = __builtin_shufflevector(v[i], next, 3, 4, 5, 6);
            const f32x4_t even = at & 2 ? two : v[i], odd = at & 2 ? three : one;
            v[i] = at & 1 ? odd : even;
        }
    }
#pragma unroll
    for (int i = 0; i < kN; ++i)
        to[i] = v[i / 4][i % 4];
}

// Rows of finished sums (bias included) on their way out through the LDS, kStride floats from row to row; row r is activation
// row row_of(r), its first sum weight row n0.  `fill` puts them there.
//   - A thread takes eight neighbouring outputs that lie on a 16-byte boundary of the residual.  A load of 16 bytes on another
//     boundary takes the texture unit several times as long: with pieces that began at multiples of eight columns, 12967 x 512 with
//     residual at 327 rows took 22.1 us where 12960 took 15.2; now 15.5 and 12.9.  (Stores do not care: without a residual the pieces
//     begin at multiples of eight columns, 12967 x 512 14.0 us; 14.4 on y's boundaries, with the ends of its rows apart.)
//   - The residual of up to four pieces is asked for together, the first ones in front of `fill`.  A piece is read
//     whole, also where only a part of it belongs to the row: what is read beside it lies in the same 16 bytes.
template <int kRows, int kCols, int kStride, class RowOf, class Fill>
__device__ __forceinline__ void emit_rows(const BlockOut& a, const float* tile, int n0, RowOf row_of, Fill fill)
{
    constexpr int kBatch = 4;
    const bool gate = a.act == MXFP4_ACT_SWIGLU;                        // rows (2 i, 2 i + 1) are (gate, up) pairs
    const bool aligned = !a.residual || rows_aligned(a.residual, a.ldr);   // (n0 is a multiple of 16)
    const int col0 = gate ? n0 >> 1 : n0, width = gate ? kCols / 2 : kCols;
    const int left = min(width, (gate ? a.n >> 1 : a.n) - col0);        // outputs of the block in a row
    // Blocks of few outputs, one or two pieces a thread, stop at the last row in front of m and at the last piece (32 x 22224 x 256 with gate and
    // residual 4.74 -> 4.50 us, 262 x 7248 x 256 7.05 -> 6.75; in larger ones 1.01, for the branches).
    constexpr bool kFew = kRows * kCols <= 8192;
    static_assert(!kFew || kRows * (kCols / 8 + 1) <= kBatch * 512, "one batch");
    const int row0 = row_of(0), live = kFew && row_of(kRows - 1) - row0 == kRows - 1 ? min(kRows, a.m - row0) : kRows;
    const int units = (width >> 3) + (aligned ? 0 : 1), total = live * units;
    const uint32_t inverse = ((1u << 20) + units - 1) / units;          // exact up to 2^20 / (units - 1) pieces
    static_assert(kRows * (kCols / 8 + 1) * (kCols / 8) < 1 << 20, "piece / units by multiplication");
    // the piece `e` of the block: its row in the LDS, activation row, first output in the row's part of the block
    struct Piece {
        int r, row, c;
        bool some;
    };
    auto piece = [&](int e) {
        Piece p;
        p.r = (int)((uint32_t)e * inverse >> 20);
        p.row = row_of(p.r);
        p.c = (e - p.r * units) * 8;
        if (!aligned)
            p.c -= (int)((reinterpret_cast<uintptr_t>(a.residual + (int64_t)p.row * a.ldr + col0) >> 1) & 7);
        p.some = e < total && p.row < a.m && p.c < left && p.c > -8;
        return p;
    };
    u32x4_t res[kBatch];
    auto ask = [&](int e0) {
        const uintptr_t any = reinterpret_cast<uintptr_t>(a.residual) & ~(uintptr_t)15;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (kFew && j * 512 >= total)
                break;
            const Piece p = piece(e0 + j * 512);
            res[j] = *reinterpret_cast<const u32x4_t*>(
                p.some ? reinterpret_cast<uintptr_t>(a.residual + (int64_t)p.row * a.ldr + col0 + p.c) : any);
        }
    };
    if (a.residual)
        ask(threadIdx.x);
    fill();
#pragma unroll 1
    for (int e0 = threadIdx.x; e0 < total; e0 += kBatch * 512) {
        if (a.residual && e0 >= 512)
            ask(e0);
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (kFew && j * 512 >= total)
                break;
            const Piece p = piece(e0 + j * 512);
            if (!p.some)
                continue;
            const float* row = tile + p.r * kStride;
            float z[8];
            if (gate) {
                float v[16];
                row_floats<16, kCols>(row, 2 * p.c, aligned, v);
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    z[i] = silu_gate(v[2 * i], v[2 * i + 1]);
            } else {
                row_floats<8, kCols>(row, p.c, aligned, z);
            }
            if (a.residual) {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    z[i] += bf16_bits_to_f32(res[j][i >> 1] >> (16 * (i & 1)) & 0xFFFFu);
            }
            uint16_t* to = a.y + (int64_t)p.row * a.ldy + col0 + p.c;
            if (p.c >= 0 && p.c + 8 <= left) {
                store_bf16<8>(to, 8, z);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (p.c + i >= 0 && p.c + i < left)
                        to[i] = f32_to_bf16_rne(z[i]);
            }
        }
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
        best_of_16(&best, &idx);
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

// The product for more activation rows than one matrix-core tile column holds (a prompt, several
// sequences verified together), and from three rows on wherever it is faster than the kernels that hold their rows in the LDS (routes.h):
// nearly always for MXFP4 weights whose K is no multiple of 128 (arXiv 2503.13565, section 3.4.3, Eq. 2 for the arithmetic; every
// weight is read once per block of rows).
//
// The tile kernels keep all of K of at most 16 activation rows in the LDS, so more rows take more
// passes, and every pass streams and decodes the weights again.  Here a workgroup of eight waves
// computes a BM x BN block of the output and walks K once: the activation rows of one phase of K
// (WK steps of 128 elements) sit in one of two LDS buffers, shared by all waves; a wave loads the weights of
// its 16 NF rows straight into registers, in the layout of the tile kernels (lane i + 16 g: block 4 T + g of row
// i), decodes them once and uses them for MF fragments of 16 activation
// rows.  The eight waves are WM x WN x WK: WM and WN split the block, WK splits the steps of a phase (few
// rows: the block is small and K is what there is to share), and then the WK partial sums of a
// fragment meet in the LDS at the end and are added in wave order.
//   - A phase's activations (16-byte chunks, one row's chunks to neighbouring threads) and its weights
//     are requested up to two phases ahead into registers.  At the start of a phase the next one's activations
//     go to the LDS, beside this one's reads and matrix instructions, and the ones after it are asked for: one
//     barrier per phase, which waits for LDS traffic only (with the writes behind the matrix instructions, in front
//     of the barrier: 4096 x 4096 at 128 rows 13.5 us against 12.2, 12288 x 4096 24.0 against 22.5, at 509 rows
//     58.5 against 55.5).  A third LDS buffer, so that the reads of a phase start before its barrier, and a second set
//     of registers for the activations were 1 to 10 % slower: the blocks that fit beside each other are worth more.
//   - Operand reads run one matrix instruction ahead.  From four fragments of activations on the next read goes into the
//     register that its fragment's instructions have just used, and the converts are spread between them: 64 x 4096
//     weight rows at K = 4096 (four tiles of 64 rows) 16.6 -> 14.4 us, 192 rows wide 27.6 -> 26.8, prompts 1 %.
//   - LDS layout [step of the phase][row][16 chunks]: chunk c of row r at position (c ^ (c & 4) * 2) ^ (r % 16).  A store
//     of 16 bytes per lane is served eight lanes at a time, half a row; a read in turns of rows 0-3 and 12-15 of one lane
//     group and rows 4-11 of its neighbour (from the counted conflicts): this position sends either to different banks.
//     Without the middle term the reads met in pairs (18 % of a prompt's cycles), with 4 j + lg in its place the stores (748 x 6528
//     at 20 rows 7.15 us against 6.85).
//   - The finished sums leave through the LDS (block_out.h): whole rows of the block, 16 bytes per thread, in a short loop.
//     Stored from the accumulators, in 32-byte pieces by code unrolled over every fragment, they took 6 us of a
//     prompt: 22016 x 128 at 509 rows with the gate 20.2 -> 14.2 us, 22016 x 4096 79.2 -> 75.8, 14000 x 6016 at 399 rows
//     77.6 -> 73.4.  Where the waves share K, a thread adds the partial sums of its outputs and stores them.
//   - Blocks of few rows keep a phase short (four or two steps instead of eight), so that several of them fit the LDS of a unit and
//     one works while another waits: 32 weight rows x 1024 at 16 rows, 512 blocks, 6.4 -> 4.6 us, 96 weight rows 11.9 -> 7.7.  The
//     short phase costs more per step, so the long one stays for a long K.
//   - The scale bytes of two phases travel together, one dword per step and row, through the LDS: as byte
//     loads by the lanes that use them (which the kernel does where K % 128 != 0 leaves the dwords
//     unaligned) every byte pulled a cache line, 104 us instead of 130 on the example below.
//   - Prompts take blocks of 128 rows with all eight waves side by side along the weight rows, so that no
//     weight is decoded or fetched twice in a block: 92 us against 104 for 2 x 4 waves.
//   - A prompt is bound by the matrix pipe and what feeds it at the clock the power limit leaves: the pipe is busy in 62 % of
//     the cycles at 2.15 GHz, the LDS in 24 %.  (When it took 86 us: 69 with the loads and the LDS reads taken out, 80 with
//     all-zero operands.)  Some tens of rows are bound by the activations' way through the L2 and LDS (at 32 rows
//     the waves wait in 45 % of their cycles).  Measured, us from launch to launch, passes of 16 rows -> here:
//     22016 x 4096 with the gate at 509 rows 436 -> 72 to 75 by the box (a library product of BF16 weights of that
//     shape: 91), 12288 x 4096 at 32 rows 18.5 -> 10.1 with three sets of weights in rotation, 22016 x 4096 with the
//     gate at 5 rows 11.0, 32000 x 4096 with the pick at 9 rows 17.0 (two launches).
//   - A block past the end of K (K % 128 != 0, the steps that round a phase up) is a load past the
//     descriptor: zero weights against zero activations.
#pragma once

#include <array>
#include <iterator>
#include <utility>

#include "block_out.h"
#include "block_ways.h"
#include "common.h"
#include "kernels.h"
#include "scale_stage.h"
#include "sum_chains.h"

namespace mxfp4 {
namespace wide {

constexpr int kOob = 0x7FFFFFF0;        // lane offset beyond any descriptor: the load returns zero

typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;
typedef __attribute__((ext_vector_type(6))) unsigned int u32x6_t;
typedef __attribute__((ext_vector_type(16))) unsigned int u32x16_t;

struct Args {
    const uint16_t* x;
    const uint8_t* q;
    const uint8_t* s;
    int n, k, m, ldx, ldw, tiles_m, tiles_n;    // ldw: BF16 weights only
    int chains;                                 // into how many an output's sum is cut (sum_chains.h)
    BlockOut out;
};

// Finished sums on their way out: floats from row to row, and how many rows of the block take a turn together where the
// waves do not share K: all of them as far as the LDS goes, which a block of eight fragments and more has to itself (its registers leave
// no room for a second one on the unit).
constexpr int tile_stride(int bn) { return bn + 4; }
constexpr int tile_rows(int wm, int mf, int nf, int bn)
{
    int pf = mf;
    while (pf > 1 && wm * pf * 16 * tile_stride(bn) * 4 > (mf * nf >= 8 ? 160 : 40) * 1024)
        pf /= 2;
    return wm * pf * 16;
}

constexpr size_t lds_bytes(Kind w, int wm, int wn, int wk, int mf, int nf)
{
    const int bm = wm * mf * 16, bn = wn * nf * 16, x = 2 * wk * bm * 256;  // two buffers of one phase
    const size_t xs = (size_t)x + (w == kBf16 ? 0 : (size_t)2 * bn * scale_row_bytes(wk));      // and two of the scales
    const size_t red = wk > 1 ? (size_t)8 * mf * nf * 1024 : 0;         // the waves' partial sums, afterwards
    const size_t tile = (size_t)(wk > 1 ? bm : tile_rows(wm, mf, nf, bn)) * tile_stride(bn) * 4;
    return xs > red + tile ? xs : red + tile;
}

// Eight codes of the 2-bit format (16 bits of `c`) -> eight MXFP4 nibbles with the same values (+-1.0 or +-0).
__device__ __forceinline__ uint32_t t2_to_nibbles(uint32_t c)
{
    c = (c | c << 8) & 0x00FF00FFu;
    c = (c | c << 4) & 0x0F0F0F0Fu;
    c = (c | c << 2) & 0x33333333u;
    return (c & 0x22222222u) << 2 | (c & 0x11111111u) << 1;
}

// The eight BF16 weights of matrix instruction j out of the dwords of a lane's block.
template <Kind kW>
__device__ __forceinline__ u32x4_t operand(const uint32_t* r, const u32x16_t& six, float scl, int j)
{
    u32x4_t w;
    if constexpr (kW == kBf16) {
        w = u32x4_t{r[4 * j], r[4 * j + 1], r[4 * j + 2], r[4 * j + 3]};
    } else if constexpr (kind_bits(kW) == 6) {
        const uint32_t w0 = six[4 * j], w1 = six[4 * j + 1], w2 = six[4 * j + 2], w3 = six[4 * j + 3];
        w = u32x4_t{w0, w1, w2, w3};
    } else if constexpr (kW == kE4m3) {
        w[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r[2 * j], scl, false));
        w[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r[2 * j], scl, true));
        w[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r[2 * j + 1], scl, false));
        w[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(r[2 * j + 1], scl, true));
    } else if constexpr (kW == kE5m2) {
        w[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(r[2 * j], scl, false));
        w[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(r[2 * j], scl, true));
        w[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(r[2 * j + 1], scl, false));
        w[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8(r[2 * j + 1], scl, true));
    } else {
        const uint32_t qd = kW == kT2 ? t2_to_nibbles(r[j >> 1] >> (16 * (j & 1)) & 0xFFFFu) : r[j];
        w[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, scl, 0));
        w[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, scl, 1));
        w[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, scl, 2));
        w[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, scl, 3));
    }
    return w;
}

// How the sums of a wave are cut into chains (what for: sum_chains.h).
//   - kSets: the matrix instructions of a step take turns on two or four sums.  Takes registers only, for one row of fragments (and
//     two or three where four waves share K).
//   - kChains: a chain of whole pairs of phases is added to the output's sum at its end, K / chains long.  (One row of fragments
//     like that: 4096 x 1024 at 5 rows 3.8 us, 3.6 with sets.)
//   - kSteps: so is every step's, which is more exact than long chains for elements of 6 bits and more (a pick's BF16 values at
//     K = 4096, against 64 bits: 0.9e-7 to 1.2e-7, 1.5e-7 in eight chains, 4.2e-7 in one).  Blocks of many rows then go through
//     one row of fragments after the other, for which two rows' sums are enough.  The largest 8-bit block has the registers for
//     kChains and not the time for this (22016 x 4096 at 509 rows: 15 % of it).
// A step's four instructions on BF16 weights make a sum each at one row of fragments, added in pairs: as exact as the vector ALUs, which
// take the shorter of these calls' neighbours (0.98 of their error at K = 512, 0.79 at 4096; 1.13 and 0.88 in one chain), and no slower.
enum Cut { kWhole, kSets, kChains, kSteps };
constexpr Cut sum_cut(Kind w, int wk, int mf, int nf)
{
    return uncut(mf, nf) || (wk == 8 && mf > 1)                              ? kWhole
           : kind_bits(w) > 4 && !(kind_bits(w) == 8 && mf * nf == 16)       ? kSteps
           : sum_sets(wk, mf) > 1 && kind_bits(w) <= 4                       ? kSets
                                                                             : kChains;
}
constexpr bool each_apart(Kind w, int mf) { return w == kBf16 && mf == 1; }

// kDirect: the activations' way into the LDS (block_ways.h).
// The leading arguments are scalars that arrive in registers when a wave starts; `out` is for the end.
template <Kind kW, int WM, int WN, int WK, int MF, int NF, bool kDirect>
__global__ __launch_bounds__(kThreads, 2) void gemm_wide_kernel(const uint16_t* __restrict__ x,
                                                                const uint8_t* __restrict__ q,
                                                                const uint8_t* __restrict__ s, int n, int k, int m,
                                                                int ldx, int ldw, int tiles_m, int tiles_n, int chains,
                                                                BlockOut out)
{
    static_assert(WM * WN * WK == 8, "eight waves");
    constexpr int BM = WM * MF * 16, BN = WN * NF * 16;
    constexpr int CA = WK * BM * 16 / kThreads;                         // activation chunks per thread and phase
    static_assert(CA >= 1 && CA * kThreads == WK * BM * 16, "whole chunks");
    static_assert(lds_bytes(kW, WM, WN, WK, MF, NF) <= 160 * 1024, "the LDS of a compute unit");
    constexpr int kRowChunks = WK * 16;                                 // chunks of one row in a phase
    constexpr int kRowStep = kThreads / kRowChunks;                     // rows between a thread's chunks
    constexpr int kBuf = WK * BM * 16;                                  // chunks of one LDS buffer
    constexpr bool kScaled = kW != kBf16, kRagged = kW == kMxRagged, kTiled = kW == kMxTiled;
    constexpr int kBits = kind_bits(kW), kBlock = 4 * kBits;            // dwords and bytes of a block of 32
    constexpr int kSRow = scale_row_bytes(WK), kSBuf = BN * kSRow;
    constexpr int SC = kScaled && !kRagged ? scale_rounds(BN, WK) : 0;  // scale dwords per thread and two phases
    extern __shared__ __align__(16) uint8_t smem[];
    u32x4_t* xs = reinterpret_cast<u32x4_t*>(smem);
    uint8_t* ss = smem + (size_t)2 * kBuf * 16;

    const int tid = threadIdx.x;
    const int lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;
    const int nblk = k >> 5, steps = (k + 127) >> 7, phases = (steps + WK - 1) / WK;
    const int n_tiles = (n + 15) >> 4, n_items = (steps + 3) >> 2;      // of the tile-major copy

    const int at = block_on_die(tiles_m * tiles_n, blockIdx.x);
    const int tm = at % tiles_m, tn = at / tiles_m;
    const int m0 = tm * BM, n0 = tn * BN;

    const int row_bytes = kW == kBf16 ? ldw * 2 : nblk * kBlock;
    const uint16_t* x0 = x + (int64_t)m0 * ldx;
    const int x_bytes = ((min(BM, m - m0) - 1) * ldx + k) * 2;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(x0), 0, x_bytes, 0x00020000);
    auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };     // (for inline assembly)
    const uint64_t x_at = reinterpret_cast<uint64_t>(x0);
    const u32x4_t rx_words = {uniform((uint32_t)x_at), uniform((uint32_t)(x_at >> 32) & 0xFFFFu), uniform((uint32_t)x_bytes), 0x00020000u};
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(q), 0, kTiled ? n_tiles * 16 * row_bytes : kW == kBf16 ? ((n - 1) * ldw + k) * 2 : n * row_bytes,
        0x00020000);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(s), 0, !kScaled ? 0 : kTiled ? n_tiles * n_items * 256 : n * nblk, 0x00020000);

    // Through registers: this thread's chunk of a row and its first row.  Direct: load i of wave w is the (8 i + w)th KiB of a
    // phase's buffer, four rows of one step, and a lane asks for the chunk whose place there it fills.
    auto chunk_at = [](int c) { return c ^ (c & 4) << 1; };
    constexpr int kRowGroups = BM / 4;
    const int xc = kDirect ? chunk_at(li ^ ((wave & 3) * 4 + lg)) : tid % kRowChunks, x_row = tid / kRowChunks;
    int x_off[CA];
#pragma unroll
    for (int i = 0; i < CA; ++i) {
        const int row = kDirect ? (i * 8 + wave) % kRowGroups * 4 + lg : x_row + i * kRowStep;
        x_off[i] = (min(m0 + row, m - 1) - m0) * ldx * 2 + xc * 16;                     // ragged M: repeat the last row
    }
    const uint32_t lds_at = (uint32_t)reinterpret_cast<uint64_t>((__attribute__((address_space(3))) uint8_t*)smem) + wave * 1024;
    int q_off[NF], s_off[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {                                      // ragged N: repeat the last row (or tile)
        const int row0 = n0 + (wn * NF + f) * 16, row = min(row0 + li, n - 1);
        q_off[f] = kTiled ? min(row0 >> 4, n_tiles - 1) * steps * 1024 + lane * 16
                          : row * row_bytes + lg * (kW == kBf16 ? 16 : kBlock);
        s_off[f] = row * nblk + lg;
    }
    int sc_off[SC + 1];
#pragma unroll
    for (int i = 0; i < SC; ++i)
        sc_off[i] = scale_row_offset(kTiled, n0 + scale_row(WK, tid, i), n, nblk, n_tiles, n_items);

    struct Slot {
        uint32_t q[NF][kBits];
        uint32_t s[kRagged ? NF : 1];
    };
    Slot buf[2];
    u32x4_t xr[CA];
    uint32_t sc[SC + 1];
    // Always the same loads, and every condition on the position arithmetic (a branch around a load makes
    // the compiler wait for all of them): what lies past K gets an offset past the descriptor.  The
    // scalar offset stays inside the descriptor then too.
    auto past = [](int last, int at) { return ((last - at) >> 31) & kOob; };    // 0 where at <= last
    int ld_x = 0, ld_q = 0;                                             // phases to ask for next
    auto issue_scales = [&](int sp) {                                   // of the phases 2 sp and 2 sp + 1
#pragma unroll
        for (int i = 0; i < SC; ++i) {
            const int T = sp * (WK * 2) + scale_step(WK, tid, i);
            sc[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, (sc_off[i] + scale_step_offset(kTiled, T)) |
                                                                 past(steps - 1, T) |
                                                                 past(BN * WK * 2 - 1, scale_index(tid, i)), 0, 0);
        }
    };
    auto store_scales = [&](int b) {
#pragma unroll
        for (int i = 0; i < SC; ++i)
            if (scale_owned(BN, WK, tid, i))
                *reinterpret_cast<uint32_t*>(ss + b * kSBuf + scale_lds(WK, tid, i)) = sc[i];
    };
    auto issue_x = [&]() {
        const int x_past = past((k >> 3) - 1, ld_x * kRowChunks + xc);
        const int x_at = ld_x < phases ? ld_x * (kRowChunks * 16) : 0;
#pragma unroll
        for (int i = 0; i < CA; ++i)
            xr[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, x_off[i] | x_past, x_at, 0);
        ++ld_x;
    };
    auto issue_direct = [&](int u, int b) {
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const int T = u * WK + (i * 8 + wave) / kRowGroups;
            const int off = x_off[i] | (kRagged ? past((k >> 3) - 1, T * 16 + xc) : T < steps ? 0 : kOob);
            // m0: where in the LDS lane 0's bytes go.  The load reads scalar registers that a vector instruction may have written just in
            // front (a read lane, a restored spill): five wait states, which the compiler does not count into assembly.
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(
                             lds_at + (b * kBuf * 16 + i * 8192)),
                         "v"(off), "s"(rx_words), "s"(T < steps ? T * 256 : 0)
                         : "memory", "m0");
        }
    };
    auto issue_q = [&](Slot& sl) {
        const int step = ld_q * WK + wk, T = step < steps ? step : 0;
        const int q_past = past(nblk - 1, 4 * step + lg);
        if constexpr (kRagged) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
                sl.s[f] = __builtin_amdgcn_raw_buffer_load_b8(rs, s_off[f] | q_past, T * 4, 0);
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            auto take = [&](int i, u32x4_t v) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    sl.q[f][4 * i + e] = v[e];
            };
            auto take2 = [&](int i, u32x2_t v) {
                sl.q[f][i] = v[0];
                sl.q[f][i + 1] = v[1];
            };
            if constexpr (kW == kBf16) {                                // 64 bytes of a row per instruction
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    take(j, __builtin_amdgcn_raw_buffer_load_b128(
                                rq, (q_off[f] + j * 64) | past((k >> 3) - 1, step * 16 + 4 * j + lg), T * 256, 0));
            } else {
                const int off = q_off[f] | q_past, row_at = T * (kTiled ? 1024 : 4 * kBlock);
                if constexpr (kBits == 2)
                    take2(0, __builtin_amdgcn_raw_buffer_load_b64(rq, off, row_at, 0));
                else
                    take(0, __builtin_amdgcn_raw_buffer_load_b128(rq, off, row_at, kTiled ? 2 : 0));
                if constexpr (kBits == 8)
                    take(1, __builtin_amdgcn_raw_buffer_load_b128(rq, (q_off[f] + 16) | q_past, row_at, 0));
                if constexpr (kBits == 6)
                    take2(4, __builtin_amdgcn_raw_buffer_load_b64(rq, (q_off[f] + 16) | q_past, row_at, 0));
            }
        }
        ++ld_q;
    };
    auto x_store = [&](int b) {
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const int r = x_row + i * kRowStep;
            xs[b * kBuf + ((xc >> 4) * BM + r) * 16 + (chunk_at(xc & 15) ^ (r & 15))] = xr[i];
        }
    };
    // The loads of one phase's weights: direct, the only ones that stay in flight across a barrier.  The counted waits below rely on
    // issue_q being this many vector memory instructions at the least, none dropped, merged or moved in front of the direct loads (the
    // scheduling barriers): with fewer behind those, a wait for the weights would not cover them.  True of every instance as compiled.
    constexpr int kQueued = NF * (kRagged ? 2 : kW == kBf16 ? 4 : kBits == 8 || kBits == 6 ? 2 : 1);
    issue_scales(0);
    if constexpr (kDirect)
        issue_direct(0, 0);
    else
        issue_x();
    __builtin_amdgcn_sched_barrier(0);                                  // keep the loads in this order
    issue_q(buf[0]);
    __builtin_amdgcn_sched_barrier(0);
    store_scales(0);
    if constexpr (!kDirect) {
        x_store(0);
        issue_x();
    }
    __builtin_amdgcn_sched_barrier(0);
    issue_q(buf[1]);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kDirect)                                              // at most the weights of both phases are younger
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kQueued) : "memory");
    lds_barrier();

    constexpr Cut kCut = sum_cut(kW, WK, MF, NF);
    constexpr bool kRoll = MF >= 4;                                     // (below)
    constexpr bool kEach = each_apart(kW, MF), kStepSums = kCut == kSteps && !kRoll;
    constexpr int kCopies = kCut == kSets ? sum_sets(WK, MF) : kCut == kChains ? 2 : kStepSums ? (kEach ? 5 : 2) : 1;
    f32x4_t sums_of[kCopies][MF][NF];                                   // [0]: the outputs' sums; kSteps, kChains: what is added to them
    auto& acc = sums_of[0];
#pragma unroll
    for (int c = 0; c < kCopies; ++c)
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f)
                sums_of[c][i][f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int chain_all = chain_pairs(phases, WK, chains);
    int chain_left = chain_all;
    auto end_chain = [&]() {
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                if constexpr (kEach)
                    acc[i][f] += (sums_of[1][i][f] + sums_of[2][i][f]) + (sums_of[3][i][f] + sums_of[4][i][f]);
                else
                    acc[i][f] += sums_of[1][i][f];
                if constexpr (kCut == kChains)
                    sums_of[1][i][f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                else                                                    // (a step starts from zero; the sum stays here)
                    asm volatile("" : "+v"(acc[i][f]));
            }
    };
    const int x_read = (wk * BM + wm * MF * 16 + li) * 16;
    const int s_read = (wn * NF * 16 + li) * kSRow + wk * 4 + lg;
    // The operand reads of matrix instructions j + 1 go out beside those of j: into a second set of registers, or, from
    // four fragments of activations on, each into the register that its fragment's instructions have just read.
    u32x4_t xf[kRoll ? 1 : 2][MF];

    for (int u0 = 0; u0 < phases; u0 += 2) {
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const Slot& sl = buf[d];
            // the next phase's activations go to the buffer that the phase before this one read, beside this
            // phase's reads and matrix instructions; the ones after them are asked for (or the next phase's, directly)
            if constexpr (kDirect) {
#pragma unroll
                for (int f = 0; f < NF; ++f)                            // this phase's weights are waited for first
                    asm volatile("" : "+v"(buf[d].q[f][kBits - 1]));
            } else {
                x_store(1 - d);
            }
            if (d == 1)
                store_scales(((u0 >> 1) + 1) & 1);
            if (d == 0)
                issue_scales((u0 >> 1) + 1);
            if constexpr (kDirect)
                issue_direct(u0 + d + 1, 1 - d);
            else
                issue_x();
            __builtin_amdgcn_sched_barrier(0);
            if ((u0 + d) * WK + wk < steps) {
                const u32x4_t* xb = xs + d * kBuf + x_read;
                const uint8_t* sb = ss + ((u0 >> 1) & 1) * kSBuf + s_read + d * (WK * 4);
                float scl[NF];
                u32x16_t six[kBits == 6 ? NF : 1] = {};                 // 6-bit: one convert for the whole block
                auto read_x = [&](int i, int j) { return xb[i * 256 + (chunk_at(kW == kBf16 ? 4 * j + lg : 4 * lg + j) ^ li)]; };
                auto weights = [&](int f, int j) { return operand<kW>(sl.q[f], six[kBits == 6 ? f : 0], scl[f], j); };
                auto multiply = [&](int i, int f, int j, u32x4_t w, u32x4_t x) {
                    f32x4_t& sum = sums_of[kCut == kSets ? j % kCopies : kCut == kChains ? 1 : kStepSums ? (kEach ? 1 + j : 1) : 0][i][f];
                    sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, x),
                        kStepSums && (kEach || j == 0) ? f32x4_t{0.f, 0.f, 0.f, 0.f} : sum, 0, 0, 0);
                };
#pragma unroll
                for (int i = 0; i < (kCut == kSteps && kRoll ? 1 : MF); ++i)
                    xf[0][i] = read_x(i, 0);
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    scl[f] = !kScaled ? 1.f : __uint_as_float((kRagged ? sl.s[f] : (uint32_t)sb[f * 16 * kSRow]) << 23);
                    if constexpr (kBits == 6) {
                        const u32x6_t packed = {sl.q[f][0], sl.q[f][1], sl.q[f][2], sl.q[f][3], sl.q[f][4], sl.q[f][5]};
                        if constexpr (kW == kE3m2)
                            six[f] = __builtin_bit_cast(u32x16_t, __builtin_amdgcn_cvt_scalef32_pk32_bf16_bf6(packed, scl[f]));
                        else
                            six[f] = __builtin_bit_cast(u32x16_t, __builtin_amdgcn_cvt_scalef32_pk32_bf16_fp6(packed, scl[f]));
                    }
                }
                if constexpr (kCut == kSteps && kRoll) {
                    // one fragment's four instructions behind each other; its sums are added beside the next one's
                    u32x4_t w[4][NF], xj[4] = {xf[0][0], read_x(0, 1), read_x(0, 2), read_x(0, 3)};
                    f32x4_t part[2][NF];
#pragma unroll
                    for (int f = 0; f < NF; ++f)
                        w[0][f] = weights(f, 0);
#pragma unroll
                    for (int i = 0; i <= MF; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
#pragma unroll
                            for (int f = 0; f < NF; ++f) {
                                f32x4_t& sum = part[i & 1][f];
                                if (i < MF)
                                    sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                        __builtin_bit_cast(bf16x8_t, w[j][f]), __builtin_bit_cast(bf16x8_t, xj[j]),
                                        j == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : sum, 0, 0, 0);
                                if (i == 0 && j < 3)
                                    w[j + 1][f] = weights(f, j + 1);
                                if (i > 0 && j == 1) {
                                    acc[i - 1][f] += part[(i - 1) & 1][f];
                                    asm volatile("" : "+v"(acc[i - 1][f]));     // (the sum stays here)
                                }
                            }
                            if (i + 1 < MF)
                                xj[j] = read_x(i + 1, j);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                } else if constexpr (kRoll) {
                    u32x4_t w[2][NF];
#pragma unroll
                    for (int f = 0; f < NF; ++f)
                        w[0][f] = weights(f, 0);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int i = 0; i < MF; ++i) {
#pragma unroll
                            for (int f = 0; f < NF; ++f)
                                multiply(i, f, j, w[j & 1][f], xf[0][i]);
                            if (j < 3) {
                                xf[0][i] = read_x(i, j + 1);
#pragma unroll
                                for (int f = 0; f < NF; ++f)            // the converts spread over the fragments
                                    if (f * (MF - 1) / NF + 1 == i)
                                        w[(j + 1) & 1][f] = weights(f, j + 1);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (j < 3)
#pragma unroll
                            for (int i = 0; i < MF; ++i)
                                xf[(j + 1) & 1][i] = read_x(i, j + 1);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int f = 0; f < NF; ++f) {
                            const u32x4_t w = weights(f, j);
#pragma unroll
                            for (int i = 0; i < MF; ++i)
                                multiply(i, f, j, w, xf[j & 1][i]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (kStepSums)
                        end_chain();
                }
            }
            if constexpr (kCut == kChains) {
                if (d == 1 && (--chain_left == 0 || u0 + 2 >= phases)) {
                    chain_left = chain_all;
                    end_chain();
                }
                if (d == 0 && cuts_phases(WK, MF) && phases <= 2)       // a single pair
                    end_chain();
            }
            issue_q(buf[d]);
            if constexpr (kDirect) {
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kQueued) : "memory");      // the activations; younger are the weights just asked for
            }
            lds_barrier();
        }
    }

    if constexpr (kCut == kSets)
#pragma unroll
        for (int c = 1; c < kCopies; ++c)
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    acc[i][f] += sums_of[c][i][f];

    // Output fragment (i, f) of block position (wm, wn): lane (li, lg) holds weight rows 4 lg + r for
    // activation row li.  The sums go through the LDS, so that whole rows are stored.
    constexpr int kStride = tile_stride(BN);
    if constexpr (WK == 1) {
        if (out.bias) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const f32x4_t bias = bias_of(out, n0 + (wn * NF + f) * 16 + 4 * lg);
#pragma unroll
                for (int i = 0; i < MF; ++i)
                    acc[i][f] += bias;
            }
        }
        float* tile = reinterpret_cast<float*>(smem);
        constexpr int PF = tile_rows(WM, MF, NF, BN) / (WM * 16);                            // fragment rows of a wave per turn
#pragma unroll
        for (int p = 0; p < MF / PF; ++p) {
            auto row_of = [&](int r) { return m0 + r / (PF * 16) * (MF * 16) + p * (PF * 16) + r % (PF * 16); };
            auto fill = [&]() {
                if (p > 0)
                    lds_barrier();
#pragma unroll
                for (int i = 0; i < PF; ++i)
#pragma unroll
                    for (int f = 0; f < NF; ++f)
                        *reinterpret_cast<f32x4_t*>(tile + ((wm * PF + i) * 16 + li) * kStride + (wn * NF + f) * 16 + 4 * lg) =
                            acc[p * PF + i][f];
                lds_barrier();
            };
            if (out.part_val != nullptr) {
                fill();
                pick_rows<WM * PF * 16, BN, kStride>(out, tile, n0, tn, row_of);
            } else if (MF * NF < 8 && out.residual && !rows_aligned(out.residual, out.ldr)) {
                // Small blocks, several on a unit: they hide each other's slow loads, and pieces on the residual's boundaries (one more to a
                // row, their sums shifted) cost more: 18577 x 256 at 64 rows 6.25 us with those, 4.62; 32011 x 512 at 141 rows 18.2, 13.4.
                fill();
                BlockOut rest = out;
                rest.bias = nullptr;                                   // (is in the sums)
                for (int e = tid; e < WM * PF * 16 * (BN / 8); e += kThreads) {
                    const int r = e / (BN / 8), c = e % (BN / 8) * 8;
                    float sums[8];
                    row_floats<8, BN>(tile + r * kStride, c, true, sums);
                    emit_sums(rest, sums, row_of(r), n0 + c);
                }
            } else {
                emit_rows<WM * PF * 16, BN, kStride>(out, tile, n0, row_of, fill);
            }
        }
    } else {
        f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);               // [position][fragment][wk][lane]
        const int base = (wm * WN + wn) * MF * NF;
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f)
                red[((base + i * NF + f) * WK + wk) * 64 + lane] = acc[i][f];
        lds_barrier();
        // the sums of fragment (at / NF, at % NF) of a position, of one lane's place, in wave order
        auto sum_of = [&](int at, int place) {
            f32x4_t sum = red[at * WK * 64 + place];
#pragma unroll
            for (int w = 1; w < WK; ++w)
                sum += red[(at * WK + w) * 64 + place];
            return sum;
        };
        if (out.part_val != nullptr) {
            float* tile = reinterpret_cast<float*>(smem + (size_t)8 * MF * NF * 1024);
            for (int e = wk; e < MF * NF; e += WK)
                *reinterpret_cast<f32x4_t*>(tile + ((wm * MF + e / NF) * 16 + li) * kStride + (wn * NF + e % NF) * 16 + 4 * lg) =
                    sum_of(base + e, lane);
            lds_barrier();
            pick_rows<BM, BN, kStride>(out, tile, n0, tn, [&](int r) { return m0 + r; });
        } else {
            // (whole rows through the LDS in pieces on a misaligned residual's boundaries, as the blocks do whose waves do not share K: 0.96 to 1.02
            // of this without the gate, 1.02 to 1.15 with it, and the code for it took 2 to 4 % of every call of 64 x 192 outputs)
            // straight from the partial sums: sixteen rows side by side, then the next columns; four sums per thread where
            // that takes one turn (748 x 6528 at 20 rows 6.85 us with eight, 6.48), else eight
            constexpr int kCols = BM * BN <= 4 * kThreads ? 4 : 8, kChunks = BN / kCols, kPerTile = 16 / kCols;
#pragma unroll 1
            for (int e = tid; e < BM * kChunks; e += kThreads) {
                const int row = e & 15, c = (e >> 4) % kChunks, i = (e >> 4) / kChunks, col = c / kPerTile;
                const int at = ((i / MF * WN + col / NF) * MF + i % MF) * NF + col % NF, place = c % kPerTile * (kCols * 4) + row;
                float sums[kCols];
#pragma unroll
                for (int h = 0; h < kCols / 4; ++h) {
                    const f32x4_t part = sum_of(at, place + 16 * h);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        sums[4 * h + r] = part[r];
                }
                emit_sums(out, sums, m0 + i * 16 + row, n0 + c * kCols);
            }
        }
    }
}

template <Kind kW, int WM, int WN, int WK, int MF, int NF, bool kDirect>
hipError_t launch_way(const Args& a, const DeviceInfo& dev, hipStream_t stream)
{
    auto kern = gemm_wide_kernel<kW, WM, WN, WK, MF, NF, kDirect>;
    static LdsLimit lds_limit;                      // of this kernel instance
    if (hipError_t e = lds_limit.raise(reinterpret_cast<const void*>(kern), dev.lds_bytes); e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3(a.tiles_m * a.tiles_n), dim3(kThreads), lds_bytes(kW, WM, WN, WK, MF, NF), stream, a.x, a.q,
                       a.s, a.n, a.k, a.m, a.ldx, a.ldw, a.tiles_m, a.tiles_n, a.chains, a.out);
    return hipGetLastError();
}
template <Kind kW, int WM, int WN, int WK, int MF, int NF>
hipError_t launch_block(const Args& a, const DeviceInfo& dev, hipStream_t stream)
{
    if constexpr (has_direct(kW, WK, MF, NF))
        if (takes_direct(kW, WK, MF, NF, a.k, a.tiles_m, a.out.part_val != nullptr))
            return launch_way<kW, WM, WN, WK, MF, NF, true>(a, dev, stream);
    if constexpr (has_registers(kW, WK, MF, NF))
        return launch_way<kW, WM, WN, WK, MF, NF, false>(a, dev, stream);
    return hipErrorInvalidValue;
}

// A block shape with what it took, in microseconds: the first block of a compute unit and every further one
// as start + step x (steps of 128 along K, whole phases).  Fitted to every shape at 3300 sizes (row-major MXFP4; 1550 each of the 8-bit,
// 6-bit, ternary and BF16 elements) of 3 to 520 rows, 128 to 65536 weight rows and K = 128 to 12288, six sets of weights in
// rotation, those near the fastest shape of a size weighing most.  (Fitted up to 34000 weight rows alone: 1.018 of the fastest on average
// beyond them.)  That was before the activations' direct way and the sums' present way out, which favour the larger blocks: the figures are up to
// 6 % above what the largest take now, and only their order counts.  On the kernel as it is, at 640 to 725 other sizes each, the choice is within
// 5 % of the fastest shape that cuts the sums far enough on 684 of 724 (MXFP4), 660 of 725 (its tile-major copy, which takes the same table), 646 of
// 694 (8 bits), 659 of 700 (6), 690 of 718 (ternary) and 602 of 639 (BF16), on average 1.010, 1.011, 1.008, 1.008, 1.007 and 1.009 of it, at
// worst 1.40 (519 x 16310 x 7936, a row of blocks for seven rows), 1.25, 1.24, 1.16, 1.42 and 1.16 (there mostly a short K under many weight rows).
struct Cost {
    int wm, wn, wk, mf, nf;
    float first_start, first_step, next_start, next_step;
};

// The launches of a table's shapes, in its order.
using Launch = hipError_t (*)(const Args&, const DeviceInfo&, hipStream_t);
template <Kind kW, auto& kTable, size_t... kAt>
constexpr std::array<Launch, sizeof...(kAt)> launches(std::index_sequence<kAt...>)
{
    return {launch_block<kW, kTable[kAt].wm, kTable[kAt].wn, kTable[kAt].wk, kTable[kAt].mf, kTable[kAt].nf>...};
}
template <Kind kW, auto& kTable>
constexpr auto launches()
{
    return launches<kW, kTable>(std::make_index_sequence<std::size(kTable)>{});
}

// The cheapest of a table's shapes for a call, of those that cut its sums as far as it wants (-1: none with at most `max_cols` block
// columns); kBits per weight.  Products and picks take the same one, but for picks with little room for partial winners.  Written
// out over the table, so that all divisions but the one by the units are by constants (0.30 us of a call's host time, 0.05 now).
template <auto& kTable, int kBits, size_t... kAt>
int pick_shape(int m, int n, int k, int cus, int max_cols, Args* a, std::index_sequence<kAt...>)
{
    const char* forced_shape = knob("MXFP4_WIDE_SHAPE");            // measurement only
    const int forced = forced_shape ? atoi(forced_shape) : -1;
    const int wanted = chains_wanted(m, n, k, cus), all_steps = (k + 127) / 128;
    int best = -1;
    float best_time = 0;
    auto consider = [&](auto at) {
        constexpr int i = at();
        constexpr Cost c = kTable[i];
        constexpr int bm = c.wm * c.mf * 16, bn = c.wn * c.nf * 16;
        const int tiles_m = (int)((uint32_t)(m + bm - 1) / bm), tiles_n = (int)((uint32_t)(n + bn - 1) / bn);
        const uint64_t blocks = (uint64_t)tiles_m * tiles_n + (uint32_t)(cus - 1);
        const int rounds = (int)(blocks >> 32 ? blocks / (uint32_t)cus : (uint32_t)blocks / (uint32_t)cus);
        const int steps = (int)((uint32_t)(all_steps + c.wk - 1) / c.wk * c.wk);
        const float time = i == forced ? -1.f
                                       : c.first_start + c.first_step * steps + (rounds - 1) * (c.next_start + c.next_step * steps);
        if (tiles_n <= max_cols && (best < 0 || time < best_time) &&
            (i == forced || cuts_enough(kBits, c.wm, c.wn, c.wk, c.mf, c.nf, m, n, k, cus, wanted))) {
            best = i;
            best_time = time;
            a->tiles_m = tiles_m;
            a->tiles_n = tiles_n;
        }
    };
    (consider(std::integral_constant<int, (int)kAt>{}), ...);
    a->chains = wanted;
    return best;
}
template <auto& kTable, int kBits>
int pick_shape(int m, int n, int k, int cus, int max_cols, Args* a)
{
    return pick_shape<kTable, kBits>(m, n, k, cus, max_cols, a, std::make_index_sequence<std::size(kTable)>{});
}

}  // namespace wide
}  // namespace mxfp4

// The product for more activation rows than one matrix-core tile column holds (a prompt, several
// sequences verified together) and, at any row count from three on, for K that is no multiple of 128
// (arXiv 2503.13565, section 3.4.3, Eq. 2 for the arithmetic; every weight is still read once per
// pass over the rows).
//
// The tile kernels keep all of K of at most 16 activation rows in the LDS, so more rows take more
// passes, and every pass streams and decodes the weights again.  Here a workgroup of eight waves
// computes a BM x BN block of the output and walks K once: the activation rows of one phase of K
// (WK steps of 128 elements) sit in one of two LDS buffers, shared by all waves; a wave loads the weights of
// its 16 NF rows straight into registers, in the layout of the tile kernels (lane i + 16 g: the 16
// bytes of block 4 T + g of row i), decodes them once and uses them for MF fragments of 16 activation
// rows.  The eight waves are WM x WN x WK: WM and WN split the block, WK splits the steps of a phase (few
// rows: the block is small and K is what there is to share), and then the WK partial sums of a
// fragment meet in the LDS at the end and are added in wave order.
//   - A phase's activations (16-byte chunks, one row's chunks to neighbouring threads) and its weights
//     are requested two phases ahead into registers, the activations written to the LDS one phase ahead:
//     one barrier per phase, which waits for LDS traffic only.
//   - LDS layout [step of the phase][row][16 chunks], chunk c of row r at position c ^ (r % 16): the
//     threads of a store cover whole rows and the 16 rows of an operand read hit different banks.
//   - The scale bytes of two phases travel together, one dword per step and row, through the LDS: as byte
//     loads by the lanes that use them (which the kernel does where K % 128 != 0 leaves the dwords
//     unaligned) every byte pulled a cache line, 104 us instead of 130 on the example below.
//   - Prompts take blocks of 128 rows with all eight waves side by side along the weight rows, so that no
//     weight is decoded or fetched twice in a block: 92 us against 104 for 2 x 4 waves.
//   - Bound by the matrix pipe at the clock the power limit leaves (with the loads and the LDS reads taken out
//     the example takes 69 us, with all-zero operands 80), by the activations' way through the L2 and LDS for some
//     tens of rows.  Measured, us per call, 16-row passes -> here: 22016 x 4096 with the gate at 509 rows
//     436 -> 79 (a library product of BF16 weights of that shape: 91), 12288 x 4096 at 32 rows 18.6 -> 12.2
//     (host time included), 4096 x 1376 at 7 rows (two rows per pass on the vector ALUs before) 18.3 -> 4.7.
//   - A block past the end of K (K % 128 != 0, the steps that round a phase up) is a load past the
//     descriptor: zero weights against zero activations.
#include <stdlib.h>

#include "common.h"
#include "kernels.h"
#include "../../include/mxfp4.h"

namespace mxfp4 {

namespace {

constexpr int kOob = 0x7FFFFFF0;        // lane offset beyond any descriptor: the load returns zero
constexpr int kThreads = 512;

struct WideArgs {
    const uint16_t* x;
    const uint8_t* q;
    const uint8_t* s;
    uint16_t* y;
    float* part_val;                    // argmax form: [M, parts], one partial winner per row and block column
    int32_t* part_idx;
    const uint16_t* bias;
    const uint16_t* residual;
    int64_t ldx, ldy;
    int n, k, m, parts, ldr, act, tiles_m, tiles_n;
};

// Scale bytes of a block's weight rows for two phases, one row behind the other with a dword of padding
// (the rows of an operand read hit different banks).
constexpr int scale_row_bytes(int wk) { return wk * 8 + 4; }

constexpr size_t wide_lds_bytes(int wm, int wn, int wk, int mf, int nf)
{
    const size_t xs = (size_t)2 * wk * wm * mf * 16 * 256 +             // two buffers of one phase
                      (size_t)2 * wn * nf * 16 * scale_row_bytes(wk);   // and two of the scales
    const size_t red = wk > 1 ? (size_t)8 * mf * nf * 1024 : 0;         // the waves' partial sums, afterwards
    const size_t table = (size_t)wm * wn * mf * nf * 16 * 8;            // argmax: a winner per fragment and row
    const size_t most = xs > red ? xs : red;
    return wk > 1 ? most + table : most > table ? most : table;         // (WK = 1: the table takes the buffers' place)
}

template <int WM, int WN, int WK, int MF, int NF, bool kRagged>
__global__ __launch_bounds__(kThreads, 2) void gemm_wide_kernel(WideArgs a)
{
    static_assert(WM * WN * WK == 8, "eight waves");
    constexpr int BM = WM * MF * 16, BN = WN * NF * 16;
    constexpr int CA = WK * BM * 16 / kThreads;                         // activation chunks per thread and phase
    static_assert(CA >= 1 && CA * kThreads == WK * BM * 16, "whole chunks");
    constexpr int kRowChunks = WK * 16;                                 // chunks of one row in a phase
    constexpr int kRowStep = kThreads / kRowChunks;                     // rows between a thread's chunks
    constexpr int kBuf = WK * BM * 16;                                  // chunks of one LDS buffer
    constexpr int kSRow = scale_row_bytes(WK), kSBuf = BN * kSRow;
    constexpr int SC = kRagged ? 0 : (BN * WK * 2 + kThreads - 1) / kThreads;   // scale dwords per thread and two phases
    extern __shared__ __align__(16) uint8_t smem[];
    u32x4_t* xs = reinterpret_cast<u32x4_t*>(smem);
    uint8_t* ss = smem + (size_t)2 * kBuf * 16;

    const int tid = threadIdx.x;
    const int lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wn = wave / WK % WN, wm = wave / WK / WN;
    const int n = a.n, k = a.k, m = a.m;
    const int nblk = k >> 5, steps = (k + 127) >> 7, phases = (steps + WK - 1) / WK;

    // Workgroups go to the eight dies round robin: a die takes a run of neighbouring blocks, the
    // blocks of one weight strip next to each other, so that the strip comes from its L2 after the first.
    const int total = a.tiles_m * a.tiles_n;
    const int die = blockIdx.x & 7, per = total >> 3, more = total & 7;
    const int at = die * per + (die < more ? die : more) + (int)(blockIdx.x >> 3);
    const int tm = at % a.tiles_m, tn = at / a.tiles_m;
    const int m0 = tm * BM, n0 = tn * BN;

    const int ldx = (int)a.ldx;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(a.x + (int64_t)m0 * a.ldx), 0, ((min(BM, m - m0) - 1) * ldx + k) * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.q), 0, n * (k >> 1), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(a.s), 0, n * nblk, 0x00020000);

    const int xc = tid % kRowChunks, xr = tid / kRowChunks;             // this thread's chunk of a row, first row
    int x_off[CA];
#pragma unroll
    for (int i = 0; i < CA; ++i)
        x_off[i] = (min(m0 + xr + i * kRowStep, m - 1) - m0) * ldx * 2 + xc * 16;       // ragged M: repeat the last row
    int q_off[NF], s_off[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int row = min(n0 + (wn * NF + f) * 16 + li, n - 1);       // ragged N: repeat the last row
        q_off[f] = row * (k >> 1) + lg * 16;
        s_off[f] = row * nblk + lg;
    }
    // (K % 128 == 0) dword e of the block's scales: step e % (2 WK) of the two phases, row e / (2 WK)
    int sc_off[SC + 1], sc_at[SC + 1];
#pragma unroll
    for (int i = 0; i < SC; ++i) {
        const int e = min(tid + i * kThreads, BN * WK * 2 - 1), r = e / (WK * 2), c = e % (WK * 2);
        sc_off[i] = min(n0 + r, n - 1) * nblk + c * 4;
        sc_at[i] = r * kSRow + c * 4;
    }

    struct Slot {
        u32x4_t x[CA];
        u32x4_t q[NF];
        uint32_t s[kRagged ? NF : 1];
    };
    Slot buf[2];
    uint32_t sc[SC + 1];
    // Always the same loads, and every condition on the position arithmetic (a branch around a load makes
    // the compiler wait for all of them): what lies past K gets an offset past the descriptor.  The
    // scalar offset stays inside the descriptor then too.
    auto past = [](int last, int at) { return ((last - at) >> 31) & kOob; };    // 0 where at <= last
    int ld_ph = 0;
    auto issue_scales = [&](int sp) {                                   // of the phases 2 sp and 2 sp + 1
        const int at = sp * (WK * 8) < nblk ? sp * (WK * 8) : 0;
#pragma unroll
        for (int i = 0; i < SC; ++i)
            sc[i] = __builtin_amdgcn_raw_buffer_load_b32(
                rs, sc_off[i] | past(nblk - 1, sp * (WK * 8) + (tid + i * kThreads) % (WK * 2) * 4), at, 0);
    };
    auto store_scales = [&](int b) {
#pragma unroll
        for (int i = 0; i < SC; ++i)
            *reinterpret_cast<uint32_t*>(ss + b * kSBuf + sc_at[i]) = sc[i];
    };
    auto issue = [&](Slot& sl) {
        const int x_past = past((k >> 3) - 1, ld_ph * kRowChunks + xc);
        const int x_at = ld_ph < phases ? ld_ph * (kRowChunks * 16) : 0;
#pragma unroll
        for (int i = 0; i < CA; ++i)
            sl.x[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, x_off[i] | x_past, x_at, 0);
        const int q_past = past(nblk - 1, 4 * (ld_ph * WK + wk) + lg);
        const int T = ld_ph * WK + wk < steps ? ld_ph * WK + wk : 0;
        if constexpr (kRagged) {
#pragma unroll
            for (int f = 0; f < NF; ++f)
                sl.s[f] = __builtin_amdgcn_raw_buffer_load_b8(rs, s_off[f] | q_past, T * 4, 0);
        }
#pragma unroll
        for (int f = 0; f < NF; ++f)
            sl.q[f] = __builtin_amdgcn_raw_buffer_load_b128(rq, q_off[f] | q_past, T * 64, 0);
        ++ld_ph;
    };
    auto x_store = [&](const Slot& sl, int b) {
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const int r = xr + i * kRowStep;
            xs[b * kBuf + ((xc >> 4) * BM + r) * 16 + ((xc & 15) ^ (r & 15))] = sl.x[i];
        }
    };
    issue_scales(0);
    issue(buf[0]);
    __builtin_amdgcn_sched_barrier(0);                                  // keep the slots' loads in issue order
    issue(buf[1]);
    __builtin_amdgcn_sched_barrier(0);
    store_scales(0);
    x_store(buf[0], 0);
    lds_barrier();

    f32x4_t acc[MF][NF];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int f = 0; f < NF; ++f)
            acc[i][f] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int x_read = (wk * BM + wm * MF * 16 + li) * 16;
    const int s_read = (wn * NF * 16 + li) * kSRow + wk * 4 + lg;

    for (int u0 = 0; u0 < phases; u0 += 2) {
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const Slot& sl = buf[d];
            if ((u0 + d) * WK + wk < steps) {
                const u32x4_t* xb = xs + d * kBuf + x_read;
                const uint8_t* sb = ss + ((u0 >> 1) & 1) * kSBuf + s_read + d * (WK * 4);
                float scl[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    scl[f] = __uint_as_float((kRagged ? sl.s[f] : (uint32_t)sb[f * 16 * kSRow]) << 23);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    u32x4_t xf[MF];
#pragma unroll
                    for (int i = 0; i < MF; ++i)
                        xf[i] = xb[i * 256 + ((4 * lg + j) ^ li)];
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        const uint32_t qd = sl.q[f][j];
                        u32x4_t w;
                        w[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, scl[f], 0));
                        w[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, scl[f], 1));
                        w[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, scl[f], 2));
                        w[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(qd, scl[f], 3));
#pragma unroll
                        for (int i = 0; i < MF; ++i)
                            acc[i][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf16x8_t, w), __builtin_bit_cast(bf16x8_t, xf[i]), acc[i][f], 0, 0, 0);
                    }
                }
            }
            // the next phase's activations go to the buffer that the phase before this one read
            x_store(buf[1 - d], 1 - d);
            if (d == 1)
                store_scales(((u0 >> 1) + 1) & 1);
            if (d == 0)
                issue_scales((u0 >> 1) + 1);
            issue(buf[d]);
            lds_barrier();
        }
    }

    // Output fragment (i, f) of block position (wm, wn): lane (li, lg) holds weight rows 4 lg + r for
    // activation row li.
    constexpr size_t kXBytes = (size_t)2 * kBuf * 16 + 2 * kSBuf, kRedBytes = WK > 1 ? (size_t)8 * MF * NF * 1024 : 0;
    float2* table = reinterpret_cast<float2*>(smem + (WK == 1 ? 0 : kXBytes > kRedBytes ? kXBytes : kRedBytes));
    const bool pick = a.part_val != nullptr, gated = a.act == MXFP4_ACT_SWIGLU;
    const bool wide_store = !gated && (a.ldy & 3) == 0 && (reinterpret_cast<uintptr_t>(a.y) & 7) == 0;
    auto emit = [&](const f32x4_t sum, int i, int f) {
        const int row = m0 + (wm * MF + i) * 16 + li, col = n0 + (wn * NF + f) * 16 + 4 * lg;
        if (pick) {
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
            if (lane < 16)
                table[((wm * MF + i) * 16 + li) * (WN * NF) + wn * NF + f] = make_float2(best, __int_as_float(idx));
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
        if (wide_store && col + 4 <= n) {
            *reinterpret_cast<uint2*>(y + col) = make_uint2(o[0] | (uint32_t)o[1] << 16, o[2] | (uint32_t)o[3] << 16);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (col + r < n)
                    y[col + r] = o[r];
        }
    };
    if constexpr (WK == 1) {
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f)
                emit(acc[i][f], i, f);
    } else {
        f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);               // [position][fragment][wk][lane]
        const int base = (wm * WN + wn) * MF * NF;
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int f = 0; f < NF; ++f)
                red[((base + i * NF + f) * WK + wk) * 64 + lane] = acc[i][f];
        lds_barrier();
        for (int e = wk; e < MF * NF; e += WK) {                        // a fragment's sums, in wave order
            f32x4_t sum = red[(base + e) * WK * 64 + lane];
#pragma unroll
            for (int w = 1; w < WK; ++w)
                sum += red[((base + e) * WK + w) * 64 + lane];
            emit(sum, e / NF, e % NF);
        }
    }
    if (pick) {
        lds_barrier();
        if (tid < BM && m0 + tid < m) {
            float best = -INFINITY;
            int idx = 0x7FFFFFFF;
            for (int e = 0; e < WN * NF; ++e) {                         // columns ascend
                const float2 c = table[tid * (WN * NF) + e];
                if (c.x > best) {
                    best = c.x;
                    idx = __float_as_int(c.y);
                }
            }
            a.part_val[(int64_t)(m0 + tid) * a.parts + tn] = best;
            a.part_idx[(int64_t)(m0 + tid) * a.parts + tn] = idx;
        }
    }
}

// The block shapes there are, each with what it took, in microseconds: the first block of a compute unit
// and every further one as start + step x (steps of 128 along K, whole phases), measured with 256, 512 and 1024
// blocks over K = 1024 and 4096.  (Two blocks share a unit where LDS and registers allow.)
struct Shape {
    int wm, wn, wk, mf, nf;
    float first_start, first_step, next_start, next_step;
    hipError_t (*launch)(const WideArgs&, const DeviceInfo&, hipStream_t);
};

template <int WM, int WN, int WK, int MF, int NF>
hipError_t launch_shape(const WideArgs& a, const DeviceInfo& dev, hipStream_t stream)
{
    auto kern = gemm_wide_kernel<WM, WN, WK, MF, NF, false>;
    auto kern_ragged = gemm_wide_kernel<WM, WN, WK, MF, NF, true>;
    static LdsLimit lds_limit, lds_limit_ragged;    // of these kernel instances
    const bool ragged = a.k % 128 != 0;
    if (hipError_t e = (ragged ? lds_limit_ragged : lds_limit)
                           .raise(reinterpret_cast<const void*>(ragged ? kern_ragged : kern), dev.lds_bytes);
        e != hipSuccess)
        return e;
    if (ragged)
        kern = kern_ragged;
    hipLaunchKernelGGL(kern, dim3(a.tiles_m * a.tiles_n), dim3(kThreads), wide_lds_bytes(WM, WN, WK, MF, NF), stream, a);
    return hipGetLastError();
}

#define MXFP4_WIDE(WM_, WN_, WK_, MF_, NF_, A_, B_, C_, D_) \
    {WM_, WN_, WK_, MF_, NF_, A_, B_, C_, D_, launch_shape<WM_, WN_, WK_, MF_, NF_>}
const Shape kShapes[] = {
    MXFP4_WIDE(1, 1, 8, 1, 1, 4.29f, 0.060f, 1.20f, 0.047f),
    MXFP4_WIDE(1, 1, 8, 1, 2, 4.71f, 0.070f, 1.46f, 0.078f),
    MXFP4_WIDE(1, 1, 8, 1, 3, 5.05f, 0.107f, 1.73f, 0.099f),
    MXFP4_WIDE(1, 1, 8, 1, 4, 5.04f, 0.145f, 1.82f, 0.125f),
    MXFP4_WIDE(1, 1, 8, 1, 6, 5.46f, 0.224f, 4.12f, 0.185f),
    MXFP4_WIDE(1, 1, 8, 1, 8, 6.23f, 0.282f, 4.93f, 0.248f),
    MXFP4_WIDE(1, 1, 8, 2, 1, 5.18f, 0.101f, 3.47f, 0.101f),
    MXFP4_WIDE(1, 1, 8, 2, 2, 5.56f, 0.145f, 3.83f, 0.134f),
    MXFP4_WIDE(1, 1, 8, 2, 3, 5.98f, 0.182f, 4.27f, 0.164f),
    MXFP4_WIDE(1, 1, 8, 2, 4, 6.22f, 0.219f, 4.80f, 0.192f),
    MXFP4_WIDE(1, 1, 8, 2, 6, 7.51f, 0.290f, 6.36f, 0.240f),
    MXFP4_WIDE(1, 2, 4, 4, 1, 4.28f, 0.332f, 2.83f, 0.297f),
    MXFP4_WIDE(1, 2, 4, 4, 2, 5.42f, 0.378f, 4.55f, 0.310f),
    MXFP4_WIDE(1, 2, 4, 4, 3, 6.60f, 0.465f, 5.28f, 0.416f),
    MXFP4_WIDE(2, 2, 2, 4, 2, 7.37f, 0.685f, 5.26f, 0.647f),
    MXFP4_WIDE(2, 2, 2, 4, 3, 9.18f, 0.845f, 5.97f, 0.860f),
    MXFP4_WIDE(2, 4, 1, 4, 2, 8.47f, 0.990f, 0.57f, 1.088f),
    MXFP4_WIDE(2, 4, 1, 4, 3, 11.68f, 1.322f, 5.43f, 1.589f),
    MXFP4_WIDE(1, 8, 1, 8, 2, 13.11f, 1.649f, 10.94f, 1.719f),
    MXFP4_WIDE(1, 8, 1, 8, 3, 17.49f, 2.228f, 15.91f, 2.251f),
    MXFP4_WIDE(1, 4, 2, 4, 1, 4.52f, 0.447f, 1.79f, 0.317f),
    MXFP4_WIDE(1, 4, 2, 4, 2, 6.33f, 0.526f, 2.02f, 0.463f),
    MXFP4_WIDE(1, 4, 2, 4, 3, 8.68f, 0.704f, 4.44f, 0.877f),
};
#undef MXFP4_WIDE

// What a call would take with a shape, in microseconds.
float shape_time(const Shape& c, int m, int n, int k, int cus, int* tiles_m, int* tiles_n)
{
    const int bm = c.wm * c.mf * 16, bn = c.wn * c.nf * 16;
    *tiles_m = (m + bm - 1) / bm;
    *tiles_n = (n + bn - 1) / bn;
    const int rounds = (int)(((int64_t)*tiles_m * *tiles_n + cus - 1) / cus);
    const int steps = ((k + 127) / 128 + c.wk - 1) / c.wk * c.wk;
    return c.first_start + c.first_step * steps + (rounds - 1) * (c.next_start + c.next_step * steps);
}

const Shape* pick_shape(int m, int n, int k, int cus, int max_cols, int* tiles_m, int* tiles_n)
{
    const char* forced_shape = knob("MXFP4_WIDE_SHAPE");            // measurement only
    const int env = forced_shape ? atoi(forced_shape) : -1;
    const Shape* best = nullptr;
    float best_time = 0;
    int i = 0;
    for (const Shape& c : kShapes) {
        int tm, tn;
        const float time = shape_time(c, m, n, k, cus, &tm, &tn);
        const bool forced = env == i++;
        if (tn <= max_cols && (!best || time < best_time || forced)) {
            best = &c;
            best_time = forced ? -1.f : time;
            *tiles_m = tm;
            *tiles_n = tn;
        }
    }
    return best;
}

}  // namespace

bool gemm_wide_can_run(const GemmArgs& a, const DeviceInfo& dev)
{
    if (a.k % 32 != 0 || a.m < 1 || a.ldx > (1 << 21))              // a block's activation rows behind one 32-bit offset
        return false;
    if (dev.lds_bytes < 160 * 1024)
        return false;
    return a.part_val == nullptr || (a.n + 127) / 128 <= a.parts;   // (a column of partial winners per 128 weight rows)
}

hipError_t launch_gemm_wide(const GemmArgs& a, const DeviceInfo& dev, int* parts_used, hipStream_t stream,
                            const Epilogue* epi)
{
    if (!gemm_wide_can_run(a, dev))
        return hipErrorInvalidValue;
    WideArgs w{};
    const Shape* c = pick_shape(a.m, a.n, a.k, dev.cus, a.part_val ? a.parts : 0x7FFFFFFF, &w.tiles_m, &w.tiles_n);
    if (!c)
        return hipErrorInvalidValue;
    w.x = a.x;
    w.q = a.q;
    w.s = a.s;
    w.y = a.y;
    w.part_val = a.part_val;
    w.part_idx = a.part_idx;
    w.ldx = a.ldx;
    w.ldy = a.ldy;
    w.n = a.n;
    w.k = a.k;
    w.m = a.m;
    w.parts = a.parts;
    if (epi) {
        w.bias = epi->bias;
        w.residual = epi->residual;
        w.ldr = epi->ldr;
        w.act = epi->act;
    }
    if (parts_used)
        *parts_used = w.tiles_n;
    return c->launch(w, dev, stream);
}

}  // namespace mxfp4

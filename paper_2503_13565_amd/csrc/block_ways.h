// How a block of gemm_wide.h brings its activations into the LDS, and which forms of a block shape there are.  Plain integer arithmetic
// without any device header, so that it can be walked on the CPU for every table and size.
//
// Through registers: asked for two phases ahead, written a phase ahead.  Or directly, by loads that put them there: asked for a phase ahead,
// into the buffer that the phase before read.  The direct way saves the registers, the writes and their waits, but its loads
// leave only when the phase's weights have arrived: the compiler counts the weights' loads exactly as long as nothing younger is in flight that
// it does not know, and a wait too many is a whole latency.  So it is for
//   - calls of few phases, which are mostly start and end: 1016 x 2016 at three rows 3.72 -> 3.42 us, 14234 x 768 at 17 4.26 -> 4.02, E3M2
//     1875 x 1152 at 24 3.85 -> 3.57; with nine phases and more 1.05 to 1.15 of the other way, and so are many rows of blocks over few weight
//     rows (302 x 4352 at 173 rows, five phases, 1.09; 542 x 2048 at 475 1.07) and picks (1.00 to 1.02);
//   - blocks whose waves all lie along the weight rows, at any K: over 1300 sizes 0.90 to 1.00 of the registers by shape and layout (128 x 384
//     outputs 0.95 at K = 1024 and at 6144, tile-major 0.93; 128 rows in two times four waves 0.92; ternary 0.93 to 0.97; 6 bits 0.97 up to K =
//     1024 and 1.00 to 1.01 beyond).  But not with eight fragments a wave and 8 bits (1.00 up to K = 1024, 1.02 at 2560, 60 x 48000 x 2048 1.04,
//     1.10 from 4096 on: E4M3 138 x 14496 x 7552 84 us, 92 directly), nor with a long K in row-major MXFP4: from 8192 on 1.07 (58 x 50677 x
//     10112 95 us, 105 directly); up to there 0.98 to 1.00, and between 5120 and 8192 1.02 to 1.04 with weights from memory, 0.95 from the last-level cache.
#pragma once

namespace mxfp4 {
namespace wide {

// The weights: MXFP4 row-major, MXFP4 tile-major, MXFP4 row-major with K % 128 != 0, E4M3 and E5M2 bytes,
// E2M3 and E3M2 blocks of 24 bytes, ternary blocks of 8 bytes, unquantised BF16 (any K % 8 == 0).
enum Kind { kMx, kMxTiled, kMxRagged, kE4m3, kE5m2, kE2m3, kE3m2, kT2, kBf16 };
constexpr int kind_bits(Kind w)
{
    return w == kBf16 ? 16 : w == kE4m3 || w == kE5m2 ? 8 : w == kE2m3 || w == kE3m2 ? 6 : w == kT2 ? 2 : 4;
}

// Steps of 128 along K up to which blocks with all waves along the weight rows take the direct way (0: at any K).
constexpr int direct_steps(Kind w, int mf, int nf) { return w == kMx && mf * nf == 8 ? 64 : 0; }

// Whether a shape has the direct form: where it is the faster, and not where a K of few phases never takes the shape (with 256 units; 65
// million sizes to 120000 rows and three million weight rows).
constexpr bool has_direct(Kind w, int wk, int mf, int nf)
{
    if (w == kBf16)
        return false;
    if (kind_bits(w) != 4)
        return !(kind_bits(w) == 8 && wk == 1 && mf * nf == 8);
    if ((wk == 4 && mf == 2 && nf == 4) || (wk == 2 && mf == 4 && nf == 2))
        return false;
    return w != kMxTiled || wk == 1 || !((nf == 2 && wk >= 4) || (wk == 8 && mf == 2) || nf == 4);
}

// Whether it has the one through registers, which takes every call that the direct one does not.
constexpr bool has_registers(Kind w, int wk, int mf, int nf) { return !has_direct(w, wk, mf, nf) || wk > 1 || direct_steps(w, mf, nf) > 0; }

// Which of them a call takes; `tiles_m` blocks of rows.
constexpr bool takes_direct(Kind w, int wk, int mf, int nf, int k, int tiles_m, bool pick)
{
    const int steps = (k + 127) / 128;
    if (!has_direct(w, wk, mf, nf) || !has_registers(w, wk, mf, nf))
        return has_direct(w, wk, mf, nf);
    if (wk == 1)
        return steps <= direct_steps(w, mf, nf);
    return !pick && steps <= (w == kMxTiled ? 3 : tiles_m > 6 ? 2 : 6) * wk;
}

}  // namespace wide
}  // namespace mxfp4

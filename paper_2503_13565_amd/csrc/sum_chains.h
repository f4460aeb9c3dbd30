// Into how many chains the block kernel (gemm_wide.h) cuts the sum of an output along K, and which block shapes cut it as
// far.  Plain integer arithmetic without any device header, so that it can be walked on the CPU for every table and size.
//
// An output is up to K / 32 matrix instructions added one behind the other in 32 bits, and the roundings of such a chain grow with
// its length: the picks' values at 64 rows and K = 4096 are off by 0.84e-7 of them in eight chains, 0.98e-7 in four, 1.3e-7 in two
// and 1.9e-7 in one (MXFP4; BF16 1.5e-7, 2.0e-7, 2.8e-7, 4.2e-7).  The waves that share K make a chain each, so how far a
// sum is cut would change with the block shape, that is with what is fastest at a size.  It does not: a call is cut
// as far as blocks of eight (few outputs, or a long K), four and two waves along K cut it, and a shape with fewer waves along K cuts its
// waves' sums further.
#pragma once

#include <cstdint>

namespace mxfp4 {
namespace wide {

// Blocks without registers for a second set of sums: one chain per wave.
constexpr bool uncut(int mf, int nf) { return mf * nf > 16; }

// Sums that the matrix instructions of a step take turns on, where there are registers for them: sixteen chains of K for blocks of
// sixteen rows, as many as the tile kernels make (eight with two waves along K), eight for the others.
constexpr int sum_sets(int wk, int mf) { return mf == 1 ? (wk == 8 ? 2 : 4) : mf <= 3 && wk == 4 ? 2 : 1; }

// Whether a block whose sums are cut at pairs of phases also cuts the only pair there is.
constexpr bool cuts_phases(int wk, int mf) { return wk == 2 && mf <= 3; }

constexpr int64_t tiles_of(int m, int n) { return (int64_t)((m + 15) / 16) * ((n + 15) / 16); }

// Chains of a call's outputs: eight up to 32 rows or 12 tiles of 16 x 16 outputs per compute unit, four up to 28, else two; twice
// that, and eight at most, where K is longer than 4096 (blocks of four waves along K went there too, and a further cut of
// so long a sum takes no time that could be measured); never more than steps of 128 along K.
constexpr int chains_wanted(int m, int n, int k, int cus)
{
    const int64_t tiles = tiles_of(m, n);
    const int few = m <= 32 || tiles <= 12 * (int64_t)cus ? 8 : tiles <= 28 * (int64_t)cus ? 4 : 2, steps = (k + 127) / 128;
    const int most = k > 4096 && few < 8 ? 2 * few : few;
    return steps < most ? steps : most;
}

// What a shape with `wk` waves along K and mf x nf fragments can make of them, for elements of `bits`; `steps` of 128 along K.
constexpr int chains_of(int bits, int wk, int mf, int nf, int steps)
{
    if (wk == 8 || uncut(mf, nf))
        return wk;                                                      // (and more at one row of fragments)
    if (wk == 1)
        return steps > 4 ? 4 : 2;
    return bits <= 4 && mf > 3 && steps <= 2 * wk ? wk : 8;             // (6 bits and more: every step is a chain)
}

// Pairs of phases in a chain of a wave whose sums are cut at pairs: an eighth (a quarter, a half) of K at most, or one pair.
constexpr int chain_pairs(int phases, int wk, int chains)
{
    const int pairs = phases * wk / (2 * chains);
    return pairs > 1 ? pairs : 1;
}

// Whether a call may take a shape.  A block that cannot cut its sums is there for the largest products alone, where its outputs
// fill their rounds over the units to 85 %: there it is the fastest by a fifth (22016 x 4096 at 509 rows 75 us,
// 94 in blocks that do).
constexpr bool cuts_enough(int bits, int wm, int wn, int wk, int mf, int nf, int m, int n, int k, int cus, int wanted)
{
    if (chains_of(bits, wk, mf, nf, (k + 127) / 128) >= wanted)
        return true;
    if (!uncut(mf, nf) || m <= 32 || tiles_of(m, n) <= 28 * (int64_t)cus)
        return false;
    const int64_t bm = 16 * wm * mf, bn = 16 * wn * nf, blocks = ((m + bm - 1) / bm) * ((n + bn - 1) / bn);
    return (int64_t)m * n * 100 >= 85 * bm * bn * ((blocks + cus - 1) / cus * cus);
}
constexpr bool cuts_enough(int bits, int wm, int wn, int wk, int mf, int nf, int m, int n, int k, int cus)
{
    return cuts_enough(bits, wm, wn, wk, mf, nf, m, n, k, cus, chains_wanted(m, n, k, cus));
}

}  // namespace wide
}  // namespace mxfp4

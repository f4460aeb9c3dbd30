// Which products take the block kernel (gemm_wide.h) and which the kernels that hold their activation rows in the LDS.
// Plain integer arithmetic without any device header, so that the rules can be checked on the CPU.
//
// The blocks win where the other kernels would stream and decode the weights several times (more rows than a
// pass, rows that do not fit the LDS whole) and where every compute unit has one block.  They lose where a matrix has
// few rows and K is long: a block walks all of K by itself, while the other kernels split K over the units or
// keep a unit's tile beside its rows.  Every line below was measured on both sides over N = 16 .. 64000 and
// K = 128 .. 65536; `unit` is a number of weight rows per compute unit.
#pragma once

namespace mxfp4 {

// What the tile kernels would do with an MXFP4 call.
struct TileCall {
    int m, n, k, cus;
    bool fits;      // a pass of 16 (8, 4) rows fits the LDS whole
    bool split;     // else: K can be split over the units through the caller's workspace
    bool tiled;     // tile-major weights
    bool fused;     // bias, gate or residual behind the product
    bool pick;      // the pick instead of the product
};

// Three to eight rows that the tiles take in one pass.  Figures: blocks as a part of what the tiles take, over 256 to 65536
// weight rows, K = 128 to 14336 and 3 to 8 rows, with and without gate and pick, on average around the size that is named.  A tile per
// unit and a short K are nothing but start and end, where the blocks are the faster (4096 x 512 0.89, 0.95 tile-major; 8192 x 512 0.73;
// 32000 x 512 0.54, 0.58; K = 128 0.41 at 57344 weight rows, 0.86 to 0.93 at one tile per unit).  From there on either side wins where the
// weight rows and the phases of its loop come out even, within a tenth mostly: blocks in rounds of 256, phases of 256 to 1024
// elements, against tiles of 16 rows per unit in groups of 512 elements.
inline bool wide_one_pass_preferred(const TileCall& c)
{
    const int m = c.m, n = c.n, k = c.k, unit = c.cus;
    const bool wide = m > 4;                        // the tiles stage eight rows instead of four
    // One tile per unit: 4096 x 1280 1.03, x 4096 0.99, x 5120 1.0 to 1.03, x 6144 0.97, x 9216 0.93 to 0.97; at four rows 1.0 or more;
    // tile-major from K = 1280 on 1.02 to 1.2.
    if (n <= 16 * unit)
        return k <= 1024 || (!c.tiled && wide && k > 5120);
    if (k <= 1024)
        return true;
    if (c.tiled) {
        // Just past a whole number of the tiles' groups: 27262 x 4224 0.73, 18268 x 4608 0.80, 13822 x 4352 0.85.
        if (k > 4096 && k <= 4608)
            return true;
        // 8192 x 3072 0.88, x 4096 0.93 (0.95 at four rows, x 3584 0.97 to 1.02), x 5120 0.91 (0.99), x 8192 1.07.
        if (n <= 32 * unit)
            return k <= (wide ? 5120 : 3072);
        // 12288 x 1536 0.97, x 2048 1.02, x 3584 1.1, x 5120 0.89 (1.05), x 7168 0.99 (1.06), x 9216 0.90.
        if (n <= 48 * unit)
            return k <= 1536 || (wide && k > 4096 && k <= 6144) || k > 8704;
        // 22016 x 4096 0.91, 24576 x 2048 0.87, x 4096 0.96, x 5120 0.75 (0.89), x 8192 0.95; 33924 x 7808 1.13; 57344 x 3584 0.97,
        // x 10240 1.0.
        return k <= 3072 || (wide && k > 4096 && k <= 7680) || (k > 7936 && (wide || k <= 9728)) ||
               (n > 80 * unit && n <= 96 * unit && k <= 4096);
    }
    // Just past a whole number of the tiles' groups: K = 4224 to 4608 at more than four rows 0.80 (20480 to 32768, 45056 weight rows)
    // to 0.92 (36864), at fewer 0.93 to 1.04, beyond 128 rows per unit 1.04 to 1.2.
    if (k > 4096 && k <= 4864 && (wide || n <= 128 * unit))
        return true;
    // 8192 x 2048 0.80, x 4096 0.85, x 7168 0.82 (0.90 at four rows), x 11008 0.75 (0.91).
    if (n <= 32 * unit)
        return k <= 11520;
    // 12288 x 3072 0.98, x 3584 0.97 to 1.0, x 4096 0.94 to 1.0, x 5120 0.90, x 8192 0.95; at four rows from 3584 on 1.0 to 1.1.
    if (n <= 48 * unit)
        return wide || k <= 3072;
    // 16384 x 4096 0.91, x 9216 0.92, x 10240 1.11 at four rows.
    if (n <= 64 * unit)
        return k <= 9728;
    // 20480 x 3072 1.02, x 3584 1.11, x 5120 0.98, x 6144 0.96; 32000 x 3072 0.99, x 3584 1.05, x 5120 0.91, x 7168 0.92, x 8192 1.09; at
    // four rows from 3584 on 1.07 to 1.2.  One round of blocks of 96 weight rows: 22016 to 24576 x 3584 0.99, x 4096 0.98 to 1.0 (pick 1.07).
    if (n <= 128 * unit)
        return k <= 3072 || (wide && k > 4096 && k <= 7680) || (n > 80 * unit && n <= 96 * unit && k <= 4096 && !c.pick);
    // Two rounds and more: K = 1280 0.95, 1536 1.0, 1664 1.08, 2048 1.08, just past the groups again 2176 0.96, 2304 0.93, 2432 0.99,
    // 2560 1.03, 3072 1.1, 4096 1.2.
    return k <= 1536 || (k > 2048 && k <= 2432);
}

// One and two rows of tile-major weights, where the tiles take them (two rows; one row with bias, gate or residual).  The decode kernels
// keep all other calls of one and two rows of quantised weights, also where a block would be faster (28000 x 512 at two rows of ternary
// codes 0.26): their lanes' short chains leave FP32 sums closer to 64 bits than a block does (blocks 1.0 to 1.7 of their rms error in row-major
// MXFP4, with ragged K 0.9 to 1.6, of 8 and 6 bits 0.9 to 1.9, ternary 1.0 to 1.1; 6000 values a size, those of the picks).  Against the tiles
// it is 0.87 to 1.01 from K = 1024 on (5000 x 640 1.1, 16000 x 256 1.2, 25600 x 2048 1.04).  Products and picks take the same lines, so that a
// pick is the largest of the sums that the product rounds.  Time, blocks as a part of the tiles' (product, pick): 300 x 1024 0.93, 0.95; 4096 x 1280
// 1.00, 0.97, x 2048 0.97, 0.96; 6000 x 1536 0.90, 0.90; 14500 x 2560 0.82, 0.88; 22016 x 1024 0.76, 0.83; 57344 x 1280 0.84, 0.86.
inline bool wide_tiled_decode_preferred(int n, int k, int cus)
{
    const int unit = cus;
    if (k < 1024)
        return false;
    return k == 1024 || (n >= 16 * unit && n <= 36 * unit && k <= 2048) || (n >= 56 * unit && n <= 96 * unit && k <= 2560) ||
           (n > 100 * unit && k <= 1280);
}

// MXFP4, K % 128 == 0.  Figures, from three rows on: us per launch, tiles -> blocks, or blocks as a part of what the tiles take.
inline bool wide_preferred(const TileCall& c)
{
    const int m = c.m, n = c.n, k = c.k, unit = c.cus, passes = (m + 15) / 16;
    const bool plain = !c.fused && !c.pick;
    if (m < 3)
        return c.tiled && c.fits && (m == 2 || c.fused) && wide_tiled_decode_preferred(n, k, unit);
    if (c.fits) {
        // Beyond 16 rows always: 12288 x 4096 at 32 rows 19.9 -> 10.1, 22016 x 4096 at 64 57 -> 19.
        if (m > 16)
            return true;
        if (m <= 8)
            return wide_one_pass_preferred(c);
        // Nine to 16: the tiles' passes of 16 rows have fewer waves in flight.  One tile per unit: K = 128 to 1024 0.86 to 0.94, 1536 1.03,
        // 2048 0.98, 2560 1.0, 3072 0.92, 4096 0.89; tile-major 0.87 to 0.97, 1.07, 1.02, 0.95, 0.96, 0.98.
        if (n <= 16 * unit)
            return k <= 1024 || (k > 2560 && !(c.tiled && c.fused));
        // 18432 x 3584 0.96, x 4096 0.98; beyond 128 rows per unit K = 3072 0.97, 3584 0.97, 3712 to 4096 1.07, 4224 to 4608 0.94;
        // tile-major never more than 0.98.
        return n <= 128 * unit || c.tiled || k <= 3584 || k > 4096;
    }
    if (m <= 8) {
        // (57344 x 10240 and 32000 x 11008 tile-major at five and eight rows 0.76 of K split; row-major 1.04)
        if (n > 96 * unit)
            return c.tiled && c.split && m > 4 && k <= 11264;
        // Plain products: K in phases inside a tile kernel, which walks one tile per unit as fast as a block and
        // starts earlier: 4096 x 11008 at 8 rows 12.4 -> 11.7, 4096 x 28672 18.9 -> 22.8 at three; tile-major 1000 x 28672
        // 15.0 -> 19.9.  Every further tile fetches the rows again: 12288 x 14336 at 5 rows 0.74 of it.
        if (plain && (n <= 16 * unit || !c.split))
            return n <= 16 * unit ? m > 4 && k <= (c.tiled ? 11264 : 14336) : c.tiled ? m > 3 || k <= 28672 : m > 4 || k <= 20480;
        // No workspace: narrower passes over the weights (five rows and more 0.6 to 0.9 of them, but 18432 x 24576 at 8
        // rows 1.12; at three and four rows 0.9 to 1.2).
        if (!c.split)
            return m > 4 && (n <= 48 * unit || k <= 14336);
        // K split: 8192 x 11008 at 5 rows 0.87 of it, 12288 x 28672 1.0, 18432 x 11008 1.07; pick 1000 x 20480 1.12;
        // tile-major pick 256 x 11008 1.07, 1000 x 11008 1.04 (taken all the same, so that it gives the row-major pick's
        // bits), 1000 x 14336 1.13, 8192 x 20480 0.84, 16384 x 32768 1.06.
        if (c.tiled)
            return k <= (n <= unit ? 10240 : n < 16 * unit ? 11264 : n < 24 * unit ? 16384 : 20480);
        return m > 4 && n <= 64 * unit && k <= 14336 && !(c.fused && n < 4 * unit);
    }
    // No workspace (row-major): narrower passes of eight or four rows, 0.3 to 0.8 of them.
    if (!c.split)
        return m > 16 || (n <= 96 * unit && k <= 16384);
    // One pass of K split over the units: at 16 rows 4096 x 11008 0.83 of it, 256 x 14336 1.13, 5000 x 11008 1.05, 18432 x 12288
    // 1.05, 1414 x 10880 0.80, 5782 x 11264 0.74, 32000 x 5120 0.70, x 7168 0.81, x 8192 1.0, x 10240 0.91, 31892 x 11392 0.89, 29836 x 8448 0.74; tile-major 1000 x 10240 1.07, 2048 x 14336 1.08, 4096 x 20480 1.03, 16384 x 28672 1.09, 24000 x 65536 0.94.
    if (passes == 1 && c.tiled)
        return n > 64 * unit ||
               k <= (n < 5 * unit ? 8192 : n < 8 * unit ? 10240 : n < 16 * unit ? 12288 : n < 32 * unit ? 16384 : 20480);
    if (passes == 1)
        return (n <= 96 * unit && (n <= 64 * unit || n >= 84 * unit) &&
                k <= (n < 5 * unit || (n > 16 * unit && n <= 20 * unit) ? 10240
                      : n < 8 * unit                                    ? 12288
                      : n > 16 * unit && n < 32 * unit                  ? 11520
                                                                        : 14336)) ||
               (n > 64 * unit && (k <= 7680 || (k > 8192 && k <= (n > 84 * unit ? 11520 : 10240))));
    // Several passes: each of them streams the weights again, so the line moves with their number.  At 17 to 32
    // rows 256 x 24576 1.0 of them, 256 x 65536 1.9, 500 x 32768 1.19, 1500 x 49152 1.14, 3000 x 65536 1.09, 4096 x 65536 0.84;
    // tile-major 64 x 20480 1.14, 64 x 65536 2.5, 1000 x 28672 1.05, 1500 x 49152 1.14; at 64 rows 16 x 65536 1.2, 1.6.
    int pass = 0x7FFFFFFF / passes;
    if (c.tiled)
        pass = n <= 2 * unit ? 8192 : n <= 4 * unit ? 12288 : n < 8 * unit ? 16384 : n < 12 * unit ? 24576 : pass;
    else
        pass = n <= unit ? 10240 : n <= 2 * unit ? 12288 : n < 16 * unit ? 16384 : pass;
    return k <= passes * pass;
}

// K that is no multiple of 128, from three rows on, where the vector ALUs take passes of two rows: 4096 x 1376 at 7 rows
// 18.7 -> 5.0.  Three rows of a handful of weight rows, or of up to four per unit with a long K, stay there while
// two rows fit the LDS (1 x 8224 6.8 -> 7.6, 256 x 28704 20.3 -> 21.9, 1000 x 40992 0.78 of it).
inline bool wide_ragged_preferred(int m, int n, int k, int cus, int lds_bytes)
{
    if (m == 3 && 4 * k <= lds_bytes && (n < 8 ? k > 4096 : n <= 4 * cus && k > 16384))
        return false;
    return m >= 3;
}

// The other formats, K % 128 == 0.  `bits` per element; `tiles`: the call's rows fit the LDS whole on the tile kernels (of
// 6 and 8 bits; the ternary codes run on the vector ALUs); `e2m3`: that 6-bit format, which has no vector ALU kernel for few weight rows.
inline bool wide_format_preferred(int m, int n, int k, int bits, bool e2m3, bool tiles, int cus, int lds_bytes)
{
    const int unit = cus;
    // Beyond 16 rows always (E4M3 12288 x 4096 at 32 rows 33 -> 19, E2M3 27 -> 19).
    if (m > 16)
        return true;
    // One and two rows of E2M3 where the tiles ran: blocks 0.81 of their time at K = 384, 0.87 at 1024, 0.93 at 4096, 0.92 at 8192, picks 0.90
    // to 0.96; the rms error of the FP32 sums 0.5 to 0.98 of theirs (K = 128 1.2, 256 0.9 to 1.1; 16 to 100 weight rows up to 1.09).
    if (m < 3)
        return e2m3 && n > unit && n < 8 * unit && k >= 384 && k <= 8192;
    // The ternary codes went over the weights once per four rows (22016 x 4096 at 8 rows 51 -> 17).  In one such pass, up
    // to eight weight rows per unit, the vector ALUs are faster from K = 4224 (1024 x 4096 0.95, 1000 x 8192 at four rows 1.14 of them) until
    // a unit has room for one copy of the four rows only (1000 x 12288 0.89); a short K leaves nothing but
    // the start of the blocks, once per tile of many (24000 x 128 1.28, 24000 x 512 1.07, 24000 x 768 0.52).
    if (bits == 2) {
        if (m > 4)
            return true;
        if (n <= 8 * unit)
            return ((m == 4 || n >= 4 * unit) && (k <= 2048 || 16 * k > lds_bytes)) || (n >= 4 * unit && k <= 4096);
        return n <= 16 * unit || k >= 768;
    }
    // Rows that do not fit ran as passes of four (E4M3 4096 x 11008 at 16 rows 55 -> 17).
    if (m >= 5 && !tiles)
        return true;
    // Else while a unit has few tiles, the 8-bit elements from five rows on: 8192 x 4096 0.57 to 0.78 of the tiles, 8448 to 12288 x 2560
    // 0.87, x 3072 0.98, x 3584 0.95, x 4096 0.88, x 4608 0.91, x 6912 1.09, 12544 to 16384 x 4608 0.83; many weight rows with a short K: 20480 x 2048 0.80, x 3072 1.09, 57344 x 2048 0.95.  Three
    // and four rows: 1024 x 3072 1.14, 2048 x 1024 0.86, x 4096 0.96, 4096 x 8192 0.75, 8192 x 3072 0.79, x 11008 1.10, 9216 x 2048
    // 0.85, x 3072 1.06, 20480 x 2048 0.90, 57344 x 2048 0.97; 8192 x 4096 0.91, x 6144 0.92.
    if (bits == 8 && m <= 4)
        return n > 4 * unit && k <= (n <= 8 * unit ? 1024 : n <= 32 * unit ? 7168 : 2048);
    if (bits == 8)
        return n <= 32 * unit || k <= 2048 || (n <= 64 * unit && k <= 4608);
    // 6-bit: 8192 x 4096 0.75 of the tiles, 8448 to 12288 x 3072 0.93 to 0.98, x 3584 0.98, x 4096 1.04, just past the groups x 4352 0.89 to 0.93,
    // x 4864 0.95, x 5632 1.07, 16384 x 6144 0.96, 20480 x 2560 1.0, x 3072 1.01 to 1.08, 24576 x 3072 0.98, 57344 x 2048
    // 0.85, x 2560 0.97 to 1.1; three and four rows not where N is small and K is not (1024 x 1024 0.87, 896 x 4864 1.04) or K is
    // long (3072 x 16384 1.06), where the decode kernel takes passes of two again from where four rows do not fit (2048 x
    // 24576 0.9, 8192 x 24576 0.6).
    if (n < 8 * unit)
        return m >= 5 || k <= 1024;
    if (m <= 4 && 8 * k > lds_bytes)
        return n <= 40 * unit;
    if (n <= 32 * unit)
        return m >= 5 || k <= 12288;
    if (n <= 48 * unit)
        return k <= 3584 || (k > 4096 && k <= 5120);
    return k <= (n <= 64 * unit ? 6144 : n <= 80 * unit ? 2560 : n <= 128 * unit ? 3072 : 2048);
}

// BF16 weights.  `tiles`: the matrix-core tiles could take a call of nine to 16 rows in one pass.
inline bool wide_bf16_preferred(int m, int n, int k, bool tiles, int cus, int lds_bytes)
{
    const int unit = cus;
    // One and two rows with a short K, products and picks, as a part of the decode kernel's time: one row 4096 x 384 1.05, 5000 x 384 0.95, x
    // 1152 1.09, 8192 x 1024 0.86, 9216 x 1024 0.98, 12288 x 1024 0.87, 20000 x 1024 0.95, x 1152 1.04, 28000 x 512 0.63, x 1024 0.82; two rows 2048 x
    // 384 1.06, 3000 x 384 0.97, x 512 1.02, 5000 x 768 0.95, 7000 x 1024 0.97, 9216 x 512 0.90, x 768 1.02.  Only where the FP32 sums are no further from 64
    // bits: one row 0.86 to 1.01 of the decode kernel's rms error, but beyond 64 rows per unit K = 128 1.07 to 1.12, 256 1.02 to 1.3; two rows up to
    // 36 per unit 0.92 to 1.01, 28000 x 256 1.24, x 384 1.02, 57344 x 128 1.07.
    if (m == 1)
        return n > 16 * unit && k <= (n < 32 * unit ? 384 : 1024) && (n <= 64 * unit || k >= 384);
    if (m == 2)
        return n > 8 * unit && n <= 36 * unit && k <= (n <= 16 * unit ? 384 : n <= 28 * unit ? 1024 : 512);
    // Beyond 16 rows always (12288 x 4096 at 32 rows 41 -> 26, 4096 x 11008 98 -> 30).  Nine to 16 rows that the tiles
    // cannot take (4096 x 11008 at 16 rows 49 -> 25, 5001 x 2056 20 -> 11), or that leave the units few of them while K is
    // whole pairs of phases (4096 x 4096 0.93 of the tiles, x 2048 0.89, 2048 x 2048 1.0, 4096 x 512 1.07), or 17 to 32 or 49 to 64 rows
    // per unit (5120 x 1024 0.92, x 3072 0.94, 8192 x 512 0.93, x 3072 0.92, 16384 x 1024 0.92, x 2048 0.93, x 4096 1.0), or a short K (12288 x 512
    // 0.94, x 768 0.97 to 1.02, x 1536 1.07, x 2304 1.01, x 3072 1.05; 20480 x 512 1.09) or a single pair of phases (12288 x 2048 0.93).
    if (m > 16)
        return true;
    if (m > 8)
        return !tiles || (k % 2048 == 0 && n >= 12 * unit && n <= 16 * unit) || (n > 16 * unit && n <= 32 * unit) ||
               (n > 32 * unit && n <= 64 * unit && (k <= 512 || k == 2048 || n > 48 * unit));
    // Five to eight rows of a matrix of middling size, against the vector ALUs in one pass: 4096 x 4096 at 8 rows 0.88 of
    // them, 8192 x 4096 0.77, x 5120 0.97, but 2048 x 5120 1.0 to 1.22, 8192 x 6144 1.09, 10240 x 2048 1.13, 22016 x 4096 37 -> 41.
    // Rows that just fit the LDS stay (4096 x 10240 at 8 rows 1.03, 8192 x 10240 1.18); those that do not ran in phases
    // (4096 x 16384 0.74 of them, 8192 x 16384 1.1).
    // A short K, where the start of a pass is most of it: three rows 4096 x 512 0.84, 12288 x 512 0.82, 57344 x 512 0.97; four 4096 x
    // 1536 0.84, 12288 x 1024 0.87, 57344 x 512 0.79; five to eight 2048 x 2048 0.85, 12288 x 1024 0.74, 32000 x 1024 0.73.
    if (m < 5)
        return n > 12 * unit && k <= (m == 3 || n > 64 * unit ? 512 : n > 32 * unit ? 1024 : 1536);
    if (n <= 8 * unit)
        return n >= 6 * unit && k <= 2048;
    if (n > 40 * unit)
        return k <= 1024;
    const bool phased = m > 6 && 16 * k > lds_bytes;
    if (n <= 16 * unit)
        return k <= (m > 6 ? 9216 : 8192) || phased;
    return k <= (n > 32 * unit ? 1024 : n > 20 * unit ? 5120 : 2048) || (phased && n <= 20 * unit);
}

// Workgroups per compute unit of a vector-ALU pass of `rows` BF16 rows: as many copies of the rows as the LDS holds, up to
// four (of four waves each, two of eight, one of 16).  Five rows and more of a long K take two where the
// matrix is not short (12288 x 4096 at five rows 20.5 us, 21.6 with three; but 1000 x 2048 at eight 7.2, 6.3 with four), three
// rows that would take three take two, 16 waves instead of 12 (4096 x 7168 12.6 us, 14.8 with three).
inline int bf16_workgroups_per_unit(int rows, int n, int k, int cus, int lds_bytes)
{
    const int bytes = rows * k * 2, fit = lds_bytes / (bytes < 256 ? 256 : bytes);      // (a pick needs a few bytes)
    const int most = rows > 4 && k > 2048 && n >= 8 * cus ? 2 : rows == 3 && fit == 3 ? 2 : 4;
    return fit < 1 ? 1 : fit < most ? fit : most;
}

}  // namespace mxfp4

// Which scale dwords a thread of the block kernel (gemm_wide.h) asks for and where it puts them in the LDS.  Plain
// integer arithmetic without any device header, so that the map can be walked on the CPU for every block shape.
//
// A block of `bn` weight rows holds bn x 2 WK dwords at a time (four scale bytes per row and step of 128, the steps of
// two phases).  They are dealt to the threads in order; where their number is no multiple of the threads, the threads
// that are left over in the last round own none: they ask for an offset past the descriptor and store nothing.
// Every dword in the LDS has one writer.
#pragma once

namespace mxfp4 {
namespace wide {

constexpr int kThreads = 512;

// Scale bytes of a block's weight rows for two phases, one row behind the other with a dword of padding
// (the rows of an operand read hit different banks).
constexpr int scale_row_bytes(int wk) { return wk * 8 + 4; }

// Rounds in which the threads fetch a block's dwords.
constexpr int scale_rounds(int bn, int wk) { return (bn * wk * 2 + kThreads - 1) / kThreads; }

// Dword of thread `tid` in round `i`: the row in the block and the step in the two phases.
constexpr int scale_index(int tid, int i) { return tid + i * kThreads; }
constexpr bool scale_owned(int bn, int wk, int tid, int i) { return scale_index(tid, i) < bn * wk * 2; }
constexpr int scale_row(int wk, int tid, int i) { return scale_index(tid, i) / (wk * 2); }
constexpr int scale_step(int wk, int tid, int i) { return scale_index(tid, i) % (wk * 2); }
constexpr int scale_lds(int wk, int tid, int i)
{
    return scale_row(wk, tid, i) * scale_row_bytes(wk) + scale_step(wk, tid, i) * 4;
}

// Byte offset of weight row `row` (past the last one: the last row, or the same row of the last tile), first step, and
// what step `step` of all of K adds.  The tile-major copy: 16 rows x four steps per 256 bytes.
constexpr int scale_row_offset(bool tiled, int row, int n, int blocks_k, int n_tiles, int n_items)
{
    const int tile = (row >> 4) < n_tiles ? row >> 4 : n_tiles - 1;
    return tiled ? (tile * n_items * 16 + (row & 15)) * 16 : (row < n ? row : n - 1) * blocks_k;
}
constexpr int scale_step_offset(bool tiled, int step) { return tiled ? (step >> 2) * 256 + (step & 3) * 4 : step * 4; }

}  // namespace wide
}  // namespace mxfp4

// Which kernel takes which list: rules on sizes, ranks and what the plans counted, apart from the kernels so that the host can be asked alone.
#pragma once

#include "tensor.hpp"

namespace comet {

// SpMM and TTM at ranks 8 and 16: the walk over whole tiles of nonzeros (k_stream_rankR), or the pieces, which take all other ranks.
constexpr int64_t kWalkNnz = int64_t(10) << 20;            // nonzeros from which on the walk is taken at all
inline bool segreduce_takes_walk(const Schedule &sc, int64_t R) {
    const int64_t n = sc.nnz;
    const PiecePlan &p = sc.pieces;
    if ((R != 8 && R != 16) || n < kWalkNnz) return false;
    if (p.ntiles == 0) return true;                        // there was no memory for the plan of the pieces
    // Very many nonzeros in short segments, of which the walk keeps more in flight.  Whole calls on the walk and on the pieces, rank 16, us:
    // TTM on 100 M (35 M of them, 5 per fiber, off the sweep) 667 and 700; 30 M at random, 7.5 per fiber, 347 and 356, 4 per fiber 420 and
    // 420.  15 M, 5 and 2.5 per fiber, 212 and 205, 281 and 266.
    if (n <= 8 * sc.nseg) return R == 16 && n >= int64_t(24) << 20;
    // Longer segments: the pieces gain where every part of the list has operand rows of its own (banded matrices: 12 M, 12 per row, rank 16, 229
    // and 137) or where the rows come from behind the L2 (11 M, 16 per row in 300 000 columns, 216 and 209), and lose where the list goes on
    // using the same rows, which the L2 then holds, and segments differ in length, so that some are cut up:
    //   rank 16   20 per row, 30 000 columns: 11 M 100 and 112, 40 M 328 and 385; 60 000 (7.6 MB of rows) 434 and 451, 120 000 610 and 603 at 16 per row;
    //             150 per row 277 and 303; columns that follow a power law (58 000 in a sample), 34 M, 290 and 357, 22 M in rows of 9, 203 and 213;
    //             every row 9 long: 24 M 253 and 231, 16 long: 200 and 201
    //   rank 8    20 per row, 30 000 columns: 11 M 90 and 91, 24 M 181 and 190, 40 M 295 and 309; 9 per row, power-law rows and columns, 19 M, 149 and 169; 120 000, 16 per row, 458 and 444; power-law
    //             columns, 31 M, 258 and 287; 32 per row 281 and 269; 150 per row 262 and 242; every row 20 long 292 and 248
    if (p.common < 0.75) return false;
    if (R == 16) return p.distinct <= 78000 && 512 * p.njoins >= sc.nseg;
    return n <= 28 * sc.nseg && p.distinct <= 67000 && 200 * p.njoins >= sc.nseg;
}

}  // namespace comet

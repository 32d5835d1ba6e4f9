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
    // TTM on 100 M (35 M of them, 5 per fiber, off the sweep) 669 and 700; 30 M at random, 7.5 per fiber, 347 and 356, 4 per fiber 420 and
    // 420.  15 M, 5 and 2.5 per fiber, 212 and 205, 281 and 266.
    if (n <= 8 * sc.nseg) return R == 16 && n >= int64_t(24) << 20;
    // Longer segments: the pieces gain where every part of the list has operand rows of its own (banded matrices: 12 M, 12 per row, rank 16, 229
    // and 137), where the rows come from behind the L2 (11 M, 16 per row in 300 000 columns, 216 and 209) and where there is little but short segments or little but
    // long ones (TTM over power-law fibers, 20 M, rank 8, 170 and 155).  They lose where the whole list uses the same rows, which the L2 then holds, and
    // segments of middle lengths differ: the pieces of a tile fill the lane groups' last turn badly.
    //   rank 16   20 per row, 30 000 columns: 11 M 100 and 112, 40 M 328 and 385; 60 000 (7.6 MB of rows) 434 and 451, 120 000 610 and 603 at 16 per row;
    //             150 per row 277 and 303; columns that follow a power law (58 000 in a sample), 34 M, 290 and 357; 9 per row, 22 M, 203 and 213;
    //             every row 9 long: 24 M 253 and 231, 16 long: 200 and 201
    //   rank 8    20 per row, 30 000 columns: 11 M 90 and 91, 24 M 181 and 190, 40 M 295 and 309; 120 000, 16 per row, 458 and 444; power-law rows and
    //             columns, 31 M, 258 and 287, 19 M, 9 per row, 149 and 169; 32 per row 281 and 269; 150 per row 262 and 242; every row 20 long 292 and 248
    // The lines are those that left fewest of 3200 calls on random lists (three kinds of lengths, uniform and power-law columns, TTM of power-law tensors) with the
    // slower kernel: 6 are more than 3 % slower than on the pieces, the worst 1.04 times; 59 than on the walk, most of them by 3 to 6 %.
    const int64_t whole = sc.nseg - p.njoins, in_parts = 30 * (p.npieces - whole);      // segments in one piece; nonzeros of the others, about
    // a power-law mode: samples share their frequent coordinates and not the rest
    const bool power = p.common <= 0.985 && p.distinct <= 72000;
    if (p.common < 0.72 || p.distinct > (p.common <= 0.8 || R == 8 ? 92000 : 85000)) return false;
    if (R == 8) return 100 * in_parts <= (power ? 48 : 42) * n && (30 * p.njoins >= sc.nseg || (power && n >= 8 * p.npieces && 90 * p.njoins >= sc.nseg));
    if (power && 100 * in_parts >= n && (n >= 8 * p.npieces || (n >= int64_t(19) << 20 && 2 * n >= 5 * p.npieces))) return true;
    return 1000 * in_parts >= n && 10 * (n - in_parts) >= 33 * whole && (2 * n >= 19 * p.npieces || (n >= int64_t(24) << 20 && 2 * n >= 17 * p.npieces));
}

// MTTKRP, lists and ranks that do not take the pieces: the wavefronts over blocks of nonzeros (k_mttkrp_wave), or the walk over nonzeros (k_stream_mttkrp).
// The wavefronts read a row of B once per fiber and block where the walk reads one per nonzero (ranks up to 16) or per fiber; they read rows 16 bytes per
// lane at every even rank (8 at odd ones), the walk only at ranks 8, 16, 32, 48, 64, 96 and 128, and they take 16 or 32 columns at a time, so that they read
// the list, and the lines in which rows begin and end, once for each.  What that gives is decided by where the rows of C come from: while a compute
// unit's and an XCD's caches hold them, the fewer loads count; where they come from behind the L2 the lines do, and the walk has more loads in flight.
//   c      different rows of C in 32768 nonzeros: power-law modes 1300 to 10 000, uniform ones of 3000 / 8000 / 15 000 / 30 000 / 300 000 rows 3000 / 7900 /
//          13 300 / 19 900 / 31 000.  b: different rows of B in 32768 fibers.  slice: most nonzeros of a slice; a block in which a slice ends
//          costs more, so that lists of short slices gain less.
// Calls on the walk and on the wavefronts, us, 44 M nonzeros; power: all modes, 3.6 per fiber; the others uniform, in slices of 25 fibers, and
// most of the 2 M rows of M cleared:
//         power        2.2 per fiber  5 per fiber  3 per fiber  3 per fiber  5 per fiber  6 per fiber
// rank    c 4000       c 3000         c 7900       c 13 300     c 19 900     c 25 300     c 31 000
//     9     782   662    802   762    736   657    760   703    783   744    766   766   1160  1194
//    10     783   537    809   641    747   583    768   581    793   688    792   834   1189  1240
//    15     812   735    918   900    838   796    876   849   1012  1074   1197  1275   1579  1658
//    16     513   460    570   571    514   502    544   541    639   683    727   773    972   986
//    20    1368   816   1338   963   1241   883   1329   951   1381  1320   1438  1474   1722  1828
//    32     985   844   1024  1019    946   922   1092  1136   1598  1690   1630  1720   1844  1897
//    34    2060  1754   2027  2137   1866  1930   2011  2448   2355  3687   2379  3863   2627  4434
//    40    2064  1569   2035  1872   1931  1734   2027  1910   2488  2954   2464  3158   2771  3739
//    62    2838  2135   2897  2521   3102  2521   3462  3778   4235  5053   4056  4988   4394  5287
//    64    1694  1669   1827  1984   1976  1832   3016  2299   3689  3373   3534  3425   3728  3784
//    96    2553  2504   2944  2990   3492  2747   5113  3872   5850  5849   5440  5645   5623  6071
//   128    4206  3318   4675  3977   5268  3709   7165  4595   7902  6746   7337  6973   7390  7644
// Rank 16: 150 M, power, 1602 and 1393; 2 per fiber, c 13 000, b 32 000, 633 and 647.  Rank 32: 2 per fiber, c 7900, 1131 and 1166.  Rank 40: 2 per fiber, c 7900, b 28 000,
// 1862 and 2115.  Rank 64: 20 M, power, 772 and 753.  3 M, 5 per fiber, c 25 300: rank 20 1.12 times as fast, 30 1.02.
// The lines below left few of 13 200 calls on random lists (uniform and power-law modes, 2 to 30 nonzeros per fiber, 2 to 10^5 fibers per slice, 1.2 M to
// 45 M nonzeros) with the slower kernel: 270 are more than 2 % slower than on the walk, and 3770 were with lines on sizes and ranks alone.
inline bool mttkrp_takes_wave(const Schedule &sc, int64_t R) {
    const int64_t n = sc.nnz, f = sc.nseg, c = sc.pieces.few, b = sc.pieces.parent_few, slice = sc.max_parent_len;
    constexpr int64_t Mi = int64_t(1) << 20;
    if (n < 2 * f || R <= 8) return false;                 // a row of B for almost every nonzero either way; rows of 64 bytes
    if (R < 16) {
        if (n < 5 * Mi) return false;
        if (R % 2 == 0) return c <= (n >= 6 * f ? 26000 : 22000);
        return c <= (R < 13 ? 22000 : 16000) && (4 * n >= 11 * f || n >= 11 * Mi || (slice >= 4096 && slice < Mi / 2));
    }
    if (R == 16) return n >= 40 * Mi && c <= 22000 && slice >= 4096 && (8 * n >= 21 * f || slice >= Mi / 4);
    if (n > 8 * f) return false;                           // the walk, too, loads few rows of B
    if (R % 32 == 0) {
        if (n < 10 * Mi) return false;
        if (R == 32) return c <= 12000 && slice >= 6144 && (b <= 32000 || 2 * n >= 5 * f);
        if (R == 64) return c <= 28500 && (c > 7800 || (2 * n <= 9 * f && slice >= Mi / 4));
        if (R == 96) return c <= 20500 && (c > 5050 || (c > 3050 && n <= 5 * f) || slice >= Mi);
        return R == 128 && c <= 28500 && (c > 3050 || 4 * n <= 11 * f || slice >= Mi / 4);
    }
    if (R % 2 || R > 64 || R == 48) return false;
    if (R < 32) return 2 * n >= 5 * Mi && (c <= (R <= 24 ? 22000 : 17000) || n < (R <= 24 ? 4 : 5) * Mi);
    if (n < Mi) return false;
    const bool long_slices = slice >= 1 << 14, thick = long_slices || 8 * n >= 17 * f;
    if (R == 56) return c <= 14000 && (slice >= 40 || 2 * n <= 7 * f);
    if (R == 40) return slice >= 128 && thick && (c <= 7900 || (c <= 13600 && (long_slices || (b <= 28000 && 2 * n >= 5 * f))));
    if (R >= 50) return thick && c <= (slice >= 1 << 15 ? 13600 : 11200) && (slice >= 70 || 2 * n <= 7 * f);
    // rows that begin and end inside lines, in three blocks of columns: power-law modes only, and short lists
    const bool power = 32 * slice >= n || (b <= 12000 && slice >= 20000), several = 8 * n >= 17 * f;
    if (R % 4 == 0)
        return b <= 32200 && ((c <= 13600 && power) || (c <= 11200 && n < 6 * Mi && slice >= 74 && several) ||
                              (c <= 9000 && slice >= 3072 && 2 * n >= 5 * f && b <= 17500));
    return (c <= 11700 && b <= 28800 && power) || (c <= 7900 && n < 3 * Mi && slice >= 104 && several);
}

}  // namespace comet

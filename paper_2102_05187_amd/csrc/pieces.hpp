// Piece plan of a compressed level: how the rank-R kernel takes its segments (built once per tensor, pieces.hip).
//
// The level is cut into tiles of `units` units -- a nonzero is a unit and a segment is one, so that a tile is the same
// work whether it holds one long segment or hundreds of single nonzeros.  Inside a tile the segments become pieces of
// at most kWhole nonzeros, sorted by length: the lane groups of a wavefront then walk pieces of (almost) equal length
// side by side, and no nonzero asks whether a segment ends behind it.  A piece that is a whole segment writes its result
// row; the sums of the pieces of a longer or cut segment meet in LDS (a join).  Segments cut by a tile boundary are
// finished by a small kernel that works off a list.  The nonzeros themselves stay where the caller has them.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "tensor.hpp"

namespace comet {

// Units per tile, and how the nonzeros are read.  Small tiles leave room for more workgroups per compute unit (LDS), which
// hides the latencies at the start of a tile; that wins while the nonzeros (12 bytes each) are still in the caches from the
// pass before.  A list that is not would only push the operand out of them: from kStreamNnz on its loads are non-temporal.
// TTM at rank 32, 8 M nonzeros in 1.6 M fibers: 177 us, and 192 with plain loads, where four tensors take turns; 184 and 147
// where one is used again and again; 6 M: 137 and 141, 136 and 112.  15 M: 318 and 352, 317 and 275.
// Large tiles end at 1472 units so that a tile full of pieces of long segments leaves room for two workgroups per compute
// unit at rank 128 (1536 units did not: SpMM on 13 M nonzeros in power-law rows 2043 us, now 1940; rank 112 1820 and 1665).
constexpr int kUnitsSmall = 768, kUnitsLarge = 1472;
constexpr int64_t kStreamNnz = int64_t(7) << 20;
constexpr int kWhole = 48;             // longest segment that is taken as one piece
constexpr int kPiece = 32;             // longest piece of any other segment
constexpr int kSnap = 32;              // a tile boundary inside a segment of at most this many nonzeros moves to its start

// Most nonzeros, pieces and pieces that are not whole segments in a tile.  The last: n > kWhole nonzeros become at most
// 3 n / 65 pieces (65 make 3), a cut segment at either end of the tile at most one more than that.
__host__ __device__ constexpr int tile_items(int units) { return units + kSnap + 1; }
__host__ __device__ constexpr int tile_pieces(int units) { return units + kSnap + 1; }
__host__ __device__ constexpr int tile_parts(int units) { return 3 * tile_items(units) / 65 + 3; }
static_assert(kWhole == 48 && kPiece == 32, "tile_parts");

// piece: start in the tile (11 bits), length (6), number (11), flag (1).  The number is the segment's number in the tile
// for a whole segment, else the piece's slot among the partial sums (and the flag is set).
static_assert(tile_items(kUnitsLarge) < 2048 && kWhole < 64, "fields of a piece");
__host__ __device__ inline unsigned piece_pack(int start, int len, int num, int part) {
    return (unsigned)start | ((unsigned)len << 11) | ((unsigned)num << 17) | ((unsigned)part << 28);
}
__device__ __forceinline__ int piece_start(unsigned p) { return (int)(p & 2047u); }
__device__ __forceinline__ int piece_len(unsigned p) { return (int)((p >> 11) & 63u); }
__device__ __forceinline__ int piece_num(unsigned p) { return (int)((p >> 17) & 2047u); }
__device__ __forceinline__ bool piece_is_part(unsigned p) { return (p >> 28) & 1u; }

// join: first slot (7 bits), slots (7), segment's number in the tile (11), where the sum goes (2)
static_assert(tile_parts(kUnitsLarge) < 128, "fields of a join");
enum JoinTo { kJoinRow = 0, kJoinHead = 1, kJoinTail = 2 };
__host__ __device__ inline unsigned join_pack(int slot, int n, int seg, int to) {
    return (unsigned)slot | ((unsigned)n << 7) | ((unsigned)seg << 14) | ((unsigned)to << 25);
}
__device__ __forceinline__ int join_slot(unsigned j) { return (int)(j & 127u); }
__device__ __forceinline__ int join_count(unsigned j) { return (int)((j >> 7) & 127u); }
__device__ __forceinline__ int join_seg(unsigned j) { return (int)((j >> 14) & 2047u); }
__device__ __forceinline__ int join_to(unsigned j) { return (int)(j >> 25); }

// Builds the plan for a level of nseg segments over nnz nonzeros with coordinates crd; parent: coordinates of the segments, if they are
// to be sampled too, else null.  Synchronises with st.
hipError_t piece_plan_build(const int32_t *pos, int64_t nseg, const int32_t *crd, int64_t nnz, const int32_t *parent, PiecePlan &plan, hipStream_t st);

}  // namespace comet

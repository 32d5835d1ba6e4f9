// Plan of the MTTKRP kernel for a [CU,CU,CU] tensor (built once per tensor, mttkrp_plan.hip).
//
// The leaf level is cut into tiles of `units` units, a nonzero and a fiber being a unit each, so that a tile is about the
// same work whatever the lengths of its fibers.  Inside a tile the fibers become pieces of at most kMtWhole nonzeros,
// sorted by length: the lane groups of a wavefront walk pieces of (almost) equal length side by side and load their rows
// of B at the same time.  The sum of piece number n in fiber order goes to row n of a table in LDS, so that the pieces of
// a slice are neighbours there; records say which of these rows make up which slice.  Slices cut by a tile boundary leave
// partial sums in memory, which a small kernel adds up.  The nonzeros themselves stay where the caller has them.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "tensor.hpp"

namespace comet {

// Lists of up to this many nonzeros have a plan (kernels_mttkrp.hip says which ranks use it).
constexpr int64_t kMtNarrow = int64_t(5) << 20;
// Units per tile: with 448 the items and sums of a tile take at most 39 KB of LDS at rank 16, so that four workgroups share a
// compute unit.  Short lists take smaller tiles, down to 128 units, so that there are about 1024 of them.
constexpr int kMtUnitsMin = 128, kMtUnitsMax = 448;
constexpr int kMtWhole = 16;           // longest fiber that is taken as one piece
constexpr int kMtPiece = 12;           // longest piece of any other fiber
constexpr int kMtSnap = 32;            // a tile boundary inside a fiber of at most this many nonzeros moves to its start
constexpr int kMtSum = 16;             // rows of sums that one lane group adds up at a time
// A fiber of n >= 1 nonzeros is n + 1 units and gives one piece, or n / 12 and a part of one; the fibers at either end may be cut.
constexpr int kMtItems = kMtUnitsMax + kMtSnap + 1, kMtPieces = kMtItems / 2 + 8;
static_assert(kMtPieces <= 256, "a thread holds one piece");

// piece {place, row of B}: start in the tile (10 bits), length (6), number in fiber order (9)
static_assert(kMtItems < 1024 && kMtWhole < 64 && kMtPieces < 512, "fields of a piece");
__host__ __device__ inline unsigned mt_piece(int start, int len, int slot) {
    return (unsigned)start | ((unsigned)len << 10) | ((unsigned)slot << 16);
}
__device__ __forceinline__ int mt_start(unsigned p) { return (int)(p & 1023u); }
__device__ __forceinline__ int mt_len(unsigned p) { return (int)((p >> 10) & 63u); }
__device__ __forceinline__ int mt_slot(unsigned p) { return (int)(p >> 16); }

// record {what, row of M}.  First the sums: first row (9 bits), rows (5), kind (2), rows of M in front of this one that are
// not stored (16, at most 65535).  A slice is one sum (kMtSlice), or several (kMtPart: the result replaces the first of its
// rows) followed by a join; kMtGap stands for unstored rows alone, those in front of the row it names.
enum MtKind { kMtSlice = 0, kMtPart = 1, kMtGap = 2 };
__host__ __device__ inline unsigned mt_sum(int first, int rows, int kind, int gap) {
    return (unsigned)first | ((unsigned)rows << 9) | ((unsigned)kind << 14) | ((unsigned)gap << 16);
}
__device__ __forceinline__ int mt_sum_rows(unsigned r) { return (int)((r >> 9) & 31u); }
__device__ __forceinline__ int mt_sum_kind(unsigned r) { return (int)((r >> 14) & 3u); }
__device__ __forceinline__ int mt_sum_gap(unsigned r) { return (int)(r >> 16); }
// Rows of M between two stored ones (from = -1: in front of the first); none where the coordinates do not increase.
__host__ __device__ inline int mt_gap(int64_t from, int64_t to) {
    const int64_t gap = to - from - 1;
    return gap < 0 ? 0 : (gap > 65535 ? 65535 : (int)gap);
}
// Then the joins: first row (9 bits), rows (9), whether the slice began in front of the tile, whether it goes on behind it.
__host__ __device__ inline unsigned mt_join(int first, int rows, bool cont, bool open) {
    return (unsigned)first | ((unsigned)rows << 9) | (cont ? 1u << 18 : 0u) | (open ? 1u << 19 : 0u);
}
__device__ __forceinline__ int mt_first(unsigned r) { return (int)(r & 511u); }
__device__ __forceinline__ int mt_join_rows(unsigned r) { return (int)((r >> 9) & 511u); }
__device__ __forceinline__ bool mt_join_cont(unsigned r) { return (r >> 18) & 1u; }
__device__ __forceinline__ bool mt_join_open(unsigned r) { return (r >> 19) & 1u; }

// tile {first nonzero, first piece, first record, joins}; pieces and records are counted without sign

// Builds the plan: slices pos2 / crd1 over fibers pos3 / crd2 over nnz nonzeros; dim0 = rows of M.  Synchronises with st.
hipError_t mttkrp_plan_build(const int32_t *pos2, const int32_t *crd1, int64_t nslice, const int32_t *pos3, const int32_t *crd2,
                             int64_t nfib, int64_t nnz, int64_t dim0, MttkrpPlan &plan, hipStream_t st);

}  // namespace comet

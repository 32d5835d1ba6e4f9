// Rank-1 kernels of the nonzero-tiled family (SpMV, TTV on CSF and on sorted coordinate lists), the
// carry fix-up kernels shared by all of them, and the host entry points of the family.
#include <atomic>

#include "pieces.hpp"
#include "routes.hpp"
#include "stream_common.hpp"

namespace comet {

namespace {


constexpr int kWaves = 4;                    // wavefronts per workgroup
constexpr int kWaveItems = kTile / kWaves;   // 1024 consecutive items per wavefront

// ---- DPP helpers (gfx9 controls: row_shr:n = 0x110+n, wave_shr:1 = 0x138, row_bcast:15 = 0x142,
//      row_bcast:31 = 0x143, quad_perm = 8-bit selector) ------------------------------------------
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_i(int old, int v) {
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_d(double old, double v) {
    int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), CTRL, ROW_MASK, 0xf, false);
    int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), CTRL, ROW_MASK, 0xf, false);
    return __hiloint2double(hi, lo);
}
// Same with every row and bank enabled and zero fill for lanes that have no source (bound_ctrl): the
// result does not depend on a previous register value, so no identity has to be materialised first.
template <int CTRL>
__device__ __forceinline__ int dpp0_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp0_d(double v) {
    int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double readlane_d(double v, int lane) {
    int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// Inclusive segmented scan over the 64 lanes.  Element = (f, v); combine(left, right) =
// (left.f | right.f, right.f ? right.v : left.v + right.v): a flagged element cuts the running sum.
__device__ __forceinline__ void segscan_inclusive(int &f, double &v) {
#define COMET_SCAN_STEP0(CTRL)                            \
    {                                                     \
        int nf = dpp0_i<CTRL>(f);                         \
        double nv = dpp0_d<CTRL>(v);                      \
        v = f ? v : nv + v;                               \
        f |= nf;                                          \
    }
#define COMET_SCAN_STEP(CTRL, RM)                         \
    {                                                     \
        int nf = dpp_i<CTRL, RM>(0, f);                   \
        double nv = dpp_d<CTRL, RM>(0.0, v);              \
        v = f ? v : nv + v;                               \
        f |= nf;                                          \
    }
    COMET_SCAN_STEP0(0x111)       // row_shr:1
    COMET_SCAN_STEP0(0x112)       // row_shr:2
    COMET_SCAN_STEP0(0x114)       // row_shr:4
    COMET_SCAN_STEP0(0x118)       // row_shr:8
    COMET_SCAN_STEP(0x142, 0xa)   // row_bcast:15 into rows 1 and 3
    COMET_SCAN_STEP(0x143, 0xc)   // row_bcast:31 into rows 2 and 3
#undef COMET_SCAN_STEP0
#undef COMET_SCAN_STEP
}

// ---- rank-1 walk ---------------------------------------------------------------------------------
// A wavefront owns 1024 consecutive items = 8 blocks of 128; in a block lane l holds items 2l, 2l+1
// (one 8-byte crd load and one 16-byte vals load per lane, consecutive lanes on consecutive bytes).
// The loads of four blocks are issued together, and the first four before the tail map is built, so
// the HBM latency overlaps the map construction and the scans of the preceding blocks.
struct Rank1Half {
    int2    c[4];
    double2 a[4];
};

__device__ __forceinline__ void rank1_load_half(Rank1Half &h, const int32_t *__restrict__ crd,
                                                const double *__restrict__ vals, int64_t base, int lane, int64_t nnz) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int64_t i0 = base + b * 128 + 2 * lane;
        if (i0 + 1 < nnz) {
            // streamed once: non-temporal, so the lines do not displace the gathered operand in L1/L2
            const long long cc = __builtin_nontemporal_load(reinterpret_cast<const long long *>(crd + i0));
            h.c[b].x = (int)(cc & 0xffffffffll); h.c[b].y = (int)(cc >> 32);
            h.a[b].x = __builtin_nontemporal_load(vals + i0);
            h.a[b].y = __builtin_nontemporal_load(vals + i0 + 1);
        } else {
            h.c[b].x = i0 < nnz ? crd[i0] : 0;   h.c[b].y = 0;
            h.a[b].x = i0 < nnz ? vals[i0] : 0.0; h.a[b].y = 0.0;
        }
    }
}

struct Rank1Carry {
    int    cf;     // a segment end was seen in the blocks done so far
    double cv;     // sum of the items after the last segment end
};

template <bool ROWMAP>
__device__ __forceinline__ void rank1_process_half(const Rank1Half &h, const double2 *xv, const int2 *tt,
                                                   int64_t base, int64_t nnz, int lane, int w,
                                                   const int32_t *__restrict__ rowmap, double *__restrict__ out,
                                                   Rank1Carry &cy, double *wsum_first, int *wsum_first_id,
                                                   const Epilogue ep = Epilogue()) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int64_t i0 = base + b * 128 + 2 * lane;
        const int2 t = tt[b];                                // segment ids of the items that end a segment, else -1
        const double p0 = i0 < nnz ? h.a[b].x * xv[b].x : 0.0;
        const double p1 = i0 + 1 < nnz ? h.a[b].y * xv[b].y : 0.0;
        const int f = (t.x >= 0) | (t.y >= 0);
        const double first = t.x >= 0 ? p0 : p0 + p1;
        const int first_id = t.x >= 0 ? t.x : t.y;
        const double open = t.y >= 0 ? 0.0 : (t.x >= 0 ? p1 : p0 + p1);
        if (t.x >= 0 && t.y >= 0) {                          // item i0+1 is a whole segment by itself
            const int64_t row = ROWMAP ? (int64_t)rowmap[t.y] : (int64_t)t.y;
            out[row] = ep_apply(ep, p1, out + row);
        }
        int sf = f;
        double sv = open;
        segscan_inclusive(sf, sv);
        // exclusive value for this lane = carry (+) inclusive value of the previous lane
        const int pf = dpp0_i<0x138>(sf);                    // wave_shr:1, lane 0 gets the identity (0, 0.0)
        const double pv = dpp0_d<0x138>(sv);
        const int ef = cy.cf | pf;
        const double ev = pf ? pv : cy.cv + pv;
        if (f) {
            const double value = ev + first;
            if (ef) {
                const int64_t row = ROWMAP ? (int64_t)rowmap[first_id] : (int64_t)first_id;
                out[row] = ep_apply(ep, value, out + row);
            } else {                                         // the first segment end of this wavefront's range
                wsum_first[w] = value;
                wsum_first_id[w] = first_id;
            }
        }
        const int tf = __builtin_amdgcn_readlane(sf, 63);
        const double tv = readlane_d(sv, 63);
        cy.cv = tf ? tv : cy.cv + tv;
        cy.cf |= tf;
    }
}

__device__ __forceinline__ void rank1_gather(const Rank1Half &h, const double *__restrict__ x, double2 *xv) {
#pragma unroll
    for (int b = 0; b < 4; ++b) { xv[b].x = x[h.c[b].x]; xv[b].y = x[h.c[b].y]; }
}

// Second part of the walk (after the map is complete); h0 holds the already issued first half.
template <bool ROWMAP>
__device__ __forceinline__ void walk_rank1(Rank1Half &h0, const int32_t *ts, const int32_t *__restrict__ crd,
                                           const double *__restrict__ vals, const double *__restrict__ x,
                                           const int32_t *__restrict__ rowmap, double *__restrict__ out, int64_t tb,
                                           int64_t nnz, int *wsum_ht, double *wsum_open, double *wsum_first,
                                           int *wsum_first_id, const Epilogue ep = Epilogue()) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t wb = tb + (int64_t)w * kWaveItems;
    Rank1Carry cy{0, 0.0};
    double2 xv[4];
    rank1_gather(h0, x, xv);
    Rank1Half h1;
    rank1_load_half(h1, crd, vals, wb + 512, lane, nnz);
    int2 tt[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) tt[b] = *reinterpret_cast<const int2 *>(ts + (wb - tb) + b * 128 + 2 * lane);
    rank1_process_half<ROWMAP>(h0, xv, tt, wb, nnz, lane, w, rowmap, out, cy, wsum_first, wsum_first_id, ep);
    rank1_gather(h1, x, xv);
#pragma unroll
    for (int b = 0; b < 4; ++b) tt[b] = *reinterpret_cast<const int2 *>(ts + (wb - tb) + 512 + b * 128 + 2 * lane);
    rank1_process_half<ROWMAP>(h1, xv, tt, wb + 512, nnz, lane, w, rowmap, out, cy, wsum_first, wsum_first_id, ep);
    if (lane == 0) { wsum_ht[w] = cy.cf; wsum_open[w] = cy.cv; }
}

// Combine the wavefront summaries of one tile in order and publish the tile summary.
template <bool ROWMAP>
__device__ __forceinline__ void finish_tile_rank1(const int *wsum_ht, const double *wsum_open, const double *wsum_first,
                                                  const int *wsum_first_id, const int32_t *__restrict__ rowmap,
                                                  double *__restrict__ out, CarryView cb, int64_t t,
                                                  const Epilogue ep = Epilogue()) {
    if (threadIdx.x != 0) return;
    int rf = 0, fid = -1;
    double rv = 0.0, tfirst = 0.0;
    for (int w = 0; w < kWaves; ++w) {
        if (wsum_ht[w]) {
            const double value = rv + wsum_first[w];
            if (rf) {
                const int64_t row = ROWMAP ? (int64_t)rowmap[wsum_first_id[w]] : (int64_t)wsum_first_id[w];
                out[row] = ep_apply(ep, value, out + row);
            } else {
                tfirst = value; fid = wsum_first_id[w]; rf = 1;
            }
            rv = wsum_open[w];
        } else {
            rv += wsum_open[w];
        }
    }
    cb.has_tail[t] = rf;
    cb.first_id[t] = fid;
    cb.first[t] = tfirst;
    cb.open[t] = rv;
}

template <bool ROWMAP>
__global__ void __launch_bounds__(256) k_stream_rank1(const int32_t *__restrict__ pos, const int32_t *__restrict__ crd,
                                                      const double *__restrict__ vals,
                                                      const int32_t *__restrict__ seg_begin,
                                                      const int32_t *__restrict__ rowmap, const double *__restrict__ x,
                                                      double *__restrict__ out, int64_t nnz, int64_t ntiles,
                                                      void *scratch, Epilogue ep) {
    __shared__ __attribute__((aligned(16))) int32_t ts[kTile];
    __shared__ int wsum_ht[kWaves], wsum_first_id[kWaves];
    __shared__ double wsum_open[kWaves], wsum_first[kWaves];
    const int64_t t = blockIdx.x;
    const int64_t tb = t * (int64_t)kTile;
    Rank1Half h0;
    rank1_load_half(h0, crd, vals, tb + (int64_t)(threadIdx.x >> 6) * kWaveItems, threadIdx.x & 63, nnz);
    build_tail_map_from_pos(ts, pos, rowmap, tb, seg_begin[t], seg_begin[t + 1], out, 1, false, ep);
    walk_rank1<ROWMAP>(h0, ts, crd, vals, x, rowmap, out, tb, nnz, wsum_ht, wsum_open, wsum_first, wsum_first_id, ep);
    __syncthreads();
    finish_tile_rank1<ROWMAP>(wsum_ht, wsum_open, wsum_first, wsum_first_id, rowmap, out, carry_view(scratch, ntiles, 1), t, ep);
}

// ---- rank-1 kernel over chunks -------------------------------------------------------------------------
// Each wavefront works alone on 1024-item chunks: it marks the segment ends of its chunk in a private 1024-bit mask,
// gets the segment id of an end as (first segment of the chunk) + (ends before it) -- valid because
// this kernel is only used when the level has no empty segment -- and writes the chunk summary
// straight to the carry buffer (one entry per chunk).
// LDSVEC: where x (SpMV) / v (TTV) fits in the 160 KB of LDS next to a few hundred bytes of bookkeeping, one
// workgroup of 16 wavefronts per CU copies it in once and every gather x[crd] becomes an LDS read: the
// L1 / texture-address path, which handles only about one scattered 8-byte gather every two clocks per CU,
// is then left to the streaming loads.
// Otherwise the vector is gathered through L1, a chunk per wavefront; coordinate lists only, whose runs are found here with all loads
// of eight rows of 64 items under way at once, and none behind a comparison: 5 M nonzeros, 60 013 values in the vector, 47.6 us a call with a
// load of both coordinates and both predecessors per item behind branches, and 44.5 with five wavefronts per SIMD (a third of the time are the gathers,
// the rest a chunk's chain of loads); 46.1 with all 16 rows unrolled (three per SIMD), 58.7 with six. Compressed levels keep
// k_stream_rank1 there: 4.7 M nonzeros in short rows, 59 us, and 62 here.
// COO = true: the input is a sorted coordinate list [CN,S,S]; segment ends come from neighbour
// comparisons of (c0, c1) instead of pos, the id of a run is (runs started before the chunk) + (runs
// started earlier in the chunk), and the result's coordinate arrays y0 / y1 are written here too.
template <bool ROWMAP, bool COO, bool LDSVEC>
__global__ void __launch_bounds__(LDSVEC ? 1024 : 256, LDSVEC ? 4 : 5) k_stream_rank1_chunk(const int32_t *__restrict__ pos, const int32_t *__restrict__ crd,
                                                              const double *__restrict__ vals,
                                                              const int32_t *__restrict__ chunk_begin,
                                                              const int32_t *__restrict__ rowmap,
                                                              const double *__restrict__ x, int64_t ncols,
                                                              double *__restrict__ out, int64_t nnz, int64_t nchunks,
                                                              void *scratch, const int32_t *__restrict__ c0,
                                                              const int32_t *__restrict__ c1, int32_t *__restrict__ y0,
                                                              int32_t *__restrict__ y1, Epilogue ep) {
    constexpr int NW = LDSVEC ? 16 : kWaves;
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    const int64_t xpad = LDSVEC ? (ncols + 1) & ~(int64_t)1 : 0;
    double *xs = reinterpret_cast<double *>(lds_raw);
    unsigned *bits_all = reinterpret_cast<unsigned *>(lds_raw + xpad * 8);            // [NW][32]
    double *wfirst_all = reinterpret_cast<double *>(lds_raw + xpad * 8 + NW * 128);   // [NW]
    int *wfirst_id_all = reinterpret_cast<int *>(lds_raw + xpad * 8 + NW * 128 + NW * 8);   // [NW]
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned *bits = bits_all + w * 32;
    const int64_t stride = (int64_t)gridDim.x * NW;
    int64_t c = (int64_t)blockIdx.x * NW + w;
    Rank1Half h0;
    if (c < nchunks) rank1_load_half(h0, crd, vals, c * kChunk, lane, nnz);          // in flight during the staging
    if constexpr (LDSVEC) {
        for (int64_t i = (int64_t)threadIdx.x * 2; i + 1 < ncols; i += 2048)
            *reinterpret_cast<double2 *>(xs + i) = *reinterpret_cast<const double2 *>(x + i);
        if ((ncols & 1) && threadIdx.x == 0) xs[ncols - 1] = x[ncols - 1];
        __syncthreads();
    }
    CarryView cb = carry_view(scratch, nchunks, 1);
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    for (; c < nchunks; c += stride) {
        const int64_t cbeg = c * kChunk;
        int base_id;
        if constexpr (COO) {
            constexpr int kRows = kChunk / 64, kBatch = LDSVEC ? 4 : 8;
            // run starts of a row of 64 items (hm), and the same with items past the end counted as starts (hx);
            // the mask of run ENDS of row r-1 is written as soon as row r is known, so only one row is kept
            unsigned long long hx_prev = 0ull;
            bool first_is_head = false;
            const int runs_before = chunk_begin[c];
            // the coordinate loads of a batch of rows are issued together; the predecessor of an item comes from
            // the neighbouring lane (wave_shr:1), of lane 0 from the previous row (or the item before the chunk)
            const int64_t inext = cbeg + kChunk;
            int before0 = -2, before1 = -2, after0 = -1, after1 = -1;
            if (cbeg > 0) { before0 = c0[cbeg - 1]; before1 = c1[cbeg - 1]; }
            if (inext < nnz) { after0 = c0[inext]; after1 = c1[inext]; }
            int running = runs_before;
            // item e ends a run when item e+1 starts one or lies past the end of the list
            auto write_ends = [&](int r, unsigned long long hx_r, unsigned long long nextbit) {
                const int64_t left = nnz - (cbeg + 64 * r);          // items of this row that exist
                const unsigned long long exist = left >= 64 ? ~0ull : (left <= 0 ? 0ull : ((1ull << left) - 1ull));
                const unsigned long long tmask = ((hx_r >> 1) | (nextbit << 63)) & exist;
                if (lane == 0) *reinterpret_cast<unsigned long long *>(bits + 2 * r) = tmask;
            };
#pragma unroll 1
            for (int rb = 0; rb < kRows; rb += kBatch) {          // (a loop: unrolled it keeps more loads in flight than there are registers)
                int a0[kBatch], a1[kBatch];
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    const int64_t i = cbeg + 64 * (rb + q) + lane;
                    a0[q] = i < nnz ? __builtin_nontemporal_load(c0 + i) : -1;
                    a1[q] = i < nnz ? __builtin_nontemporal_load(c1 + i) : -1;
                }
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    const int r = rb + q;
                    const int64_t i = cbeg + 64 * r + lane;
                    const int p0 = dpp_i<0x138, 0xf>(before0, a0[q]);
                    const int p1 = dpp_i<0x138, 0xf>(before1, a1[q]);
                    const bool differs = a0[q] != p0 || a1[q] != p1;
                    const unsigned long long hm = __ballot(differs && i < nnz);
                    const unsigned long long hx = __ballot(differs);
                    before0 = __builtin_amdgcn_readlane(a0[q], 63);
                    before1 = __builtin_amdgcn_readlane(a1[q], 63);
                    if ((hm >> lane) & 1ull) {
                        const int id = running + __popcll(hm & lt_mask);
                        y0[id] = a0[q]; y1[id] = a1[q];
                    }
                    running += __popcll(hm);
                    if (r == 0) first_is_head = (hm & 1ull) != 0ull;
                    else write_ends(r - 1, hx_prev, hx & 1ull);
                    hx_prev = hx;
                }
            }
            write_ends(kRows - 1, hx_prev, (after0 != before0 || after1 != before1) ? 1ull : 0ull);
            base_id = runs_before - (first_is_head ? 0 : 1);          // the run that holds the chunk's first item
        } else {
            if (lane < 32) bits[lane] = 0u;
            __builtin_amdgcn_wave_barrier();
            const int32_t s0 = chunk_begin[c], s1 = chunk_begin[c + 1];
            for (int32_t sgm = s0 + lane; sgm < s1; sgm += 64) {
                const int64_t idx = (int64_t)pos[sgm + 1] - 1 - cbeg;                  // in [0, 1024): the segment ends here
                atomicOr(&bits[idx >> 5], 1u << (idx & 31));
            }
            base_id = s0;
        }
        __builtin_amdgcn_wave_barrier();
        Rank1Carry cy{0, 0.0};
        auto tails_of_half = [&](int half, int2 *tt) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const unsigned word = bits[(half * 4 + b) * 4 + (lane >> 4)];
                const int sh = (2 * lane) & 31;
                const bool t0 = (word >> sh) & 1u, t1 = (word >> (sh + 1)) & 1u;
                const unsigned long long b0 = __ballot(t0), b1 = __ballot(t1);
                const int id0 = base_id + __popcll(b0 & lt_mask) + __popcll(b1 & lt_mask);
                tt[b].x = t0 ? id0 : -1;
                tt[b].y = t1 ? id0 + (t0 ? 1 : 0) : -1;
                base_id += __popcll(b0) + __popcll(b1);
            }
        };
        auto gather = [&](const Rank1Half &h, double2 *xv) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                if constexpr (LDSVEC) { xv[b].x = xs[h.c[b].x]; xv[b].y = xs[h.c[b].y]; }
                else { xv[b].x = x[h.c[b].x]; xv[b].y = x[h.c[b].y]; }
            }
        };
        double2 xv[4];
        int2 tt[4];
        Rank1Half h1;
        rank1_load_half(h1, crd, vals, cbeg + 512, lane, nnz);
        gather(h0, xv);
        tails_of_half(0, tt);
        rank1_process_half<ROWMAP>(h0, xv, tt, cbeg, nnz, lane, w, rowmap, out, cy, wfirst_all, wfirst_id_all, ep);
        if (c + stride < nchunks) rank1_load_half(h0, crd, vals, (c + stride) * kChunk, lane, nnz);   // next chunk
        gather(h1, xv);
        tails_of_half(1, tt);
        rank1_process_half<ROWMAP>(h1, xv, tt, cbeg + 512, nnz, lane, w, rowmap, out, cy, wfirst_all, wfirst_id_all, ep);
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) {
            cb.has_tail[c] = cy.cf;
            cb.open[c] = cy.cv;
            cb.first[c] = cy.cf ? wfirst_all[w] : 0.0;
            cb.first_id[c] = cy.cf ? wfirst_id_all[w] : -1;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---- fix-up: finish the first segment end of every tile -------------------------------------------
// value = first[t] + open[t-1] + open[t-2] + ... up to and including the nearest tile that contains a segment end.  A thread per
// (tile, r) walks back; for levels whose segments are cut over kShortChain tiles at most.
__global__ void __launch_bounds__(256) k_stream_fixup(void *scratch, int64_t ntiles, int R, const int32_t *__restrict__ rowmap,
                                                      double *__restrict__ out, Epilogue ep) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= ntiles * R) return;
    const int64_t t = g / R;
    const int r = (int)(g - t * R);
    CarryView cb = carry_view(scratch, ntiles, R);
    if (!cb.has_tail[t]) return;
    double v = cb.first[t * R + r];
    for (int64_t u = t - 1; u >= 0; --u) {
        v += cb.open[u * R + r];
        if (cb.has_tail[u]) break;
    }
    const int32_t id = cb.first_id[t];
    const int64_t row = rowmap ? (int64_t)rowmap[id] : (int64_t)id;
    out[row * R + r] = ep_apply(ep, v, out + row * R + r);
}

// The same for longer chains (the head slice of a power-law tensor is cut over thousands of tiles): eight summaries at a time,
// whose loads do not depend on what they hold, and from kFixSerial tiles on the whole workgroup, sixteen at a time per thread.
// A workgroup finishes up to kFixTiles tiles, among which no two chains that long can end, in a block of columns: whole rows (150 M
// nonzeros, rank 64, 36 600 tiles: 58 us, in blocks of 16 columns 69), but 16 columns where one chain may hold an eighth of all
// tiles, so that 64 threads and more share it at every rank.  Whole calls with a launch per level of 64 summaries, which took two
// to four, with workgroups of 1024 threads' worth of tiles in whole rows always, and now: TTV of 12 M nonzeros in 40 fibers
// 69 / 103 / 67 us; MTTKRP at rank 64, one slice of 37 M, 1575 / 1630 / 1581; rank 128, two slices of 18 M in all, 2024 / 2047 / 2017;
// 20 M in power-law slices, rank 64, 815 / 774 / 772; 150 M, rank 16, 1641 / 1603 / 1601.
constexpr int kFixSerial = 64, kFixTiles = 64, kFixColumns = 16;
static_assert(kFixTiles <= kFixSerial, "one long chain per workgroup");
__host__ __device__ inline int fix_tiles(int block) { return 1024 / block < kFixTiles ? 1024 / block : kFixTiles; }   // a thread per tile and column
__global__ void __launch_bounds__(1024) k_stream_fixup_long(void *scratch, int64_t ntiles, int R, int block,
                                                       const int32_t *__restrict__ rowmap, double *__restrict__ out, Epilogue ep) {
    __shared__ double sums[1024];
    __shared__ int chain, newest;
    const CarryView cb = carry_view(scratch, ntiles, R);
    const int tiles = fix_tiles(block), c0 = (int)blockIdx.y * block, cols = R - c0 < block ? R - c0 : block;
    const int lanes = 1024 / cols, lane = (int)threadIdx.x / cols, col = (int)threadIdx.x - lane * cols, r = c0 + col;
    if (threadIdx.x == 0) chain = -1;
    __syncthreads();
    auto finish = [&](int64_t t, double v) {
        const int32_t id = cb.first_id[t];
        double *o = out + (rowmap ? (int64_t)rowmap[id] : (int64_t)id) * R + r;
        *o = ep_apply(ep, v, o);
    };
    const int64_t t0 = (int64_t)blockIdx.x * tiles, mine = t0 + lane;
    if (lane < tiles && mine < ntiles && cb.has_tail[mine]) {
        double v = cb.first[mine * R + r];
        bool done = false;
        int64_t u = mine - 1;
        for (int step = 0; !done && u >= 0 && step < kFixSerial; step += 8) {
            int ht[8];
            double op[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int64_t w = u - q > 0 ? u - q : 0;
                ht[q] = cb.has_tail[w];
                op[q] = cb.open[w * R + r];
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (!done && u - q >= 0) { v += op[q]; done = ht[q] != 0; }
            u -= 8;
        }
        if (done || u < 0) finish(mine, v);
        else if (col == 0) chain = lane;
    }
    __syncthreads();
    if (chain < 0) return;
    const int64_t t = t0 + chain;
    int64_t from = 0;                                             // the nearest tile in front of t that contains a segment end, or the first
    auto look = [&](auto count, int64_t base) {                   // among count * 1024 tiles up to base
        constexpr int N = decltype(count)::value;
        int ht[N], nearest = -1;
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int64_t u = base - q * 1024 - (int)threadIdx.x;
            ht[q] = cb.has_tail[u > 0 ? u : 0];
        }
#pragma unroll
        for (int q = N - 1; q >= 0; --q) {
            const int64_t u = base - q * 1024 - (int)threadIdx.x;
            if (u >= 0 && ht[q]) nearest = (int)u;
        }
        __syncthreads();
        if (threadIdx.x == 0) newest = -1;
        __syncthreads();
        if (nearest >= 0) atomicMax(&newest, nearest);
        __syncthreads();
        if (newest >= 0) from = newest;
        return newest >= 0;
    };
    if (!look(IntC<1>{}, t - 1))
        for (int64_t base = t - 1 - 1024; base >= 0 && !look(IntC<8>{}, base); base -= 8 * 1024) {}
    double v = 0.0;
    int64_t u = from + lane;
    auto sum = [&](auto count) {                                  // (no load under a condition: a last round would go one by one)
        constexpr int N = decltype(count)::value;
        double x[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int64_t w = u + q * (int64_t)lanes;
            x[q] = cb.open[(w < t ? w : t - 1) * R + r];
        }
#pragma unroll
        for (int q = 0; q < N; ++q) v += u + q * (int64_t)lanes < t ? x[q] : 0.0;
        u += N * (int64_t)lanes;
    };
    if (lane < lanes) {
        while (u + 4 * (int64_t)lanes < t) sum(IntC<16>{});
        if (u < t) sum(IntC<4>{});
    }
    sums[threadIdx.x] = v;
    for (int k = lanes; k > 1;) {
        const int h = (k + 1) / 2;
        __syncthreads();
        if (lane < k - h) sums[threadIdx.x] += sums[threadIdx.x + h * cols];
        k = h;
    }
    if (lane == 0) finish(t, cb.first[t * R + r] + sums[threadIdx.x]);
}


}  // namespace

// Finish every segment that a tile boundary cut.  max_chain bounds the number of tiles that one of them is cut over (0: unknown).
hipError_t run_fixup(void *scratch, int64_t ntiles, int R, const int32_t *rowmap, double *out, int64_t max_chain, hipStream_t st,
                     Epilogue ep) {
    if (max_chain > 0 && max_chain <= kShortChain) {
        hipLaunchKernelGGL(k_stream_fixup, dim3((unsigned)((ntiles * R + 255) / 256)), dim3(256), 0, st, scratch, ntiles, R, rowmap, out, ep);
    } else {
        const int block = max_chain <= 0 || max_chain * 8 > ntiles ? kFixColumns : R, tiles = fix_tiles(block);
        hipLaunchKernelGGL(k_stream_fixup_long, dim3((unsigned)((ntiles + tiles - 1) / tiles), (unsigned)((R + block - 1) / block)), dim3(1024), 0, st, scratch, ntiles, R, block, rowmap, out, ep);
    }
    return hipGetLastError();
}


// Allows a kernel to use up to the whole 160 KB of LDS as dynamic shared memory; done once per kernel
// (it is not a stream operation, but calling it once keeps it out of captured regions after the first call).
template <auto Kernel>
static hipError_t allow_full_lds() {
    static hipError_t status = hipFuncSetAttribute((const void *)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    return status;
}

int current_device_cu_count() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return 256; }
    if (dev >= 0 && dev < 64 && cached[dev].load() > 0) return cached[dev].load();
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) { (void)hipGetLastError(); n = 256; }
    if (dev >= 0 && dev < 64) cached[dev].store(n);
    return n;
}

namespace {

struct Rank1Args {
    const int32_t *pos, *crd;
    const double *vals;
    const int32_t *chunk_begin, *rowmap;
    const double *x;
    int64_t ncols;
    double *out;
    int64_t nnz, nchunks;
    void *scratch;
    const int32_t *c0, *c1;
    int32_t *y0, *y1;
    hipStream_t st;
    Epilogue ep;
};

constexpr size_t kChunkWaveLds = 128 + 8 + 4;                     // per wavefront
size_t rank1_lds(int64_t ncols) { return (size_t)((ncols + 1) & ~(int64_t)1) * 8 + 16 * kChunkWaveLds; }
// There is a workgroup's worth of chunks, and the vector fits in LDS.
bool vector_in_lds(int64_t nchunks, int64_t ncols) { return nchunks >= 16 && rank1_lds(ncols) <= 160 * 1024; }

template <bool ROWMAP, bool COO, bool LDSVEC>
hipError_t launch_rank1_chunks(const Rank1Args &a) {
    const int64_t nw = LDSVEC ? 16 : kWaves, want = (a.nchunks + nw - 1) / nw, ncu = LDSVEC ? current_device_cu_count() : want;
    if (LDSVEC) {
        const hipError_t e = allow_full_lds<k_stream_rank1_chunk<ROWMAP, COO, LDSVEC>>();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_stream_rank1_chunk<ROWMAP, COO, LDSVEC>), dim3((unsigned)(want < ncu ? want : ncu)), dim3((unsigned)(64 * nw)),
                       (unsigned)(LDSVEC ? rank1_lds(a.ncols) : kWaves * kChunkWaveLds), a.st, a.pos, a.crd, a.vals, a.chunk_begin, a.rowmap, a.x,
                       a.ncols, a.out, a.nnz, a.nchunks, a.scratch, a.c0, a.c1, a.y0, a.y1, a.ep);
    return hipGetLastError();
}

}  // namespace

bool stream_supports_rank(int64_t R) { return R >= 1 && R <= 128; }
bool stream_mttkrp_supports_rank(int64_t R) { return R >= 1 && R <= 128; }
bool stream_supports_coo() { return true; }

size_t stream_scratch_bytes(int64_t ntiles, int64_t R) { return carry_bytes(ntiles < 1 ? 1 : ntiles, R) + 256; }

bool segreduce_supports(const Schedule &sc, int64_t R) {
    return sc.ntiles <= 0 || R == 1 || segreduce_takes_walk(sc, R) || sc.pieces.ntiles > 0;
}

size_t segreduce_scratch_bytes(const Schedule &sc, int64_t R) {
    if (R == 1) return stream_scratch_bytes(sc.nchunks, 1);
    const size_t a = stream_scratch_bytes(sc.ntiles, R), b = piece_scratch_bytes(sc.pieces, R);
    return a > b ? a : b;
}

hipError_t stream_segreduce(const Schedule &sc, const int32_t *pos, const int32_t *crd, const double *vals,
                            const int32_t *rowmap, const double *Dn, int64_t dense_rows, int64_t R, double *out,
                            void *scratch, bool plain, hipStream_t st, Epilogue ep) {
    if (sc.ntiles <= 0) return hipSuccess;
    if (!stream_supports_rank(R)) return hipErrorNotSupported;
    const int32_t *sb = (const int32_t *)sc.seg_begin->ptr;
    hipError_t e = hipSuccess;
    if (R == 1) {
        if (sc.empty_segments == 0 && sc.chunk_seg_begin && !plain && vector_in_lds(sc.nchunks, dense_rows)) {
            // the dense vector fits in LDS and every segment holds a nonzero: wavefront-per-chunk kernel
            const Rank1Args a{pos, crd, vals, (const int32_t *)sc.chunk_seg_begin->ptr, rowmap, Dn, dense_rows, out, sc.nnz, sc.nchunks, scratch,
                              nullptr, nullptr, nullptr, nullptr, st, ep};
            e = rowmap ? launch_rank1_chunks<true, false, true>(a) : launch_rank1_chunks<false, false, true>(a);
            if (e != hipSuccess) return e;
            return run_fixup(scratch, sc.nchunks, 1, rowmap, out, sc.max_seg_len / kChunk + 2, st, ep);
        }
        if (rowmap)
            hipLaunchKernelGGL(k_stream_rank1<true>, dim3((unsigned)sc.ntiles), dim3(256), 0, st, pos, crd, vals, sb,
                               rowmap, Dn, out, sc.nnz, sc.ntiles, scratch, ep);
        else
            hipLaunchKernelGGL(k_stream_rank1<false>, dim3((unsigned)sc.ntiles), dim3(256), 0, st, pos, crd, vals, sb,
                               rowmap, Dn, out, sc.nnz, sc.ntiles, scratch, ep);
        e = hipGetLastError();
    } else {
        if (!segreduce_takes_walk(sc, R))
            return piece_rows(sc.pieces, crd, vals, sc.nnz, rowmap, Dn, dense_rows, (int)R, out, scratch, st, ep);
        e = stream_segreduce_rankR(sc, pos, crd, vals, rowmap, Dn, (int)R, out, scratch, st, ep);
    }
    if (e != hipSuccess) return e;
    // the rank-R kernel publishes result rows as ids, the rank-1 kernel segment numbers
    return run_fixup(scratch, sc.ntiles, (int)R, R == 1 ? rowmap : nullptr, out, sc.max_seg_len / kTile + 2, st, ep);
}

hipError_t stream_ttv_coo(const Schedule &sc, const int32_t *c0, const int32_t *c1, const int32_t *c2,
                          const double *vals, const double *v, int64_t dense_rows, int32_t *y0, int32_t *y1, double *yv,
                          void *scratch, bool plain, hipStream_t st) {
    if (sc.ntiles <= 0) return hipSuccess;
    // a run of equal (c0, c1) holds at most one nonzero per coordinate of the last mode
    const int64_t max_run = dense_rows;
    const Rank1Args a{nullptr, c2, vals, (const int32_t *)sc.chunk_run_base->ptr, nullptr, v, dense_rows, yv, sc.nnz, sc.nchunks, scratch,
                      c0, c1, y0, y1, st, Epilogue()};
    const hipError_t e = !plain && vector_in_lds(sc.nchunks, dense_rows) ? launch_rank1_chunks<false, true, true>(a) : launch_rank1_chunks<false, true, false>(a);
    if (e != hipSuccess) return e;
    return run_fixup(scratch, sc.nchunks, 1, nullptr, yv, max_run / kChunk + 2, st);
}

}  // namespace comet

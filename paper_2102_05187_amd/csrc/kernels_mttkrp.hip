// MTTKRP kernels.  Short lists: lane groups of 4, 8 or 16 walk the pieces of the fibers of a tile (k_mttkrp_pieces, mttkrp_plan.hpp);
// a tile is a chain of dependent loads -- its descriptor, its nonzeros, rows of B and C, the sums -- and what bounds the kernel is how
// many of them are in flight.  Long lists: wavefronts over blocks of nonzeros (kernels_mttkrp_wave.hip), or lane groups that walk runs of nonzeros over two
// nested segment levels (k_stream_mttkrp); mttkrp_route chooses.
// A piece loads rows of C in groups of four, none behind its batch's last group; with up to seven more rows per piece, fibers of 12 / 30 /
// 200 nonzeros, rank 10, 2.3 M, took 39 / 40 / 37 us instead of 36 / 35 / 32, rank 33 107 / 117 / 108 instead of 90 / 87 / 79.
#include "mttkrp_plan.hpp"
#include "routes.hpp"
#include "stream_common.hpp"

namespace comet {

namespace {

struct MtItem { unsigned off, pad; double val; };                 // a nonzero: where its row of C starts, and its value

// A workgroup takes a tile and a block of L * E columns.
template <int L, int E, bool FULL, bool BIG>
__global__ void __launch_bounds__(256, 3) k_mttkrp_pieces(const int4 *__restrict__ tiles, const uint2 *__restrict__ pieces,
                                                       const uint2 *__restrict__ recs, int ntiles, int items_cap,
                                                       const int32_t *__restrict__ crd, const double *__restrict__ vals,
                                                       const double *__restrict__ Bm, const double *__restrict__ Cm,
                                                       double *__restrict__ M, int64_t nnz, int R, int gaps, double *__restrict__ head,
                                                       double *__restrict__ tail, Epilogue ep) {
    constexpr int V = E, KP = 64 / L, NG = 256 / L, kRow = L * E;
    constexpr int G = 4;                                          // rows of C in flight per group, next to as many being used
    extern __shared__ __attribute__((aligned(16))) char lds[];
    MtItem *item = reinterpret_cast<MtItem *>(lds);
    double *slots = reinterpret_cast<double *>(item + items_cap);
    const int cb = (int)(blockIdx.x / (unsigned)ntiles), t = (int)(blockIdx.x % (unsigned)ntiles);
    const int c0 = cb * kRow;
    const int k = threadIdx.x % L, gw = (threadIdx.x & 63) / L, gid = threadIdx.x / L, wave = threadIdx.x >> 6;
    const RowOf<L, E, 1, FULL> rw(R - c0 < kRow ? R - c0 : kRow, k);
    const char *Cl = reinterpret_cast<const char *>(Cm + c0), *Bl = reinterpret_cast<const char *>(Bm + c0);
    const unsigned unit = (unsigned)R * (BIG ? 1u : 8u);          // row offsets: bytes, or doubles for operands of 4 GiB and more
    auto from_lane = [&](unsigned v, int lane) { return (unsigned)__shfl((int)v, gw * L + lane); };

    const int4 d0 = tiles[t], d1 = tiles[t + 1];
    const int p0 = d0.x & ~1, np = (int)((unsigned)d1.y - (unsigned)d0.y), njoin = d0.w;
    const unsigned nr = (unsigned)d1.z - (unsigned)d0.z, nsum = nr - (unsigned)njoin;
    const MtItem *items = item + (d0.x - p0);
    // two nonzeros, a piece and a record per thread; lane k of a group keeps what the group takes in its k-th turn
    const int pi = (4 * k + wave) * KP + gw;
    const unsigned ri = (unsigned)(k * NG + gid);
    const uint2 pcs = pi < np ? pieces[(size_t)(unsigned)d0.y + pi] : make_uint2(0u, 0u);
    const uint2 rcs = ri < nr ? recs[(size_t)(unsigned)d0.z + ri] : make_uint2(0u, 0u);
    {
        const int i = (int)threadIdx.x * 2;
        if (i < d1.x - p0) {
            int c[2] = {0, 0};
            double a[2] = {0.0, 0.0};
            if ((int64_t)p0 + i + 2 <= nnz) {
                const int2 cc = *reinterpret_cast<const int2 *>(crd + p0 + i);
                const double2 x = *reinterpret_cast<const double2 *>(vals + p0 + i);
                c[0] = cc.x; c[1] = cc.y;
                a[0] = x.x; a[1] = x.y;
            } else {
                c[0] = crd[p0 + i]; a[0] = vals[p0 + i];
            }
            item[i] = MtItem{(unsigned)c[0] * unit, 0u, a[0]};
            item[i + 1] = MtItem{(unsigned)c[1] * unit, 0u, a[1]};
        }
    }
    __syncthreads();
    // Longest pieces first: a piece per group at a time until the longest of them is short.
    int m = 0;
    for (; m < L && (4 * m + wave) * KP < np; ++m) {
        const int longest = mt_len((unsigned)__builtin_amdgcn_readlane((int)pcs.x, m));
        if (longest <= 2 * G) break;
        const unsigned pd = from_lane(pcs.x, m), br = from_lane(pcs.y, m);
        const int shortest = mt_len((unsigned)__builtin_amdgcn_readlane((int)pcs.x, 64 - L + m));
        const int len = mt_len(pd), last = len > 0 ? len - 1 : 0;
        const MtItem *it = items + mt_start(pd);
        double acc[V], b[V], row[2][G][V], val[2][G];
        rw.template load<BIG>(Bl, br * unit, b);
#pragma unroll
        for (int q = 0; q < V; ++q) acc[q] = 0.0;
        auto issue = [&](int j, double (*d)[V], double *v) {
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const MtItem x = it[j + u < last ? j + u : last];
                v[u] = x.val;
                rw.template load<BIG>(Cl, x.off, d[u]);
            }
        };
        auto consume = [&](int j, const double (*d)[V], const double *v) {
            if (j + G <= shortest) {
#pragma unroll
                for (int u = 0; u < G; ++u)
#pragma unroll
                    for (int q = 0; q < V; ++q) acc[q] = fma(v[u], d[u][q], acc[q]);
            } else {
#pragma unroll
                for (int u = 0; u < G; ++u)
                    if (j + u < len) {
#pragma unroll
                        for (int q = 0; q < V; ++q) acc[q] = fma(v[u], d[u][q], acc[q]);
                    }
            }
        };
        // one group in flight behind the one being used, none behind the batch's last one
        issue(0, row[0], val[0]);
        int j = 0;
        for (; j + 2 * G < longest; j += 2 * G) {
            issue(j + G, row[1], val[1]);
            consume(j, row[0], val[0]);
            issue(j + 2 * G, row[0], val[0]);
            consume(j + G, row[1], val[1]);
        }
        if (j + G < longest) {
            issue(j + G, row[1], val[1]);
            consume(j, row[0], val[0]);
            consume(j + G, row[1], val[1]);
        } else {
            consume(j, row[0], val[0]);
        }
#pragma unroll
        for (int q = 0; q < V; ++q) acc[q] *= b[q];
        if (len > 0) rw.put(slots + mt_slot(pd) * kRow, acc);
    }
    // Short pieces: several of them per group at the same time.
    auto short_pieces = [&](auto count) {
        constexpr int KB = decltype(count)::value;
        const int longest = mt_len((unsigned)__builtin_amdgcn_readlane((int)pcs.x, m));
        unsigned pd[KB];
        int len[KB];
        double acc[KB][V], b[KB][V], row[2][KB][V], val[2][KB];
        auto issue = [&](int j, double (*d)[V], double *v) {
#pragma unroll
            for (int q = 0; q < KB; ++q) {
                const MtItem x = items[j < len[q] ? mt_start(pd[q]) + j : 0];
                v[q] = x.val;
                rw.template load<BIG>(Cl, x.off, d[q]);
            }
        };
        auto consume = [&](int j, const double (*d)[V], const double *v) {
#pragma unroll
            for (int q = 0; q < KB; ++q)
                if (j < len[q]) {
#pragma unroll
                    for (int e = 0; e < V; ++e) acc[q][e] = fma(v[q], d[q][e], acc[q][e]);
                }
        };
#pragma unroll
        for (int q = 0; q < KB; ++q) {
            pd[q] = from_lane(pcs.x, m + q);
            len[q] = mt_len(pd[q]);
            rw.template load<BIG>(Bl, from_lane(pcs.y, m + q) * unit, b[q]);
#pragma unroll
            for (int e = 0; e < V; ++e) acc[q][e] = 0.0;
        }
        issue(0, row[0], val[0]);
        for (int j = 0; j < longest; j += 2) {
            if (j + 1 < longest) issue(j + 1, row[1], val[1]);
            consume(j, row[0], val[0]);
            if (j + 1 >= longest) break;
            if (j + 2 < longest) issue(j + 2, row[0], val[0]);
            consume(j + 1, row[1], val[1]);
        }
#pragma unroll
        for (int q = 0; q < KB; ++q)
            if (len[q] > 0) {
#pragma unroll
                for (int e = 0; e < V; ++e) acc[q][e] *= b[q][e];
                rw.put(slots + mt_slot(pd[q]) * kRow, acc[q]);
            }
        m += KB;
    };
    const int turns = ((np + KP - 1) / KP - wave + 3) >> 2;    // pieces of this wavefront's groups
    while (m < turns) {
        if (turns - m >= 4) short_pieces(IntC<4>{});
        else if (turns - m >= 2) short_pieces(IntC<2>{});
        else short_pieces(IntC<1>{});
    }
    __syncthreads();
    auto add_rows = [&](int first, int n, int step, double *s) {
        for (int i = 0; i < n; i += 4 * step) {
            double v[4][V];
#pragma unroll
            for (int u = 0; u < 4; ++u) rw.get(slots + (first + (i + u * step < n ? i + u * step : i)) * kRow, v[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u * step < n) {
#pragma unroll
                    for (int q = 0; q < V; ++q) s[q] += v[u][q];
                }
        }
    };
    auto do_sum = [&](const uint2 r) {
        const int kind = mt_sum_kind(r.x), first = mt_first(r.x), n = mt_sum_rows(r.x);
        double s[V];
#pragma unroll
        for (int q = 0; q < V; ++q) s[q] = 0.0;
        add_rows(first, n, 1, s);
        double *o = M + (int64_t)(int)r.y * R + c0;
        if (kind == kMtPart) rw.put(slots + first * kRow, s);
        else if (kind == kMtSlice) rw.store_result(o, s, ep, n == 0);
        if (gaps)
            for (int g = mt_sum_gap(r.x); g > 0; --g) {       // rows that are not stored
#pragma unroll
                for (int q = 0; q < V; ++q) s[q] = 0.0;
                rw.store_result(o - (int64_t)g * R, s, ep, true);
            }
    };
    auto do_join = [&](const uint2 r) {
        const bool cont = mt_join_cont(r.x), open = mt_join_open(r.x);
        double s[V];
#pragma unroll
        for (int q = 0; q < V; ++q) s[q] = 0.0;
        add_rows(mt_first(r.x), mt_join_rows(r.x), kMtSum, s);
        const int64_t at = (int64_t)t * R + c0;
        if (cont) rw.store(head + at, s);
        else if (open) rw.store(tail + at, s);
        else rw.store_result(M + (int64_t)(int)r.y * R + c0, s, ep);
    };
    auto record = [&](int q) { return make_uint2(from_lane(rcs.x, q), from_lane(rcs.y, q)); };
    int q = 0;
    for (; q < L; ++q) {
        if ((unsigned)(q * NG + gid) >= nsum) break;
        do_sum(record(q));
    }
    for (unsigned i = 256 + gid; i < nsum; i += NG) do_sum(recs[(size_t)(unsigned)d0.z + i]);
    if (njoin) {
        __syncthreads();
        for (; q < L; ++q) {
            if ((unsigned)(q * NG + gid) >= nr) break;
            do_join(record(q));
        }
        for (unsigned i = 256 + gid; i < nr; i += NG)
            if (i >= nsum) do_join(recs[(size_t)(unsigned)d0.z + i]);
    }
}

// Slices cut by tile boundaries: what the first tile holds of one behind its boundary, then what the following tiles hold in
// front of theirs.  A thread per (slice, column); the last workgroups take the slices over many tiles, a block of 16 columns
// each, with the tiles dealt over 64 threads per column.  A thread does little else than wait for its loads: those of four tiles are under way
// at once, the last one's again behind the end (100 000 nonzeros in slices over up to 16 tiles, rank 10: 5.2 us, and 4.0 with them; whole calls 13.9 and 12.5).
__global__ void __launch_bounds__(1024) k_mttkrp_cut_sums(const int4 *__restrict__ cuts, int ncut, int nlong, int64_t ntiles,
                                                          const double *__restrict__ head, const double *__restrict__ tail, int R,
                                                          double *__restrict__ M, Epilogue ep) {
    __shared__ double sums[1024];
    const int nblocks = (R + 15) / 16, narrow = (int)gridDim.x - nlong * nblocks;
    if ((int)blockIdx.x < narrow) {
        const unsigned g = blockIdx.x * 1024u + threadIdx.x, i = g / (unsigned)R;
        const int r = (int)(g - i * (unsigned)R);
        if (i >= (unsigned)ncut) return;
        const int4 c = cuts[i];
        double s = tail[(int64_t)c.y * R + r];
        for (int u = c.y + 1; u <= c.z; u += 4) {
            double v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = head[(int64_t)(u + q < c.z ? u + q : c.z) * R + r];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (u + q <= c.z) s += v[q];
        }
        double *o = M + (int64_t)c.x * R + r;
        *o = ep_apply(ep, s, o);
        return;
    }
    const int w = (int)blockIdx.x - narrow;
    const int4 c = cuts[ntiles - 1 - w / nblocks];
    const int lane = threadIdx.x >> 4, r = (w % nblocks) * 16 + (threadIdx.x & 15);
    double s = 0.0;
    if (r < R) {
        if (lane == 0) s = tail[(int64_t)c.y * R + r];
        int64_t u = c.y + 1 + lane;
        for (; u + 7 * 64 <= c.z; u += 8 * 64) {
            double v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = head[(u + 64 * q) * R + r];
#pragma unroll
            for (int q = 0; q < 8; ++q) s += v[q];
        }
        for (; u <= c.z; u += 64) s += head[u * R + r];
    }
    sums[threadIdx.x] = s;
    for (int d = 32; d > 0; d >>= 1) {
        __syncthreads();
        if (lane < d) sums[threadIdx.x] += sums[threadIdx.x + 16 * d];
    }
    if (lane != 0 || r >= R) return;
    double *o = M + (int64_t)c.x * R + r;
    *o = ep_apply(ep, sums[threadIdx.x], o);
}

// ---- MTTKRP: the same walk, two nested segment levels ---------------------------------------------
// Inner level: fibers (segments of pos3); the per-fiber sum of vals * C[crd3, :] is scaled by the row
// B[crd2[fiber], :] when the fiber ends and folded into the slice accumulator.  Scaling is linear,
// so a fiber cut by a walker or tile boundary is folded piecewise (each piece times the same B row);
// only the slice level needs carries.  Outer level: slices (segments of pos2); a slice end writes
// row crd1[slice] of M.  Two LDS maps, both keyed by tile item: ts = the fiber's coordinate crd2[fiber]
// (its row of B) at a fiber's last nonzero, tm = output row at a slice's last nonzero (-1 elsewhere).  Both
// are looked up while the maps are built, with coalesced loads, so that the walk has no dependent index load.
// TILE: kTile, or kChunk for lists below kChunkWalkNnz.
template <int L, int V, bool WIDE, int TILE>
__global__ void __launch_bounds__(256) k_stream_mttkrp(const int32_t *__restrict__ pos2, const int32_t *__restrict__ crd1,
                                                       const int32_t *__restrict__ pos3, const int32_t *__restrict__ crd2,
                                                       const int32_t *__restrict__ crd3, const double *__restrict__ vals,
                                                       const int32_t *__restrict__ seg_begin,
                                                       const int32_t *__restrict__ slice_begin,
                                                       const double *__restrict__ Bm, const double *__restrict__ Cm,
                                                       double *__restrict__ M, int64_t nnz, int64_t nfib, int64_t ntiles,
                                                       int R, void *scratch, Epilogue ep) {
    constexpr int NW = 256 / L, WI = TILE / NW, SB = 4 * L;
    constexpr int kMapInts = 2 * TILE;
    constexpr int kOpenInts = 256 * V * 2;
    constexpr int kLdsInts = kMapInts > kOpenInts ? kMapInts : kOpenInts;
    __shared__ __attribute__((aligned(16))) int32_t lds[kLdsInts];
    __shared__ int wht[NW], wfirst_j[NW];
    int32_t *ts = lds, *tm = lds + TILE;
    double *wopen = reinterpret_cast<double *>(lds);              // reused once the maps are dead
    const int64_t t = blockIdx.x;
    const int64_t tb = t * (int64_t)TILE, te = tb + TILE;
    const int g = threadIdx.x / L, j = threadIdx.x % L;
    const int64_t gb = tb + (int64_t)g * WI;
    LaneItems cur;
    lane_load_items(cur, crd3, vals, gb + 4 * j, nnz);            // in flight while the maps are built

    for (int i = threadIdx.x * 4; i < 2 * TILE; i += blockDim.x * 4)
        *reinterpret_cast<int4 *>(lds + i) = make_int4(-1, -1, -1, -1);
    __syncthreads();
    for (int32_t f = seg_begin[t] + threadIdx.x; f < seg_begin[t + 1]; f += blockDim.x) {
        int32_t b = pos3[f], e = pos3[f + 1];
        if (e > b) ts[(int64_t)e - 1 - tb] = crd2[f];
    }
    for (int32_t sl = slice_begin[t] + threadIdx.x; sl < slice_begin[t + 1]; sl += blockDim.x) {
        int32_t fb = pos2[sl], fe = pos2[sl + 1];
        int64_t il = -1;                                          // last nonzero of the slice
        for (int32_t f = fe - 1; f >= fb; --f) {
            int32_t b = pos3[f], e = pos3[f + 1];
            if (e > b) { il = (int64_t)e - 1; break; }
        }
        if (il >= tb && il < te) tm[il - tb] = crd1[sl];
        if (il < 0) {                                             // a stored slice without any nonzero: its row is zero
            double *row = M + (int64_t)crd1[sl] * R;
            for (int r = 0; r < R; ++r) row[r] = ep_empty(ep, row + r);
        }
    }
    __syncthreads();

    double facc[V], sacc[V], first[V];
#pragma unroll
    for (int q = 0; q < V; ++q) { facc[q] = 0.0; sacc[q] = 0.0; first[q] = 0.0; }
    int ht = 0, first_row = -1, first_j = -1, last_is_tail = 1;

    // narrow rows: two steps per pipeline group instead of four keeps the kernel under 128 registers
    // (four wavefronts per SIMD instead of three), which is worth more here than the deeper gather queue
    constexpr int G = V <= 2 ? 2 : StepGroup<V>::value, NG = SB / G;
    for (int sb = 0; sb < WI / SB; ++sb) {
        const int64_t i0 = gb + SB * sb + 4 * j;
        LaneItems nxt;
        if (sb + 1 < WI / SB) lane_load_items(nxt, crd3, vals, i0 + SB, nnz);
        int tl[4], tr[4];
        {
            const int4 t4 = *reinterpret_cast<const int4 *>(ts + (i0 - tb));
            const int4 m4 = *reinterpret_cast<const int4 *>(tm + (i0 - tb));
            tl[0] = t4.x; tl[1] = t4.y; tl[2] = t4.z; tl[3] = t4.w;
            tr[0] = m4.x; tr[1] = m4.y; tr[2] = m4.z; tr[3] = m4.w;
        }
        const bool any_item = gb + SB * sb < nnz;
        RowBuf<V> cbuf[2][G], bbuf[2][G];
        auto issue = [&](auto gc, RowBuf<V> *cb_, RowBuf<V> *bb_) {
            static_for<0, G>([&](auto sc) {
                constexpr int k = decltype(gc)::value * G + decltype(sc)::value;
                constexpr int s_ = decltype(sc)::value;
                const int c = grp_bcast_i<L, k / 4>(cur.cr[k % 4]);
                grp_load_row<L, V, WIDE>(Cm, c, R, j, cb_[s_].d);
                const int tf = grp_bcast_i<L, k / 4>(tl[k % 4]);
                // The B row is needed where a fiber ends.  Narrow rows: loaded at every item (row 0, a cache hit,
                // where no fiber ends), so that the number of loads in flight is fixed and the gathers of the next
                // group really overlap these FMAs (a load under a branch makes the wait for the rows of this group
                // cover part of the next group's loads): 1.74 -> 1.61 ms at rank 16.  Wide rows pay more for the
                // extra load instructions than they gain (5.18 -> 5.32 ms at rank 64) and keep the branch.
                if constexpr (V <= 2) grp_load_row<L, V, WIDE>(Bm, tf >= 0 ? tf : 0, R, j, bb_[s_].d);
                else if (tf >= 0) grp_load_row<L, V, WIDE>(Bm, tf, R, j, bb_[s_].d);
            });
        };
        auto consume = [&](auto gc, const RowBuf<V> *cb_, const RowBuf<V> *bb_) {
            static_for<0, G>([&](auto sc) {
                constexpr int k = decltype(gc)::value * G + decltype(sc)::value;
                constexpr int s_ = decltype(sc)::value;
                const double a = grp_bcast_d<L, k / 4>(cur.va[k % 4]);
                const int tf = grp_bcast_i<L, k / 4>(tl[k % 4]);
                const int tmr = grp_bcast_i<L, k / 4>(tr[k % 4]);
#pragma unroll
                for (int q = 0; q < V; ++q) facc[q] = fma(a, cb_[s_].d[q], facc[q]);
                if (any_item) last_is_tail = tf >= 0;
                if (tf >= 0) {
                    if (first_j < 0) first_j = tf;
#pragma unroll
                    for (int q = 0; q < V; ++q) { sacc[q] = fma(bb_[s_].d[q], facc[q], sacc[q]); facc[q] = 0.0; }
                    if (tmr >= 0) {
                        if (!ht) {
#pragma unroll
                            for (int q = 0; q < V; ++q) first[q] = sacc[q];
                            first_row = tmr; ht = 1;
                        } else {
                            grp_store_row_stream<L, V, WIDE>(M, tmr, R, j, sacc, ep);
                        }
#pragma unroll
                        for (int q = 0; q < V; ++q) sacc[q] = 0.0;
                    }
                }
            });
        };
        issue(IntC<0>{}, cbuf[0], bbuf[0]);
        static_for<0, NG>([&](auto gc) {
            constexpr int gi = decltype(gc)::value;
            if constexpr (gi + 1 < NG) issue(IntC<gi + 1>{}, cbuf[(gi + 1) & 1], bbuf[(gi + 1) & 1]);
            consume(gc, cbuf[gi & 1], bbuf[gi & 1]);
        });
        if (sb + 1 < WI / SB) cur = nxt;
    }

    // A fiber left open at the end of this walker's range ends at the next fiber end of the tile, or,
    // if there is none, it is the fiber that contains the first nonzero of the next tile.
    if (j == 0) wfirst_j[g] = first_j;
    __syncthreads();                                              // also: every walk is done, the maps are dead
    if (!last_is_tail) {
        int jrow = -1;
        for (int g2 = g + 1; g2 < NW; ++g2) { const int j2 = wfirst_j[g2]; if (j2 >= 0) { jrow = j2; break; } }
        if (jrow < 0 && (int64_t)seg_begin[t + 1] < nfib) jrow = crd2[seg_begin[t + 1]];
        if (jrow >= 0) {
            double bw[V];
            grp_load_row<L, V, WIDE>(Bm, jrow, R, j, bw);
#pragma unroll
            for (int q = 0; q < V; ++q) sacc[q] = fma(bw[q], facc[q], sacc[q]);
        }
    }
    {
        double *wo = wopen + (g * L + j) * V;
#pragma unroll
        for (int q = 0; q < V; ++q) wo[q] = sacc[q];
        if (j == 0) wht[g] = ht;
    }
    __syncthreads();
    finish_tile_walkers<L, V, WIDE>(wopen, wht, g, j, ht, first, first_row, first_row, sacc, M, R,
                                    carry_view(scratch, ntiles, R), t, ep);
}

struct MtArgs {
    const MttkrpPlan &plan;
    const int32_t *pos2, *crd1, *pos3, *crd2;
    const int32_t *crd;
    const double *vals, *B, *C;
    double *M;
    int64_t nnz;
    int R, gaps;
    double *head, *tail;
    hipStream_t st;
    Epilogue ep;
};

template <int L, int E, bool FULL, bool BIG>
hipError_t launch_mttkrp(const MtArgs &a) {
    constexpr int kRow = L * E;
    const int nblocks = (a.R + kRow - 1) / kRow, items_cap = a.plan.max_items + 3;
    const size_t lds = (size_t)items_cap * sizeof(MtItem) + (size_t)a.plan.max_pieces * kRow * 8;
    hipLaunchKernelGGL((k_mttkrp_pieces<L, E, FULL, BIG>), dim3((unsigned)(a.plan.ntiles * nblocks)), dim3(256), (unsigned)lds, a.st,
                       (const int4 *)a.plan.tiles(), (const uint2 *)a.plan.pieces(), (const uint2 *)a.plan.recs(), (int)a.plan.ntiles,
                       items_cap, a.crd, a.vals, a.B, a.C, a.M, a.nnz, a.R, a.gaps, a.head, a.tail, a.ep);
    return hipGetLastError();
}

template <int L, int V, bool WIDE>
hipError_t launch_walk(const MtArgs &a, const Schedule &sc, void *scratch) {
    auto go = [&](auto kernel, int64_t ntiles, const DevRef &fibers, const DevRef &slices) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)ntiles), dim3(256), 0, a.st, a.pos2, a.crd1, a.pos3, a.crd2, a.crd, a.vals,
                           (const int32_t *)fibers->ptr, (const int32_t *)slices->ptr, a.B, a.C, a.M, sc.nnz, sc.nseg, ntiles, a.R,
                           scratch, a.ep);
    };
    if (sc.nnz < kChunkWalkNnz) go(k_stream_mttkrp<L, V, WIDE, kChunk>, sc.nchunks, sc.chunk_seg_begin, sc.chunk_slice_begin);
    else go(k_stream_mttkrp<L, V, WIDE, kTile>, sc.ntiles, sc.seg_begin, sc.slice_begin);
    return hipGetLastError();
}

// Calls F<L, E, FULL, BIG>(args) for rank R: blocks of 16 columns, 16 bytes per lane where the rank is even.
#define COMET_DISPATCH_BLOCKS(F, R, big, args)                                \
    (big ? ((R) & 1 ? F<16, 1, false, true>(args) : F<8, 2, false, true>(args)) \
     : (R) & 1 ? ((R) <= 4 ? F<4, 1, false, false>(args) : (R) <= 8 ? F<8, 1, false, false>(args) : F<16, 1, false, false>(args)) \
               : ((R) <= 8 ? F<4, 2, false, false>(args) : (R) % 16 ? F<8, 2, false, false>(args) : F<8, 2, true, false>(args)))

// Tiles that the slices of the walk are cut over at most.
int64_t mttkrp_chain(const Schedule &sc) { return sc.max_parent_len / (sc.nnz < kChunkWalkNnz ? kChunk : kTile) + 2; }

// Which lists and ranks take the pieces; all others the walk over tiles of nonzeros or the wavefronts (routes.hpp), which keep more rows in flight once their tiles
// fill the chip, while a tile of pieces needs several rounds of loads one after the other.  Calls of the walk and of the pieces in us,
// three tensors taking turns.  Power: power-law modes, 2.5 to 4 nonzeros per fiber, slices cut over many tiles, for which the walk's
// carry fix-up is longer; ones: uniform modes, a nonzero per fiber, so that the pieces read a row of B for each; fives, thirties: so
// many per fiber, short slices.
//   nonzeros         rank 8     16        32        64         10        20        7         9         33        40
//   0.2 M power      27   19   29   25   37   35   61   64    30   22   39   30   28   19   30   22   55   42   59   46
//         ones       18   15   20   17   24   23   35   37    25   17   30   25   20   15   25   17   41   38   40   33
//         fives      15   15   15   15   15   16   16   24    15   15   18   15   15   15   15   15   24   20   24   20
//         thirties   15   15   15   15   15   16   16   23    16   15   18   16   16   15   16   14   22   19   22   19
//   0.6 M power      37   25   42   34   66   59  101  103    44   30   67   48   38   26   44   35  102   88  109   83
//         ones       25   22   26   27   45   45   83   94    34   29   52   49   30   24   33   32   74   86   75   69
//         fives      15   15   15   16   23   24   30   38    21   16   32   24   16   15   21   18   43   32   43   30
//         thirties   18   15   17   15   22   21   27   33    22   15   28   20   20   15   23   16   36   29   36   27
//   1.2 M power      42   34   49   49   89   88  136  158    55   43   93   79   47   34   54   51  141  140  146  124
//         ones       34   34   37   43   71   82  135  159    47   46   73   83   41   37   47   54  111  158  114  124
//         fives      17   21   20   25   32   41   46   74    29   25   46   41   21   21   30   27   64   60   64   57
//         thirties   22   17   21   22   31   34   40   58    30   21   41   34   25   19   30   24   53   49   53   46
//   2.3 M power      55   51   67   75  122  133  193  252    76   68  144  127   60   50   76   82  206  228  213  192
//         ones       53   57   56   76  117  149  248  286    72   78  114  154   64   62   72   96  179  291  182  228
//         fives      28   33   30   40   53   72   77  136    46   40   75   72   33   32   47   43  107  105  108  103
//         thirties   29   27   30   34   49   59   64  108    46   35   67   59   35   28   47   37   87   87   87   84
//   4.9 M power      88   98  124  131  198  239  327  460   154  127  253  234  107   97  151  153  370  425  379  350
//         ones      108  119  126  153  244  292  538  574   157  162  244  317  137  127  155  190  372  609  385  466
//         fives      47   62   63   75   95  145  152  285    95   76  142  143   61   58   97   78  210  213  210  212
//         thirties   48   47   61   62   73  116  109  224    92   63  106  116   62   50   92   67  151  174  152  170
// Ranks 2 and 4 go with 8, 48 with 32, 96 and 128 with 64; 1, 3, 6 with 7; 12 with 10; 15 with 9; 17 between 9 and 33; 24 with 20; 80 with 40.
bool mttkrp_takes_pieces(const Schedule &sc, int64_t R) {
    const int64_t n = sc.nnz, blocks = (R + 15) / 16;
    const bool long_slices = sc.max_parent_len <= 0 || mttkrp_chain(sc) > kShortChain;
    // ranks whose rows the walk reads 16 bytes per lane, with no lane idle
    if (R == 2 || R == 4 || R == 8 || R % 16 == 0) {
        if (long_slices) return R <= 48 && n <= (R <= 8 ? int64_t(9) << 18 : int64_t(9) << 17) && n * blocks <= int64_t(9) << 18;
        return R <= 32 && n * (R > 8 ? R : 8) <= int64_t(25) << 18;
    }
    if (n < 2 * sc.nseg) return n * (R % 2 ? blocks : (R + 31) / 32) <= int64_t(3) << 18;
    if (R > 32 || (R % 2 && R > 16)) return n * blocks <= int64_t(9) << 18;
    if (R % 2 && R > 8) return n <= (long_slices ? int64_t(5) << 18 : int64_t(9) << 18);
    return R < 16 || long_slices || n <= int64_t(9) << 18;
}

}  // namespace

MttkrpRoute mttkrp_route(const Schedule &sc, int64_t dense_rows, int64_t R, bool plain) {
    // row offsets of the pieces and of the wavefronts are 32-bit counts of doubles; the walk forms 64-bit addresses
    if (plain || dense_rows * R >= (int64_t(1) << 32)) return MttkrpRoute::kWalk;
    if (sc.mttkrp.ntiles > 0 && mttkrp_takes_pieces(sc, R)) return MttkrpRoute::kPieces;
    return sc.empty_segments == 0 && sc.empty_slices == 0 && mttkrp_takes_wave(sc, R) ? MttkrpRoute::kWave : MttkrpRoute::kWalk;
}

static int64_t walk_tiles(const Schedule &sc) { return sc.nnz < kChunkWalkNnz ? sc.nchunks : sc.ntiles; }

size_t mttkrp_call_bytes(const Schedule &sc, int64_t R, MttkrpRoute route) {
    if (route == MttkrpRoute::kPieces) return (size_t)sc.mttkrp.ntiles * (size_t)R * 2 * sizeof(double);
    return stream_scratch_bytes(route == MttkrpRoute::kWave ? sc.nchunks : walk_tiles(sc), R);
}

size_t mttkrp_scratch_bytes(const Schedule &sc, int64_t R) {
    // the walk, which serves variant 3 and the largest factors at every rank, and what each rank up to R takes otherwise
    size_t need = stream_scratch_bytes(walk_tiles(sc), R);
    for (int64_t r = 1; r <= R; ++r) {
        const size_t b = mttkrp_call_bytes(sc, r, mttkrp_route(sc, 0, r, false));
        if (b > need) need = b;
    }
    return need;
}

hipError_t stream_mttkrp(const Schedule &sc, const int32_t *pos2, const int32_t *crd1, int64_t nslice, const int32_t *pos3, const int32_t *crd2,
                         const int32_t *crd3, const double *vals, const double *B, const double *C, int64_t dense_rows, int64_t R,
                         double *M, MttkrpRoute route, bool gaps, void *scratch, hipStream_t st, Epilogue ep) {
    if (sc.ntiles <= 0) return hipSuccess;
    if (!stream_mttkrp_supports_rank(R) || !sc.slice_begin) return hipErrorNotSupported;
    const MttkrpPlan &plan = sc.mttkrp;
    double *head = (double *)scratch, *tail = head + plan.ntiles * R;
    const MtArgs a{plan, pos2, crd1, pos3, crd2, crd3, vals, B, C, M, sc.nnz, (int)R, gaps ? 1 : 0, head, tail, st, ep};
    if (route == MttkrpRoute::kPieces) {
        const bool wide = dense_rows * R * 8 >= (int64_t(1) << 32);   // row offsets in bytes no longer fit 32 bits
        const hipError_t e = COMET_DISPATCH_BLOCKS(launch_mttkrp, a.R, wide, a);
        if (e != hipSuccess || plan.ncut + plan.ncut_long == 0) return e;
        const int64_t narrow = (plan.ncut * R + 1023) / 1024;
        hipLaunchKernelGGL(k_mttkrp_cut_sums, dim3((unsigned)(narrow + plan.ncut_long * ((R + 15) / 16))), dim3(1024), 0, st,
                           (const int4 *)plan.cuts(), (int)plan.ncut, (int)plan.ncut_long, plan.ntiles, (const double *)head,
                           (const double *)tail, (int)R, M, ep);
        return hipGetLastError();
    }
    if (route == MttkrpRoute::kWave)
        return mttkrp_wave(sc, pos2, nslice, crd1, pos3, crd2, crd3, vals, B, C, dense_rows * R * 8 >= (int64_t(1) << 32), (int)R, M, scratch, st, ep);
    const hipError_t e = COMET_DISPATCH_GROUPS(launch_walk, a.R, a, sc, scratch);
    if (e != hipSuccess) return e;
    return run_fixup(scratch, walk_tiles(sc), (int)R, nullptr, M,
                     sc.max_parent_len > 0 ? mttkrp_chain(sc) : 0, st, ep);
}

}  // namespace comet

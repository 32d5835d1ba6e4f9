// Rank-R kernel (SpMM, TTM): lane groups of 4, 8 or 16 walk the pieces of a level (pieces.hpp).
//
// What bounds it.  Every vector memory instruction keeps the texture-address unit of a compute unit busy for 16 clocks and
// more, however few of its lanes are active, and the vector L1 behind it returns data in order, so that the times for
// gathering operand rows, reading nonzeros and writing results add up rather than overlap.  The kernel therefore spends as
// few instructions as it can: rows 16 bytes per lane, nonzeros 16 bytes per lane into LDS, from where a lane group reads one
// with a broadcast, and result rows stored for all groups of a wavefront at once, which pieces of equal length make possible.
// A walk that asks at every nonzero whether a segment ends (kernels_rankR.hip) stores few rows at a time.
// Measured before and after, that walk and this, for whole calls whose inputs change from call to call: SpMM on 11.3 M
// nonzeros within 2000 columns of the diagonal, rank 20, added to the old result, 358 and 236 us; TTM on 8 M nonzeros in
// 1.6 M fibers, rank 32, 180 and 172 us (the result's 415 MB and nonzeros that come from memory leave little to gain);
// 200 000 nonzeros, rank 16, 29 and 14 us.
// The loads of a long piece.  Where a part of the list comes back to the same operand rows, as many as its batch has steps:
// 3.6 M nonzeros, 12 per row near the diagonal, three states taking turns, ranks 20 / 32 / 128, 59 / 75 / 260 us, and 72 / 86 / 292
// with up to eight loads behind its end; 9 M, nine per row, rank 32, 210 and 260; 11.3 M in power-law rows, rank 64, 367 and 402.
// Where almost every row is a new one from memory it is the other way round: nine nonzeros per row at random, 7.2 M, ranks 10 / 32,
// 198 and 192, 296 and 280 us; 1 to 120 per row, rank 64, 531 and 519.  The loads behind the end read the piece's last row again;
// other rows there, fewer wavefronts or fewer loads in flight do not give the same, and why it does was not found (spread_rows).
#include "pieces.hpp"
#include "stream_common.hpp"

namespace comet {

namespace {

struct Item { unsigned off, pad; double val; };                   // a nonzero: where its operand row starts, and its value

// Bytes of LDS: the tile's nonzeros (up to 7 more for the 16-byte boundaries around them), its pieces, its partial sums.
__host__ __device__ inline int lds_pieces_at(int units) { return (tile_items(units) + 7) * (int)sizeof(Item); }
__host__ __device__ inline int lds_parts_at(int units) { return lds_pieces_at(units) + ((tile_pieces(units) + 3) & ~3) * 4; }

// stream: the nonzeros are read around the caches (kStreamNnz); spread: spread_rows
template <int L, int E, int NL, bool FULL, bool BIG, bool ROWMAP>
__global__ void __launch_bounds__(256) k_pieces(const int4 *__restrict__ tiles, const uint32_t *__restrict__ pieces,
                                                const uint32_t *__restrict__ joins, int units, int stream, int spread,
                                                const int32_t *__restrict__ crd, const double *__restrict__ vals,
                                                const int32_t *__restrict__ rowmap, const double *__restrict__ Dn,
                                                double *__restrict__ out, int64_t nnz, int R, double *__restrict__ head,
                                                double *__restrict__ tail, Epilogue ep) {
    constexpr int V = E * NL, KP = 64 / L, kRow = L * V;          // pieces side by side in a wavefront
    // Gathers of a piece in flight, next to as many being used.  More cost wavefronts: with 6 at two values per lane, band of 12 per
    // row, 3.6 M nonzeros, ranks 16 / 32 go from 31 / 61 us to 50 / 64; with 2 and 1 instead of 3 at four and eight values ranks 64 / 128
    // of 11.3 M nonzeros near the diagonal and of the band take 396 and 276 instead of 381 and 250.
    constexpr int G = V <= 2 ? 4 : 3;
    constexpr int KB = V <= 2 ? 4 : (V <= 4 ? 2 : 1);             // pieces of a group at a time, when they are short
    extern __shared__ __attribute__((aligned(16))) char lds[];
    Item *item = reinterpret_cast<Item *>(lds);
    uint32_t *piece = reinterpret_cast<uint32_t *>(lds + lds_pieces_at(units));
    double *part = reinterpret_cast<double *>(lds + lds_parts_at(units));
    // Workgroups go to the eight XCDs in turn.  Each XCD gets a contiguous eighth of the tiles, so that operand rows which
    // neighbouring segments share are shared in its L2 (12 M nonzeros within 2000 columns, rank 32: 403 -> 284 us).
    const int n8 = (int)gridDim.x / 8;
    const int t = (int)blockIdx.x < 8 * n8 ? ((int)blockIdx.x & 7) * n8 + ((int)blockIdx.x >> 3) : (int)blockIdx.x;
    const int4 t0 = tiles[t], t1 = tiles[t + 1];
    // a level of almost 2^31 segments has more pieces than that: their numbers are unsigned
    const uint32_t first_piece = (uint32_t)t0.z;
    const int np = (int)((uint32_t)t1.z - first_piece), nj = t1.w - t0.w;
    const unsigned unit = (unsigned)R * (BIG ? 1u : 8u);          // row offsets: bytes, or doubles for operands of 4 GiB and more
    // nonzeros of the tile from the 16-byte boundary in front of them
    const int p0 = t0.x & ~3, lead = t0.x - p0, n_items = t1.x - p0;
    // (two loops: the compiler folds a plain and a non-temporal load of one address into a plain one)
    auto stage = [&](auto around) {
        for (int i = (int)threadIdx.x * 4; i < n_items; i += 1024) {
            int c[4];
            double a[4];
            if ((int64_t)p0 + i + 4 <= nnz) {
                typedef int v4i __attribute__((ext_vector_type(4)));
                typedef double v2d __attribute__((ext_vector_type(2)));
                const v4i *pc = reinterpret_cast<const v4i *>(crd + p0 + i);
                const v2d *pv = reinterpret_cast<const v2d *>(vals + p0 + i);
                v4i cv;
                v2d x, y;
                if constexpr (decltype(around)::value) {
                    cv = __builtin_nontemporal_load(pc); x = __builtin_nontemporal_load(pv); y = __builtin_nontemporal_load(pv + 1);
                } else {
                    cv = pc[0]; x = pv[0]; y = pv[1];
                }
                c[0] = cv.x; c[1] = cv.y; c[2] = cv.z; c[3] = cv.w;
                a[0] = x.x; a[1] = x.y; a[2] = y.x; a[3] = y.y;
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) { const bool in = i + u < n_items; c[u] = in ? crd[p0 + i + u] : 0; a[u] = in ? vals[p0 + i + u] : 0.0; }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) item[i + u] = Item{(unsigned)c[u] * unit, 0u, a[u]};
        }
    };
    if (stream) stage(IntC<1>{}); else stage(IntC<0>{});
    for (int i = threadIdx.x; i < np; i += 256) piece[i] = pieces[(size_t)first_piece + i];
    __syncthreads();

    // The wavefront's number and the length of a short batch: in scalar registers for wide rows (60 000 nonzeros, rank 53, level with
    // vector ones at 20 us); narrow ones are slower with them (the 10^6 x 10^6 matrix, rank 32, 447.4 and 445.8).
    auto uniform = [](int x) { if constexpr (V > 2) return __builtin_amdgcn_readfirstlane(x); else return x; };
    const int k = threadIdx.x % L, gw = (threadIdx.x & 63) / L, wave = uniform(threadIdx.x >> 6);
    const RowOf<L, E, NL, FULL> rw(R, k);
    const char *base = reinterpret_cast<const char *>(Dn);
    const Item *items = item + lead;
    auto result_row = [&](uint32_t pd) {
        const int s = t0.y + (piece_is_part(pd) ? 0 : piece_num(pd));
        return ROWMAP ? rowmap[s] : s;
    };
    auto finish = [&](uint32_t pd, int r, const double *acc) {
        if (piece_is_part(pd)) rw.put(part + piece_num(pd) * kRow, acc);
        else rw.store_result(out + (int64_t)r * R, acc, ep, piece_len(pd) == 0);
    };
    // Longest pieces first: batches of one piece per group until the longest piece of a batch is short.
    int b = wave * KP;
    for (; b < np; b += 4 * KP) {
        const int longest = __builtin_amdgcn_readfirstlane(piece_len(piece[b]));
        if (longest <= 2 * G) break;
        const bool mine = b + gw < np;
        const uint32_t pd = piece[mine ? b + gw : b];
        const int len = mine ? piece_len(pd) : 0;
        const int shortest = b + KP <= np ? __builtin_amdgcn_readfirstlane(piece_len(piece[b + KP - 1])) : 0;
        const int r = result_row(pd);
        const Item *it = items + piece_start(pd);
        const int last = len > 0 ? len - 1 : 0;
        // Groups of loads, and the nonzeros that fill none: wide rows have them first in the queue of loads, narrow ones, whose
        // kernels would lose a wavefront per SIMD to the registers that costs, last.
        constexpr bool kEarly = V > 2;
        const int full = spread ? 2 * ((longest + 2 * G - 1) / (2 * G)) + 1 : longest / G, left = spread ? 0 : longest - full * G;
        double acc[V], row[2][G][V], val[2][G], rrow[G][V], rval[G];
#pragma unroll
        for (int q = 0; q < V; ++q) acc[q] = 0.0;
        auto issue_left = [&](double (*d)[V], double *v) {
#pragma unroll
            for (int u = 0; u < G - 1; ++u)
                if (u < left) {
                    const Item x = it[full * G + u < last ? full * G + u : last];
                    v[u] = x.val;
                    rw.template load<BIG>(base, x.off, d[u]);
                }
        };
        auto consume_left = [&](const double (*d)[V], const double *v) {
#pragma unroll
            for (int u = 0; u < G - 1; ++u)
                if (u < left && full * G + u < len) {
#pragma unroll
                    for (int q = 0; q < V; ++q) acc[q] = fma(v[u], d[u][q], acc[q]);
                }
        };
        if constexpr (kEarly) issue_left(rrow, rval);
        auto issue = [&](int g, double (*d)[V], double *v) {
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const Item x = it[g * G + u < last ? g * G + u : last];
                v[u] = x.val;
                rw.template load<BIG>(base, x.off, d[u]);
            }
        };
        auto consume = [&](int g, const double (*d)[V], const double *v) {
            if (g * G + G <= shortest) {
#pragma unroll
                for (int u = 0; u < G; ++u)
#pragma unroll
                    for (int q = 0; q < V; ++q) acc[q] = fma(v[u], d[u][q], acc[q]);
            } else {
#pragma unroll
                for (int u = 0; u < G; ++u)
                    if (g * G + u < len) {
#pragma unroll
                        for (int q = 0; q < V; ++q) acc[q] = fma(v[u], d[u][q], acc[q]);
                    }
            }
        };
        // a group is in flight while the one before it is used; none of these loads is under a condition, which would make
        // the wait for a group cover the next one too
        issue(0, row[0], val[0]);
        int g = 0;
        for (; g + 2 < full; g += 2) {
            issue(g + 1, row[1], val[1]);
            consume(g, row[0], val[0]);
            issue(g + 2, row[0], val[0]);
            consume(g + 1, row[1], val[1]);
        }
        if (g + 1 < full) {
            issue(g + 1, row[1], val[1]);
            consume(g, row[0], val[0]);
            if constexpr (!kEarly) issue_left(row[0], val[0]);
            consume(g + 1, row[1], val[1]);
            if constexpr (!kEarly) consume_left(row[0], val[0]);
        } else {
            if constexpr (!kEarly) issue_left(row[1], val[1]);
            consume(g, row[0], val[0]);
            if constexpr (!kEarly) consume_left(row[1], val[1]);
        }
        if constexpr (kEarly) consume_left(rrow, rval);
        if (mine) finish(pd, r, acc);
    }
    // Short pieces: KB of them per group at the same time.
    for (; b < np; b += 4 * KP * KB) {
        const int longest = uniform(piece_len(piece[b]));
        uint32_t pd[KB];
        int len[KB], r[KB];
        double acc[KB][V];
#pragma unroll
        for (int m = 0; m < KB; ++m) {
            const int i = b + 4 * KP * m + gw;
            pd[m] = i < np ? piece[i] : 0u;
            len[m] = i < np ? piece_len(pd[m]) : -1;
            r[m] = result_row(pd[m]);
#pragma unroll
            for (int q = 0; q < V; ++q) acc[m][q] = 0.0;
        }
        double row[2][KB][V], val[2][KB];
        auto issue = [&](int j, double (*d)[V], double *v) {
#pragma unroll
            for (int m = 0; m < KB; ++m) {
                const Item x = items[j < len[m] ? piece_start(pd[m]) + j : 0];
                v[m] = x.val;
                rw.template load<BIG>(base, x.off, d[m]);
            }
        };
        auto consume = [&](int j, const double (*d)[V], const double *v) {
#pragma unroll
            for (int m = 0; m < KB; ++m)
                if (j < len[m]) {
#pragma unroll
                    for (int q = 0; q < V; ++q) acc[m][q] = fma(v[m], d[m][q], acc[m][q]);
                }
        };
        if (longest > 0) issue(0, row[0], val[0]);
        for (int j = 0; j < longest; j += 2) {
            if (j + 1 < longest) issue(j + 1, row[1], val[1]);
            consume(j, row[0], val[0]);
            if (j + 1 >= longest) break;
            if (j + 2 < longest) issue(j + 2, row[0], val[0]);
            consume(j + 1, row[1], val[1]);
        }
#pragma unroll
        for (int m = 0; m < KB; ++m)
            if (len[m] >= 0) finish(pd[m], r[m], acc[m]);
    }
    if (nj == 0) return;
    __syncthreads();
    for (int i = threadIdx.x / L; i < nj; i += 256 / L) {
        const uint32_t jn = joins[t0.w + i];
        const double *ps = part + join_slot(jn) * kRow;
        double sum[V], v[V];
#pragma unroll
        for (int q = 0; q < V; ++q) sum[q] = 0.0;
        const int n = join_count(jn);
        for (int m = 0; m < n; ++m) {
            rw.get(ps + m * kRow, v);
#pragma unroll
            for (int q = 0; q < V; ++q) sum[q] += v[q];
        }
        const int to = join_to(jn);
        if (to == kJoinRow) {
            const int s = t0.y + join_seg(jn);
            rw.store_result(out + (int64_t)(ROWMAP ? rowmap[s] : s) * R, sum, ep);
        } else {
            rw.store((to == kJoinHead ? head : tail) + (int64_t)t * R, sum);
        }
    }
}

// Segments cut by tile boundaries: what the first tile holds of one behind its boundary, then what the following tiles
// hold in front of theirs.  A thread per (segment, column); the last workgroups of the grid take the segments over many
// tiles, one each, with the tiles dealt over 256 / R threads per column.
__global__ void __launch_bounds__(256) k_piece_cut_sums(const int4 *__restrict__ cuts, int ncut, int nlong, int64_t ntiles,
                                                        const double *__restrict__ head, const double *__restrict__ tail, int R,
                                                        const int32_t *__restrict__ rowmap, double *__restrict__ out, Epilogue ep) {
    __shared__ double sums[256];
    const int narrow = (int)gridDim.x - nlong;
    if ((int)blockIdx.x < narrow) {
        const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
        if (g >= (int64_t)ncut * R) return;
        const int i = (int)(g / R), r = (int)(g - (int64_t)i * R);
        const int4 c = cuts[i];
        double s = tail[(int64_t)c.y * R + r];
        for (int t = c.y + 1; t <= c.z; ++t) s += head[(int64_t)t * R + r];
        double *o = out + (int64_t)(rowmap ? rowmap[c.x] : c.x) * R + r;
        *o = ep_apply(ep, s, o);
        return;
    }
    const int4 c = cuts[ntiles - 1 - ((int)blockIdx.x - narrow)];
    // thread (lane, r): tiles lane, lane + nl, ...; R <= 128, so at least two lanes of tiles
    const int nl = 256 / R, lane = threadIdx.x / R, r = threadIdx.x - lane * R;
    double s = 0.0;
    if (lane < nl) {
        if (lane == 0) s = tail[(int64_t)c.y * R + r];
        for (int64_t t = c.y + 1 + lane; t <= c.z; t += nl) s += head[t * R + r];
        sums[threadIdx.x] = s;
    }
    __syncthreads();
    if (lane != 0) return;
    for (int m = 1; m < nl; ++m) s += sums[m * R + r];
    double *o = out + (int64_t)(rowmap ? rowmap[c.x] : c.x) * R + r;
    *o = ep_apply(ep, s, o);
}

struct PieceArgs {
    const PiecePlan &plan;
    const int32_t *crd;
    const double *vals;
    const int32_t *rowmap;
    const double *Dn;
    double *out;
    int64_t nnz;
    int R, spread;
    double *head, *tail;
    hipStream_t st;
    Epilogue ep;
};

template <int L, int E, int NL, bool FULL, bool BIG>
hipError_t launch_pieces(const PieceArgs &a) {
    const int lds = lds_parts_at(a.plan.units) + a.plan.max_parts * L * E * NL * 8;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)a.plan.ntiles), dim3(256), (unsigned)lds, a.st, (const int4 *)a.plan.tiles(),
                           (const uint32_t *)a.plan.pieces(), (const uint32_t *)a.plan.joins(), a.plan.units, a.plan.units == kUnitsLarge,
                           a.spread, a.crd, a.vals, a.rowmap, a.Dn, a.out, a.nnz, a.R, a.head, a.tail, a.ep);
    };
    if (lds > 64 * 1024) {
        static const hipError_t allowed[2] = {
            hipFuncSetAttribute((const void *)k_pieces<L, E, NL, FULL, BIG, false>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024),
            hipFuncSetAttribute((const void *)k_pieces<L, E, NL, FULL, BIG, true>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)};
        if (allowed[a.rowmap ? 1 : 0] != hipSuccess) return allowed[a.rowmap ? 1 : 0];
    }
    if (a.rowmap) go(k_pieces<L, E, NL, FULL, BIG, true>); else go(k_pieces<L, E, NL, FULL, BIG, false>);
    return hipGetLastError();
}

// Whether a part of the list as long as an XCD works on at a time reads more of the operand than its L2 gives back, so that most
// rows come from behind it; in whole lines of 128 bytes.  With the loads behind the pieces' ends and without: nine nonzeros per row
// at random, rank 32, 100 000 columns (24 MB by this count) 37.7 and 36.5 us, 150 000 (32 MB) 53.3 and 54.0, 300 000 105 and 110;
// rank 10, 300 000 (35 MB) 68.9 and 69.0, 500 000 118 and 120; 1 M columns, rank 32, at most 20 000 from the diagonal (18 MB) 278 and 253,
// 100 000 (38 MB) 323 and 338; TTM over 400 000 rows that follow a power law (25 MB and less) 242 and 240, 199 and 193.
int spread_rows(const PiecePlan &plan, int R) {
    const int64_t row = R % 16 ? R * 8 + 120 : R * 8;
    return plan.distinct * row >= int64_t(30) << 20;
}

}  // namespace

size_t piece_scratch_bytes(const PiecePlan &plan, int64_t R) { return (size_t)plan.ntiles * (size_t)R * 2 * sizeof(double); }

hipError_t piece_rows(const PiecePlan &plan, const int32_t *crd, const double *vals, int64_t nnz, const int32_t *rowmap, const double *Dn,
                      int64_t dense_rows, int R, double *out, void *scratch, hipStream_t st, Epilogue ep) {
    double *head = (double *)scratch, *tail = head + plan.ntiles * R;
    const PieceArgs a{plan, crd, vals, rowmap, Dn, out, nnz, R, spread_rows(plan, R), head, tail, st, ep};
    const bool big = dense_rows * R * 8 >= (int64_t(1) << 32);    // row offsets in bytes no longer fit 32 bits
    const hipError_t e = COMET_DISPATCH_RANK(launch_pieces, R, big, a);
    if (e != hipSuccess || plan.ncut + plan.ncut_long == 0) return e;
    const int64_t narrow = (plan.ncut * R + 255) / 256;
    hipLaunchKernelGGL(k_piece_cut_sums, dim3((unsigned)(narrow + plan.ncut_long)), dim3(256), 0, st, (const int4 *)plan.cuts(),
                       (int)plan.ncut, (int)plan.ncut_long, plan.ntiles, (const double *)head, (const double *)tail, R, rowmap, out, ep);
    return hipGetLastError();
}

}  // namespace comet

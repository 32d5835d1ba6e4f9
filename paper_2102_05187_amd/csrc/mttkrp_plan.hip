// Builds the plan of the MTTKRP kernel (see mttkrp_plan.hpp); runs once per tensor.
#include "mttkrp_plan.hpp"

#include "kernels.hpp"

namespace comet {

namespace {

// Boundary of tile t: the first nonzero behind it, the fiber it lies in (or starts at), and how many slices have ended in
// front of it.  In the order "a fiber's nonzeros, then the fiber itself" the boundary is unit t * units.
__global__ void __launch_bounds__(256) k_mt_bounds(const int32_t *__restrict__ pos2, int64_t nslice, const int32_t *__restrict__ pos3,
                                                   int64_t nfib, int64_t nnz, int units, int64_t ntiles, int4 *__restrict__ bounds) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t > ntiles) return;
    const int64_t d = t * units;
    if (t == 0) { bounds[0] = make_int4(0, 0, 0, 0); return; }
    if (t == ntiles || d >= nnz + nfib) { bounds[t] = make_int4((int)nnz, (int)nfib, (int)nslice, 0); return; }
    int64_t lo = 0, hi = nfib - 1;                           // smallest fiber f with pos3[f + 1] + f + 1 > d
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)pos3[mid + 1] + mid + 1 > d) hi = mid; else lo = mid + 1;
    }
    int64_t f = lo;
    const int64_t b = pos3[f], e = pos3[f + 1];
    int64_t p = d - f;
    if (p > e) p = e;
    if (e - b <= kMtSnap) p = b;                             // the whole short fiber goes to this tile
    if (p == e && e > b) f += 1;                             // all of it belongs to the tile before
    lo = 0; hi = nslice;                                     // slices whose last fiber lies in front of f
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)pos2[mid + 1] <= f) lo = mid + 1; else hi = mid;
    }
    bounds[t] = make_int4((int)p, (int)f, (int)lo, 0);
}

// Whether slice s, which has not ended in front of the boundary, has nonzeros in front of it.
__device__ __forceinline__ bool crosses(const int4 &bound, int64_t s, int64_t nslice, const int32_t *pos2, const int32_t *pos3) {
    return s < nslice && pos3[pos2[s]] < bound.x;
}

// The pieces and records of tile t; FILL = false only counts them.
template <bool FILL>
__global__ void __launch_bounds__(256) k_mt_fill(const int32_t *__restrict__ pos2, const int32_t *__restrict__ crd1, int64_t nslice,
                                                 const int32_t *__restrict__ pos3, const int32_t *__restrict__ crd2, int64_t nfib,
                                                 int64_t ntiles, int64_t dim0, const int4 *__restrict__ bounds,
                                                 uint64_t *__restrict__ counts, int *__restrict__ most, int4 *__restrict__ tiles,
                                                 uint2 *__restrict__ pieces, uint2 *__restrict__ recs) {
    __shared__ int before[kMtItems + 2];                       // pieces in front of each fiber of the tile
    __shared__ int bin[64], wave_sum[4], nsum, njoin, at_sum, at_join;
    const int64_t t = blockIdx.x;
    const int4 a = bounds[t], b = bounds[t + 1];
    const int p0 = a.x, p1 = b.x, f0 = a.y;
    const int f1 = b.y + (b.y < nfib && pos3[b.y] < p1 ? 1 : 0);           // fibers [f0, f1), the last of them possibly continued
    const int nf = f1 - f0, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x < 64) bin[threadIdx.x] = 0;
    if (threadIdx.x == 0) { nsum = 0; njoin = 0; at_sum = 0; at_join = 0; before[0] = 0; }
    __syncthreads();
    auto cut = [&](int f, int &lo, int &n, int &np) {
        const int fb = pos3[f], fe = pos3[f + 1], hi = fe < p1 ? fe : p1;
        lo = fb > p0 ? fb : p0;
        n = hi - lo;
        np = n <= 0 ? 0 : (n <= kMtWhole ? 1 : (n + kMtPiece - 1) / kMtPiece);
    };
    int total = 0;
    for (int i0 = 0; i0 < nf; i0 += 256) {
        const int i = i0 + (int)threadIdx.x;
        int lo = 0, n = 0, np = 0;
        if (i < nf) cut(f0 + i, lo, n, np);
        int sum = np;
        for (int d = 1; d < 64; d *= 2) { const int y = __shfl_up(sum, d); if (lane >= d) sum += y; }
        if (lane == 63) wave_sum[wave] = sum;
        __syncthreads();
        int front = total;
        for (int w = 0; w < wave; ++w) front += wave_sum[w];
        if (i < nf) before[i + 1] = front + sum;
        total += wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
        __syncthreads();
    }
    if (FILL) {
        for (int i = threadIdx.x; i < nf; i += 256) {
            int lo, n, np;
            cut(f0 + i, lo, n, np);
            if (np == 0) continue;
            const int base = n / np, extra = n - np * base;    // `extra` pieces of base + 1 nonzeros, the others of base
            if (extra) atomicAdd(&bin[base + 1], extra);
            atomicAdd(&bin[base], np - extra);
        }
        __syncthreads();
        if (threadIdx.x < 64) {                                // first place of every length, longest first
            const int n = bin[63 - lane];
            int at = n;
            for (int d = 1; d < 64; d *= 2) { const int y = __shfl_up(at, d); if (lane >= d) at += y; }
            bin[63 - lane] = at - n;
        }
        __syncthreads();
        uint2 *pc = pieces + (uint32_t)counts[t];
        for (int i = threadIdx.x; i < nf; i += 256) {
            int lo, n, np;
            cut(f0 + i, lo, n, np);
            if (np == 0) continue;
            const int base = n / np, extra = n - np * base;
            int at = lo - p0;
            for (int q = 0; q < np; ++q) {
                const int len = base + (q < extra ? 1 : 0);
                pc[atomicAdd(&bin[len], 1)] = make_uint2(mt_piece(at, len, before[i] + q), (unsigned)crd2[f0 + i]);
                at += len;
            }
        }
    }
    // slices that end in the tile, and the one that goes on behind it
    const bool cont = crosses(a, a.z, nslice, pos2, pos3), open = crosses(b, b.z, nslice, pos2, pos3);
    const int64_t nend = (int64_t)b.z - a.z, nsl = nend + (open ? 1 : 0);
    auto each = [&](auto &&sum, auto &&join) {
        for (int64_t q = threadIdx.x; q < nsl; q += 256) {
            const int64_t s = a.z + q;
            int lo = pos2[s] - f0, hi = pos2[s + 1] - f0;      // fibers of the slice inside the tile
            lo = lo < 0 ? 0 : (lo > nf ? nf : lo);
            hi = hi < lo ? lo : (hi > nf ? nf : hi);
            const int r0 = before[lo], n = before[hi] - r0, row = crd1[s];
            const bool cn = cont && q == 0, op = q == nend;
            const int gap = op ? 0 : mt_gap(s > 0 ? crd1[s - 1] : -1, row);
            if (!cn && !op && n <= kMtSum) { sum(mt_sum(r0, n, kMtSlice, gap), row); continue; }
            if (gap > 0) sum(mt_sum(0, 0, kMtGap, gap), row);
            for (int c = 0; c < n; c += kMtSum)
                if (n - c > 1) sum(mt_sum(r0 + c, n - c < kMtSum ? n - c : kMtSum, kMtPart, 0), row);
            join(mt_join(r0, n, cn, op), row);
        }
        if (threadIdx.x == 0 && t == ntiles - 1) {             // rows of M behind the last stored one
            const int gap = mt_gap(crd1[nslice - 1], dim0);
            if (gap > 0) sum(mt_sum(0, 0, kMtGap, gap), (int)dim0);
        }
    };
    each([&](unsigned, int) { atomicAdd(&nsum, 1); }, [&](unsigned, int) { atomicAdd(&njoin, 1); });
    __syncthreads();
    if (!FILL) {
        if (threadIdx.x == 0) {
            counts[t] = (uint64_t)(uint32_t)total | ((uint64_t)(uint32_t)(nsum + njoin) << 32);
            // few tiles raise a maximum; atomics of all of them on one address would queue up
            if (total > __hip_atomic_load(most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(most, total);
            if (p1 - p0 > __hip_atomic_load(most + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(most + 1, p1 - p0);
        }
        return;
    }
    if (threadIdx.x == 0)
        tiles[t] = make_int4(p0, (int)(uint32_t)counts[t], (int)(uint32_t)(counts[t] >> 32),
                             njoin);
    uint2 *sums = recs + (uint32_t)(counts[t] >> 32), *joins = sums + nsum;
    each([&](unsigned what, int row) { sums[atomicAdd(&at_sum, 1)] = make_uint2(what, (unsigned)row); },
         [&](unsigned what, int row) { joins[atomicAdd(&at_join, 1)] = make_uint2(what, (unsigned)row); });
}

__global__ void k_mt_end(int4 *__restrict__ tiles, int64_t ntiles, int nnz, int npieces, int nrecs) {
    tiles[ntiles] = make_int4(nnz, npieces, nrecs, 0);
}

// Slices that begin in a tile and go on behind it: {row of M, first tile, last tile}.
__global__ void __launch_bounds__(256) k_mt_cuts(const int32_t *__restrict__ pos2, const int32_t *__restrict__ crd1, int64_t nslice,
                                                 const int32_t *__restrict__ pos3, const int4 *__restrict__ bounds, int64_t ntiles,
                                                 int4 *__restrict__ cuts, int *__restrict__ counters) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t + 1 >= ntiles) return;
    const int4 begin = bounds[t], bound = bounds[t + 1];
    const int64_t s = bound.z;
    if (!crosses(bound, s, nslice, pos2, pos3)) return;
    if (begin.z == s && crosses(begin, s, nslice, pos2, pos3)) return;      // it began in front of the tile
    const int end = pos2[s + 1];
    int64_t lo = t + 1, hi = ntiles - 1;                       // last tile that starts before the slice's end
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (bounds[mid].y < end) lo = mid; else hi = mid - 1;
    }
    const int4 c = make_int4(crd1[s], (int)t, (int)lo, 0);
    if (c.z - c.y < kMtLongCut) cuts[atomicAdd(&counters[0], 1)] = c;
    else cuts[ntiles - 1 - atomicAdd(&counters[1], 1)] = c;
}

unsigned grid_for(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t mttkrp_plan_build(const int32_t *pos2, const int32_t *crd1, int64_t nslice, const int32_t *pos3, const int32_t *crd2,
                             int64_t nfib, int64_t nnz, int64_t dim0, MttkrpPlan &plan, hipStream_t st) {
    plan = MttkrpPlan();
    if (nfib < 1 || nnz < 1 || nslice < 1) return hipSuccess;
    auto fail = [&](hipError_t e) { plan = MttkrpPlan(); return e; };
    int64_t units = (nnz + nfib) / 1024;
    units = units < kMtUnitsMin ? kMtUnitsMin : (units > kMtUnitsMax ? kMtUnitsMax : units);
    const int64_t ntiles = (nnz + nfib + units - 1) / units;
    plan.ntiles = ntiles;
    plan.tiles_mem = dev_alloc(sizeof(int4) * (2 * ntiles + 1));
    // temporary: the boundaries, pieces and records of each tile, their sums before each tile, counters (short cuts, long
    // cuts, most pieces and nonzeros in a tile), and what the scan asks for
    size_t tb = 0;
    hipError_t e = reorder_scan_flags(nullptr, &tb, (uint64_t *)nullptr, (uint64_t *)nullptr, ntiles + 1, st);
    if (e != hipSuccess) return fail(e);
    const size_t bounds_at = ((size_t)(2 * (ntiles + 1) + 2) * sizeof(uint64_t) + 255) & ~(size_t)255;
    const size_t scan_at = (bounds_at + (size_t)(ntiles + 1) * sizeof(int4) + 255) & ~(size_t)255;
    DevRef temp = dev_alloc(scan_at + tb);
    if (!plan.tiles_mem || !temp) return fail(hipErrorOutOfMemory);
    uint64_t *cn = (uint64_t *)temp->ptr, *bf = cn + ntiles + 1;
    int *counters = (int *)(bf + ntiles + 1);
    int4 *bounds = (int4 *)((char *)temp->ptr + bounds_at);
    hipLaunchKernelGGL(k_mt_bounds, dim3(grid_for(ntiles + 1)), dim3(256), 0, st, pos2, nslice, pos3, nfib, nnz, (int)units, ntiles, bounds);
    e = hipMemsetAsync(cn + ntiles, 0, sizeof(uint64_t), st);
    if (e == hipSuccess) e = hipMemsetAsync(counters, 0, 4 * sizeof(int), st);
    if (e != hipSuccess) return fail(e);
    hipLaunchKernelGGL((k_mt_fill<false>), dim3((unsigned)ntiles), dim3(256), 0, st, pos2, crd1, nslice, pos3, crd2, nfib, ntiles, dim0,
                       (const int4 *)bounds, cn, counters + 2, (int4 *)nullptr, (uint2 *)nullptr, (uint2 *)nullptr);
    hipLaunchKernelGGL(k_mt_cuts, dim3(grid_for(ntiles)), dim3(256), 0, st, pos2, crd1, nslice, pos3, (const int4 *)bounds, ntiles,
                       plan.cuts(), counters);
    e = reorder_scan_flags((char *)temp->ptr + scan_at, &tb, cn, bf, ntiles + 1, st);
    struct { uint64_t total; int short_cuts, long_cuts, pieces, items; } sums = {0, 0, 0, 0, 0};    // bf[ntiles] and the counters
    if (e == hipSuccess) e = hipMemcpyAsync(&sums, bf + ntiles, sizeof sums, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(e);
    plan.npieces = (int64_t)(uint32_t)sums.total;
    plan.nrecs = (int64_t)(uint32_t)(sums.total >> 32);
    plan.ncut = sums.short_cuts;
    plan.ncut_long = sums.long_cuts;
    plan.max_pieces = sums.pieces;
    plan.max_items = sums.items;
    plan.pieces_mem = dev_alloc(sizeof(uint2) * (size_t)(plan.npieces + plan.nrecs));
    if (!plan.pieces_mem) return fail(hipErrorOutOfMemory);
    hipLaunchKernelGGL((k_mt_fill<true>), dim3((unsigned)ntiles), dim3(256), 0, st, pos2, crd1, nslice, pos3, crd2, nfib, ntiles, dim0,
                       (const int4 *)bounds, bf, (int *)nullptr, plan.tiles(), plan.pieces(), plan.recs());
    hipLaunchKernelGGL(k_mt_end, dim3(1), dim3(1), 0, st, plan.tiles(), ntiles, (int)nnz, (int)plan.npieces, (int)plan.nrecs);
    e = hipStreamSynchronize(st);                              // the temporaries go out of scope
    return e == hipSuccess ? hipGetLastError() : fail(e);
}

}  // namespace comet

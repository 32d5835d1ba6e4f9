// Builds the piece plan of a compressed level (see pieces.hpp); runs once per tensor.
#include "pieces.hpp"

#include <cmath>

#include "kernels.hpp"

namespace comet {

namespace {

// Boundary of tile t: the segment s it lies in (or starts at) and the first nonzero of the tile.  In the order "a
// segment's nonzeros, then the segment itself" the boundary is unit t * units: the smallest s whose end lies beyond it.
__global__ void __launch_bounds__(256) k_piece_tiles(const int32_t *__restrict__ pos, int64_t nseg, int64_t nnz, int units,
                                                     int64_t ntiles, int4 *__restrict__ tiles) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t > ntiles) return;
    int64_t s = nseg, p = nnz;
    const int64_t d = t * units;
    if (d < nnz + nseg) {
        int64_t lo = 0, hi = nseg - 1;                       // smallest s with pos[s + 1] + s + 1 > d
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if ((int64_t)pos[mid + 1] + mid + 1 > d) hi = mid; else lo = mid + 1;
        }
        s = lo;
        const int64_t b = pos[s], e = pos[s + 1];
        p = d - s;
        if (p > e) p = e;
        if (e - b <= kSnap) p = b;                           // the whole short segment goes to this tile
        if (p == e && e > b) { p = e; s += 1; }              // all of it belongs to the tile before
    }
    tiles[t] = make_int4((int)p, (int)s, 0, 0);
}

// The pieces and joins of tile t; FILL = false only counts them.
template <bool FILL>
__global__ void __launch_bounds__(256) k_piece_fill(const int32_t *__restrict__ pos, int64_t nseg, int64_t ntiles, int4 *__restrict__ tiles,
                                                    uint64_t *__restrict__ counts, int *__restrict__ max_parts,
                                                    uint32_t *__restrict__ pieces, uint32_t *__restrict__ joins) {
    __shared__ int bin[64], nwhole, npart, njoin;
    const int64_t t = blockIdx.x;
    const int4 a = tiles[t], b = tiles[t + 1];
    const int p0 = a.x, p1 = b.x, s0 = a.y;
    // segments of the tile: [s0, s1), the last of them possibly continued
    const int s1 = b.y + (b.y < nseg && pos[b.y] < p1 ? 1 : 0);
    if (threadIdx.x < 64) bin[threadIdx.x] = 0;
    if (threadIdx.x == 0) { nwhole = 0; npart = 0; njoin = 0; }
    __syncthreads();
    auto each = [&](auto &&whole, auto &&cut) {
        for (int i = threadIdx.x; i < s1 - s0; i += 256) {      // a count: segment numbers end just below 2^31
            const int s = s0 + i, sb = pos[s], se = pos[s + 1];
            const int lo = sb > p0 ? sb : p0, hi = se < p1 ? se : p1, n = hi - lo;
            const bool begins = sb >= p0, ends = se <= p1;
            if (begins && ends && n <= kWhole) whole(s, lo, n);
            else cut(s, lo, n, ends ? (begins ? kJoinRow : kJoinHead) : (begins ? kJoinTail : kJoinHead));
        }
    };
    if (!FILL) {
        each([&](int, int, int) { atomicAdd(&nwhole, 1); },
             [&](int, int, int n, int) { atomicAdd(&npart, (n + kPiece - 1) / kPiece); atomicAdd(&njoin, 1); });
        __syncthreads();
        if (threadIdx.x == 0) {
            counts[t] = (uint64_t)(uint32_t)(nwhole + npart) | ((uint64_t)(uint32_t)njoin << 32);
            // few tiles raise the maximum; atomics of all of them on one address would queue up
            if (npart > __hip_atomic_load(max_parts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(max_parts, npart);
        }
        return;
    }
    // a segment in np pieces: `extra` of them hold base + 1 nonzeros, the others base
    each([&](int, int, int n) { atomicAdd(&bin[n], 1); },
         [&](int, int, int n, int) {
             const int np = (n + kPiece - 1) / kPiece, base = n / np, extra = n - np * base;
             if (extra) atomicAdd(&bin[base + 1], extra);
             atomicAdd(&bin[base], np - extra);
         });
    __syncthreads();
    if (threadIdx.x < 64) {                                     // first place of every length, longest first
        const int lane = threadIdx.x, n = bin[63 - lane];
        int at = n;
        for (int d = 1; d < 64; d *= 2) { const int y = __shfl_up(at, d); if (lane >= d) at += y; }
        bin[63 - lane] = at - n;
    }
    if (threadIdx.x == 0) {
        tiles[t].z = (int)(uint32_t)counts[t];
        tiles[t].w = (int)(uint32_t)(counts[t] >> 32);
    }
    __syncthreads();
    uint32_t *pc = pieces + (uint32_t)counts[t], *jn = joins + (uint32_t)(counts[t] >> 32);
    // an empty segment starts nowhere: behind the tile's last nonzero there is none that its lanes could read beside longer pieces
    each([&](int s, int lo, int n) { pc[atomicAdd(&bin[n], 1)] = piece_pack(n ? lo - p0 : 0, n, s - s0, 0); },
         [&](int s, int lo, int n, int to) {
             const int np = (n + kPiece - 1) / kPiece, base = n / np, extra = n - np * base;
             const int slot = atomicAdd(&npart, np);
             int at = lo - p0;
             for (int q = 0; q < np; ++q) {
                 const int len = base + (q < extra ? 1 : 0);
                 pc[atomicAdd(&bin[len], 1)] = piece_pack(at, len, slot + q, 1);
                 at += len;
             }
             jn[atomicAdd(&njoin, 1)] = join_pack(slot, np, s - s0, to);
         });
}

__global__ void k_piece_end(int4 *__restrict__ tiles, int64_t ntiles, int npieces, int njoins) {
    tiles[ntiles].z = npieces;
    tiles[ntiles].w = njoins;
}

constexpr int kLongCut = 16;           // tiles from which on a cut segment is summed by a whole workgroup

// Segments that begin in a tile and go on behind it.
__global__ void __launch_bounds__(256) k_piece_cuts(const int32_t *__restrict__ pos, int64_t nseg, const int4 *__restrict__ tiles,
                                                    int64_t ntiles, int4 *__restrict__ cuts, int *__restrict__ counters) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t + 1 >= ntiles) return;
    const int p0 = tiles[t].x, p1 = tiles[t + 1].x, s = tiles[t + 1].y;
    if (s >= nseg || pos[s] >= p1 || pos[s] < p0) return;
    const int e = pos[s + 1];
    int64_t lo = t + 1, hi = ntiles - 1;                     // last tile that starts before the segment's end
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (tiles[mid].x < e) lo = mid; else hi = mid - 1;
    }
    const int4 c = make_int4(s, (int)t, (int)lo, 0);
    if (lo - t < kLongCut) cuts[atomicAdd(&counters[0], 1)] = c;
    else cuts[ntiles - 1 - atomicAdd(&counters[1], 1)] = c;
}

// A workgroup sets a bit per coordinate of a sample (samples spread evenly over the list).  kSamples of kSampleNnz nonzeros, of all
// together, sums[0]: the bits that are set; sums[1]: how many of the first kSampleLook of the sample behind find theirs set.  Behind these, kLooks
// of kSampleLook, sums[2]: the bits that are set; and as many of the coordinates `parent` of the segments, sums[3].
constexpr int kSampleBits = 1 << 18;
__global__ void __launch_bounds__(1024) k_piece_sample(const int32_t *__restrict__ leaf, int64_t nnz, const int32_t *__restrict__ parent, int64_t nseg,
                                                       int *__restrict__ sums) {
    __shared__ uint32_t bits[kSampleBits / 32];
    const int look = (int)blockIdx.x - kSamples;                 // negative: one of the large samples
    const int32_t *crd = look < kLooks ? leaf : parent;
    const int64_t total = look < kLooks ? nnz : nseg, most = look < 0 ? kSampleNnz : kSampleLook, n = total < most ? total : most;
    const int samples = look < 0 ? kSamples : kLooks, mine = look < 0 ? (int)blockIdx.x : look % kLooks;
    for (int i = threadIdx.x; i < kSampleBits / 32; i += 1024) bits[i] = 0u;
    __syncthreads();
    auto begin = [&](int s) { return (total - n) / (samples - 1) * (s % samples); };
    auto batch = [&](int64_t at, int64_t i, auto use) {          // nonzeros i, i + 1024, ... of the sample that begins at `at`
        uint32_t c[32];
#pragma unroll
        for (int q = 0; q < 32; ++q) c[q] = (uint32_t)crd[at + (i + q * 1024 < n ? i + q * 1024 : i)];
#pragma unroll
        for (int q = 0; q < 32; ++q) use((c[q] * 0x9E3779B1u) >> 14);
    };
    auto add_up = [&](int v, int *to) {
        for (int d = 32; d > 0; d >>= 1) v += __shfl_down(v, d);
        if ((threadIdx.x & 63) == 0) atomicAdd(to, v);
    };
    for (int64_t i = threadIdx.x; i < n; i += 32 * 1024)
        batch(begin(mine), i, [&](uint32_t h) { atomicOr(&bits[h >> 5], 1u << (h & 31u)); });
    __syncthreads();
    int set = 0, found = 0;
    for (int i = threadIdx.x; i < kSampleBits / 32; i += 1024) set += __popc(bits[i]);
    add_up(set, &sums[look < 0 ? 0 : look < kLooks ? 2 : 3]);
    if (look >= 0) return;
    static_assert(kSampleLook == 32 * 1024, "one batch");
    if (threadIdx.x < n) batch(begin(mine + 1), threadIdx.x, [&](uint32_t h) { found += (bits[h >> 5] >> (h & 31u)) & 1u; });
    add_up(found, &sums[1]);
}

unsigned grid_for(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t piece_plan_build(const int32_t *pos, int64_t nseg, const int32_t *crd, int64_t nnz, const int32_t *parent, PiecePlan &plan, hipStream_t st) {
    plan = PiecePlan();
    if (nseg < 1 || nnz < 1) return hipSuccess;
    auto fail = [&](hipError_t e) { plan = PiecePlan(); return e; };
    const int64_t units = nnz >= kStreamNnz ? kUnitsLarge : kUnitsSmall, ntiles = (nnz + nseg + units - 1) / units;
    plan.nseg = nseg;
    plan.units = (int)units;
    plan.ntiles = ntiles;
    plan.tiles_mem = dev_alloc(sizeof(int4) * (2 * ntiles + 1));
    // temporary: pieces and joins of each tile, their sums before each tile, counters (short cuts, long cuts, most partial
    // sums in a tile, bits set by the samples and found in them), and what the scan asks for.  One allocation: each costs a small handle's creation 10 us and more
    size_t tb = 0;
    hipError_t e = reorder_scan_flags(nullptr, &tb, (uint64_t *)nullptr, (uint64_t *)nullptr, ntiles + 1, st);
    if (e != hipSuccess) return fail(e);
    const size_t scan_at = ((size_t)(2 * (ntiles + 1) + 4) * sizeof(uint64_t) + 255) & ~(size_t)255;
    DevRef temp = dev_alloc(scan_at + tb);
    if (!plan.tiles_mem || !temp) return fail(hipErrorOutOfMemory);
    uint64_t *cn = (uint64_t *)temp->ptr, *bf = cn + ntiles + 1;
    int *counters = (int *)(bf + ntiles + 1);
    hipLaunchKernelGGL(k_piece_tiles, dim3(grid_for(ntiles + 1)), dim3(256), 0, st, pos, nseg, nnz, plan.units, ntiles, plan.tiles());
    e = hipMemsetAsync(cn + ntiles, 0, sizeof(uint64_t), st);
    if (e == hipSuccess) e = hipMemsetAsync(counters, 0, 8 * sizeof(int), st);
    if (e != hipSuccess) return fail(e);
    hipLaunchKernelGGL((k_piece_fill<false>), dim3((unsigned)ntiles), dim3(256), 0, st, pos, nseg, ntiles, plan.tiles(), cn,
                       counters + 2, (uint32_t *)nullptr, (uint32_t *)nullptr);
    hipLaunchKernelGGL(k_piece_cuts, dim3(grid_for(ntiles)), dim3(256), 0, st, pos, nseg, (const int4 *)plan.tiles(), ntiles,
                       plan.cuts(), counters);
    // (a list shorter than a sample is not worth the 40 us that the kernel costs a small handle)
    if (nnz >= kSampleNnz)
        hipLaunchKernelGGL(k_piece_sample, dim3(kSamples + (parent ? 2 : 1) * kLooks), dim3(1024), 0, st, crd, nnz, parent, nseg, counters + 3);
    e = reorder_scan_flags((char *)temp->ptr + scan_at, &tb, cn, bf, ntiles + 1, st);
    struct { uint64_t total; int short_cuts, long_cuts, max_parts, set, found, few, parent_few, pad; } sums = {};    // bf[ntiles] and the counters
    if (e == hipSuccess) e = hipMemcpyAsync(&sums, bf + ntiles, sizeof sums, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail(e);
    plan.npieces = (int64_t)(uint32_t)sums.total;
    plan.njoins = (int64_t)(uint32_t)(sums.total >> 32);
    plan.ncut = sums.short_cuts;
    plan.ncut_long = sums.long_cuts;
    plan.max_parts = sums.max_parts;
    // m coordinates set kSampleBits * (1 - exp(-m / kSampleBits)) bits, and as large a share of the others finds a bit set by chance
    if (nnz >= kSampleNnz) {
        auto unset = [](int set, int samples) { return 1.0 - (double)set / ((double)samples * kSampleBits); };
        const double left = unset(sums.set, kSamples);
        plan.distinct = left > 0.0 ? (int64_t)(-std::log(left) * kSampleBits) : kSampleNnz;
        plan.common = left > 0.0 ? 1.0 - (1.0 - (double)sums.found / ((double)kSamples * kSampleLook)) / left : 0.0;
        plan.few = (int64_t)(-std::log(unset(sums.few, kLooks)) * kSampleBits);      // (an eighth of the bits at most)
        if (parent) plan.parent_few = (int64_t)(-std::log(unset(sums.parent_few, kLooks)) * kSampleBits);
    }
    plan.pieces_mem = dev_alloc(sizeof(uint32_t) * (plan.npieces + plan.njoins));
    if (!plan.pieces_mem) return fail(hipErrorOutOfMemory);
    hipLaunchKernelGGL((k_piece_fill<true>), dim3((unsigned)ntiles), dim3(256), 0, st, pos, nseg, ntiles, plan.tiles(), bf,
                       (int *)nullptr, plan.pieces(), plan.joins());
    hipLaunchKernelGGL(k_piece_end, dim3(1), dim3(1), 0, st, plan.tiles(), ntiles, (int)plan.npieces, (int)plan.njoins);
    e = hipStreamSynchronize(st);                            // the temporaries go out of scope
    return e == hipSuccess ? hipGetLastError() : fail(e);
}

}  // namespace comet

// MTTKRP, long lists: a wavefront works alone on kChunk consecutive nonzeros (k_mttkrp_wave).
//
// What bounds it.  A load of 64 lanes keeps the texture-address unit for 16 to 18 clocks, whatever it hits, and every kernel of this file's
// kind spends most of its time on that (84 % busy here on average, the busiest 97 %), so what counts is how many such loads a nonzero costs.  The walk over two levels
// (kernels_mttkrp.hip) loads a row of C and a row of B for each, because it cannot know which of the lane groups of a wavefront end a fiber.
// Here the nonzeros are taken in blocks of 8 per lane group.  The fibers of a block are consecutive, so their rows of B are loaded for all lane
// groups together, one per fiber, into LDS, from where each nonzero reads the one of its fiber.  Per block: 8 loads of C for 64 nonzeros (rank 16) and
// one of B for 8 fibers, 2.6 on average for the power-law tensor of 150 M nonzeros; 30.7 M loads in all where the walk has 40.7 M,
// 1602 us before and 1393 now.  The rows of C of the next block are loaded as those of the current one are used, one for one, and its rows of
// B in front of them, so that loads are in flight all the time without a wait of their own; blocks of 16 per lane group, with the loads
// of a block issued and used inside it, took 1591.  Runs of 4096 nonzeros per wavefront are level for 150 M and leave the chip unevenly filled for 20 M (820 us
// at rank 64, and 753).
//
// Sums.  No nonzero asks whether its fiber ends: (value * C) * B is added to the lane group's part of the open slice (the other kernels add up
// value * C over a fiber, or a part of it, first; for factors that are not finite this makes an infinity there a NaN here or the reverse, see comet.h).  Where no slice
// ends in a block (85 % of the blocks of that tensor) the parts of the lane groups just go on; where some do, those that lie in one lane group's
// nonzeros are stored by it, and the others are put together in LDS in the order of the nonzeros.  What is open at either end of the run goes through the carry
// fix-up of the other walks.  The order of every sum is the program's.
#include "stream_common.hpp"

namespace comet {

namespace {

// The value is computed here: without this the compiler moves the sums of a block behind the branches of the next block's loads,
// and keeps all of its rows in registers until then.
__device__ __forceinline__ void stay(double &x) { asm volatile("" : "+v"(x)); }

// What a wavefront wrote to LDS is there for all of its lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int L, int E, bool FULL, bool BIG>
__global__ void __launch_bounds__(64, 4) k_mttkrp_wave(const int32_t *__restrict__ pos2, const int32_t *__restrict__ crd1,
                                                       const int32_t *__restrict__ pos3, const int32_t *__restrict__ crd2,
                                                       const int32_t *__restrict__ crd3, const double *__restrict__ vals,
                                                       const int32_t *__restrict__ fiber_begin, const int32_t *__restrict__ slice_begin,
                                                       const double *__restrict__ Bm, const double *__restrict__ Cm,
                                                       double *__restrict__ M, int64_t nnz, int64_t nfib, int64_t nslice, int nruns,
                                                       int R, void *scratch, Epilogue ep) {
    // a block is ST nonzeros for each of the KP lane groups, those of a group consecutive; LB blocks are loaded at a time, IPL nonzeros per lane
    constexpr int V = E, KP = 64 / L, ST = 8, SB = KP * ST, W = SB / 32, kRow = L * E;
    constexpr int NB = 4, LB = 2, IPL = SB * LB / 64;
    constexpr int kBlocks = kChunk / SB;
    static_assert(L == 8 || L == 16, "a block has 64 or 32 nonzeros");
    static_assert(SB * kRow * 8 >= kChunk / 4, "the masks have room in the slots");
    __shared__ __attribute__((aligned(16))) double slots[SB * kRow];
    __shared__ __attribute__((aligned(16))) double ival[2][SB];
    __shared__ __attribute__((aligned(16))) unsigned ioff[2][SB];
    __shared__ int held[SB];                                      // rows of M of the slices that end in the block
    unsigned *fbits = reinterpret_cast<unsigned *>(slots), *sbits = fbits + kChunk / 32;
    const int lane = threadIdx.x, k = lane % L, gw = lane / L;
    const int run = (int)blockIdx.x, c0 = (int)blockIdx.y * kRow;
    const RowOf<L, E, 1, FULL> rw(R - c0 < kRow ? R - c0 : kRow, k);
    const char *Cl = reinterpret_cast<const char *>(Cm + c0), *Bl = reinterpret_cast<const char *>(Bm + c0);
    const unsigned unit = (unsigned)R * (BIG ? 1u : 8u);
    const CarryView cv = carry_view(scratch, nruns, R);
    unsigned front[W];                                            // nonzeros of the block in front of this group's, as a mask
#pragma unroll
    for (int w = 0; w < W; ++w) front[w] = gw / 4 > w ? ~0u : gw / 4 == w ? (1u << (gw % 4 * 8)) - 1u : 0u;

    struct Items { int crd[IPL]; double val[IPL]; };
    auto load_items = [&](Items &it, int64_t at) {                // LB blocks from nonzero `at` on
        const int32_t *pc = crd3 + at;
        const double *pv = vals + at;
        const unsigned i = (unsigned)lane * IPL;
        if (at + SB * LB <= nnz) {
            typedef int v2i __attribute__((ext_vector_type(2)));
            typedef double v2d __attribute__((ext_vector_type(2)));
            if constexpr (IPL == 1) {
                it.crd[0] = __builtin_nontemporal_load(pc + i);
                it.val[0] = __builtin_nontemporal_load(pv + i);
            } else {
                const v2i cc = __builtin_nontemporal_load(reinterpret_cast<const v2i *>(pc + i));
                const v2d x = __builtin_nontemporal_load(reinterpret_cast<const v2d *>(pv + i));
                it.crd[0] = cc.x; it.crd[1] = cc.y;
                it.val[0] = x.x; it.val[1] = x.y;
            }
        } else {
#pragma unroll
            for (int u = 0; u < IPL; ++u) { const bool in = at + i + u < nnz; it.crd[u] = in ? pc[i + u] : 0; it.val[u] = in ? pv[i + u] : 0.0; }
        }
    };
    // block h of the loaded ones to LDS
    auto stage = [&](const Items &it, int h, int to) {
        const int i = lane * IPL - h * SB;
        if (i >= 0 && i < SB) {
#pragma unroll
            for (int u = 0; u < IPL; ++u) { ioff[to][i + u] = (unsigned)it.crd[u] * unit; ival[to][i + u] = it.val[u]; }
        }
    };
    // rows of B of 64 consecutive fibers, one per lane
    auto load_fibers = [&](int64_t first) {
        const int64_t f = first + lane;
        return crd2[f < nfib ? f : nfib - 1];
    };

    double base[V];                                               // this group's part of the slice that is open in front of the block
#pragma unroll
    for (int e = 0; e < V; ++e) base[e] = 0.0;
    bool run_ht = false;                                          // a slice has ended in the run
    {
        const int64_t cbeg = (int64_t)run * kChunk;
        const int f0 = fiber_begin[run], s0 = slice_begin[run], f1 = fiber_begin[run + 1], s1 = slice_begin[run + 1];
        Items it;
        load_items(it, cbeg);
        int wbase = f0;                                           // the fibers from here on
        int win = load_fibers(wbase), ahead = load_fibers((int64_t)wbase + 64), later = load_fibers((int64_t)wbase + 128);
        for (int i = lane; i < kChunk / 16; i += 64) fbits[i] = 0u;
        wave_sync();
        for (int f = f0 + lane; f < f1; f += 64) {
            const int i = (int)((int64_t)pos3[f + 1] - 1 - cbeg);
            atomicOr(&fbits[i >> 5], 1u << (i & 31));
        }
        for (int s = s0 + lane; s < s1; s += 64) {
            const int i = (int)((int64_t)pos3[pos2[s + 1]] - 1 - cbeg);
            atomicOr(&sbits[i >> 5], 1u << (i & 31));
        }
        wave_sync();
        const unsigned fword = fbits[lane & 31], sword = sbits[lane & 31];
        wave_sync();
        const int nblk = nnz - cbeg >= kChunk ? kBlocks : (int)((nnz - cbeg + SB - 1) / SB);

        double br[NB][V], ring[ST][V];
        struct Block { int nrows, fibers, slow; unsigned fw[W], sw[W]; };
        auto look = [&](int blk) {
            Block b;
            unsigned any = 0;
            b.fibers = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                b.fw[w] = (unsigned)__builtin_amdgcn_readlane((int)fword, blk * W + w);
                b.sw[w] = (unsigned)__builtin_amdgcn_readlane((int)sword, blk * W + w);
                any |= b.sw[w];
                b.fibers += __builtin_popcount(b.fw[w]);
            }
            b.slow = any != 0u ? 1 : 0;
            b.nrows = b.fibers + 1 - (int)(b.fw[W - 1] >> 31);
            return b;
        };
        // rows i * KP ... of the block whose first fiber is number `at` (below 64) of the window
        auto b_row = [&](int at, auto ic, double *d) {
            constexpr int i = decltype(ic)::value;
            const int n = at + i * KP + gw, c = __shfl(win, n & 63), c1 = __shfl(ahead, n & 63);
            rw.template load<BIG>(Bl, (unsigned)(n < 64 ? c : c1) * unit, d);
        };
        auto load_b = [&](int at, int nrows) {
            static_for<0, NB>([&](auto ic) {
                if (decltype(ic)::value * KP < nrows) b_row(at, ic, br[decltype(ic)::value]);
            });
        };
        auto put_b = [&](int nrows) {
            static_for<0, NB>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if (i * KP < nrows) rw.put(slots + (i * KP + gw) * kRow, br[i]);
            });
        };
        Block cur = look(0);
        int fat = f0, sat = s0;                                   // fibers and slices that ended in front of the block
        int row = 0;                                              // row of M of the slice that ends as number `lane` of the block
        stage(it, 0, 0);
        wave_sync();
        load_b(0, cur.nrows);
        {
            const uint4 o0 = *reinterpret_cast<const uint4 *>(ioff[0] + gw * ST), o1 = *reinterpret_cast<const uint4 *>(ioff[0] + gw * ST + 4);
            const unsigned o[ST] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
            static_for<0, ST>([&](auto jc) { rw.template load<BIG>(Cl, o[decltype(jc)::value], ring[decltype(jc)::value]); });
        }
        if (cur.slow) row = crd1[sat + lane < nslice ? sat + lane : nslice - 1];
        for (int blk = 0; blk < nblk; ++blk) {
            const int par = blk & 1;
            const bool more = blk + 1 < nblk;
            put_b(cur.nrows);
            if (cur.nrows > NB * KP) {                            // more rows of B than are kept in registers
                static_for<NB, ST>([&](auto ic) {
                    if (decltype(ic)::value * KP < cur.nrows) b_row(fat - wbase, ic, br[decltype(ic)::value - NB]);
                });
                __builtin_amdgcn_s_waitcnt(0x0f70);               // vmcnt(0), whichever of them there were
                static_for<NB, ST>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    if (i * KP < cur.nrows) rw.put(slots + (i * KP + gw) * kRow, br[i - NB]);
                });
            }
            if (cur.slow && lane < SB) held[lane] = row;
            Block next = cur;
            if (more) {
                next = look(blk + 1);
                stage(it, (blk + 1) % LB, (blk + 1) & 1);
                const bool shift = fat + cur.fibers - wbase >= 64;
                if (shift) { win = ahead; ahead = later; wbase += 64; }
                load_b(fat + cur.fibers - wbase, next.nrows);
                if (shift) later = load_fibers((int64_t)wbase + 128);
                if (blk % LB == LB - 2 && blk + 2 < nblk) load_items(it, cbeg + (int64_t)(blk + 2) * SB);
                if (next.slow) {
                    int n = 0;
#pragma unroll
                    for (int w = 0; w < W; ++w) n += __builtin_popcount(cur.sw[w]);
                    const int64_t s = (int64_t)sat + n + lane;
                    row = crd1[s < nslice ? s : nslice - 1];
                }
            } else {
                if (lane < SB) ioff[par ^ 1][lane] = 0u;          // the rows that the walk loads ahead
            }
            wave_sync();
            unsigned fm = cur.fw[0], sm = 0;
            int slot = 0, srank = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                slot += __popc(cur.fw[w] & front[w]);
                if (w > 0) fm = gw / 4 == w ? cur.fw[w] : fm;
            }
            fm >>= gw % 4 * 8;
            if (cur.slow) {
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    srank += __popc(cur.sw[w] & front[w]);
                    sm = gw / 4 == w ? cur.sw[w] : sm;
                }
                sm >>= gw % 4 * 8;
            }
            const double *gv = ival[par] + gw * ST;
            const unsigned *go = ioff[par ^ 1] + gw * ST;
            double loc[V], first[V];
            int ends = 0;
#pragma unroll
            for (int e = 0; e < V; ++e) { loc[e] = 0.0; first[e] = 0.0; }
            unsigned anyend = cur.sw[0];
#pragma unroll
            for (int w = 1; w < W; ++w) anyend |= cur.sw[w];
            anyend |= anyend >> 16;
            anyend |= anyend >> 8;
            {
                const double *sp = slots + slot * kRow;
                double b[2][V];
                double2 vq;
                uint4 oq;
                rw.get(sp, b[0]);
                static_for<0, ST>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (j % 2 == 0) vq = *reinterpret_cast<const double2 *>(gv + j);
                    if constexpr (j % 4 == 0) oq = *reinterpret_cast<const uint4 *>(go + j);
                    if constexpr (j + 1 < ST) { sp += ((fm >> j) & 1u) * kRow; rw.get(sp, b[(j + 1) & 1]); }
                    const double a = j % 2 ? vq.y : vq.x;
#pragma unroll
                    for (int e = 0; e < V; ++e) { loc[e] = fma(a * ring[j][e], b[j & 1][e], loc[e]); stay(loc[e]); }
                    rw.template load<BIG>(Cl, j % 4 == 0 ? oq.x : j % 4 == 1 ? oq.y : j % 4 == 2 ? oq.z : oq.w, ring[j]);
                    if ((anyend >> j) & 1u) {
                        asm volatile("");                         // a scalar branch of its own
                        if ((sm >> j) & 1u) {
                            if (ends == 0) {
#pragma unroll
                                for (int e = 0; e < V; ++e) first[e] = loc[e];
                            } else {
                                rw.store_result(M + (int64_t)held[srank + ends] * R + c0, loc, ep);
                            }
                            ++ends;
#pragma unroll
                            for (int e = 0; e < V; ++e) loc[e] = 0.0;
                        }
                    }
                });
            }
            if (!cur.slow) {
#pragma unroll
                for (int e = 0; e < V; ++e) base[e] += loc[e];
            } else {
                const bool ht = ends > 0;
                const int first_row = held[srank & (SB - 1)];
                const unsigned long long ended = __ballot(ht);
                double all[V];
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    all[e] = base[e];
#pragma unroll
                    for (int d = L; d < 64; d *= 2) all[e] += __shfl_xor(all[e], d);
                }
                wave_sync();
                rw.put(slots + gw * kRow, loc);
                wave_sync();
                if (ht) {
                    double sum[V];
#pragma unroll
                    for (int e = 0; e < V; ++e) sum[e] = first[e];
                    bool found = false;
                    for (int g = gw - 1; g >= 0 && !found; --g) {
                        double x[V];
                        rw.get(slots + g * kRow, x);
#pragma unroll
                        for (int e = 0; e < V; ++e) sum[e] += x[e];
                        found = (ended >> (g * L)) & 1ull;
                    }
                    if (!found) {
#pragma unroll
                        for (int e = 0; e < V; ++e) sum[e] += all[e];
                    }
                    if (found || run_ht) {
                        rw.store_result(M + (int64_t)first_row * R + c0, sum, ep);
                    } else {                                      // it may have begun in front of the run
                        rw.store(cv.first + (int64_t)run * R + c0, sum);
                        if (k == 0 && c0 == 0) cv.first_id[run] = first_row;
                    }
                }
                const int latest = (63 - __clzll((long long)ended)) / L;
#pragma unroll
                for (int e = 0; e < V; ++e) base[e] = gw >= latest ? loc[e] : 0.0;
                run_ht = true;
            }
            wave_sync();                                          // before LDS is written again
            fat += cur.fibers;
#pragma unroll
            for (int w = 0; w < W; ++w) sat += __builtin_popcount(cur.sw[w]);
            cur = next;
        }
    }
#pragma unroll
    for (int e = 0; e < V; ++e)
#pragma unroll
        for (int d = L; d < 64; d *= 2) base[e] += __shfl_xor(base[e], d);
    if (gw == 0) rw.store(cv.open + (int64_t)run * R + c0, base);
    if (lane == 0 && c0 == 0) cv.has_tail[run] = run_ht ? 1 : 0;
}

struct WaveArgs {
    const Schedule &sc;
    const int32_t *pos2, *crd1, *pos3, *crd2, *crd;
    const double *vals, *B, *C;
    double *M;
    int64_t nslice;
    int R;
    void *scratch;
    hipStream_t st;
    Epilogue ep;
};

template <int L, int E, bool FULL, bool BIG>
hipError_t launch_wave(const WaveArgs &a) {
    constexpr int kRow = L * E;
    const int nruns = (int)a.sc.nchunks, nblocks = (a.R + kRow - 1) / kRow;
    hipLaunchKernelGGL((k_mttkrp_wave<L, E, FULL, BIG>), dim3((unsigned)nruns, (unsigned)nblocks), dim3(64), 0, a.st, a.pos2, a.crd1, a.pos3,
                       a.crd2, a.crd, a.vals, (const int32_t *)a.sc.chunk_seg_begin->ptr, (const int32_t *)a.sc.chunk_slice_begin->ptr, a.B,
                       a.C, a.M, a.sc.nnz, a.sc.nseg, a.nslice, nruns, a.R, a.scratch, a.ep);
    return hipGetLastError();
}

}  // namespace

hipError_t mttkrp_wave(const Schedule &sc, const int32_t *pos2, int64_t nslice, const int32_t *crd1, const int32_t *pos3, const int32_t *crd2,
                       const int32_t *crd3, const double *vals, const double *B, const double *C, bool big, int R, double *M, void *scratch,
                       hipStream_t st, Epilogue ep) {
    const WaveArgs a{sc, pos2, crd1, pos3, crd2, crd3, vals, B, C, M, nslice, R, scratch, st, ep};
    hipError_t e;
    if (R & 1) e = big ? launch_wave<16, 1, false, true>(a) : launch_wave<16, 1, false, false>(a);
    else if (big) e = launch_wave<8, 2, false, true>(a);
    else if (R % 32 == 0) e = launch_wave<16, 2, true, false>(a);
    else if ((R + 15) / 16 % 2 == 0) e = launch_wave<16, 2, false, false>(a);   // the list is read half as often as in blocks of 16 columns
    else if (R % 16) e = launch_wave<8, 2, false, false>(a);
    else e = launch_wave<8, 2, true, false>(a);
    if (e != hipSuccess) return e;
    return run_fixup(scratch, sc.nchunks, R, nullptr, M, sc.max_parent_len > 0 ? sc.max_parent_len / kChunk + 2 : 0, st, ep);
}

}  // namespace comet

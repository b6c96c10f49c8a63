// Plan kernels (uv -> tile-sorted work lists) and the permutations between
// caller order and entry order.
#include "dev_common.h"

namespace lmg {
namespace dev {


// Set (never cleared by a kernel) when a plan meets non-finite coordinates;
// read and cleared by lmg_sync_status through the runtime's symbol copies.
__device__ int g_data_error;

// The constants a plan keeps (coefficients, twiddles, correction) and, for a
// batch, the block tables, read from pinned host memory in 16-byte pieces (one
// per thread, all in flight at once) by the workgroups of the plan's first
// launch that have no visibilities to count: i is the thread's number among
// them. (A launch of its own took 8 us per plan, copies and a fill 30 to 40.)
__device__ __forceinline__ void copy_constants(const PlanSetup& a, int i) {
    int at = i;
#pragma unroll
    for (int q = 0; q < PlanSetup::kCopies; ++q) {
        const int n = (a.bytes[q] + 15) / 16;
        if (at >= 0 && at < n) {
            const char* src = static_cast<const char*>(a.src[q]) + static_cast<size_t>(at) * 16;
            char* dst = static_cast<char*>(a.dst[q]) + static_cast<size_t>(at) * 16;
            const int left = a.bytes[q] - at * 16;
            if (left >= 16) {
                *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
            } else {
                for (int w = 0; w < left; w += 4) *reinterpret_cast<int*>(dst + w) = *reinterpret_cast<const int*>(src + w);
            }
        }
        at -= n;
    }
}

// Plan block b: (channel, first visibility, count, 0); from the batch's table, or for a single channel (no table) by
// its size.
__device__ __forceinline__ int4 plan_block(const PlanBlocks& p, int b) {
    if (p.table) return p.table[b];
    return make_int4(0, b * p.block_vis, min(p.block_vis, p.nvis - b * p.block_vis), 0);
}

// Visibilities base .. base + count of one channel: one count each in hist (slot g.ntiles: coordinates that are not
// finite). True if this thread met such coordinates.
__device__ __forceinline__ bool count_run(const double2* __restrict__ uv, int64_t base, int count, const PlanGeom& g,
                                          int* hist) {
    const int64_t end = base + count;
    bool bad = false;
    constexpr int kB = 8;
    for (int i0 = 0; i0 < count; i0 += kB * kPlanThreads) {
        double2 c[kB];
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            const int64_t k = base + i0 + u * kPlanThreads + threadIdx.x;
            if (k < end) c[u] = uv[k];
        }
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            const int64_t k = base + i0 + u * kPlanThreads + threadIdx.x;
            if (k >= end) break;
            int cu, cv;
            double du, dv;
            if (tap_geometry(c[u].x, g.W, g.ref, g.N, &cu, &du) && tap_geometry(c[u].y, g.W, g.ref, g.N, &cv, &dv)) {
                atomicAdd(&hist[((cv >> g.lb) << g.lbx) + (cu >> g.lb)], 1);
            } else {
                atomicAdd(&hist[g.ntiles], 1);
                bad = true;
            }
        }
    }
    return bad;
}

// Pass 1: count visibilities per tile, per plan block (a run of at most
// plan_block_vis() visibilities of one channel, kept per block so that pass 3
// can place each block's visibilities of a tile in one contiguous run). The
// slot after the tiles counts visibilities whose coordinates are not finite
// (they are dropped). Workgroups nb .. copy the plan's constants.
__global__ __launch_bounds__(kPlanThreads) void k_plan_count(const double2* __restrict__ uv, PlanBlocks blocks, int nb,
                                                             PlanGeom g, int* __restrict__ blockhist, PlanSetup setup) {
    extern __shared__ int hist[];
    if (static_cast<int>(blockIdx.x) >= nb) {                // uniform across the workgroup
        copy_constants(setup, (blockIdx.x - nb) * kPlanThreads + threadIdx.x);
        return;
    }
    const int hs = g.ntiles + 1;
    for (int t = threadIdx.x; t < hs; t += blockDim.x) hist[t] = 0;
    __syncthreads();
    const int chunk = xcd_chunk(blockIdx.x, nb);
    const int4 bd = plan_block(blocks, chunk);
    if (count_run(uv, bd.y, bd.z, g, hist)) atomicOr(&g_data_error, 1);
    __syncthreads();
    int* row = blockhist + static_cast<size_t>(chunk) * hs;
    for (int t = threadIdx.x; t < hs; t += blockDim.x) row[t] = hist[t];
}

// Pass 1b: per slot (channel c, tile t), the exclusive prefix of the counts of
// the channel's blocks [chan_blocks[c], chan_blocks[c + 1]) (in place) and
// their total; slot nchan * ntiles (dropped visibilities) runs over all
// blocks. Workgroups of kScanGroups x 64 threads: 64 slots, each split into
// kScanGroups runs of blocks.
constexpr int kScanGroups = 16;
__global__ __launch_bounds__(64 * kScanGroups) void k_plan_colscan(PlanGeom g, int* __restrict__ blockhist,
                                                                   const int* __restrict__ chan_blocks, int nb,
                                                                   int* __restrict__ tile_count) {
    __shared__ int part[kScanGroups][64];
    const int64_t tot = static_cast<int64_t>(g.ntiles) * g.nchan;
    const int hs = g.ntiles + 1;
    const int64_t slot = static_cast<int64_t>(blockIdx.x) * 64 + (threadIdx.x & 63);
    const int grp = threadIdx.x >> 6;
    const bool live = slot <= tot;
    int b0 = 0, b1 = 0, col = 0;
    if (live) {
        if (slot == tot) {
            b0 = 0;
            b1 = nb;
            col = g.ntiles;
        } else if (g.nchan == 1) {
            b1 = nb;
            col = static_cast<int>(slot);
        } else {
            const int c = static_cast<int>(slot >> (2 * g.lbx));
            b0 = chan_blocks[c];
            b1 = chan_blocks[c + 1];
            col = static_cast<int>(slot) & (g.ntiles - 1);
        }
    }
    const int len = b1 - b0;
    const int lo = b0 + static_cast<int>((static_cast<int64_t>(len) * grp) / kScanGroups);
    const int hi = b0 + static_cast<int>((static_cast<int64_t>(len) * (grp + 1)) / kScanGroups);
    // Both passes take kU blocks' counts at a time, all loads issued before the first is used.
    constexpr int kU = 8;
    int sum = 0;
    int b = lo;
    for (; b + kU <= hi; b += kU) {
        int x[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) x[u] = blockhist[static_cast<size_t>(b + u) * hs + col];
#pragma unroll
        for (int u = 0; u < kU; ++u) sum += x[u];
    }
    for (; b < hi; ++b) sum += blockhist[static_cast<size_t>(b) * hs + col];
    part[grp][threadIdx.x & 63] = sum;
    __syncthreads();
    int run = 0;
    for (int q = 0; q < grp; ++q) run += part[q][threadIdx.x & 63];
    b = lo;
    for (; b + kU <= hi; b += kU) {
        int x[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) x[u] = blockhist[static_cast<size_t>(b + u) * hs + col];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            blockhist[static_cast<size_t>(b + u) * hs + col] = run;
            run += x[u];
        }
    }
    for (; b < hi; ++b) {
        int* p = blockhist + static_cast<size_t>(b) * hs + col;
        const int x = *p;
        *p = run;
        run += x;
    }
    if (live && grp == kScanGroups - 1) tile_count[slot] = run;
}

constexpr int kScanSums = 96;    // ints of LDS for the block sums and reductions of the scan
struct ScanAcc {
    int s, si, busy, rmin, rmax, cmin, cmax;
};

// Work items of a slot with c visibilities: ceil(c / cap); the division is
// only taken for the rare slots above cap (this single-workgroup pass is
// bound by its instruction count).
__device__ __forceinline__ int slot_items(int c, int cap) {
    return c <= cap ? (c > 0 ? 1 : 0) : (c + cap - 1) / cap;
}

__device__ __forceinline__ void scan_sum(int t, int c, int tot, int cap, int& s, int& si) {
    s += c;
    if (t < tot) si += slot_items(c, cap);
}

// Offsets of slot t (count c) and its work items; slot tot holds the dropped visibilities.
__device__ __forceinline__ void scan_place(const PlanGeom& g, int t, int c, int tot, int cap, int* tile_start,
                                           int* item_start, int4* items, int* flags, ScanAcc& a, bool write_items) {
    tile_start[t] = a.s;
    if (t == tot) {
        flags[0] = c > 0;
        flags[2] = a.s;
        a.s += c;
        return;
    }
    const int ni = slot_items(c, cap);
    item_start[t] = a.si;
    if (c > 0) {
        const int lt = t & (g.ntiles - 1);
        const int tr = lt >> g.lbx, tc = lt & (g.ntx - 1);
        a.rmin = min(a.rmin, tr);
        a.rmax = max(a.rmax, tr);
        a.cmin = min(a.cmin, tc);
        a.cmax = max(a.cmax, tc);
    }
    if (!write_items) {
    } else if (ni == 1) {
        items[a.si] = make_int4(t, a.s, c, 0);
    } else if (ni > 1) {
        // even split: the first c % ni items take one visibility more (32-bit arithmetic: the dense
        // central tiles are consecutive slots of one thread, and a wide division per item serialises it)
        const int base = c / ni, extra = c - base * ni;
        int lo = 0;
        for (int q = 0; q < ni; ++q) {
            const int n = base + (q < extra ? 1 : 0);
            items[a.si + q] = make_int4(t, a.s + lo, n, 0);
            lo += n;
        }
    }
    a.busy += (c > 0);
    a.s += c;
    a.si += ni;
}

// Pass 2 (one workgroup): slot offsets, work items of at most `cap`
// visibilities, counts and the occupied band (flags[0] any dropped, [1] items, [2] valid
// visibilities, [3] busy tiles, [4..7] min / max occupied tile row and
// column). tile_start has nslots + 1 entries (the last is nvis).
// Each thread scans a contiguous run of slots. With `staged` (slots fit
// twice in LDS) the counts come in, and the slot and item offsets go out,
// through LDS, so that global accesses are coalesced and the per-slot loop
// waits only on LDS, not on the global stores of the work items.
template <bool kStaged>
__device__ __forceinline__ void scan_slots(const PlanGeom& g, const int* cnt, int* start_out, int* items_out, int lo,
                                           int hi, int tot, int cap, int4* items, int* flags, int* sh, int* nvis,
                                           int* nitems, ScanAcc& acc) {
    int s = 0, si = 0;
#pragma unroll 1
    for (int t = lo; t < hi; ++t) scan_sum(t, cnt[t], tot, cap, s, si);
    // (the barriers inside also order every read of staged counts by other threads before the
    // overwrites below; a thread reads its own slot before overwriting it)
    s = block_excl_sum(s, sh, nvis);
    si = block_excl_sum(si, sh, nitems);
    acc = ScanAcc{s, si, 0, 1 << 30, -1, 1 << 30, -1};
#pragma unroll 1
    for (int t = lo; t < hi; ++t) {
        const int c = cnt[t];
        scan_place(g, t, c, tot, cap, start_out, items_out, items, flags, acc, !kStaged);
    }
}

// With the counts of all slots in s_start (LDS, ns of them): the slot offsets take their place, the item offsets go to
// s_items, both are copied out, and the work items are written.
__device__ __forceinline__ void scan_staged(const PlanGeom& g, int* s_start, int* s_items, int lo, int hi, int ns, int cap,
                                            int* tile_start, int* item_start, int4* items, int* flags, int* sh, int* nvis,
                                            int* n_items, ScanAcc& acc) {
    const int tot = ns - 1;
    __syncthreads();
    scan_slots<true>(g, s_start, s_start, s_items, lo, hi, tot, cap, items, flags, sh, nvis, n_items, acc);
    const int nitems = *n_items;
    if (threadIdx.x == 0) s_items[tot] = nitems;
    __syncthreads();
    for (int t = threadIdx.x; t < ns; t += blockDim.x) tile_start[t] = s_start[t];
    for (int t = threadIdx.x; t < tot; t += blockDim.x) item_start[t] = s_items[t];
    // Work items in parallel (a tile above cap has several, and the dense tiles are neighbours in
    // one thread's run): item i belongs to the last slot whose first item is <= i.
    for (int i = threadIdx.x; i < nitems; i += blockDim.x) {
        int a = 0, b = tot;          // s_items[a] <= i < s_items[b]
        while (b - a > 1) {
            const int m = (a + b) >> 1;
            if (s_items[m] <= i) a = m; else b = m;
        }
        const int c = s_start[a + 1] - s_start[a];
        const int ni = slot_items(c, cap);
        const int q = i - s_items[a];
        const int base = c / ni, extra = c - base * ni;     // the first extra items take one more
        const int first = q * base + min(q, extra);
        items[i] = make_int4(a, s_start[a] + first, base + (q < extra ? 1 : 0), 0);
    }
}

// The plan's counts and occupied band.
__device__ __forceinline__ void scan_flags(const ScanAcc& acc, int ns, int nvis, int nitems, int* tile_start,
                                           int* item_start, int* flags, int* host_flags, int* sh) {
    int v[5] = {acc.busy, -acc.rmin, acc.rmax, -acc.cmin, acc.cmax};     // a sum and four maxima
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const int o = __shfl_xor(v[q], d, 64);
            v[q] = q == 0 ? v[q] + o : max(v[q], o);
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < 5; ++q) sh[q * 16 + wave] = v[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            for (int w = 1; w < nw; ++w) v[q] = q == 0 ? v[q] + sh[w] : max(v[q], sh[q * 16 + w]);
        }
        tile_start[ns] = nvis;
        item_start[ns - 1] = nitems;
        flags[1] = nitems;
        flags[3] = v[0];
        flags[4] = -v[1];
        flags[5] = v[2];
        flags[6] = -v[3];
        flags[7] = v[4];
        if (host_flags) {                        // the host's copy, in pinned memory
            host_flags[0] = flags[0];
            host_flags[1] = nitems;
            host_flags[2] = flags[2];
            host_flags[3] = v[0];
            host_flags[4] = -v[1];
            host_flags[5] = v[2];
            host_flags[6] = -v[3];
            host_flags[7] = v[4];
            __threadfence_system();
        }
    }
}

__global__ __launch_bounds__(1024) void k_plan_scan(PlanGeom g, const int* __restrict__ tile_count,
                                                    int* __restrict__ tile_start, int* __restrict__ item_start,
                                                    int4* __restrict__ items, int* __restrict__ flags, int cap,
                                                    int staged, int* __restrict__ host_flags) {
    extern __shared__ int lds[];
    int* sh = lds;
    const int tot = g.ntiles * g.nchan;          // tile slots, channel-major; slot tot = dropped
    const int ns = tot + 1;
    const int per = (ns + blockDim.x - 1) / blockDim.x;
    const int lo = threadIdx.x * per, hi = min(ns, lo + per);
    int nvis = 0, nitems = 0;
    ScanAcc acc;
    if (staged) {
        int* s_start = lds + kScanSums;          // counts, then slot offsets
        int* s_items = s_start + ns;             // item offsets
        constexpr int kL = 8;                    // loads in flight per thread
        for (int t0 = 0; t0 < ns; t0 += kL * blockDim.x) {
            int v[kL];
#pragma unroll
            for (int u = 0; u < kL; ++u) {
                const int t = t0 + u * blockDim.x + threadIdx.x;
                v[u] = t < ns ? tile_count[t] : 0;
            }
#pragma unroll
            for (int u = 0; u < kL; ++u) {
                const int t = t0 + u * blockDim.x + threadIdx.x;
                if (t < ns) s_start[t] = v[u];
            }
        }
        scan_staged(g, s_start, s_items, lo, hi, ns, cap, tile_start, item_start, items, flags, sh, &nvis, &nitems, acc);
    } else {
        scan_slots<false>(g, tile_count, tile_start, item_start, lo, hi, tot, cap, items, flags, sh, &nvis, &nitems,
                          acc);
    }
    scan_flags(acc, ns, nvis, nitems, tile_start, item_start, flags, host_flags, sh);
}

// Pass 3: give each visibility its tile-order position (index = inv0, by
// caller index) and its packed offsets (offs, by caller index): both writes are
// coalesced. The scattered store of the offsets into tile order is a pass of
// its own (k_plan_place): here each XCD runs 32 plan blocks, that is 32
// time windows, at once, and their partly written lines would overflow L2.
// Positions are ranks taken from the block's LDS cursors. The waves of the
// workgroup hold consecutive runs of the caller order and take their ranks in
// a fixed turn (wave 0 first, a barrier between turns), so that a tile's
// visibilities stay in the caller's order: every later summation order is the
// same on every run and for every size of block.
//
// kDirect (plans of at most kDirectPlanVis visibilities, whose arrays stay in
// L2, so that scattered stores need no order of their own): the offsets go
// straight to tile order (off0) with the caller index beside them (perm0), and
// the item sort writes caller index -> entry itself; the place and compose
// passes are not run.
template <typename R, bool kDirect>
__device__ __forceinline__ void scatter_run(const double2* __restrict__ uv, int64_t base, int count, const PlanGeom& g,
                                            int* cur, double dlo, int ms, int kb, int* __restrict__ index,
                                            typename Pack<R>::T2* __restrict__ offs) {
    const int wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int64_t end = base + count;
    constexpr int kB = 8;                                    // most coordinates loaded together per thread
    const int kb_run = min(kB, (count + kPlanThreads - 1) / kPlanThreads);     // coordinates per thread and step
    const int first = wave * 64 * kb_run + (threadIdx.x & 63);
    for (int i0 = 0; i0 < count; i0 += kb_run * kPlanThreads) {  // uniform across the workgroup
        double2 c[kB];
        const int64_t k0 = base + i0 + first;                // this thread's coordinates: k0 + 64 u, u < kb_run
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            const int64_t k = k0 + u * 64;
            if (u < kb_run && k < end) c[u] = nt_load(uv + k);     // the coordinates' last read
        }
        int key[kB];                                         // tile slot (ntiles: dropped), -1 past the run
        typename Pack<R>::T2 packed[kB];
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            const int64_t k = k0 + u * 64;
            key[u] = -1;
            if (u >= kb_run || k >= end) continue;
            int cu, cv;
            double du, dv;
            if (tap_geometry(c[u].x, g.W, g.ref, g.N, &cu, &du) && tap_geometry(c[u].y, g.W, g.ref, g.N, &cv, &dv)) {
                key[u] = ((cv >> g.lb) << g.lbx) + (cu >> g.lb);
                typename Pack<R>::T2 o;
                o.x = pack_axis<R>(cu & (g.T - 1), du, dlo, g.lb, ms, kb);
                o.y = pack_axis<R>(cv & (g.T - 1), dv, dlo, g.lb, ms, kb);
                packed[u] = o;
                if (!kDirect) offs[k] = o;
            } else {
                key[u] = g.ntiles;                           // dropped: a position after the valid ones
            }
        }
        int dst[kB];
        for (int w = 0; w < nwaves; ++w) {
            if (wave == w) {
#pragma unroll
                for (int u = 0; u < kB; ++u)
                    if (key[u] >= 0) dst[u] = atomicAdd(&cur[key[u]], 1);
            }
            __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < kB; ++u) {
            if (key[u] < 0) continue;
            if constexpr (kDirect) {
                if (key[u] != g.ntiles) offs[dst[u]] = packed[u];
                index[dst[u]] = static_cast<int>(k0 + u * 64);
            } else {
                index[k0 + u * 64] = dst[u];
            }
        }
    }
}

template <typename R, bool kDirect>
__global__ __launch_bounds__(kPlanThreads) void k_plan_scatter(const double2* __restrict__ uv, PlanBlocks blocks, int nb,
                                                               PlanGeom g, const int* __restrict__ tile_start,
                                                               const int* __restrict__ blockhist, double dlo, int ms,
                                                               int kb, int* __restrict__ index,
                                                               typename Pack<R>::T2* __restrict__ offs) {
    extern __shared__ int cur[];
    const int hs = g.ntiles + 1;
    const int chunk = xcd_chunk(blockIdx.x, nb);
    const int4 bd = plan_block(blocks, chunk);
    const int* row = blockhist + static_cast<size_t>(chunk) * hs;
    const int* ts = tile_start + static_cast<size_t>(bd.x) * g.ntiles;
    for (int t = threadIdx.x; t < g.ntiles; t += blockDim.x) cur[t] = ts[t] + row[t];
    if (threadIdx.x == 0) cur[g.ntiles] = tile_start[static_cast<size_t>(g.ntiles) * g.nchan] + row[g.ntiles];
    __syncthreads();
    scatter_run<R, kDirect>(uv, bd.y, bd.z, g, cur, dlo, ms, kb, index, offs);
}

// Passes 1 to 3 of a plan of one channel and at most kSmallPlanVis
// visibilities, by one workgroup, with the counts and offsets of all tiles in
// LDS (workgroups 1 .. copy the plan's constants). Such a plan is bound by its
// launches (2,000 visibilities on 128^2: 50 us in five, 43 in two).
template <typename R>
__global__ __launch_bounds__(kPlanThreads) void k_plan_small(const double2* __restrict__ uv, PlanGeom g, int nvis,
                                                             int* __restrict__ tile_start, int* __restrict__ item_start,
                                                             int4* __restrict__ items, int* __restrict__ flags, int cap,
                                                             int* __restrict__ host_flags, double dlo, int ms, int kb,
                                                             int* __restrict__ perm0,
                                                             typename Pack<R>::T2* __restrict__ off0, PlanSetup setup) {
    extern __shared__ int lds[];
    if (blockIdx.x > 0) {                        // uniform across the workgroup
        copy_constants(setup, (blockIdx.x - 1) * kPlanThreads + threadIdx.x);
        return;
    }
    const int ns = g.ntiles + 1;
    int* sh = lds;
    int* s_start = lds + kScanSums;              // counts, then slot offsets, then cursors
    int* s_items = s_start + ns;
    for (int t = threadIdx.x; t < ns; t += blockDim.x) s_start[t] = 0;
    __syncthreads();
    if (count_run(uv, 0, nvis, g, s_start)) atomicOr(&g_data_error, 1);
    const int per = (ns + blockDim.x - 1) / blockDim.x;
    const int lo = threadIdx.x * per, hi = min(ns, lo + per);
    int n = 0, nitems = 0;
    ScanAcc acc;
    scan_staged(g, s_start, s_items, lo, hi, ns, cap, tile_start, item_start, items, flags, sh, &n, &nitems, acc);
    scan_flags(acc, ns, n, nitems, tile_start, item_start, flags, host_flags, sh);
    __syncthreads();                             // the offsets have been read
    scatter_run<R, true>(uv, 0, nvis, g, s_start, dlo, ms, kb, perm0, off0);
}

// Threads per workgroup of the permutation passes (place, compose, permute in / out).
constexpr int kPermThreads = 1024;     // (256 / 512 / 1024: place 123 / 123 / 119 us, compose 104 / 103 / 100 us)

// Pass 3b: packed offsets into tile order, off0[inv0[k]] = offk[k] for the
// valid visibilities (flags[2] of them; dropped ones sit above). Consecutive
// workgroups take consecutive indices on one XCD, so its L2 sees one window
// of the caller order at a time and merges the scattered writes into lines.

template <typename R>
__global__ __launch_bounds__(kPermThreads) void k_plan_place(const int* __restrict__ inv0,
                                                    const typename Pack<R>::T2* __restrict__ offk,
                                                    const int* __restrict__ flags, int64_t nvis,
                                                    typename Pack<R>::T2* __restrict__ off0) {
    const int64_t k = static_cast<int64_t>(xcd_chunk(blockIdx.x, gridDim.x)) * blockDim.x + threadIdx.x;
    if (k >= nvis) return;
    const int d = nt_load(inv0 + k);
    if (d < flags[2]) off0[d] = nt_load(offk + k);
}

// Pass 4 (workgroups loop over items): order the item's visibilities into
// pieces (at most kPiece visibilities of one footprint cell) and lay the
// entries out in piece order, so that a turn of the gridding kernel, which
// takes 64 of them, reads one contiguous range. Piece order: the full
// pieces, cell by cell (cell c's f = n / kPiece pieces at F(c) .. F(c)+f-1,
// F an exclusive prefix of f), then the tails, longest first (a wave's lanes
// run loops of similar length). With lsub = 1 the item is cut into the four
// quadrants of its tile, laid out one after the other, and each becomes a work
// item of its own (a 64-cell tile's patch would leave a compute unit one or
// two workgroups). Outputs: packed offsets `off` by entry, map (pos2,
// tile-order position -> entry; with perm0, tile-order position -> caller
// index, it is inv, caller index -> entry), pieces[] (first entry, length |
// cell << 16, the cell within the quadrant) and the work items sub[]: (tile or
// quadrant, first entry, visibilities, number of pieces | (full pieces / 64)
// << 16). Dropped visibilities (tile-order positions n_valid .. nvis) get -1.
// Ranks within a cell follow the item's tile order in a fixed way: the item
// is cut into `groups` contiguous chunks, one per group of waves, each with
// its own LDS cell counters whose bases are the counts of the chunks before
// it; the waves of one group take their turns in order (a barrier between
// turns), so with one wave per group no barrier is needed at all.
// What bounds it is latency: an item's phases follow one another, and a dense item's rounds of load, LDS rank and store
// (a plan of few items runs as long as its densest). So a lane has kSortU entries in flight (16.8M visibilities on
// 4096^2: 1 144 us, 2 124, 4 119, 8 146, where the registers cost a workgroup), and the tails' slots come from cursors of
// each wave, not in turns (105 us; 201,600 on 1024^2: 32 -> 23 us). 256 threads: 108 and 26 us; 128: 120 and 36.
constexpr int kSortU = 4;
constexpr int kSortThreads = 512;
template <typename R, int kLsub>
__global__ __launch_bounds__(kSortThreads) void k_plan_sort_items(PlanGeom g, const int4* items, int4* sub,
                                                         const int* __restrict__ flags, int nvis, int lb, int groups,
                                                         const typename Pack<R>::T2* __restrict__ off0,
                                                         const int* __restrict__ perm0,
                                                         typename Pack<R>::T2* __restrict__ off,
                                                         int* __restrict__ map, int2* __restrict__ pieces) {
    extern __shared__ int sm[];
    constexpr int Q = 1 << (2 * kLsub);    // items cut from one
    __shared__ int scan_sh[17];            // block scan
    __shared__ int fstart[Q + 1];         // full pieces of the cells before each quadrant
    __shared__ int lcnt[kSortThreads / 64][kPiece];   // per wave: tails per length of its cells, then slot cursors
    __shared__ int lfirst[Q][kPiece];     // first tail slot of each length
    __shared__ int lbase[Q][kPiece];      // first entry of each length's tails
    __shared__ int npiece[Q], etail[Q];  // pieces of each quadrant, entries of its tails
    const int TT = g.T * g.T;
    const int sh = pack_cell_shift<R>(lb);            // position of the cell bits
    int* cnt = sm;             // per cell: count (low half); with one group, ranks given out (high half)
    int* cinfo = sm + TT;      // per cell: first full entry | (first tail entry) << 16   (both < 2^16: cap <= 16384)
    int* gcnt = groups > 1 ? sm + 2 * TT : sm;       // per group and cell: counts, then the group's next rank
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nwaves = blockDim.x >> 6;
    const int wpg = nwaves / groups;                 // waves per group
    const int grp = wave / wpg, wig = wave % wpg;
    int* gc = gcnt + grp * TT;
    // Cells quadrant by quadrant: index m = quadrant (TT / Q) + i; each thread takes a run of m, so a quadrant's
    // cells belong to `wpq` neighbouring waves (or to part of one).
    const int lbs = lb - kLsub, lbc = 2 * lbs;      // log2 of a quadrant's edge and cells
    const int ms = (1 << lbs) - 1;
    auto cell_of = [&](int m) {
        if constexpr (kLsub == 0) return m;
        const int k = m >> lbc, i = m & ((1 << lbc) - 1);
        const int y = ((k >> kLsub) << lbs) + (i >> lbs), x = ((k & ((1 << kLsub) - 1)) << lbs) + (i & ms);
        return (y << lb) + x;
    };
    const int seg = (TT + blockDim.x - 1) / blockDim.x;
    const int c0 = threadIdx.x * seg, c1 = min(TT, c0 + seg);
    const int wpq = max(1, TT / Q / seg / 64);
    const int n_items = flags[1];
    for (int e = flags[2] + blockIdx.x * blockDim.x + threadIdx.x; e < nvis; e += gridDim.x * blockDim.x)
        map[perm0 ? perm0[e] : e] = -1;
    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {     // uniform across the workgroup
        const int4 it = items[item];
        for (int c = threadIdx.x; c < groups * TT; c += blockDim.x) gcnt[c] = 0;
        if (lane < kPiece) lcnt[wave][lane] = 0;
        __syncthreads();
        // chunk of each group: a multiple of the group's 64 wpg lanes, the same for all groups
        const int chunk = ((it.z + groups - 1) / groups + 64 * wpg - 1) / (64 * wpg) * (64 * wpg);
        const int g0 = grp * chunk, g1 = min(it.z, g0 + chunk);
        // entries of a lane per round, all loaded before the first is used: e0 + 64 u, u < ku (waves of a group take
        // runs of 64 ku in turn, so a round's entries are in order of wave, u, lane)
        const int ku = min(kSortU, chunk / (64 * wpg));
        const int step = 64 * wpg * ku;
        for (int e0 = g0 + wig * 64 * ku + lane; e0 < g1; e0 += step) {
            typename Pack<R>::T2 r[kSortU];
#pragma unroll
            for (int u = 0; u < kSortU; ++u)
                if (u < ku && e0 + 64 * u < g1) r[u] = off0[it.y + e0 + 64 * u];
#pragma unroll
            for (int u = 0; u < kSortU; ++u)
                if (u < ku && e0 + 64 * u < g1)
                    atomicAdd(&gc[(static_cast<int>(r[u].y >> sh) << lb) + static_cast<int>(r[u].x >> sh)], 1);
        }
        __syncthreads();
        if (groups > 1) {
            for (int c = threadIdx.x; c < TT; c += blockDim.x) {     // group bases: counts of the chunks before
                int base = 0;
                for (int q = 0; q < groups; ++q) {
                    const int n = gcnt[q * TT + c];
                    gcnt[q * TT + c] = base;
                    base += n;
                }
                cnt[c] = base;
            }
            __syncthreads();
        }
        // full pieces: exclusive prefix F over cells (each thread a run of cells); tails counted by length
        int fsum = 0;
        for (int m = c0; m < c1; ++m) {
            const int n = cnt[cell_of(m)];
            fsum += n / kPiece;
            if (n % kPiece) atomicAdd(&lcnt[wave][n % kPiece], 1);
        }
        int nf_all = 0;
        int F = block_excl_sum(fsum, scan_sh, &nf_all);     // (its barriers also publish lcnt)
        if (threadIdx.x == 0) fstart[Q] = nf_all;
        for (int m = c0; m < c1; ++m) {
            if ((m & ((1 << lbc) - 1)) == 0) fstart[m >> lbc] = F;
            cinfo[cell_of(m)] = F;
            F += cnt[cell_of(m)] / kPiece;
        }
        __syncthreads();
        if (wave < Q) {                                  // tail slots and entries of a quadrant, longest first
            const int k = wave;
            const int nf = fstart[k + 1] - fstart[k];
            const int t = kPiece - 1 - lane;             // lengths 31 .. 1 on lanes 0 .. 30
            int before[kSortThreads / 64], n = 0;        // tails of this length in the quadrant's waves before each
#pragma unroll
            for (int w = 0; w < kSortThreads / 64; ++w) {
                before[w] = n;
                if (lane < kPiece - 1 && w < wpq) n += lcnt[k * wpq + w][t];
            }
            const int inc_n = wave_incl_sum(n);
            const int inc_e = wave_incl_sum(n * t);
            if (lane < kPiece - 1) {
                lfirst[k][t] = nf + inc_n - n;
#pragma unroll
                for (int w = 0; w < kSortThreads / 64; ++w)
                    if (w < wpq) lcnt[k * wpq + w][t] = nf + inc_n - n + before[w];
                lbase[k][t] = nf * kPiece + inc_e - n * t;
            }
            if (lane == 63) {
                npiece[k] = nf + inc_n;
                etail[k] = inc_e;
            }
        }
        __syncthreads();
        // First entry of each quadrant (its pieces start there too), and the work items.
        int ebase[Q];
        {
            int e = 0;
#pragma unroll
            for (int k = 0; k < Q; ++k) {
                ebase[k] = e;
                {
                    const int nf = fstart[k + 1] - fstart[k], count = nf * kPiece + etail[k];
                    if (threadIdx.x == k) {
                        // quadrants numbered as the tiles of a grid of T / 2-cell tiles
                        const int lt = it.x & (g.ntiles - 1), chan = it.x >> (2 * g.lbx);
                        const int r = ((lt >> g.lbx) << kLsub) + (k >> kLsub);
                        const int c = ((lt & (g.ntx - 1)) << kLsub) + (k & ((1 << kLsub) - 1));
                        const int id = (((chan << (g.lbx + kLsub)) + r) << (g.lbx + kLsub)) + c;
                        sub[item * Q + k] = make_int4(id, it.y + e, count, npiece[k] | ((nf >> 6) << 16));
                    }
                    e += count;
                }
            }
        }
        // Tail slots come from the wave's own LDS cursors, so that the layout, and with it the summation order of the
        // gridding kernel, is the same on every run.
        for (int m = c0; m < c1; ++m) {
            const int c = cell_of(m), n = cnt[c];
            if (!n) continue;
            const int k = m >> lbc;
            const int f = n / kPiece, t = n % kPiece;
            const int lc = (((c >> lb) & ms) << 8) | (c & ms);
            int eb = ebase[0];
#pragma unroll
            for (int q = 1; q < Q; ++q)
                if (k == q) eb = ebase[q];
            const int Fc = cinfo[c] - fstart[k];             // full pieces of the quadrant before this cell
            const int fe = eb + Fc * kPiece;
            for (int q = 0; q < f; ++q)
                pieces[it.y + eb + Fc + q] = make_int2(it.y + fe + q * kPiece, kPiece | (lc << 16));
            int first = 0;
            if (t) {
                const int slot = atomicAdd(&lcnt[wave][t], 1);
                first = eb + lbase[k][t] + t * (slot - lfirst[k][t]);
                pieces[it.y + eb + slot] = make_int2(it.y + first, t | (lc << 16));
            }
            cinfo[c] = fe | (first << 16);
        }
        __syncthreads();
        const int rounds = (chunk + step - 1) / step;
        for (int rd = 0; rd < rounds; ++rd) {            // uniform across the workgroup
            const int e0 = g0 + rd * step + wig * 64 * ku + lane;
            typename Pack<R>::T2 r[kSortU];
            int c[kSortU], rank[kSortU], n[kSortU], from[kSortU];
#pragma unroll
            for (int u = 0; u < kSortU; ++u) {
                from[u] = -1;
                if (u < ku && e0 + 64 * u < g1) {
                    r[u] = off0[it.y + e0 + 64 * u];
                    from[u] = perm0 ? perm0[it.y + e0 + 64 * u] : it.y + e0 + 64 * u;
                }
            }
#pragma unroll
            for (int u = 0; u < kSortU; ++u)
                c[u] = from[u] < 0 ? 0 : (static_cast<int>(r[u].y >> sh) << lb) + static_cast<int>(r[u].x >> sh);
            if (wpg == 1) {                              // the group's counters are the wave's own
#pragma unroll
                for (int u = 0; u < kSortU; ++u)
                    if (from[u] >= 0) {
                        rank[u] = atomicAdd(&gc[c[u]], 1);
                        n[u] = cnt[c[u]];
                    }
            } else {
                for (int w = 0; w < wpg; ++w) {          // uniform: every group has wpg waves
                    if (wig == w) {
#pragma unroll
                        for (int u = 0; u < kSortU; ++u)
                            if (from[u] >= 0) {
                                n[u] = atomicAdd(&gc[c[u]], 1 << 16);  // one group: gc is cnt
                                rank[u] = n[u] >> 16;
                                n[u] &= 0xffff;
                            }
                    }
                    __syncthreads();
                }
            }
#pragma unroll
            for (int u = 0; u < kSortU; ++u) {
                if (from[u] < 0) continue;
                const int ci = cinfo[c[u]];
                const int full = n[u] & ~(kPiece - 1);
                const int pos = rank[u] < full ? (ci & 0xffff) + rank[u] : (ci >> 16) + rank[u] - full;
                const int dst = it.y + pos;
                off[dst] = r[u];
                map[from[u]] = dst;
            }
        }
        __syncthreads();                                 // LDS counters are reused by the next item
    }
}

// Pass 5: caller index -> entry index, composed once so that the per-call
// permutations need a single lookup: inv[k] = pos2[inv0[k]] (-1: dropped).
// Each thread handles kComposeE indices a block apart, so that that many
// independent gathers are in flight per thread.
constexpr int kComposeE = 8;
__global__ __launch_bounds__(kPermThreads) void k_plan_compose(const int* __restrict__ inv0, const int* __restrict__ pos2,
                                                      int64_t nvis, int* __restrict__ inv) {
    const int64_t base = static_cast<int64_t>(xcd_chunk(blockIdx.x, gridDim.x)) * (blockDim.x * kComposeE) + threadIdx.x;
    int d[kComposeE];
#pragma unroll
    for (int e = 0; e < kComposeE; ++e) {
        const int64_t k = base + e * blockDim.x;
        d[e] = k < nvis ? nt_load(inv0 + k) : 0;     // 0: a valid position (nvis > 0), result unused
    }
    int r[kComposeE];
#pragma unroll
    for (int e = 0; e < kComposeE; ++e) r[e] = pos2[d[e]];
#pragma unroll
    for (int e = 0; e < kComposeE; ++e) {
        const int64_t k = base + e * blockDim.x;
        if (k < nvis) inv[k] = r[e];
    }
}

// Caller order -> entry order: vs[inv[k]] = w_k V_k. Reads are sequential;
// the writes of one block land in a few runs per footprint cell. `zero` (or
// nullptr): the work-item counter of the gridding launch that follows, which
// would otherwise take a launch of its own.
template <typename R>
__global__ __launch_bounds__(kPermThreads) void k_permute_in(const typename C2<R>::T* __restrict__ vis, const float* __restrict__ w,
                                                    const int* __restrict__ inv, int64_t nvis,
                                                    typename C2<R>::T* __restrict__ vs, int* zero) {
    const int64_t k = static_cast<int64_t>(xcd_chunk(blockIdx.x, gridDim.x)) * blockDim.x + threadIdx.x;
    if (zero && k == 0) *zero = 0;
    if (k >= nvis) return;
    const int d = nt_load(inv + k);
    if (d < 0) return;
    typename C2<R>::T v = nt_load(vis + k);
    if (w) {
        const R wk = static_cast<R>(nt_load(w + k));
        v.x *= wk;
        v.y *= wk;
    }
    vs[d] = v;
}

// Entry order -> caller order: out[k] = vs[inv[k]], zero for dropped
// visibilities. kPermOutE indices a block apart per thread, so that several
// gathers are in flight per thread. (The scattering direction, k_permute_in,
// keeps one index per thread: there more in flight spreads the writes to a
// line over a longer time and L2 merges fewer of them.)
constexpr int kPermOutE = 4;
template <typename R>
__global__ __launch_bounds__(kPermThreads) void k_permute_out(const typename C2<R>::T* __restrict__ vs, const int* __restrict__ inv,
                                                     int64_t nvis, typename C2<R>::T* __restrict__ out) {
    const int64_t base = static_cast<int64_t>(xcd_chunk(blockIdx.x, gridDim.x)) * (blockDim.x * kPermOutE) + threadIdx.x;
    int d[kPermOutE];
#pragma unroll
    for (int e = 0; e < kPermOutE; ++e) {
        const int64_t k = base + e * blockDim.x;
        d[e] = k < nvis ? nt_load(inv + k) : -1;
    }
    typename C2<R>::T v[kPermOutE];
#pragma unroll
    for (int e = 0; e < kPermOutE; ++e) {
        v[e].x = 0;
        v[e].y = 0;
        if (d[e] >= 0) v[e] = vs[d[e]];
    }
#pragma unroll
    for (int e = 0; e < kPermOutE; ++e) {
        const int64_t k = base + e * blockDim.x;
        if (k < nvis) out[k] = v[e];
    }
}

// Zero n ints (work counters) with vector stores.
__global__ void k_zero_ints(int* __restrict__ p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

}  // namespace dev

namespace {
unsigned copy_groups(const PlanSetup& a) {
    int n = 0;
    for (int q = 0; q < PlanSetup::kCopies; ++q) n += (a.bytes[q] + 15) / 16;
    return static_cast<unsigned>((n + kPlanThreads - 1) / kPlanThreads);
}
// LDS of the scan over ns slots with their counts and two offset arrays in it; 0 if it does not fit.
size_t staged_scan_bytes(size_t ns) {
    const size_t bytes = (dev::kScanSums + 2 * ns) * sizeof(int);
    return bytes <= kMaxDynLds ? bytes : 0;
}
}  // namespace

hipError_t launch_plan_count(const double* uv, const PlanBlocks& blocks, int nb, const PlanGeom& g, int* blockhist,
                             const PlanSetup& setup, hipStream_t s) {
    const unsigned groups = nb + copy_groups(setup);
    if (groups == 0) return hipSuccess;
    hipLaunchKernelGGL(dev::k_plan_count, dim3(groups), dim3(kPlanThreads), (g.ntiles + 1) * sizeof(int), s,
                       reinterpret_cast<const double2*>(uv), blocks, nb, g, blockhist, setup);
    return hipGetLastError();
}

bool small_plan(const PlanGeom& g, int64_t nvis) {
    return g.nchan == 1 && nvis <= kSmallPlanVis && staged_scan_bytes(static_cast<size_t>(g.ntiles) + 1) != 0;
}

hipError_t launch_plan_small(bool f64, const double* uv, const PlanGeom& g, int nvis, int* tile_start, int* item_start,
                             int4* items, int* flags, int cap, int* host_flags, double dlo, int ms, int kb, int* perm0,
                             void* off0, const PlanSetup& setup, hipStream_t s) {
    const size_t shm = staged_scan_bytes(static_cast<size_t>(g.ntiles) + 1);
    const dim3 groups(1 + copy_groups(setup));
    const double2* c = reinterpret_cast<const double2*>(uv);
    if (f64)
        hipLaunchKernelGGL(dev::k_plan_small<double>, groups, dim3(kPlanThreads), shm, s, c, g, nvis, tile_start, item_start,
                           items, flags, cap, host_flags, dlo, ms, kb, perm0, reinterpret_cast<ulonglong2*>(off0), setup);
    else
        hipLaunchKernelGGL(dev::k_plan_small<float>, groups, dim3(kPlanThreads), shm, s, c, g, nvis, tile_start, item_start,
                           items, flags, cap, host_flags, dlo, ms, kb, perm0, reinterpret_cast<uint2*>(off0), setup);
    return hipGetLastError();
}

hipError_t launch_plan_colscan(const PlanGeom& g, int* blockhist, const int* chan_blocks, int nb, int* tile_count,
                               hipStream_t s) {
    const int64_t ns = static_cast<int64_t>(g.ntiles) * g.nchan + 1;
    hipLaunchKernelGGL(dev::k_plan_colscan, dim3(static_cast<unsigned>((ns + 63) / 64)), dim3(64 * dev::kScanGroups),
                       0, s, g, blockhist, chan_blocks, nb, tile_count);
    return hipGetLastError();
}

hipError_t launch_plan_scan(const PlanGeom& g, const int* tile_count, int* tile_start, int* item_start, int4* items,
                            int* flags, int cap, int* host_flags, hipStream_t s) {
    // Staged through LDS when the counts and two offset arrays fit.
    const size_t staged = staged_scan_bytes(static_cast<size_t>(g.ntiles) * g.nchan + 1);
    const size_t shm = staged ? staged : dev::kScanSums * sizeof(int);
    hipLaunchKernelGGL(dev::k_plan_scan, dim3(1), dim3(1024), shm, s, g, tile_count, tile_start, item_start, items,
                       flags, cap, staged ? 1 : 0, host_flags);
    return hipGetLastError();
}

size_t packed_offset_bytes(bool f64) { return f64 ? sizeof(dev::Pack<double>::T2) : sizeof(dev::Pack<float>::T2); }
int packed_cell_shift(bool f64, int lb) {
    return f64 ? dev::pack_cell_shift<double>(lb) : dev::pack_cell_shift<float>(lb);
}

namespace {
template <typename R, bool kDirect>
void scatter(const double* uv, const PlanBlocks& blocks, int nb, const PlanGeom& g, const int* tile_start,
             const int* blockhist, double dlo, int ms, int kb, int* index, void* offs, hipStream_t s) {
    hipLaunchKernelGGL((dev::k_plan_scatter<R, kDirect>), dim3(nb), dim3(kPlanThreads), (g.ntiles + 1) * sizeof(int), s,
                       reinterpret_cast<const double2*>(uv), blocks, nb, g, tile_start, blockhist, dlo, ms, kb,
                       index, reinterpret_cast<typename dev::Pack<R>::T2*>(offs));
}
}  // namespace

hipError_t launch_plan_scatter(bool f64, bool direct, const double* uv, const PlanBlocks& blocks, int nb, const PlanGeom& g,
                               const int* tile_start, const int* blockhist, double dlo, int ms, int kb,
                               int* index, void* offs, hipStream_t s) {
    if (nb == 0) return hipSuccess;
    if (f64 && direct) scatter<double, true>(uv, blocks, nb, g, tile_start, blockhist, dlo, ms, kb, index, offs, s);
    else if (f64) scatter<double, false>(uv, blocks, nb, g, tile_start, blockhist, dlo, ms, kb, index, offs, s);
    else if (direct) scatter<float, true>(uv, blocks, nb, g, tile_start, blockhist, dlo, ms, kb, index, offs, s);
    else scatter<float, false>(uv, blocks, nb, g, tile_start, blockhist, dlo, ms, kb, index, offs, s);
    return hipGetLastError();
}

hipError_t launch_plan_place(bool f64, const int* inv0, const void* offk, const int* flags, int64_t nvis, void* off0,
                             hipStream_t s) {
    if (nvis == 0) return hipSuccess;
    const unsigned nb = static_cast<unsigned>((nvis + dev::kPermThreads - 1) / dev::kPermThreads);
    if (f64)
        hipLaunchKernelGGL(dev::k_plan_place<double>, dim3(nb), dim3(dev::kPermThreads), 0, s, inv0,
                           reinterpret_cast<const ulonglong2*>(offk), flags, nvis, reinterpret_cast<ulonglong2*>(off0));
    else
        hipLaunchKernelGGL(dev::k_plan_place<float>, dim3(nb), dim3(dev::kPermThreads), 0, s, inv0,
                           reinterpret_cast<const uint2*>(offk), flags, nvis, reinterpret_cast<uint2*>(off0));
    return hipGetLastError();
}

namespace {
template <typename R, int kLsub>
void sort_items(unsigned nb, size_t shm, const PlanGeom& g, const int4* items, int4* sub, const int* flags, int nvis, int lb,
                int groups, const void* off0, const int* perm0, void* off, int* map, int2* pieces, hipStream_t s) {
    using P2 = typename dev::Pack<R>::T2;
    hipLaunchKernelGGL((dev::k_plan_sort_items<R, kLsub>), dim3(nb), dim3(dev::kSortThreads), shm, s, g, items, sub, flags,
                       nvis, lb, groups, reinterpret_cast<const P2*>(off0), perm0, reinterpret_cast<P2*>(off), map, pieces);
}
}  // namespace

hipError_t launch_plan_sort(bool f64, const PlanGeom& g, const int4* items, int4* sub, int max_items, const int* flags, int nvis,
                            int lb, const void* off0, const int* perm0, void* off, int* map, int2* pieces,
                            hipStream_t s) {
    // One counter group per wave while the counters fit in 40 KB with the per-cell arrays (T <= 32),
    // else one group whose waves take turns.
    const size_t TT = static_cast<size_t>(g.T) * g.T;
    const int waves = dev::kSortThreads / 64;
    const int groups = (2 + waves) * TT * sizeof(int) <= 40 * 1024 ? waves : 1;
    const size_t shm = (2 + (groups > 1 ? groups : 0)) * TT * sizeof(int);
    const unsigned nb = static_cast<unsigned>(std::max(1, std::min(max_items, 8192)));
    if (f64 && g.lsub) sort_items<double, 1>(nb, shm, g, items, sub, flags, nvis, lb, groups, off0, perm0, off, map, pieces, s);
    else if (f64) sort_items<double, 0>(nb, shm, g, items, sub, flags, nvis, lb, groups, off0, perm0, off, map, pieces, s);
    else if (g.lsub) sort_items<float, 1>(nb, shm, g, items, sub, flags, nvis, lb, groups, off0, perm0, off, map, pieces, s);
    else sort_items<float, 0>(nb, shm, g, items, sub, flags, nvis, lb, groups, off0, perm0, off, map, pieces, s);
    return hipGetLastError();
}

hipError_t launch_plan_compose(const int* inv0, const int* pos2, int64_t nvis, int* inv, hipStream_t s) {
    if (nvis == 0) return hipSuccess;
    const int64_t per = dev::kPermThreads * dev::kComposeE;
    hipLaunchKernelGGL(dev::k_plan_compose, dim3(static_cast<unsigned>((nvis + per - 1) / per)), dim3(dev::kPermThreads), 0,
                       s, inv0, pos2, nvis, inv);
    return hipGetLastError();
}

hipError_t launch_permute_in(bool f64, const void* vis, const float* w, const int* inv, int64_t nvis, void* vs,
                             int* zero, hipStream_t s) {
    if (nvis == 0) return hipSuccess;
    const unsigned nb = static_cast<unsigned>((nvis + dev::kPermThreads - 1) / dev::kPermThreads);
    if (f64)
        hipLaunchKernelGGL(dev::k_permute_in<double>, dim3(nb), dim3(dev::kPermThreads), 0, s,
                           reinterpret_cast<const double2*>(vis), w, inv, nvis, reinterpret_cast<double2*>(vs), zero);
    else
        hipLaunchKernelGGL(dev::k_permute_in<float>, dim3(nb), dim3(dev::kPermThreads), 0, s,
                           reinterpret_cast<const float2*>(vis), w, inv, nvis, reinterpret_cast<float2*>(vs), zero);
    return hipGetLastError();
}

hipError_t launch_permute_out(bool f64, const void* vs, const int* inv, int64_t nvis, void* out, hipStream_t s) {
    if (nvis == 0) return hipSuccess;
    const int64_t per = dev::kPermThreads * dev::kPermOutE;
    const unsigned nb = static_cast<unsigned>((nvis + per - 1) / per);
    if (f64)
        hipLaunchKernelGGL(dev::k_permute_out<double>, dim3(nb), dim3(dev::kPermThreads), 0, s,
                           reinterpret_cast<const double2*>(vs), inv, nvis, reinterpret_cast<double2*>(out));
    else
        hipLaunchKernelGGL(dev::k_permute_out<float>, dim3(nb), dim3(dev::kPermThreads), 0, s,
                           reinterpret_cast<const float2*>(vs), inv, nvis, reinterpret_cast<float2*>(out));
    return hipGetLastError();
}

hipError_t launch_zero_ints(int* p, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(dev::k_zero_ints, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t set_kernel_attributes() {
    hipError_t e = hipSuccess;
#define LMG_ATTR(bytes, ...) do { hipError_t r = hipFuncSetAttribute(reinterpret_cast<const void*>(__VA_ARGS__), \
        hipFuncAttributeMaxDynamicSharedMemorySize, bytes); if (r != hipSuccess) e = r; } while (0)
    // Per-tile histograms of up to 128 x 128 ints; the item sort keeps two per-cell arrays of up to 128 x 128.
    LMG_ATTR(72 * 1024, &dev::k_plan_count);
    LMG_ATTR(kMaxDynLds, &dev::k_plan_scan);
    LMG_ATTR(kMaxDynLds, &dev::k_plan_small<float>);
    LMG_ATTR(kMaxDynLds, &dev::k_plan_small<double>);
    LMG_ATTR(72 * 1024, &dev::k_plan_scatter<float, false>);
    LMG_ATTR(72 * 1024, &dev::k_plan_scatter<float, true>);
    LMG_ATTR(72 * 1024, &dev::k_plan_scatter<double, false>);
    LMG_ATTR(72 * 1024, &dev::k_plan_scatter<double, true>);
    LMG_ATTR(128 * 1024, &dev::k_plan_sort_items<float, 0>);
    LMG_ATTR(128 * 1024, &dev::k_plan_sort_items<float, 1>);
    LMG_ATTR(128 * 1024, &dev::k_plan_sort_items<double, 0>);
    LMG_ATTR(128 * 1024, &dev::k_plan_sort_items<double, 1>);
#undef LMG_ATTR
    return e;
}

hipError_t take_data_error(int* flag) {
    int v = 0;
    hipError_t e = hipMemcpyFromSymbol(&v, HIP_SYMBOL(dev::g_data_error), sizeof(int), 0, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return e;
    *flag = v;
    if (v) {
        const int zero = 0;
        e = hipMemcpyToSymbol(HIP_SYMBOL(dev::g_data_error), &zero, sizeof(int), 0, hipMemcpyHostToDevice);
    }
    return e;
}

}  // namespace lmg

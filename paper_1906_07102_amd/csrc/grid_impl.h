// Gridding kernels: the persistent item kernel and the assemble kernel,
// templated on the accumulation mode. Included by one translation unit per
// mode (grid_f32.hip, grid_kahan.hip, grid_f64.hip) so that they compile in
// parallel.
#pragma once

#include <type_traits>

#include "dev_common.h"

namespace lmg {
namespace dev {

// ------------------------------------------------------------ gridding
// Accumulation policies. `Reg` accumulates one footprint cell over a piece
// in registers; `Cell` is the LDS patch element. One wave at a time
// flushes into a patch, so a flush is a plain read-modify-write. Lanes of one wave
// may flush overlapping footprints, so one tap's store must reach LDS before another
// tap's load: the patch is accessed with 64-bit atomic loads and stores of
// wavefront scope and sequential consistency, which the compiler neither
// merges nor reorders (LDS executes one wave's operations in order, so they
// cost no waits). `Sum` adds the wave patches of a workgroup, and the patches
// covering a grid cell: FP64 for plain FP32 and FP64, compensated FP32 (TwoSum
// into (hi, lo) pairs) for the compensated form.
using u64 = unsigned long long;

__device__ __forceinline__ u64 lds_ld(const void* p) {
    return __hip_atomic_load(reinterpret_cast<const u64*>(p), __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ void lds_st(void* p, u64 v) {
    __hip_atomic_store(reinterpret_cast<u64*>(p), v, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
__device__ __forceinline__ float2 as_f2(u64 v) {
    float2 f;
    __builtin_memcpy(&f, &v, 8);
    return f;
}
__device__ __forceinline__ u64 as_u64(float2 f) {
    u64 v;
    __builtin_memcpy(&v, &f, 8);
    return v;
}
__device__ __forceinline__ double as_d(u64 v) { return __builtin_bit_cast(double, v); }
__device__ __forceinline__ u64 as_u64(double d) { return __builtin_bit_cast(u64, d); }

struct AccF32 {
    using Cell = float2;
    using Reg = float2;
    static constexpr int kAccRegs = 112;
    __device__ static void zero_cell(Cell* c) { *c = make_float2(0.f, 0.f); }
    __device__ static void set(Reg& r, float re, float im) { r = make_float2(re, im); }
    __device__ static void add(Reg& r, float re, float im) {
        r.x += re;
        r.y += im;
    }
    __device__ static void rmw(Cell* c, const Reg& r) {
        float2 v = as_f2(lds_ld(c));
        v.x += r.x;
        v.y += r.y;
        lds_st(c, as_u64(v));
    }
    // Sum of cells (the patches of an item, then the patches covering a grid cell), in FP64, rounded once: the merges
    // add no error to the flushes' own (16.8M visibilities, W = 7: relative RMS against FP64 6.41e-8 with FP32 merges,
    // 5.47e-8; assembling a 4096^2 grid of 4.2M 36 us and 37).
    struct Sum {
        double2 s = make_double2(0.0, 0.0);
        __device__ void add(const Cell& c) {
            s.x += c.x;
            s.y += c.y;
        }
        __device__ Cell cell() const { return make_float2(static_cast<float>(s.x), static_cast<float>(s.y)); }
        __device__ float2 value(float2 old) const {
            const Cell c = cell();
            return make_float2(old.x + c.x, old.y + c.y);
        }
    };
};

// Compensated FP32 tile sums. A lane sums one piece (at most kPiece terms of
// one cell) in plain FP32 registers, and each flush adds that sum to the
// patch cell's (hi, lo) pair with TwoSum (Knuth: the rounding error of the
// addition, exactly), which goes to lo. So the many flushes that reach a patch
// cell, and the merges of patches, add no rounding error beyond the pieces'
// own short sums. A cell's value is hi + lo. Two registers per tap (as FP32)
// keep W = 7 in one pass over each piece.
struct AccKahan {
    using Cell = float4;      // (hi re, hi im, lo re, lo im)
    using Reg = float2;
    static constexpr int kAccRegs = 112;
    __device__ static void zero_cell(Cell* c) { *c = make_float4(0.f, 0.f, 0.f, 0.f); }
    __device__ static void set(Reg& r, float re, float im) { r = make_float2(re, im); }
    __device__ static void add(Reg& r, float re, float im) {
        r.x += re;
        r.y += im;
    }
    __device__ static void two_sum(float a, float b, float& s, float& e) {
        s = a + b;
        const float bp = s - a;
        e = (a - (s - bp)) + (b - bp);
    }
    __device__ static void rmw(Cell* c, const Reg& r) {
        float2* h = reinterpret_cast<float2*>(c);
        const float2 s = as_f2(lds_ld(h));
        const float2 k = as_f2(lds_ld(h + 1));
        float nx, ex, ny, ey;
        two_sum(s.x, r.x, nx, ex);
        two_sum(s.y, r.y, ny, ey);
        lds_st(h, as_u64(make_float2(nx, ny)));
        lds_st(h + 1, as_u64(make_float2(k.x + ex, k.y + ey)));
    }
    // Compensated sum of cells in FP32: the high parts are added with TwoSum, and their rounding errors
    // together with the cells' compensation terms go to the low part (value = hi + lo).
    struct Sum {
        float hr = 0.f, hi = 0.f, lr = 0.f, li = 0.f;
        __device__ void add(const Cell& c) {
            float t, e;
            two_sum(hr, c.x, t, e);
            hr = t;
            lr += e + c.z;
            two_sum(hi, c.y, t, e);
            hi = t;
            li += e + c.w;
        }
        // renormalised (hi, lo) pair: hi the rounded value, lo what it leaves out
        __device__ Cell cell() const {
            float a, ea, b, eb;
            two_sum(hr, lr, a, ea);
            two_sum(hi, li, b, eb);
            return make_float4(a, b, ea, eb);
        }
        // old + hi + lo, with the addition of old to hi compensated as well
        __device__ float2 value(float2 old) const {
            float a, ea, b, eb;
            two_sum(old.x, hr, a, ea);
            two_sum(old.y, hi, b, eb);
            return make_float2(a + (ea + lr), b + (eb + li));
        }
    };
};

struct AccF64 {
    using Cell = double2;
    using Reg = double2;
    static constexpr int kAccRegs = 224;
    __device__ static void zero_cell(Cell* c) { *c = make_double2(0.0, 0.0); }
    __device__ static void set(Reg& r, double re, double im) { r = make_double2(re, im); }
    __device__ static void add(Reg& r, double re, double im) {
        r.x += re;
        r.y += im;
    }
    __device__ static void rmw(Cell* c, const Reg& r) {
        double* d = reinterpret_cast<double*>(c);
        const double x = as_d(lds_ld(d));
        const double y = as_d(lds_ld(d + 1));
        lds_st(d, as_u64(x + r.x));
        lds_st(d + 1, as_u64(y + r.y));
    }
    struct Sum {
        double2 s = make_double2(0.0, 0.0);
        __device__ void add(const Cell& c) {
            s.x += c.x;
            s.y += c.y;
        }
        __device__ Cell cell() const { return s; }
        __device__ double2 value(double2 old) const { return make_double2(old.x + s.x, old.y + s.y); }
    };
};

// Register accumulation: a lane sums one piece's contributions to a group of
// RG footprint rows (RG x W accumulators) and then adds them to the patch;
// footprints wider than the mode's register budget (kBudget) take
// several such passes over the piece. The FP32 forms keep the accumulators
// near 112 registers, so that three waves fit a SIMD, but for W = 8, whose 128
// in one pass leave room for two (3.0M of one density on 2048^2, two passes of
// four rows / one, FP32 143 / 108 us, compensated 185 / 160). FP64 takes 224,
// one pass at W = 7, where two waves fit (16.8M visibilities, 0.59 -> 0.48 ms
// with one pass instead of two), and 160 above, which leave room for two waves
// as well: more passes over a piece, but twice the waves and the patches that a
// compute unit works on (4.2M on 4096^2, W = 8 445 us; 3.0M of one density on
// 2048^2, one wave per SIMD with 224 / two with 160, W = 9 275 / 231 us, W = 14
// 863 / 631).
template <typename Acc, int W>
struct RowGroup {
    static constexpr bool kF64 = sizeof(typename Acc::Reg) == 16;
    static constexpr int kRegsPerTap = static_cast<int>(sizeof(typename Acc::Reg) / 4);
    static constexpr int kBudget = kF64 ? (W >= 8 ? 160 : Acc::kAccRegs) : W == 8 ? 128 : Acc::kAccRegs;
    static constexpr int kRG0 = kBudget / (kRegsPerTap * W);
    static constexpr int kRG1 = kRG0 < 1 ? 1 : (kRG0 > W ? W : kRG0);
    static constexpr int kPasses = (W + kRG1 - 1) / kRG1;
    static constexpr int RG = (W + kPasses - 1) / kPasses;     // the passes' rows as even as they go
};
// Waves per SIMD the compiler keeps room for. (The compensated form at W = 7 needs a few registers more than three leave
// it; with two, 3.0M visibilities of one density on 2048^2 147 -> 113 us, 4.2M of tracks on 4096^2 140 -> 119.)
template <typename Acc, int W, int kTab>
constexpr int waves_per_simd() {
    using G = RowGroup<Acc, W>;
    constexpr int widest = std::is_same<Acc, AccKahan>::value ? 6 : 7;
    return (!G::kF64 && W <= widest && kTab != kTabDirect) ? 3 : 2;
}

// Add the piece's accumulated rows r0 .. r0 + RG - 1 (those below W) to the
// patch. Lanes holding the same cell take turns: each round one of them wins
// the cell (the last store to its owner byte) and adds its values.
template <typename Acc, int W, int RG>
__device__ __forceinline__ void flush_rows(typename Acc::Cell* patch, unsigned char* owner, int P, int lane, bool have,
                                           int l, int r0, const typename Acc::Reg* acc) {
    bool pending = have;
    const int cidx = (l >> 8) * P + (l & 255);
    while (__any(pending)) {
        if (pending)
            __hip_atomic_store(&owner[cidx], static_cast<unsigned char>(lane), __ATOMIC_SEQ_CST,
                               __HIP_MEMORY_SCOPE_WAVEFRONT);
        const int who = pending ? static_cast<int>(__hip_atomic_load(&owner[cidx], __ATOMIC_SEQ_CST,
                                                                     __HIP_MEMORY_SCOPE_WAVEFRONT))
                                : -1;
        if (pending && who == lane) {
            typename Acc::Cell* row = patch + cidx + r0 * P;
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                if (r0 + r >= W) break;
#pragma unroll
                for (int c = 0; c < W; ++c) Acc::rmw(&row[r * P + c], acc[r * W + c]);
            }
            pending = false;
        }
    }
}

// Persistent: a fixed set of workgroups takes work items from a counter
// (a.counter, zero at launch) until none are left, so the table is staged
// once per workgroup and uneven items (many channels of very different
// sizes) balance dynamically.
//
// Pieces are taken 64 at a time (a "turn"; neighbouring full pieces, often of
// one cell, go to different turns), the shortest first: a cell's plain FP32 sum
// then rounds while it is small, which halves the error that the flushes add
// (relative RMS of the grid against FP64, W = 7, longest first / shortest first
// with the FP64 merges: 201,600 visibilities on 1024^2 8.19e-8 / 6.37e-8, 16.8M on
// 4096^2 6.82e-8 / 5.47e-8), and the waves of a patch flush one after another
// while the longer pieces are still summed (compensated, W = 7, 201,600 on
// 1024^2 55 / 46 us, 1.0M on 2048^2 79 / 66). A workgroup has S = a.npatch patches and
// `waves` waves, a multiple of S; turn j is accumulated in registers by wave
// j mod waves and flushed into patch j mod S, after the turns before it on
// that patch (s_turn counts them). So the order of every sum is that of the
// plan's pieces, whatever the number of waves. With as many waves as patches
// nothing waits; more waves hide more latency where LDS holds few patches or
// the launch has few items.
template <typename R, typename Acc, int W, int kTab>
__global__ __launch_bounds__(64 * kMaxGridWaves)
__attribute__((amdgpu_waves_per_eu(waves_per_simd<Acc, W, kTab>()))) void k_grid_items(GridArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_item, s_turn[kMaxGridWaves];
    using VT = typename C2<R>::T;
    using PT2 = typename Pack<R>::T2;
    using Cell = typename Acc::Cell;
    constexpr int RG = RowGroup<Acc, W>::RG;
    constexpr int NPASS = RowGroup<Acc, W>::kPasses;
    const int P = a.T + W - 1;
    const int P2 = P * P;
    const unsigned inv_p = 0xffffffffu / P + 1;             // i / P = umulhi(i, inv_p) for i < P2
    R* tab = reinterpret_cast<R*>(smem);
    const int ntab = kTab == kTabLds ? (a.Ms + 1) * W * 4 : 0;
    Cell* patches = reinterpret_cast<Cell*>(smem + ((ntab * sizeof(R) + 15) & ~size_t(15)));
    const int S = a.npatch;
    unsigned char* owners = reinterpret_cast<unsigned char*>(patches + S * P2);   // a lane id per cell
    // The wave's number, and with it its patch, turns and order of flushes, in scalar registers: in vector registers they
    // spilled at W = 7, where three waves share a SIMD's (3.0M visibilities of one density on 2048^2, FP32
    // 76 -> 70 us, compensated 152 -> 141).
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    Cell* patch = patches + (wave % S) * P2;
    unsigned char* owner = owners + (wave % S) * P2;
    int* turn_of = &s_turn[wave % S];
    const R* gtab = reinterpret_cast<const R*>(a.coef);
    for (int i = threadIdx.x; i < ntab; i += blockDim.x) tab[i] = gtab[i];
    const VT* vis = reinterpret_cast<const VT*>(a.vis);     // entry order, weights applied
    const PT2* off = reinterpret_cast<const PT2*>(a.off);   // packed offsets, entry order
    const int nitems = *a.n_items << (2 * a.lsub);
    for (bool first = true;; first = false) {
        // the first items are dealt by workgroup, the others (if there can be any) from the counter
        if (threadIdx.x == 0) {
            if (first) s_item = blockIdx.x;
            else s_item = static_cast<int>(gridDim.x) < a.max_items ? gridDim.x + atomicAdd(a.counter, 1) : nitems;
        }
        if (threadIdx.x < S) s_turn[threadIdx.x] = 0;
        for (int i = threadIdx.x; i < S * P2; i += blockDim.x) Acc::zero_cell(&patches[i]);
        __syncthreads();
        const int item = s_item;
        if (item >= nitems) break;                       // uniform across the workgroup
        const int4 it = a.items[item];
        // entries whose loads are issued together: FP64, 8.4M visibilities on 4096^2 with 1 / 4, W = 3 188 / 125 us, W = 5
        // 222 / 163; at W = 7 with 1 / 2, 16.8M 453 / 460 us, 3.0M of one density 138 / 145 (4 spills, and above W = 8
        // leaves one wave per SIMD). Direct weights with 1 / 2 / 4: FP64, 8.4M, W = 5 772 / 702 / 705 us, W = 8 2165 /
        // 1928 / 2321; FP32, 4.2M, W = 6 2 / 4 434 / 636 us.
        // In the FP32 forms the code for four entries in every pass outgrows the instruction cache from W = 14 on (13 in
        // the compensated form, whose flush is longer; there two do from W = 15): 4.2M with 4 / 2 / 1, FP32 W = 13 294 /
        // 306 / 323 us, 14 428 / 336 / 351, 16 1150 / 741 / 781; compensated 12 330 / 335 / 343, 13 464 / 372 / 386, 15 580
        // / 603 / 509, 16 1273 / 1300 / 895.
        constexpr bool kComp = std::is_same<Acc, AccKahan>::value;
        constexpr int kWide = kComp && W >= 15 ? 1 : W >= (kComp ? 13 : 14) ? 2 : 4;
        constexpr int kB = kTab == kTabDirect ? 2 : sizeof(R) == 8 && W >= 6 ? 1 : kWide;
        const int np = it.w & 0xffff, fturns = it.w >> 16;  // pieces; turns of full pieces only
        const int turns = (np + 63) >> 6;
        // the lane's piece of turn j: turns count from the shortest tails (a ragged last run of 64) to the full pieces; from
        // the full pieces where direct weights make a long last turn the item's time and sums are not plain FP32 (8.4M on
        // 4096^2, shortest / longest first: compensated W = 2 374 / 330 us, 6 846 / 713; FP64 W = 1 310 / 279, 4 559 / 520).
        // Dealt: S runs, each of another patch, take 64 S pieces by turns (such groups count from the longest pieces).
        constexpr bool kPlain = std::is_same<Acc, AccF32>::value, kLongFirst = kTab == kTabDirect && !kPlain;
        const bool deal = kPlain && a.deal && fturns == 0;
        const int nth = deal ? (turns - 1 + S - wave % S) % S : 0;      // of the wave's runs in their groups
        auto piece_of = [&](int j) {
            const int run = kLongFirst ? (j < turns ? j : -1) : turns - 1 - j;
            if (run < 0) return np;
            if (deal) return (run - nth) * 64 + lane * min(S, turns - run + nth) + nth;
            return run < fturns ? lane * fturns + run : run * 64 + lane;
        };
#pragma unroll
        for (int pass = 0; pass < NPASS; ++pass) {
            const int r0 = pass * RG;
            int2 pc_next = make_int2(0, 0);                 // a lane's piece of the next turn is loaded a turn ahead
            if (piece_of(wave) < np) pc_next = a.pieces[it.y + piece_of(wave)];
            for (int j = wave; j < turns; j += nw) {        // uniform across the wave
                const bool have = piece_of(j) < np;
                const int2 pc = pc_next;
                pc_next = make_int2(0, 0);
                const int pn = piece_of(j + nw);
                if (pn < np) pc_next = a.pieces[it.y + pn];
                const int len = pc.y & 0xffff;
                const int l = static_cast<int>(static_cast<unsigned>(pc.y) >> 16);
                typename Acc::Reg acc[RG * W];
                // One batch of kB entries from entry j0 of the piece. The first batch sets the accumulators
                // from its first entry instead of adding to zeros; every lane runs that entry (a lane without
                // a piece reads entry 0 of the arrays and never flushes), so no accumulator is ever zeroed.
                auto batch = [&](int j0, auto first) {
                    constexpr bool kFirst = decltype(first)::value;
                    PT2 dv[kB];
                    VT vv[kB];
                    load_run<kB>(off + pc.x + j0, dv);
                    load_run<kB>(vis + pc.x + j0, vv);
#pragma unroll
                    for (int u = 0; u < kB; ++u) {
                        if (!(kFirst && u == 0) && j0 + u >= len) break;
                        R cu[W], cv[W];
                        if constexpr (kTab == kTabDirect) {
                            weights_direct<R, W>(static_cast<const double*>(a.coef), dv[u].x, a.Ft, cu);
                            weights_direct<R, W>(static_cast<const double*>(a.coef), dv[u].y, a.Ft, cv);
                        } else if constexpr (kTab == kTabGlobal) {
                            weights<R, W>(gtab, a.Ms, a.degree, dv[u].x, a.Ft, a.kb, cu);
                            weights<R, W>(gtab, a.Ms, a.degree, dv[u].y, a.Ft, a.kb, cv);
                        } else {
                            weights<R, W>(tab, a.Ms, a.degree, dv[u].x, a.Ft, a.kb, cu);
                            weights<R, W>(tab, a.Ms, a.degree, dv[u].y, a.Ft, a.kb, cv);
                        }
#pragma unroll
                        for (int r = 0; r < RG; ++r) {
                            if (r0 + r >= W) break;
                            const R ar = vv[u].x * cv[r0 + r], ai = vv[u].y * cv[r0 + r];
#pragma unroll
                            for (int c = 0; c < W; ++c) {
                                if (kFirst && u == 0)
                                    Acc::set(acc[r * W + c], ar * cu[c], ai * cu[c]);
                                else
                                    Acc::add(acc[r * W + c], ar * cu[c], ai * cu[c]);
                            }
                        }
                    }
                };
                batch(0, std::true_type{});
                for (int j0 = kB; j0 < len; j0 += kB) batch(j0, std::false_type{});
                // The patch's turns are numbered in the order (pass, j); each is flushed by a wave that waits for
                // none after it.
                const int turn = pass * ((turns - wave % S + S - 1) / S) + j / S;
                if (nw > S)
                    while (__hip_atomic_load(turn_of, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != turn)
                        __builtin_amdgcn_s_sleep(1);
                flush_rows<Acc, W, RG>(patch, owner, P, lane, have && len > 0, l, r0, acc);
                if (nw > S && lane == 0)
                    __hip_atomic_store(turn_of, turn + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        __syncthreads();
        Cell* out = reinterpret_cast<Cell*>(a.patches) + static_cast<size_t>(item) * P2;
        int nout = P2;
        if (a.by_entry) {
            const int4 q = a.items[item];                   // read again: held over the turns it costs registers
            out = reinterpret_cast<Cell*>(a.patches) + static_cast<size_t>(q.y) * P2;
            if (q.z == 0) nout = 0;
        }
        for (int i = threadIdx.x; i < nout; i += blockDim.x) {
            const int row = __umulhi(static_cast<unsigned>(i), inv_p);
            const int from = a.transpose ? (i - row * P) * P + row : i;
            typename Acc::Sum sum;
            for (int w = 0; w < S; ++w) sum.add(patches[w * P2 + from]);
            out[i] = sum.cell();
        }
        __syncthreads();                                    // the patches, s_item and s_turn are reused
    }
}

// Sum the patches covering each tile (own tile, left, upper, upper-left
// neighbours, in that fixed order; the plan keeps T >= W, so no footprint
// reaches a tile two away) in the mode's own arithmetic and write every grid
// cell of the window once: overwriting it, or adding to what it holds
// (a.accumulate). When adding, a workgroup whose tile receives no patch
// returns at once, so cells outside the data's footprint are neither read nor
// written. One workgroup per a.rows rows of a tile (chosen by the launcher).

// Patches of the items that cover tile (r, c) of a channel whose first plan tile is cbase: numbers first, first + step,
// ... before end. A transposed grid's tile rows run along u, while plan tiles are numbered along v.
struct TilePatches {
    int first, end;
    __device__ __forceinline__ TilePatches(const AssembleArgs& a, int cbase, int r, int c) {
        const int tv = a.transpose ? c : r, tu = a.transpose ? r : c;
        const int t = cbase + (tv >> a.lsub) * (a.ntx >> a.lsub) + (tu >> a.lsub), m = (1 << a.lsub) - 1;
        const int q = ((tv & m) << a.lsub) + (tu & m);
        first = (a.item_start[t] << (2 * a.lsub)) + q;
        end = a.item_start[t + 1] << (2 * a.lsub);
    }
};

// Cells of one tile, rows rb .. of it (ncell cells of them), written from the patches that cover them (own tile, left,
// upper, upper-left: numbers first[s], first[s] + step, ... before end[s]); dst: the first of them. A thread takes KC
// cells a few rows apart and a batch of patches at a time, all loads issued before the first is added: what bounds the
// occupied tiles is the latency of a cell's chain of patches, not their bytes (one 4096^2 grid of 16.8M visibilities
// 64 us with one cell per thread, 51 with four; its occupied band 32, 27 with two; 4.2M on 8192^2 in FP32 164, 143).
// kSub: patches are numbered by their items' first entries (a.sub), not by item.
template <typename R, typename Acc, int KC, bool kSub>
__device__ __forceinline__ void tile_cells(const AssembleArgs& a, typename C2<R>::T* dst, int rb, int ncell, int lbT,
                                           const int* first, const int* end, int step) {
    using VT = typename C2<R>::T;
    using Cell = typename Acc::Cell;
    constexpr int kU = KC >= 4 ? 1 : 4 / KC;               // patches per batch
    const int P = a.T + a.W - 1, halo = a.W - 1;
    const Cell* patches = reinterpret_cast<const Cell*>(a.patches);
    const int lc = threadIdx.x & (a.T - 1);                // 256 threads: whole rows of a tile
    for (int base = threadIdx.x; base < ncell; base += KC * kAssembleThreads) {
        typename Acc::Sum sum[KC];
        VT old[KC];
        bool on[KC];
        int lr[KC];
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const int cell = base + k * kAssembleThreads;
            on[k] = cell < ncell;
            lr[k] = rb + (cell >> lbT);
            old[k].x = 0;
            old[k].y = 0;
            if (a.accumulate && on[k]) old[k] = dst[static_cast<size_t>(cell >> lbT) * a.N + lc];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if ((s & 1) && lc >= halo) continue;
            const int pc = lc + ((s & 1) ? a.T : 0);
            for (int it = first[s]; it < end[s]; it += kU * step) {
                Cell c[kU][KC];
                int slot[kU];                                    // the patch of item it + u step
                bool have[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    slot[u] = it + u * step;
                    have[u] = slot[u] < end[s];
                    if constexpr (kSub) {
                        const int4 q = have[u] ? a.sub[slot[u]] : make_int4(0, 0, 0, 0);     // uniform
                        slot[u] = q.y;
                        have[u] = q.z > 0;
                    }
                }
#pragma unroll
                for (int u = 0; u < kU; ++u)
#pragma unroll
                    for (int k = 0; k < KC; ++k)
                        if (have[u] && on[k] && (s < 2 || lr[k] < halo))
                            c[u][k] = patches[(static_cast<size_t>(slot[u]) * P + lr[k] + (s >= 2 ? a.T : 0)) * P + pc];
#pragma unroll
                for (int u = 0; u < kU; ++u)
#pragma unroll
                    for (int k = 0; k < KC; ++k)
                        if (have[u] && on[k] && (s < 2 || lr[k] < halo)) sum[k].add(c[u][k]);
            }
        }
#pragma unroll
        for (int k = 0; k < KC; ++k)
            if (on[k])
                dst[static_cast<size_t>((base + k * kAssembleThreads) >> lbT) * a.N + lc] = sum[k].value(old[k]);
    }
}

template <typename R, typename Acc, int KC, bool kSub>
__global__ __launch_bounds__(kAssembleThreads) void k_assemble(AssembleArgs a) {
    using VT = typename C2<R>::T;
    const int ar = a.rows;
    const int nblk = a.T / ar;
    const int per_chan = a.trows * a.tcols;
    const int chan = blockIdx.x / (nblk * per_chan);
    const int wt = (blockIdx.x / nblk) % per_chan;          // tile within the written window
    const int rb = (blockIdx.x % nblk) * ar;
    const int tm = (a.tr0 + wt / a.tcols) & (a.ntx - 1), tn = (a.tc0 + wt % a.tcols) & (a.ntx - 1);
    const int cbase = chan * ((a.ntx * a.ntx) >> (2 * a.lsub));    // plan tiles of the channels before
    const int tmu = (tm - 1) & (a.ntx - 1), tnl = (tn - 1) & (a.ntx - 1);     // ntx is a power of two, as T is
    const int lbT = __builtin_ctz(static_cast<unsigned>(a.T));
    const int step = 1 << (2 * a.lsub);
    VT* grid = reinterpret_cast<VT*>(a.grid) + static_cast<size_t>(chan) * a.N * a.N;
    const TilePatches src[4] = {{a, cbase, tm, tn}, {a, cbase, tm, tnl}, {a, cbase, tmu, tn}, {a, cbase, tmu, tnl}};
    bool any = false;
    for (int s = 0; s < 4; ++s) any = any || src[s].end > src[s].first;
    if (a.accumulate && !any) return;                       // uniform across the workgroup
    if (!any) {                                             // no patch: zeros, two cells per store
        for (int pair = threadIdx.x; pair < ar * a.T / 2; pair += blockDim.x) {
            const int lr = rb + ((2 * pair) >> lbT), lc = (2 * pair) & (a.T - 1);
            VT* dst = grid + static_cast<size_t>(tm * a.T + lr) * a.N + tn * a.T + lc;
            VT z[2];
            z[0].x = 0; z[0].y = 0; z[1] = z[0];
            __builtin_memcpy(dst, z, sizeof(z));
        }
        return;
    }
    const int first[4] = {src[0].first, src[1].first, src[2].first, src[3].first};
    const int end[4] = {src[0].end, src[1].end, src[2].end, src[3].end};
    tile_cells<R, Acc, KC, kSub>(a, grid + static_cast<size_t>(tm * a.T + rb) * a.N + tn * a.T, rb, ar << lbT, lbT, first, end,
                           step);
}

// Whole grids of many channels: one workgroup per a.rows consecutive grid
// rows of one channel, which it writes tile by tile along the row, so that a
// batch of grids takes nchan N / a.rows workgroups instead of one per tile
// (most tiles of a batch's grids receive no patch, and per-workgroup costs
// dominate). The item ranges of the two tile rows its cells read (its own
// and the one above) are staged in LDS once; a tile's ranges are then the
// same for every lane. Cells sum the same sources in the same order as
// k_assemble, so the two give the same bits; overwrite (a tile without
// patches takes zeros two cells per store), or accumulate (such a tile is
// skipped).
template <typename R, typename Acc, int KC, bool kSub>
__global__ __launch_bounds__(kAssembleThreads) void k_assemble_rows(AssembleArgs a) {
    extern __shared__ int rng[];                           // [2][ntx + 1]: item_start of plan tile rows of tm, tm - 1
    using VT = typename C2<R>::T;
    const int per_chan = a.N / a.rows;
    const int chan = blockIdx.x / per_chan;
    const int r0 = (blockIdx.x % per_chan) * a.rows;       // first grid row (storage order)
    const int tm = r0 / a.T, rb = r0 % a.T;
    const int tmu = (tm - 1) & (a.ntx - 1);
    const int nptx = a.ntx >> a.lsub;                      // plan tiles per axis
    const int cbase = chan * nptx * nptx;
    for (int i = threadIdx.x; i <= nptx; i += blockDim.x) {
        rng[i] = a.item_start[cbase + (tm >> a.lsub) * nptx + i];
        rng[nptx + 1 + i] = a.item_start[cbase + (tmu >> a.lsub) * nptx + i];
    }
    __syncthreads();
    const int* own = rng;
    const int* up = rng + nptx + 1;
    const int sm1 = (1 << a.lsub) - 1, step = 1 << (2 * a.lsub);
    const int qown = (tm & sm1) << a.lsub, qup = (tmu & sm1) << a.lsub;
    const int lbT = __builtin_ctz(static_cast<unsigned>(a.T));
    const int ncell = a.rows << lbT;                       // cells of one tile in the workgroup's rows
    VT* grid = reinterpret_cast<VT*>(a.grid) + static_cast<size_t>(chan) * a.N * a.N + static_cast<size_t>(r0) * a.N;
    for (int tn = 0; tn < a.ntx; ++tn) {                   // uniform across the workgroup
        const int tl = (tn - 1) & (a.ntx - 1);
        int i0[4], i1[4];
        const int pn = tn >> a.lsub, pl = tl >> a.lsub, qn = tn & sm1, ql = tl & sm1;
        i0[0] = own[pn] * step + qown + qn; i1[0] = own[pn + 1] * step;   // own tile, left, upper, upper-left
        i0[1] = own[pl] * step + qown + ql; i1[1] = own[pl + 1] * step;
        i0[2] = up[pn] * step + qup + qn;   i1[2] = up[pn + 1] * step;
        i0[3] = up[pl] * step + qup + ql;   i1[3] = up[pl + 1] * step;
        const bool any = i1[0] > i0[0] || i1[1] > i0[1] || i1[2] > i0[2] || i1[3] > i0[3];
        if (!any) {
            if (a.accumulate) continue;
            for (int pair = threadIdx.x; pair < ncell / 2; pair += blockDim.x) {
                VT* dst = grid + static_cast<size_t>((2 * pair) >> lbT) * a.N + (tn << lbT) + ((2 * pair) & (a.T - 1));
                VT z[2];
                z[0].x = 0; z[0].y = 0; z[1] = z[0];
                __builtin_memcpy(dst, z, sizeof(z));
            }
            continue;
        }
        tile_cells<R, Acc, KC, kSub>(a, grid + (tn << lbT), rb, ncell, lbT, i0, i1, step);
    }
}

}  // namespace dev

namespace grid_impl {
template <typename R, typename Acc, int W, int kTab>
hipError_t launch_grid_w(const GridArgs& a, hipStream_t s) {
    const int P = a.T + W - 1;
    const size_t tab = kTab == kTabLds ? ((static_cast<size_t>(a.Ms + 1) * W * 4 * sizeof(R)) + 15) & ~size_t(15) : 0;
    const size_t shm = tab + static_cast<size_t>(P) * P * (sizeof(typename Acc::Cell) + 1) * a.npatch;
    const void* fn = reinterpret_cast<const void*>(&dev::k_grid_items<R, Acc, W, kTab>);
    static const hipError_t attr = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxDynLds);
    if (attr != hipSuccess) return attr;
    static std::atomic<uint64_t> resident{0};
    const int nb = std::min(a.max_items, resident_blocks(fn, 64 * a.waves, shm, resident));
    if (nb < a.max_items && !a.counter_zero) {
        const hipError_t e = launch_zero_ints(a.counter, 1, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((dev::k_grid_items<R, Acc, W, kTab>), dim3(nb), dim3(64 * a.waves), shm, s, a);
    return hipGetLastError();
}
template <typename R, typename Acc>
hipError_t dispatch_grid(const GridArgs& a, hipStream_t s) {
    switch (a.W) {
#define LMG_CASE(w) \
    case w:                                                                                            \
        return a.degree < 0 ? launch_grid_w<R, Acc, w, kTabDirect>(a, s)                              \
               : a.tab_global ? launch_grid_w<R, Acc, w, kTabGlobal>(a, s)                           \
                              : launch_grid_w<R, Acc, w, kTabLds>(a, s);
        LMG_CASE(1) LMG_CASE(2) LMG_CASE(3) LMG_CASE(4) LMG_CASE(5) LMG_CASE(6) LMG_CASE(7) LMG_CASE(8)
        LMG_CASE(9) LMG_CASE(10) LMG_CASE(11) LMG_CASE(12) LMG_CASE(13) LMG_CASE(14) LMG_CASE(15) LMG_CASE(16)
#undef LMG_CASE
    }
    return hipErrorInvalidValue;
}
template <typename R, typename Acc, int KC, bool kSub>
hipError_t launch_assemble_kc(const AssembleArgs& a, unsigned nt, hipStream_t s) {
    if (a.rows_kernel) {
        const unsigned nb = static_cast<unsigned>(a.nchan) * static_cast<unsigned>(a.N / a.rows);
        const size_t shm = 2 * (static_cast<size_t>(a.ntx) + 1) * sizeof(int);
        hipLaunchKernelGGL((dev::k_assemble_rows<R, Acc, KC, kSub>), dim3(nb), dim3(kAssembleThreads), shm, s, a);
    } else {
        hipLaunchKernelGGL((dev::k_assemble<R, Acc, KC, kSub>), dim3(nt), dim3(kAssembleThreads), 0, s, a);
    }
    return hipGetLastError();
}
template <typename R, typename Acc, bool kSub>
hipError_t assemble_cells(const AssembleArgs& a, unsigned nt, hipStream_t s) {
    const int cells = a.rows * a.T;                         // of one tile per workgroup
    if (cells >= 4 * kAssembleThreads) return launch_assemble_kc<R, Acc, 4, kSub>(a, nt, s);
    if (cells >= 2 * kAssembleThreads) return launch_assemble_kc<R, Acc, 2, kSub>(a, nt, s);
    return launch_assemble_kc<R, Acc, 1, kSub>(a, nt, s);
}
template <typename R, typename Acc>
hipError_t assemble(const AssembleArgs& a, unsigned nt, hipStream_t s) {
    if constexpr (sizeof(typename Acc::Cell) == 16)         // the modes whose tiles are gridded by quadrants
        if (a.sub) return assemble_cells<R, Acc, true>(a, nt, s);
    return assemble_cells<R, Acc, false>(a, nt, s);
}
}  // namespace grid_impl
}  // namespace lmg

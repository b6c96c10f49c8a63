// Launch interfaces between the C-ABI host code and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "lmg_internal.h"

namespace lmg {

// The plan's streaming passes over the visibilities: blocks of kPlanThreads
// threads, each handling a run of at most plan_block_vis() consecutive
// visibilities of one channel.
constexpr int kPlanThreads = 1024;
constexpr int kPlanBlockVis = 65536;
// A block per compute unit while blocks hold at least 1,024 visibilities (2,048 where a block's tile histogram may
// have 16,384 entries, which it zeroes and writes), at most kPlanBlockVis: the passes take a block's time as long as
// the blocks fit the chip at once.
inline int plan_block_vis(int N, int64_t nvis) {
    const int64_t least = N >= 4096 ? 2048 : 1024;
    const int64_t v = (std::max(least, (nvis + 255) / 256) + 1023) / 1024 * 1024;
    return static_cast<int>(std::min<int64_t>(v, kPlanBlockVis));
}
// Plans of at most this many visibilities scatter directly (k_plan_scatter): the scattered stores cost less than the two
// passes that order them while the arrays stay in L2 (whole plans, two more passes / directly, W = 7: 200,000 visibilities
// on 1024^2 78 and 72 us, 1.0M 92 and 86, 2.0M 109 and 115; on 4096^2 1.0M 134 and 122, in FP64 145 and 132, 2.0M 165 and
// 172; one density on 1024^2 1.0M 91 and 89, 2.0M 116 and 133; 1.0M in 24 channels of 512^2 107 and 100).
constexpr int64_t kDirectPlanVis = 1 << 20;
// Plans of one channel and at most this many visibilities take one launch up to the scatter (k_plan_small): up to there
// one workgroup is no slower than the general passes' four launches (2,000 visibilities 43 us, general 50; 8,000 52 and
// 52; 16,000 74 and 57; the whole plan with its item sort).
constexpr int64_t kSmallPlanVis = 1 << 12;
// Longest run of one footprint cell handled by one lane (a "piece").
constexpr int kPiece = 32;
// Elements of padding after the entry-order arrays the item kernels read in runs.
constexpr int kRunPad = 4;
// Largest work item (visibilities); bounded by the 16-bit in-item offsets.
constexpr int kMaxCap = 16384;

struct PlanGeom {
    int N;        // grid size
    int W;        // support
    int T;        // tile edge (cells)
    int ntx;      // tiles per axis, N / T
    int ntiles;   // ntx * ntx, per channel
    int lb, lbx;  // log2 of T and of ntx (both powers of two)
    int lsub;     // 1: work items are quadrants of tiles, 0: whole tiles
    int nchan;    // channels, each with its own grid; global tile = channel * ntiles + tile
    double ref;   // offset of the reference tap from the first tap
};

// How the kernels get the tap weights: from the coefficient table staged in
// LDS, evaluated directly per visibility (the table's FP64 expansion), or
// from a coefficient table read through the caches (too large for LDS).
constexpr int kTabLds = 0, kTabDirect = 1, kTabGlobal = 2;

// Ms: table intervals (staged in LDS unless tab_global); degree: interpolation
// degree. A direct table has Ms = -1 (nothing staged) and degree = -1, and coef
// holds its FP64 expansion (the weights are computed per visibility).
// T, ntx: edge of a work item's tile (a quadrant of the plan's tile with lsub = 1) and such tiles per axis.
struct GridArgs {
    int N, W, T, ntx, Ms, degree;
    int lsub;              // work items: n_items << (2 lsub)
    int tab_global;        // 1: read the coefficient table from device memory, not LDS
    const int* n_items;    // device: number of work items (written by the plan)
    int max_items;         // most work items the plan can have (sizes the launch), quadrants counted
    int npatch, waves;     // LDS patches per workgroup; waves per workgroup, a multiple of it up to kMaxGridWaves
    int deal;              // 1: the pieces of npatch consecutive turns are dealt to them one by one (plain FP32)
    int Ft, kb;            // packed offsets: bits of the in-interval fraction t and of the interval k
    const int4* items;     // (tile, first position, count, pieces)
    const int2* pieces;    // (first entry, length | cell << 16)
    const void* off;       // packed offsets (uint2 or ulonglong2), entry order
    const void* coef;      // coefficient table, float or double; FP64 expansion for a direct table
    const void* vis;       // complex, entry order, weights applied
    void* patches;         // patches of (T + W - 1)^2 cells, one per work item
    int by_entry;          // 1: an item's patch is numbered by its first entry (and an empty item has none), 0: by the item
    int transpose;         // 1: patches are written transposed (a grid stored with rows along u)
    int* counter;          // work-item counter
    int counter_zero;      // 1: an earlier launch zeroed it; 0: the launcher does, where it is read at all
};

// Threads of an assemble workgroup (512 / 1024 threads: band 37 -> 47 / 72 us, batched 0.84 -> 1.19 /
// 2.19 ms).
constexpr int kAssembleThreads = 256;

struct AssembleArgs {
    int N, W, T, ntx, nchan;
    int lsub;                     // item_start counts items of tiles of 2^lsub T cells, each 4^lsub patches
    int tr0, tc0, trows, tcols;   // window of tiles written (rows tr0.., columns tc0.., wrapping)
    int rows;                     // tile rows per workgroup (set by the launcher)
    int rows_kernel;              // 1: whole grids by runs of rows (k_assemble_rows; set by the launcher)
    int transpose;                // 1: patches and grid are transposed (grid rows along u, tiles' rows along u)
    int accumulate;               // 1: add to the grid's values; 0: overwrite every cell of the window
    const int* item_start;   // per plan tile, ntiles + 1
    const int4* sub;         // the work items, where patches are numbered by their first entries; else nullptr
    const void* patches;
    void* grid;
};

struct DegridArgs {
    int N, W, T, ntx, Ms, degree;
    int lsub;              // work items: n_items << (2 lsub)
    int tab_global;        // 1: read the coefficient table from device memory, not LDS
    const int* n_items;
    int max_items;
    int Ft, kb;            // packed offsets: bits of the in-interval fraction t and of the interval k
    const int4* items;
    const int2* pieces;
    const void* off;
    const void* coef;
    const void* grid;      // nchan grids of N x N
    int transpose;         // 1: the grid is stored transposed (rows along u)
    void* vis_out;         // entry order
    int* counter;          // work-item counter
    int counter_zero;      // 1: an earlier launch zeroed it; 0: the launcher does, where it is read at all
    int one_group;         // 1: one workgroup per compute unit
};

struct FftArgs {
    int N;
    int sign;
    int nrows;             // source rows transformed
    const void* src;
    int src_pitch;         // elements between source rows
    int in_count, in_pos;  // loaded values and their first FFT position
    void* dst;
    int dst_pitch;         // elements between destination rows
    // The intermediate of two passes, written transposed by the first and read by rows by the second, may be blocked
    // (see k_fft_pass): columns src_col / dst_col on of rows of src_pitch / dst_pitch elements, multiples of two.
    int src_blocked, src_col, dst_blocked, dst_col;
    int straight;          // 1: a source row's outputs go to one destination row; 0: transposed
    int out_count, out_pos;
    const void* twiddle;   // N complex values: the stages' twiddles, in the order the stages read them
    const void* h_in;      // per input position, or nullptr
    const void* h_out;     // per output position, or nullptr
    const void* h_row;     // per source row (index row + row_off), or nullptr
    int row_off;
    int* zero;             // an int to zero (the work-item counter of the kernel that follows), or nullptr
};

// What a plan's first launch copies from pinned host memory: up to five arrays (16-byte aligned on both sides, sizes
// multiples of four).
struct PlanSetup {
    static constexpr int kCopies = 5;
    const void* src[kCopies];
    void* dst[kCopies];
    int bytes[kCopies];
};
// The plan blocks: a batch's table, or (nullptr) runs of block_vis of nvis visibilities.
struct PlanBlocks {
    const int4* table;
    int block_vis, nvis;
};
hipError_t launch_plan_count(const double* uv, const PlanBlocks& blocks, int nb, const PlanGeom& g, int* blockhist,
                             const PlanSetup& setup, hipStream_t s);
// One launch for the passes up to the scatter (which is direct): one channel of at most kSmallPlanVis visibilities.
bool small_plan(const PlanGeom& g, int64_t nvis);
hipError_t launch_plan_small(bool f64, const double* uv, const PlanGeom& g, int nvis, int* tile_start, int* item_start,
                             int4* items, int* flags, int cap, int* host_flags, double dlo, int ms, int kb, int* perm0,
                             void* off0, const PlanSetup& setup, hipStream_t s);
hipError_t launch_plan_colscan(const PlanGeom& g, int* blockhist, const int* chan_blocks, int nb, int* tile_count,
                               hipStream_t s);
// host_flags (or nullptr): pinned host copy of flags[0 .. 7].
hipError_t launch_plan_scan(const PlanGeom& g, const int* tile_count, int* tile_start, int* item_start, int4* items,
                            int* flags, int cap, int* host_flags, hipStream_t s);
// By caller index: index[k] = tile-order position, offs[k] = packed offsets, packed for a table of ms intervals (1 for
// a direct table), kb = bits of ms. With `direct`, by tile-order position: index[p] = caller index, offs[p].
hipError_t launch_plan_scatter(bool f64, bool direct, const double* uv, const PlanBlocks& blocks, int nb, const PlanGeom& g,
                               const int* tile_start, const int* blockhist, double dlo, int ms, int kb, int* index,
                               void* offs, hipStream_t s);
// off0[inv0[k]] = offk[k] for the valid visibilities (flags[2] of them).
hipError_t launch_plan_place(bool f64, const int* inv0, const void* offk, const int* flags, int64_t nvis, void* off0,
                             hipStream_t s);
// sub: the work items (items itself, with piece counts, or four quadrants of each).
hipError_t launch_plan_sort(bool f64, const PlanGeom& g, const int4* items, int4* sub, int max_items, const int* flags, int nvis,
                            int lb, const void* off0, const int* perm0, void* off, int* map, int2* pieces,
                            hipStream_t s);
hipError_t launch_plan_compose(const int* inv0, const int* pos2, int64_t nvis, int* inv, hipStream_t s);
// Bytes of one visibility's packed offsets (both axes).
size_t packed_offset_bytes(bool f64);
// Position of the cell bits in a packed offset word for tile edge 2^lb.
int packed_cell_shift(bool f64, int lb);
hipError_t launch_permute_in(bool f64, const void* vis, const float* w, const int* inv, int64_t nvis, void* vs,
                             int* zero, hipStream_t s);
hipError_t launch_zero_ints(int* p, int n, hipStream_t s);
hipError_t launch_permute_out(bool f64, const void* vs, const int* inv, int64_t nvis, void* out, hipStream_t s);
hipError_t launch_grid(lmg_precision prec, const GridArgs& a, hipStream_t s);
hipError_t launch_assemble(lmg_precision prec, const AssembleArgs& a, hipStream_t s);
hipError_t launch_degrid(lmg_precision prec, const DegridArgs& a, hipStream_t s);
// The library's own device copy of the N host twiddles (FFT stage order) on the current device, for a transform outside
// of a plan. Every call enqueues the copy before its passes; calls on several streams write the same bytes.
hipError_t fft2_twiddles(bool f64, int N, const void* host, void** out, hipStream_t s);
hipError_t launch_fft_pass(bool f64, const FftArgs& a, hipStream_t s);
hipError_t set_kernel_attributes();
// Read (and, if set, clear) the device-wide flag the plans raise on non-finite coordinates, on the
// current device. Synchronous.
hipError_t take_data_error(int* flag);
// LDS bytes of the gridding kernel with `npatch` patches (the degridding
// kernel needs no more than one patch).
size_t grid_lds_bytes(lmg_precision prec, int W, int T, int Ms, int npatch);
constexpr int kMaxGridWaves = 8;
constexpr size_t kMaxLds = 160 * 1024;
// Dynamic LDS the item kernels may request: they also hold a few bytes of
// static LDS (the current work item), and both must fit the 160 KB.
constexpr size_t kMaxDynLds = kMaxLds - 256;

}  // namespace lmg

// C ABI: plans, gridding, degridding, dirty images and prediction.
//
// Host-side argument checking, workspace layout and kernel sequencing. Every
// device buffer is caller-owned; the library never allocates device memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include "kernels.h"
#include "lmg_internal.h"
#include "trace.h"

using namespace lmg;

struct lmg_plan {
    const lmg_table* table = nullptr;
    lmg_precision prec = LMG_F32;
    PlanGeom g{};
    int64_t nvis = 0;
    // Counts the plan kernels leave in flags[]; read back asynchronously into
    // host_flags and parsed on the first host query (ensure_flags).
    mutable int64_t n_valid = 0;
    mutable int n_items = 0;
    mutable int n_busy = 0;
    mutable bool flags_read = false;
    mutable std::mutex flags_mu;
    int* host_flags = nullptr;     // pinned slot of 8 ints
    hipEvent_t ready = nullptr;    // recorded after the plan's last kernel and the readback
    int max_items = 0;
    int cap = 0;
    int M = 0;                  // retained image size 2 x0 N
    int npatch = 1;             // LDS patches per gridding workgroup
    int waves = 0;              // waves per gridding workgroup
    bool by_entry = false;      // patches numbered by their items' first entries, not by item
    int nchan = 1;              // channels (grids), each with its own run of visibilities
    int nblocks = 0;            // plan blocks (runs of <= plan_block_vis() visibilities of one channel)
    mutable bool bad_data = false;
    // Occupied band of the grid (storage rows / columns [lo, hi)) and the
    // window of tiles that covers it (first tile, number of tiles).
    mutable int band_r0 = 0, band_r1 = 0, band_c0 = 0, band_c1 = 0;
    mutable int win_r0 = 0, win_rn = 0, win_c0 = 0, win_cn = 0;
    int* flags = nullptr;
    int* tile_count = nullptr;
    int* tile_start = nullptr;
    int* item_start = nullptr;
    int* blockhist = nullptr;      // per plan block and tile: counts, then offsets
    int4* blocks = nullptr;        // per plan block: (channel, first visibility, count, 0)
    int* chan_blocks = nullptr;    // per channel, its first plan block; nchan + 1 entries
    int4* items = nullptr;         // per tile: runs of at most cap visibilities
    int4* sub = nullptr;           // work items: items, or four quadrants of each
    int* inv0 = nullptr;           // caller index -> tile-order position
    void* off0 = nullptr;          // packed offsets, by tile-order position
    void* off = nullptr;           // packed offsets, by entry (piece order within items)
    int* pos2 = nullptr;           // tile-order position -> entry (-1: dropped)
    int* inv = nullptr;            // caller index -> entry (-1: dropped)
    int2* pieces = nullptr;
    int lb = 0;                    // log2 of the tile edge
    int ms_enc = 1;                // packed offsets: table intervals they are packed for (1: direct table)
    int kb = 1;                    // packed offsets: bits of the interval index (bits of ms_enc)
    int Ft = 0;                    // packed offsets: bits of the in-interval fraction
    void* coef = nullptr;
    void* twiddle = nullptr;
    void* hpix = nullptr;
    ~lmg_plan();
};

namespace {

thread_local char g_last_error[256] = "";

lmg_status hip_failed(hipError_t e, const char* what, int line) {
    std::snprintf(g_last_error, sizeof(g_last_error), "%s (capi.cpp:%d): %s", what, line, hipGetErrorString(e));
    return LMG_EHIP;
}

#define LMG_HIP(call)                                                  \
    do {                                                               \
        const hipError_t lmg_e_ = (call);                              \
        if (lmg_e_ != hipSuccess) return hip_failed(lmg_e_, #call, __LINE__); \
    } while (0)

size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

bool is_pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }

int env_int(const char* name, int fallback) {
    const char* v = std::getenv(name);
    if (!v || !*v) return fallback;
    const int x = std::atoi(v);
    return x > 0 ? x : fallback;
}

// Smallest tile edge the plan accepts for support W: a power of two >= W,
// and at least 8. The assemble kernel adds a tile's patch to its right and
// lower neighbours only, so a footprint (W cells) must not reach two tiles
// away (Eq. 6: S_k has W cells).
int min_tile(int W) {
    int T = 8;
    while (T < W) T *= 2;
    return T;
}

int choose_tile(int N, int W) {
    int T = env_int("LMG_TILE", 32);
    if (!is_pow2(T) || T < 8) T = 32;
    T = std::max(T, min_tile(W));
    T = std::min(T, 128);
    while (T > N) T /= 2;
    while (N / T > 128) T *= 2;    // keeps the plan's LDS histogram at <= 16384 tiles
    return T;
}

// Largest tile <= T of which the table and four patches fit a compute unit's LDS, so that several workgroups share
// it (and the patches of a sparse plan stay small enough for the allocation-free call's fixed scratch); where the
// tile cannot shrink (at most 128 x 128 tiles), fewer.
int fit_tile(int T, int N, lmg_precision prec, int W, int Ms) {
    while (T / 2 >= min_tile(W) && grid_lds_bytes(prec, W, T, Ms, 4) > kMaxDynLds && N / (T / 2) <= 128) T /= 2;
    return T;
}
// LDS patches of a gridding workgroup, among which it divides each sum: two where two workgroups of two patches share a
// compute unit (tiles of 32 cells), else one (64-cell tiles: 4.2M visibilities on 8192^2 in FP32 154 us with one, 207
// with two). With one patch the flushes of a workgroup's waves wait for each other: four waves on one / two patches,
// W = 7 kernel times, 16.8M visibilities FP32 206 / 187 us, compensated 293 / 274, FP64 474 / 450; 3.0M of one density
// on 2048^2 FP32 114 / 84, compensated 176 / 122, FP64 188 / 147. (256 sparse channels, compensated, are the exception:
// W = 5 438 with one patch and three waves, 507 with two and four.) A function of the grid, mode, support, table and
// tile: the number of patches fixes the order of the sums, which a batch and a single channel share.
//
// Wide plain FP32 and FP64 sums take more, as many more flushes reach a cell: from W = 9 on four in FP32 where two
// workgroups of four fit (1.0M visibilities on 2048^2, W = 14: two 8.8e-8 against FP64, four 6.6e-8), three on 64-cell
// tiles (1.0M on 8192^2, W = 12: one 1.05e-7, three 7.2e-8; with six waves also the faster, 283 and 230 us); in FP64 two
// where only one workgroup of two fits (W = 15 and 16). Four also at W = 5 and 6 on grids of up to 128^2, whose few tiles
// hold an array's whole centre (4,500 crowded visibilities with a strong source, relative RMS against FP64 at W = 6: two
// 5.71e-8, four 4.84e-8; 13.7 and 15.1 us at W = 5, 15.1 and 17.7 at W = 6 with 2,162 of tracks).
int fit_patches(int N, int T, int lsub, lmg_precision prec, int W, int Ms) {
    auto groups = [&](int s) { return static_cast<int>(kMaxLds / (grid_lds_bytes(prec, W, T, Ms, s) + 256)); };
    const int two = groups(2) >= 2 ? 2 : 1;
    if (prec == LMG_F32 && N <= 128 && (W == 5 || W == 6) && groups(4) >= 2) return 4;
    if (prec == LMG_F32 && W >= 9) return groups(4) >= 2 ? 4 : T > 32 && groups(3) >= 1 ? 3 : two;
    if (prec == LMG_F64 && T <= 32 && lsub == 0 && groups(2) >= 1) return 2;
    return two;
}
// Work items to be expected of a plan: a quarter of the tiles, as an image's data occupy, and one for every cap visibilities.
int64_t expected_items(int T, int N, int nchan, int64_t nvis, int cap) {
    const int64_t tiles = static_cast<int64_t>(N / T) * (N / T) * nchan;
    return std::min((tiles + 3) / 4, nvis) + nvis / cap;
}
// Waves per gridding workgroup, a multiple of its patches: four, as an item has about four turns (16.8M visibilities:
// 4.1) and the waves beyond an item's turns only wait (4.2M, W = 10, compensated: 234 us with four, 344 with six).
// A launch of few items, which does not fill the chip, so that an item's latency is what counts, gets eight, two to each
// SIMD (six leave two SIMDs with twice the work of the others): in FP32 with four / six / eight, tracks of 202K on 1024^2
// 45 / 38 / 37 us at W = 7, of 300K on 2048^2 at W = 6 38 / 41 / 33, of 1.0M on 2048^2 51 / 62 / 48, at W = 5 38 / 32 /
// 30; but data of one density, whose items have few turns, 300K on 1024^2 at W = 7 26 / 39 / 31. More items than five to
// a compute unit do better with four where the flush of W^2 cells takes longer than the sums before it (1.0M in 24
// channels of 512^2, W = 6 53 / 67 / 66 us; W = 5 41 / 38 / 37; FP64, W = 8 300 / 238 / 235). The estimate takes a
// quarter of the tiles as occupied, as an image's data are. On grids of up to four tiles an edge that quarter's items are
// alike and all take their time at once: from two to a compute unit on (in FP64 from W = 8 four) they do better with four
// waves (eight / four, 500,000 visibilities in 128 channels of 128^2, W = 6 compensated 52 / 42 us, W = 8 FP64 189 / 243;
// 1.0M in 256, W = 7 FP32 86 / 55, compensated 98 / 75, FP64 127 / 98). Plain FP32 at W = 8, where registers hold a
// compute unit to eight waves, works on four items at a time with two waves each rather than on two (15.8M in 256
// channels of 1024^2 662 us, with four waves 834; 4.0M 390 and 507; 4.0M of one density on 4096^2 178 and 207; 4.2M of
// tracks 131 and 126).
// (env LMG_GRID_WAVES overrides, 1 .. kMaxGridWaves, to the next multiple of the patches)
int fit_waves(int T, int N, int nchan, int64_t nvis, int cap, lmg_precision prec, int W, int npatch) {
    const int forced = env_int("LMG_GRID_WAVES", 0);
    if (forced >= 1 && forced <= kMaxGridWaves)
        return std::min((forced + npatch - 1) / npatch, kMaxGridWaves / npatch) * npatch;
    if (npatch == 3) return 6;
    const int64_t even = prec == LMG_F64 && W >= 8 ? 1024 : 512;
    const int64_t few = N / T <= 4 && (prec == LMG_F64 || W >= 6) ? even : prec != LMG_F64 && W >= 6 ? 1280 : 2048;
    if (nvis <= (int64_t{1} << 20) && expected_items(T, N, nchan, nvis, cap) <= few) return 8;
    return prec == LMG_F32 && W == 8 && npatch == 2 && nvis > (int64_t{1} << 20) ? 2 : 4;
}

int choose_cap() { return std::min(env_int("LMG_CAP", 8192), kMaxCap); }

constexpr int kMaxChannels = 65536;

size_t real_size(lmg_precision p) { return p == LMG_F64 ? 8 : 4; }
size_t cplx_size(lmg_precision p) { return 2 * real_size(p); }
size_t patch_cell_size(lmg_precision p) { return p == LMG_F32 ? 8 : 16; }

// Gridding work items are the quadrants of 64-cell tiles (1 = log2 2) on 8192^2 grids, where 128 x 128 tiles cannot be
// smaller, in the modes with 16-byte patch cells: a 64-cell patch leaves a compute unit one workgroup (gridding 16.8M
// visibilities, compensated, W = 7: 694 us whole, 578 as quadrants; 4.2M, FP64, W = 6: 283 and 229; FP32's 8-byte cells
// leave three, 154 and 156).
int tile_lsub(int N, int T, lmg_precision prec) { return N == 8192 && T == 64 && prec != LMG_F32 ? 1 : 0; }

struct Layout {
    size_t flags, tile_count, tile_start, item_start, blockhist, blocks, chan_blocks, items, sub, inv0, off0, off, pos2, inv, pieces, coef,
        twiddle, hpix, total;
    int max_items;
    int max_blocks;
};

// Most plan blocks for nvis visibilities over nchan channels.
int64_t max_plan_blocks(int N, int64_t nvis, int nchan) {
    const int v = plan_block_vis(N, nvis);
    return (nvis + v - 1) / v + nchan;
}

// Tile arrays are sized for the smallest tile any plan may pick (N / T <= 128,
// T >= 8), so the size query need not know the table.
Layout plan_layout(int N, int64_t nvis, lmg_precision prec, int cap, int nchan = 1) {
    Layout L{};
    const int64_t ntiles = std::min<int64_t>(16384, static_cast<int64_t>(N / 8) * (N / 8));
    const int64_t tot = ntiles * nchan;
    L.max_items = static_cast<int>(std::min<int64_t>(tot, nvis) + (nvis + cap - 1) / cap + 1);
    L.max_blocks = static_cast<int>(max_plan_blocks(N, nvis, nchan));
    size_t o = 0;
    auto take = [&o](size_t bytes) { const size_t at = o; o = align_up(o + bytes); return at; };
    L.flags = take(16 * sizeof(int));
    L.tile_count = take((tot + 1) * sizeof(int));
    L.tile_start = take((tot + 2) * sizeof(int));
    L.item_start = take((tot + 1) * sizeof(int));
    L.blockhist = take(static_cast<size_t>(L.max_blocks) * (ntiles + 1) * sizeof(int));
    L.blocks = take(static_cast<size_t>(L.max_blocks) * sizeof(int4));
    L.chan_blocks = take((static_cast<size_t>(nchan) + 1) * sizeof(int));
    L.items = take(static_cast<size_t>(L.max_items) * sizeof(int4));
    L.sub = take(tile_lsub(N, 64, prec) ? static_cast<size_t>(L.max_items) * 4 * sizeof(int4) : 0);
    L.inv0 = take(static_cast<size_t>(nvis) * sizeof(int));
    L.off0 = take(static_cast<size_t>(nvis) * packed_offset_bytes(prec == LMG_F64));
    L.off = take(static_cast<size_t>(nvis + kRunPad) * packed_offset_bytes(prec == LMG_F64));
    L.pos2 = take(static_cast<size_t>(nvis) * sizeof(int));
    L.inv = take(static_cast<size_t>(nvis) * sizeof(int));
    L.pieces = take(static_cast<size_t>(nvis) * sizeof(int2));
    L.coef = take(kMaxLdsTableBytes * 2);
    L.twiddle = take(static_cast<size_t>(N) * cplx_size(prec));
    L.hpix = take(static_cast<size_t>(N) * real_size(prec));
    L.total = o;
    return L;
}

// Scratch of a planned call: [work counters][grid][fft tmp][visibilities in plan order][patches].
struct Scratch {
    size_t counters, grid, tmp, vs, patches, total;
};
constexpr int kCounters = 2;    // work-item counters of the gridding and degridding kernels

// Most work items of a plan: its tiles (only those with visibilities have items), plus one per cap visibilities.
int64_t most_items(int N, int T, int nchan, int64_t nvis, int cap) {
    return std::min<int64_t>(static_cast<int64_t>(N / T) * (N / T) * nchan, nvis) + (nvis + cap - 1) / cap + 1;
}

// Quadrants' patches are numbered by their first entries where a plan has fewer visibilities than quadrants (most are
// empty then): a sparse plan's scratch is no larger than with whole tiles, and the allocation-free call takes it.
bool patches_by_entry(int lsub, int64_t items, int64_t nvis) { return lsub > 0 && nvis < (items << (2 * lsub)); }

Scratch scratch_layout(int N, int W, int T, int lsub, int M, int64_t items, int64_t nvis, lmg_precision prec, int op) {
    const size_t P = static_cast<size_t>((T >> lsub) + W - 1);
    const int64_t npatches = patches_by_entry(lsub, items, nvis) ? nvis : items << (2 * lsub);
    const size_t patches = align_up(static_cast<size_t>(npatches) * P * P * patch_cell_size(prec));
    const size_t grid = align_up(static_cast<size_t>(N) * N * cplx_size(prec));
    const size_t tmp = align_up(static_cast<size_t>((M + 3) / 4 * 4) * N * cplx_size(prec));     // blocks of four rows
    const size_t vs = align_up(static_cast<size_t>(nvis + kRunPad) * cplx_size(prec));
    Scratch s{};
    size_t o = align_up(kCounters * sizeof(int));
    s.counters = 0;
    const bool image = op == LMG_OP_DIRTY || op == LMG_OP_PREDICT;
    if (image) { s.grid = o; o += grid; s.tmp = o; o += tmp; }
    s.vs = o;
    o += vs;
    if (op == LMG_OP_GRID || op == LMG_OP_DIRTY) { s.patches = o; o += patches; }
    s.total = o;
    return s;
}

size_t scratch_for(int N, int W, int T, int M, int items, int64_t nvis, lmg_precision prec, int op) {
    size_t b = 0;
    for (int lsub = 0; lsub <= tile_lsub(N, T, prec); ++lsub)
        b = std::max(b, scratch_layout(N, W, T, lsub, M, items, nvis, prec, op).total);
    return b;
}

bool valid_grid(int N, int W, double x0, int* M) {
    if (!is_pow2(N) || N < 64 || N > 8192 || N < 2 * W) return false;
    const double m = 2.0 * x0 * N;
    if (std::fabs(m - std::round(m)) > 1e-9) return false;
    *M = static_cast<int>(std::lround(m));
    return *M >= 2 && *M <= N && (*M % 2) == 0;
}

// Host caches (never freed) of FFT twiddles and correction vectors.
std::mutex g_cache_mu;
std::map<int, std::vector<double>>& twiddle_cache() {
    static std::map<int, std::vector<double>> c;
    return c;
}
// N complex values (cos, -sin): the twiddles of the transform's stages after the first, in the order the stages read
// them. A stage of radix RAD after Ns = 8, 64, ... combined points holds e^{-2 pi i r k / (RAD Ns)} at Ns - 8 +
// (r - 1) Ns + k for r = 1 .. RAD - 1, k < Ns.
const std::vector<double>& twiddles_f64(int N) {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto& c = twiddle_cache();
    auto it = c.find(N);
    if (it != c.end()) return it->second;
    std::vector<double> tw(2 * static_cast<size_t>(N), 0.0);
    for (int Ns = 8; Ns < N; Ns *= 8) {
        const int rad = std::min(8, N / Ns);
        for (int r = 1; r < rad; ++r)
            for (int k = 0; k < Ns; ++k) {
                const double a = 2.0 * 3.14159265358979323846 * (static_cast<double>(r * k) / (rad * Ns));
                const size_t at = static_cast<size_t>(Ns) - 8 + static_cast<size_t>(r - 1) * Ns + k;
                tw[2 * at] = std::cos(a);
                tw[2 * at + 1] = -std::sin(a);
            }
    }
    return c.emplace(N, std::move(tw)).first->second;
}
std::map<int, std::vector<float>>& twiddle32_cache() {
    static std::map<int, std::vector<float>> c;
    return c;
}
const std::vector<float>& twiddles_f32(int N) {
    const std::vector<double>& d = twiddles_f64(N);
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto& c = twiddle32_cache();
    auto it = c.find(N);
    if (it != c.end()) return it->second;
    std::vector<float> f(d.begin(), d.end());
    return c.emplace(N, std::move(f)).first->second;
}

std::once_flag g_attr_once;
hipError_t g_attr_err = hipSuccess;
hipError_t ensure_attributes() {
    std::call_once(g_attr_once, [] { g_attr_err = set_kernel_attributes(); });
    return g_attr_err;
}

lmg_status upload(void* dst, const void* src, size_t bytes, hipStream_t s) {
    if (bytes == 0) return LMG_OK;
    LMG_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s));
    return LMG_OK;
}

// The coefficients a plan uploads: the interval polynomials of a table in
// the plan's precision, or for a direct table the FP64 expansion (pq).
const void* coef_host(const lmg_table* t, lmg_precision prec) {
    if (t->direct) return t->pq.data();
    return prec == LMG_F64 ? static_cast<const void*>(t->coef64.data()) : static_cast<const void*>(t->coef32.data());
}
size_t coef_bytes(const lmg_table* t, lmg_precision prec) {
    if (t->direct) return t->pq.size() * sizeof(double);
    return prec == LMG_F64 ? t->coef64.size() * sizeof(double) : t->coef32.size() * sizeof(float);
}
// A table too large for LDS: the kernels read its coefficients from the attached device copy.
bool table_global(const lmg_table* t, lmg_precision prec) {
    return !t->direct && coef_bytes(t, prec) > kMaxLdsTableBytes;
}
// Coefficient bytes a plan copies into its workspace (none for a table read from device memory).
size_t plan_coef_bytes(const lmg_table* t, lmg_precision prec) {
    return table_global(t, prec) ? 0 : coef_bytes(t, prec);
}
// Table intervals the kernels stage in LDS (-1: none, for a direct table or one read from device
// memory), the intervals of the table, and the kernels' table mode (-1: direct).
int staged_ms(const lmg_table* t, lmg_precision prec) { return (t->direct || table_global(t, prec)) ? -1 : t->Ms; }
int table_ms(const lmg_table* t) { return t->direct ? -1 : t->Ms; }
int kernel_degree(const lmg_table* t) { return t->direct ? -1 : t->degree; }

// The plan constants of (table, N, precision) in pinned host memory, built on
// first use: copies from it are asynchronous. nullptr if pinned memory is
// unavailable (the caller then uploads from pageable memory).
const lmg_table::Pinned* pinned_constants(const lmg_table* t, int N, lmg_precision prec, const std::vector<double>& h) {
    std::lock_guard<std::mutex> lk(t->cache_mu);
    const auto key = std::make_pair(N, static_cast<int>(prec));
    auto it = t->pinned.find(key);
    if (it != t->pinned.end()) return it->second.host ? &it->second : nullptr;
    lmg_table::Pinned pc;
    const bool f64 = prec == LMG_F64;
    pc.coef_bytes = plan_coef_bytes(t, prec);
    pc.twiddle_bytes = 2 * static_cast<size_t>(N) * (f64 ? 8 : 4);
    pc.hpix_bytes = static_cast<size_t>(N) * (f64 ? 8 : 4);
    pc.coef = 0;
    pc.twiddle = align_up(pc.coef_bytes);
    pc.hpix = pc.twiddle + align_up(pc.twiddle_bytes);
    const size_t total = pc.hpix + align_up(pc.hpix_bytes);
    if (hipHostMalloc(&pc.host, total, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        pc.host = nullptr;
        t->pinned.emplace(key, pc);
        return nullptr;
    }
    char* b = static_cast<char*>(pc.host);
    if (pc.coef_bytes) std::memcpy(b + pc.coef, coef_host(t, prec), pc.coef_bytes);
    if (f64) {
        std::memcpy(b + pc.twiddle, twiddles_f64(N).data(), pc.twiddle_bytes);
        std::memcpy(b + pc.hpix, h.data(), pc.hpix_bytes);
    } else {
        std::memcpy(b + pc.twiddle, twiddles_f32(N).data(), pc.twiddle_bytes);
        float* hf = reinterpret_cast<float*>(b + pc.hpix);
        for (int i = 0; i < N; ++i) hf[i] = static_cast<float>(h[i]);
    }
    return &t->pinned.emplace(key, pc).first->second;
}

// Pinned staging for the per-plan block tables, one per host thread. Plan
// creation does not wait for its uploads; the next creation on the thread
// waits for the previous one's (an event) before reusing the buffer.
struct Staging {
    hipEvent_t done = nullptr;
    bool pending = false;
};
thread_local Staging g_staging;

void* block_staging(size_t bytes) {
    thread_local void* buf = nullptr;
    thread_local size_t cap = 0;
    if (g_staging.pending) {
        (void)hipEventSynchronize(g_staging.done);
        g_staging.pending = false;
    }
    if (bytes > cap) {
        if (buf) (void)hipHostFree(buf);
        buf = nullptr;
        cap = 0;
        if (hipHostMalloc(&buf, bytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            buf = nullptr;
            return nullptr;
        }
        cap = bytes;
    }
    return buf;
}

// Pinned slots of 8 ints for the plans' flag readback, from chunks that live
// until the process ends.
std::mutex g_slot_mu;
std::vector<int*> g_free_slots;

int* take_flag_slot() {
    std::lock_guard<std::mutex> lk(g_slot_mu);
    if (g_free_slots.empty()) {
        constexpr int kSlots = 1024;
        void* chunk = nullptr;
        if (hipHostMalloc(&chunk, kSlots * 16 * sizeof(int), hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        for (int i = 0; i < kSlots; ++i) g_free_slots.push_back(static_cast<int*>(chunk) + 16 * i);
    }
    int* s = g_free_slots.back();
    g_free_slots.pop_back();
    return s;
}

void give_flag_slot(int* s) {
    std::lock_guard<std::mutex> lk(g_slot_mu);
    g_free_slots.push_back(s);
}

}  // namespace

lmg_plan::~lmg_plan() {
    if (ready) {
        (void)hipEventSynchronize(ready);          // the counts have reached the pinned slot
        (void)hipEventDestroy(ready);
        if (host_flags) give_flag_slot(host_flags);    // (a plan that failed before its event keeps its slot)
    }
}

namespace {

// Grid rows (or columns) touched by footprints of tiles lo..hi (inclusive),
// as [r0, r1); the whole range if the footprints wrap around the grid edge.
void axis_band(int lo, int hi, int T, int W, int N, int ntx, int* r0, int* r1, int* w0, int* wn) {
    if (hi < lo) {                    // nothing gridded
        *r0 = *r1 = 0;
        *w0 = 0;
        *wn = 0;
        return;
    }
    const int end = (hi + 1) * T + W - 1;
    if (end > N) {
        *r0 = 0;
        *r1 = N;
        *w0 = 0;
        *wn = ntx;
        return;
    }
    *r0 = lo * T;
    *r1 = end;
    *w0 = lo;
    *wn = std::min(hi + (W > 1 ? 1 : 0), ntx - 1) - lo + 1;
}

void set_band(const lmg_plan* p, int rmin, int rmax, int cmin, int cmax) {
    if (p->n_busy == 0) { rmax = -1; cmax = -1; rmin = 0; cmin = 0; }
    axis_band(rmin, rmax, p->g.T, p->g.W, p->g.N, p->g.ntx, &p->band_r0, &p->band_r1, &p->win_r0, &p->win_rn);
    axis_band(cmin, cmax, p->g.T, p->g.W, p->g.N, p->g.ntx, &p->band_c0, &p->band_c1, &p->win_c0, &p->win_cn);
}

// Parse the plan's counts, waiting for its readback the first time.
lmg_status ensure_flags(const lmg_plan* p) {
    std::lock_guard<std::mutex> lk(p->flags_mu);
    if (p->flags_read) return LMG_OK;
    LMG_HIP(hipEventSynchronize(p->ready));
    const int* f = p->host_flags;
    p->bad_data = f[0] != 0;
    p->n_items = f[1];
    p->n_valid = f[2];
    p->n_busy = f[3];
    set_band(p, f[4], f[5], f[6], f[7]);
    p->flags_read = true;
    if (p->n_items > p->max_items) return LMG_EHIP;     // cannot happen; guards the scratch bound
    return LMG_OK;
}

// A planned call on another stream than the plan's creation waits (on the
// device) for the plan's kernels.
lmg_status wait_plan(const lmg_plan* p, hipStream_t s) {
    LMG_HIP(hipStreamWaitEvent(s, p->ready, 0));
    return LMG_OK;
}

// Plain FP32 grids of up to 1024^2, whose items have few turns: an item without a turn of full pieces deals its pieces one
// by one to the turns, and with them the patches, of a group. Taken 64 neighbours at a time, the flushes of a few dense
// cells fall to one patch and round against a large sum (relative RMS against FP64 with a strong source at the centre, 64
// at a time / dealt: W = 6, 12,000 visibilities on 256^2 6.9e-8 / 5.7e-8; W = 7, 60,000 on 512^2 8.0e-8 / 5.9e-8). A turn
// then takes as long as the longest of more pieces: 201,600 on 1024^2, W = 7 36.7 / 37.9 us, 3.0M in 48 channels 125 /
// 127; on larger grids, whose items have enough turns without it, 8.4M on 4096^2, W = 7 112 / 116.
bool deal_pieces(const lmg_plan* p) { return p->prec == LMG_F32 && p->g.N <= 1024; }

// Gridding of visibilities already in entry order (weights applied) through
// the plan: overwrite the grid (every cell of the window written), or add to
// it (accumulate: only tiles that receive patches are read and written).
lmg_status run_grid_entries(const lmg_plan* p, const void* vs, void* grid, void* patches, int* counters, hipStream_t s,
                            bool counter_zero, bool band_only, bool accumulate) {
    const lmg_table* t = p->table;
    if (wait_plan(p, s) != LMG_OK) return LMG_EHIP;
    GridArgs a{};
    a.N = p->g.N; a.W = p->g.W; a.T = p->g.T >> p->g.lsub; a.ntx = p->g.ntx << p->g.lsub; a.lsub = p->g.lsub;
    a.Ms = table_ms(t); a.degree = kernel_degree(t);
    a.tab_global = table_global(t, p->prec) ? 1 : 0;
    a.n_items = p->flags + 1; a.max_items = p->max_items << (2 * p->g.lsub); a.npatch = p->npatch; a.waves = p->waves;
    a.deal = deal_pieces(p) ? 1 : 0; a.Ft = p->Ft; a.kb = p->kb;
    a.items = p->sub; a.pieces = p->pieces; a.off = p->off; a.coef = p->coef;
    a.vis = vs; a.patches = patches; a.by_entry = p->by_entry ? 1 : 0;
    a.counter = counters; a.counter_zero = counter_zero ? 1 : 0;
    a.transpose = band_only ? 1 : 0;
    {
        TraceScope ts("grid_items", s);
        LMG_HIP(launch_grid(p->prec, a, s));
    }
    AssembleArgs b{};
    b.transpose = a.transpose;
    b.N = p->g.N; b.W = p->g.W; b.T = a.T; b.ntx = a.ntx; b.lsub = p->g.lsub; b.nchan = p->nchan;
    b.accumulate = accumulate ? 1 : 0;
    if (band_only) {                  // an internal grid, stored transposed: only the occupied window is ever read
        const lmg_status st = ensure_flags(p);     // the grid kernels are already queued
        if (st != LMG_OK) return st;
        const int l = p->g.lsub;                    // the window is in plan tiles; rows along u
        b.tr0 = p->win_c0 << l; b.trows = p->win_cn << l; b.tc0 = p->win_r0 << l; b.tcols = p->win_rn << l;
    } else {
        b.tr0 = 0; b.trows = a.ntx; b.tc0 = 0; b.tcols = a.ntx;
    }
    b.item_start = p->item_start; b.sub = p->by_entry ? p->sub : nullptr; b.patches = patches; b.grid = grid;
    TraceScope ts("assemble", s);
    LMG_HIP(launch_assemble(p->prec, b, s));
    return LMG_OK;
}

// Caller order -> entry order (vs = w V), then gridding.
lmg_status run_grid(const lmg_plan* p, const void* vis, const float* w, void* grid, void* vs, void* patches,
                    int* counters, hipStream_t s, bool band_only, bool accumulate) {
    if (wait_plan(p, s) != LMG_OK) return LMG_EHIP;
    {
        TraceScope ts("permute_in", s);
        LMG_HIP(launch_permute_in(p->prec == LMG_F64, vis, w, p->inv, p->nvis, vs, counters, s));
    }
    return run_grid_entries(p, vs, grid, patches, counters, s, p->nvis > 0, band_only, accumulate);
}

// Degridding by the quadrants of a plan that grids by quadrants: dense FP64 data at W = 6 .. 8. The fill of four small
// patches costs more than that of a large one, so sparse data go by whole tiles: 8192^2 in FP64, whole / quadrants, 1.0M
// visibilities at W = 7 70 / 119 us, 3.0M 113 / 132 (but W = 8 240 / 226), 6.0M 234 / 219, 16.8M 348 / 317 (W = 5
// 267 / 250, but 6.0M 187 / 215; W = 3 151 / 199, 9 488 / 547). FP32 grids' patches are half as large (16.8M 195 / 223).
// Each visibility's sum is its own, so the results are the same bits.
bool degrid_by_quadrants(const lmg_plan* p) {
    return p->prec == LMG_F64 && p->g.W >= 6 && p->g.W <= 8 && p->nvis >= (p->g.W == 8 ? 3000000 : 6000000);
}

// One degridding workgroup per compute unit, where registers and LDS would hold two (of 1,024 threads, whose reads of W^2
// cells per visibility compete): launches of one to seven items to a compute unit, which then balance over twice the
// rounds (one / two, 500,000 visibilities in 128 channels of 128^2, FP32 W = 10 52 / 77 us, FP64 W = 7 44 / 57; 1.0M in
// 24 channels of 512^2, FP32 W = 8 69 / 89, W = 14 96 / 130). With more items the second workgroup fills its patch while
// the first sums (3.0M in 48 channels of 1024^2, W = 10 174 / 153), with fewer or sparse ones nothing competes. Below
// W = 8 FP32 gains on few of these and loses on others (1.0M on 1024^2 of one density, W = 7 0.79 of two's time; 4.0M on
// 2048^2 1.04); FP64 above W = 8 has registers for one only.
bool one_degrid_group(const lmg_plan* p) {
    const int64_t items = expected_items(p->g.T, p->g.N, p->nchan, p->nvis, p->cap);
    const bool two = p->prec == LMG_F64 ? p->g.W <= 8 : p->g.W >= 8;
    return two && items > 340 && items <= (p->g.W >= 14 ? 4096 : 1700) && p->nvis >= 128 * items;
}

// Degridding into entry order.
lmg_status run_degrid_entries(const lmg_plan* p, const void* grid, bool transposed, void* vs, int* counters,
                              bool counter_zero, hipStream_t s) {
    const lmg_table* t = p->table;
    if (wait_plan(p, s) != LMG_OK) return LMG_EHIP;
    DegridArgs a{};
    const int lsub = degrid_by_quadrants(p) ? p->g.lsub : 0;
    a.N = p->g.N; a.W = p->g.W; a.T = p->g.T >> lsub; a.ntx = p->g.ntx << lsub; a.lsub = lsub;
    a.Ms = table_ms(t); a.degree = kernel_degree(t);
    a.tab_global = table_global(t, p->prec) ? 1 : 0;
    a.n_items = p->flags + 1; a.max_items = p->max_items << (2 * lsub); a.Ft = p->Ft; a.kb = p->kb;
    a.items = lsub ? p->sub : p->items; a.pieces = p->pieces; a.off = p->off; a.coef = p->coef;
    a.grid = grid; a.transpose = transposed ? 1 : 0; a.vis_out = vs; a.counter = counters + 1;
    a.counter_zero = counter_zero ? 1 : 0; a.one_group = one_degrid_group(p) ? 1 : 0;
    TraceScope ts("degrid_items", s);
    LMG_HIP(launch_degrid(p->prec, a, s));
    return LMG_OK;
}

// Degridding, then entry order -> caller order.
lmg_status run_degrid(const lmg_plan* p, const void* grid, bool transposed, void* vis_out, void* vs, int* counters,
                      bool counter_zero, hipStream_t s) {
    const lmg_status st = run_degrid_entries(p, grid, transposed, vs, counters, counter_zero, s);
    if (st != LMG_OK) return st;
    TraceScope ts("permute_out", s);
    LMG_HIP(launch_permute_out(p->prec == LMG_F64, vs, p->inv, p->nvis, vis_out, s));
    return LMG_OK;
}

FftArgs fft_args(int N, int sign, const void* tw) {
    FftArgs f{};
    f.N = N;
    f.sign = sign;
    f.twiddle = tw;
    return f;
}

Scratch plan_scratch(const lmg_plan* p, int op) {
    // Sized for the most work items this plan can have, so that no query waits for its counts.
    return scratch_layout(p->g.N, p->g.W, p->g.T, p->g.lsub, p->M, most_items(p->g.N, p->g.T, p->nchan, p->nvis, p->cap),
                          p->nvis, p->prec, op);
}

bool scratch_ok(const lmg_plan* p, int op, void* scratch, size_t bytes) {
    const size_t need = plan_scratch(p, op).total;
    return need == 0 || (scratch && bytes >= need);
}

// Plan for nchan channels; channel c owns visibilities [offsets[c], offsets[c + 1]) and grid c.
// tile = 0 picks the default tile edge; otherwise a power of two in [8, min(128, N)] with N / tile <= 128.
// With `counts` false the host never learns the plan's counts, and images are made over the whole grid: no call through
// the plan waits for the device (its end does, for the plan's kernels).
lmg_status create_plan(const lmg_table* table, int N, lmg_precision prec, int nchan, const int64_t* offsets,
                       const double* uv, int tile, void* workspace, size_t ws_bytes, void* stream, lmg_plan** out,
                       bool counts = true) {
    int M = 0;
    if (!table || !out || !offsets || prec < LMG_F32 || prec > LMG_F64 || nchan < 1 || nchan > kMaxChannels ||
        !valid_grid(N, table->W, table->x0, &M))
        return LMG_EINVAL;
    if (offsets[0] != 0) return LMG_EINVAL;
    for (int c = 0; c < nchan; ++c)
        if (offsets[c + 1] < offsets[c]) return LMG_EINVAL;
    const int64_t nvis = offsets[nchan];
    if (nvis < 0 || nvis > INT32_MAX || (nvis > 0 && !uv)) return LMG_EINVAL;
    if (tile != 0 && (!is_pow2(tile) || tile < 8 || tile < table->W || tile > 128 || tile > N || N / tile > 128))
        return LMG_EINVAL;
    const size_t tab_bytes = plan_coef_bytes(table, prec);
    if (table_global(table, prec) && !table->dev_coef[prec == LMG_F64 ? 1 : 0]) return LMG_ENOTSUP;
    const int T = tile ? tile : fit_tile(choose_tile(N, table->W), N, prec, table->W, staged_ms(table, prec));
    if (T < table->W || N / T > 128) return LMG_ENOTSUP;      // cannot happen for N >= 2W, N <= 8192
    const int cap = choose_cap();
    const int Ms = staged_ms(table, prec);
    // A function of the grid, the tile and the mode: the order of the sums depends on it, and a batch's channel has the
    // bits of that channel alone. (Item numbers past 31 bits take more channels than a device holds grids of.)
    const int64_t items = most_items(N, T, nchan, nvis, cap);
    const int lsub = items <= INT32_MAX / 4 ? tile_lsub(N, T, prec) : 0;
    const int Tq = T >> lsub;
    const int npatch = fit_patches(N, Tq, lsub, prec, table->W, Ms);
    const int waves = fit_waves(Tq, N, nchan, nvis, cap, prec, table->W, npatch);
    if (grid_lds_bytes(prec, table->W, Tq, Ms, npatch) > kMaxDynLds) return LMG_ENOTSUP;
    const Layout L = plan_layout(N, nvis, prec, cap, nchan);
    if (!workspace || ws_bytes < L.total) return LMG_EWORKSPACE;
    if (ensure_attributes() != hipSuccess) return LMG_EHIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    std::unique_ptr<lmg_plan> p(new (std::nothrow) lmg_plan);
    if (!p) return LMG_EINVAL;
    char* base = static_cast<char*>(workspace);
    p->table = table;
    p->prec = prec;
    p->g.N = N; p->g.W = table->W; p->g.T = T; p->g.ntx = N / T; p->g.ntiles = (N / T) * (N / T);
    p->g.nchan = nchan;
    p->g.lsub = lsub;
    p->by_entry = patches_by_entry(lsub, items, nvis);
    p->g.ref = tap_reference(table->W);
    p->waves = waves;
    p->npatch = npatch;
    p->nchan = nchan;
    p->nvis = nvis;
    p->cap = cap;
    p->max_items = L.max_items;
    p->M = M;
    p->flags = reinterpret_cast<int*>(base + L.flags);
    p->tile_count = reinterpret_cast<int*>(base + L.tile_count);
    p->tile_start = reinterpret_cast<int*>(base + L.tile_start);
    p->item_start = reinterpret_cast<int*>(base + L.item_start);
    p->blockhist = reinterpret_cast<int*>(base + L.blockhist);
    p->blocks = reinterpret_cast<int4*>(base + L.blocks);
    p->chan_blocks = reinterpret_cast<int*>(base + L.chan_blocks);
    p->items = reinterpret_cast<int4*>(base + L.items);
    p->sub = p->g.lsub ? reinterpret_cast<int4*>(base + L.sub) : p->items;
    p->inv0 = reinterpret_cast<int*>(base + L.inv0);
    p->off0 = base + L.off0;
    p->off = base + L.off;
    p->pos2 = reinterpret_cast<int*>(base + L.pos2);
    p->inv = reinterpret_cast<int*>(base + L.inv);
    p->pieces = reinterpret_cast<int2*>(base + L.pieces);
    p->lb = 0;
    while ((1 << p->lb) < T) ++p->lb;
    p->g.lb = p->lb;
    while ((1 << p->g.lbx) < p->g.ntx) ++p->g.lbx;
    // Packed offsets hold the interval index in kb <= 24 bits over Ft >= 2 fraction bits.
    p->ms_enc = table->direct ? 1 : table->Ms;
    p->kb = 0;
    while (p->kb < 31 && (p->ms_enc >> p->kb) != 0) ++p->kb;
    p->Ft = packed_cell_shift(prec == LMG_F64, p->lb) - p->kb;
    if (p->kb > 24 || p->Ft < 2) return LMG_ENOTSUP;
    p->coef = table_global(table, prec) ? table->dev_coef[prec == LMG_F64 ? 1 : 0] : base + L.coef;
    p->twiddle = base + L.twiddle;
    p->hpix = base + L.hpix;

    // Plan blocks: runs of at most plan_block_vis() visibilities of one channel. A batch's tables are staged in
    // pinned memory; a single channel's blocks follow from their size.
    const int block_vis = plan_block_vis(N, nvis);
    std::vector<int4> blocks;
    std::vector<int> chan_blocks;
    if (nchan == 1) {
        p->nblocks = static_cast<int>((nvis + block_vis - 1) / block_vis);
    } else {
        chan_blocks.resize(static_cast<size_t>(nchan) + 1);
        for (int c = 0; c < nchan; ++c) {
            chan_blocks[c] = static_cast<int>(blocks.size());
            for (int64_t a = offsets[c]; a < offsets[c + 1]; a += block_vis)
                blocks.push_back(make_int4(c, static_cast<int>(a),
                                           static_cast<int>(std::min<int64_t>(block_vis, offsets[c + 1] - a)), 0));
        }
        chan_blocks[nchan] = static_cast<int>(blocks.size());
        p->nblocks = static_cast<int>(blocks.size());
    }
    if (p->nblocks > L.max_blocks) return LMG_EINVAL;       // cannot happen; guards the workspace bound

    // Constant tables: kernel coefficients, FFT twiddles, correction h(x_p); block tables.
    std::vector<double> h(N);
    if (lmg_correction(table, N, h.data()) != LMG_OK) return LMG_EINVAL;
    PlanSetup su{};
    PlanBlocks bl{};
    bl.block_vis = block_vis;
    bl.nvis = static_cast<int>(nvis);
    int copies = 0;
    auto from_pinned = [&](void* dst, const void* src, size_t bytes) {
        su.dst[copies] = dst;
        su.src[copies] = src;
        su.bytes[copies++] = static_cast<int>(bytes);
    };
    std::vector<float> hf;
    if (const lmg_table::Pinned* pc = pinned_constants(table, N, prec, h)) {
        const char* b = static_cast<const char*>(pc->host);
        from_pinned(p->coef, b + pc->coef, pc->coef_bytes);
        from_pinned(p->twiddle, b + pc->twiddle, pc->twiddle_bytes);
        from_pinned(p->hpix, b + pc->hpix, pc->hpix_bytes);
    } else if (prec == LMG_F64) {
        if (upload(p->coef, coef_host(table, prec), tab_bytes, s) != LMG_OK) return LMG_EHIP;
        if (upload(p->twiddle, twiddles_f64(N).data(), 2 * sizeof(double) * N, s) != LMG_OK) return LMG_EHIP;
        if (upload(p->hpix, h.data(), sizeof(double) * N, s) != LMG_OK) return LMG_EHIP;
    } else {
        hf.assign(h.begin(), h.end());
        if (upload(p->coef, coef_host(table, prec), tab_bytes, s) != LMG_OK) return LMG_EHIP;
        if (upload(p->twiddle, twiddles_f32(N).data(), 2 * sizeof(float) * N, s) != LMG_OK) return LMG_EHIP;
        if (upload(p->hpix, hf.data(), sizeof(float) * N, s) != LMG_OK) return LMG_EHIP;
    }
    bool staged = false;
    if (nchan > 1) {
        const size_t bb = blocks.size() * sizeof(int4), cb = chan_blocks.size() * sizeof(int);
        if (char* st = static_cast<char*>(block_staging(align_up(bb) + cb))) {
            if (bb) std::memcpy(st, blocks.data(), bb);
            std::memcpy(st + align_up(bb), chan_blocks.data(), cb);
            from_pinned(p->blocks, st, bb);
            from_pinned(p->chan_blocks, st + align_up(bb), cb);
            bl.table = reinterpret_cast<const int4*>(st);      // the first launch reads it where it lies
            staged = true;
        } else {
            if (upload(p->blocks, blocks.data(), bb, s) != LMG_OK) return LMG_EHIP;
            if (upload(p->chan_blocks, chan_blocks.data(), cb, s) != LMG_OK) return LMG_EHIP;
            bl.table = p->blocks;
        }
    }
    const bool direct = nvis <= kDirectPlanVis;
    if (counts) p->host_flags = take_flag_slot();
    if (small_plan(p->g, nvis)) {
        TraceScope ts("plan_small", s);
        LMG_HIP(launch_plan_small(prec == LMG_F64, uv, p->g, static_cast<int>(nvis), p->tile_start, p->item_start, p->items,
                                  p->flags, cap, p->host_flags, delta_low(table->W), p->ms_enc, p->kb, p->inv0, p->off0,
                                  su, s));
    } else {
        {
            TraceScope ts("plan_count", s);
            LMG_HIP(launch_plan_count(uv, bl, p->nblocks, p->g, p->blockhist, su, s));
        }
        if (staged) {
            if (!g_staging.done) LMG_HIP(hipEventCreateWithFlags(&g_staging.done, hipEventDisableTiming));
            LMG_HIP(hipEventRecord(g_staging.done, s));
            g_staging.pending = true;
            bl.table = p->blocks;
        }
        {
            TraceScope ts("plan_colscan", s);
            LMG_HIP(launch_plan_colscan(p->g, p->blockhist, p->chan_blocks, p->nblocks, p->tile_count, s));
        }
        {
            TraceScope ts("plan_scan", s);
            LMG_HIP(launch_plan_scan(p->g, p->tile_count, p->tile_start, p->item_start, p->items, p->flags, cap,
                                     p->host_flags, s));
        }
        TraceScope ts("plan_scatter", s);
        // packed offsets by caller index go to `off` for now (the item sort overwrites it)
        LMG_HIP(launch_plan_scatter(prec == LMG_F64, direct, uv, bl, p->nblocks, p->g, p->tile_start, p->blockhist,
                                    delta_low(table->W), p->ms_enc, p->kb, p->inv0, direct ? p->off0 : p->off, s));
    }
    if (!direct) {
        TraceScope ts("plan_place", s);
        LMG_HIP(launch_plan_place(prec == LMG_F64, p->inv0, p->off, p->flags, nvis, p->off0, s));
    }
    {
        TraceScope ts("plan_sort_items", s);
        LMG_HIP(launch_plan_sort(prec == LMG_F64, p->g, p->items, p->sub, L.max_items, p->flags, static_cast<int>(nvis),
                                 p->lb, p->off0, direct ? p->inv0 : nullptr, p->off, direct ? p->inv : p->pos2,
                                 p->pieces, s));
    }
    if (!direct) {
        TraceScope ts("plan_compose", s);
        LMG_HIP(launch_plan_compose(p->inv0, p->pos2, nvis, p->inv, s));
    }
    if (!counts) {
        p->n_busy = nvis > 0 ? 1 : 0;
        set_band(p.get(), 0, p->g.ntx - 1, 0, p->g.ntx - 1);
        p->flags_read = true;
    }
    // The counts came back with the scan; the host reads them when it first needs them.
    hipEvent_t ready = nullptr;
    LMG_HIP(hipEventCreateWithFlags(&ready, hipEventDisableTiming));
    const hipError_t rec = hipEventRecord(ready, s);
    if (rec != hipSuccess) (void)hipEventDestroy(ready);
    LMG_HIP(rec);
    p->ready = ready;
    if (counts && !p->host_flags) {                        // no pinned memory: read back synchronously
        static thread_local int fallback[8];
        LMG_HIP(hipMemcpyAsync(fallback, p->flags, sizeof(fallback), hipMemcpyDeviceToHost, s));
        LMG_HIP(hipStreamSynchronize(s));
        p->host_flags = fallback;
        const lmg_status st = ensure_flags(p.get());
        p->host_flags = nullptr;
        if (st != LMG_OK) return st;
    }
    *out = p.release();
    return LMG_OK;
}

}  // namespace

extern "C" {

lmg_status lmg_plan_workspace_size(int N, int W, int64_t nvis, lmg_precision prec, size_t* bytes) {
    if (!bytes || !is_pow2(N) || N < 64 || N > 8192 || W < 1 || W > kMaxW || nvis < 0 || nvis > INT32_MAX ||
        prec < LMG_F32 || prec > LMG_F64)
        return LMG_EINVAL;
    *bytes = plan_layout(N, nvis, prec, choose_cap()).total;
    return LMG_OK;
}

lmg_status lmg_plan_create(const lmg_table* table, int N, lmg_precision prec, int64_t nvis, const double* uv,
                           void* workspace, size_t ws_bytes, void* stream, lmg_plan** out) {
    const int64_t offsets[2] = {0, nvis};
    return create_plan(table, N, prec, 1, offsets, uv, 0, workspace, ws_bytes, stream, out);
}

lmg_status lmg_batch_workspace_size(int N, int W, int nchan, int64_t nvis, lmg_precision prec, size_t* bytes) {
    if (!bytes || !is_pow2(N) || N < 64 || N > 8192 || W < 1 || W > kMaxW || nchan < 1 || nchan > kMaxChannels ||
        nvis < 0 || nvis > INT32_MAX || prec < LMG_F32 || prec > LMG_F64)
        return LMG_EINVAL;
    *bytes = plan_layout(N, nvis, prec, choose_cap(), nchan).total;
    return LMG_OK;
}

lmg_status lmg_batch_plan_create(const lmg_table* table, int N, lmg_precision prec, int nchan, const int64_t* offsets,
                                 const double* uv, int tile, void* workspace, size_t ws_bytes, void* stream,
                                 lmg_plan** out) {
    return create_plan(table, N, prec, nchan, offsets, uv, tile, workspace, ws_bytes, stream, out);
}

lmg_status lmg_batch_info(const lmg_plan* p, int* nchan, int* tile, int* waves) {
    if (!p) return LMG_EINVAL;
    if (nchan) *nchan = p->nchan;
    if (tile) *tile = p->g.T;
    if (waves) *waves = p->waves;
    return LMG_OK;
}

const char* lmg_last_error(void) { return g_last_error; }

lmg_status lmg_sync_status(void* stream) {
    LMG_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
    int flag = 0;
    LMG_HIP(take_data_error(&flag));
    return flag ? LMG_EDATA : LMG_OK;
}

lmg_status lmg_plan_check(const lmg_plan* p) {
    if (!p) return LMG_EINVAL;
    const lmg_status st = ensure_flags(p);
    if (st != LMG_OK) return st;
    return p->bad_data ? LMG_EDATA : LMG_OK;
}

lmg_status lmg_plan_info(const lmg_plan* p, int* tile, int* n_items, int* n_busy, int64_t* n_valid) {
    if (!p) return LMG_EINVAL;
    const lmg_status st = ensure_flags(p);
    if (st != LMG_OK) return st;
    if (tile) *tile = p->g.T;
    if (n_items) *n_items = p->n_items;
    if (n_busy) *n_busy = p->n_busy;
    if (n_valid) *n_valid = p->n_valid;
    return LMG_OK;
}

void lmg_plan_destroy(lmg_plan* p) { delete p; }

lmg_status lmg_plan_scratch_size(const lmg_plan* p, int op, size_t* bytes) {
    if (!p || !bytes || op < LMG_OP_GRID || op > LMG_OP_PREDICT) return LMG_EINVAL;
    *bytes = plan_scratch(p, op).total;
    return LMG_OK;
}

lmg_status lmg_grid_planned(const lmg_plan* p, const void* vis, const float* w, void* grid, int accumulate,
                            void* scratch, size_t scratch_bytes, void* stream) {
    if (!p || !grid || (p->nvis > 0 && !vis) || (accumulate != 0 && accumulate != 1)) return LMG_EINVAL;
    if (!scratch_ok(p, LMG_OP_GRID, scratch, scratch_bytes)) return LMG_EWORKSPACE;
    const Scratch L = plan_scratch(p, LMG_OP_GRID);
    char* sc = static_cast<char*>(scratch);
    return run_grid(p, vis, w, grid, sc + L.vs, sc + L.patches, reinterpret_cast<int*>(sc + L.counters),
                    static_cast<hipStream_t>(stream), false, accumulate != 0);
}

lmg_status lmg_degrid_planned(const lmg_plan* p, const void* grid, void* vis_out, void* scratch, size_t scratch_bytes,
                              void* stream) {
    if (!p || !grid || (p->nvis > 0 && !vis_out)) return LMG_EINVAL;
    if (!scratch_ok(p, LMG_OP_DEGRID, scratch, scratch_bytes)) return LMG_EWORKSPACE;
    const Scratch L = plan_scratch(p, LMG_OP_DEGRID);
    char* sc = static_cast<char*>(scratch);
    return run_degrid(p, grid, false, vis_out, sc + L.vs, reinterpret_cast<int*>(sc + L.counters), false,
                      static_cast<hipStream_t>(stream));
}

lmg_status lmg_plan_order_length(const lmg_plan* p, int64_t* n) {
    if (!p || !n) return LMG_EINVAL;
    *n = p->nvis + kRunPad;
    return LMG_OK;
}

lmg_status lmg_to_plan_order(const lmg_plan* p, const void* vis, const float* w, void* vis_plan, void* stream) {
    if (!p || (p->nvis > 0 && (!vis || !vis_plan))) return LMG_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (wait_plan(p, s) != LMG_OK) return LMG_EHIP;
    TraceScope ts("permute_in", s);
    LMG_HIP(launch_permute_in(p->prec == LMG_F64, vis, w, p->inv, p->nvis, vis_plan, nullptr, s));
    return LMG_OK;
}

lmg_status lmg_from_plan_order(const lmg_plan* p, const void* vis_plan, void* vis, void* stream) {
    if (!p || (p->nvis > 0 && (!vis || !vis_plan))) return LMG_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (wait_plan(p, s) != LMG_OK) return LMG_EHIP;
    TraceScope ts("permute_out", s);
    LMG_HIP(launch_permute_out(p->prec == LMG_F64, vis_plan, p->inv, p->nvis, vis, s));
    return LMG_OK;
}

lmg_status lmg_grid_planned_ordered(const lmg_plan* p, const void* vis_plan, void* grid, int accumulate, void* scratch,
                                    size_t scratch_bytes, void* stream) {
    if (!p || !grid || (p->nvis > 0 && !vis_plan) || (accumulate != 0 && accumulate != 1)) return LMG_EINVAL;
    if (!scratch_ok(p, LMG_OP_GRID, scratch, scratch_bytes)) return LMG_EWORKSPACE;
    const Scratch L = plan_scratch(p, LMG_OP_GRID);
    char* sc = static_cast<char*>(scratch);
    return run_grid_entries(p, vis_plan, grid, sc + L.patches, reinterpret_cast<int*>(sc + L.counters),
                            static_cast<hipStream_t>(stream), false, false, accumulate != 0);
}

lmg_status lmg_degrid_planned_ordered(const lmg_plan* p, const void* grid, void* vis_plan_out, void* scratch,
                                      size_t scratch_bytes, void* stream) {
    if (!p || !grid || (p->nvis > 0 && !vis_plan_out)) return LMG_EINVAL;
    if (!scratch_ok(p, LMG_OP_DEGRID, scratch, scratch_bytes)) return LMG_EWORKSPACE;
    const Scratch L = plan_scratch(p, LMG_OP_DEGRID);
    char* sc = static_cast<char*>(scratch);
    return run_degrid_entries(p, grid, false, vis_plan_out, reinterpret_cast<int*>(sc + L.counters), false,
                              static_cast<hipStream_t>(stream));
}

lmg_status lmg_make_dirty_image_planned(const lmg_plan* p, const void* vis, const float* w, void* image, void* scratch,
                                        size_t scratch_bytes, void* stream) {
    if (!p || !image || (p->nvis > 0 && !vis)) return LMG_EINVAL;
    if (p->nchan != 1) return LMG_ENOTSUP;
    if (!scratch_ok(p, LMG_OP_DIRTY, scratch, scratch_bytes)) return LMG_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int N = p->g.N, M = p->M;
    const Scratch L = plan_scratch(p, LMG_OP_DIRTY);
    char* sc = static_cast<char*>(scratch);
    void* grid = sc + L.grid;
    void* tmp = sc + L.tmp;
    lmg_status st = run_grid(p, vis, w, grid, sc + L.vs, sc + L.patches, reinterpret_cast<int*>(sc + L.counters), s,
                             true, false);
    if (st != LMG_OK) return st;
    const bool f64 = p->prec == LMG_F64;
    const size_t cs = cplx_size(p->prec);
    const int r0 = p->band_r0, nr = p->band_r1 - p->band_r0, c0 = p->band_c0, nc = p->band_c1 - p->band_c0;
    if (nr == 0) {                     // nothing gridded: the image is zero
        LMG_HIP(launch_zero_ints(static_cast<int*>(image), static_cast<int>(static_cast<size_t>(M) * M * cs / 4), s));
        return LMG_OK;
    }
    // The grid is stored transposed (rows n). Rows n of the occupied band: transform over m (only the occupied rows m
    // are non-zero), keep the central M outputs, write transposed (tmp is M x N, blocked; only columns c0 .. c0 + nc
    // are written).
    FftArgs a = fft_args(N, +1, p->twiddle);
    a.nrows = nc; a.src = static_cast<char*>(grid) + (static_cast<size_t>(c0) * N + r0) * cs; a.src_pitch = N;
    a.in_count = nr; a.in_pos = r0;
    a.dst = tmp; a.dst_pitch = N; a.dst_blocked = 1; a.dst_col = c0; a.out_count = M; a.out_pos = N / 2 - M / 2;
    {
        TraceScope ts("fft_cols_inverse", s);
        LMG_HIP(launch_fft_pass(f64, a, s));
    }
    // Rows q of tmp: transform over n (zero outside the band), keep the central M outputs, apply
    // h(x_p) h(y_q), write image[q][p].
    FftArgs b = fft_args(N, +1, p->twiddle);
    b.nrows = M; b.src = tmp; b.src_pitch = N; b.src_blocked = 1; b.src_col = c0; b.in_count = nc; b.in_pos = c0;
    b.dst = image; b.dst_pitch = M; b.out_count = M; b.out_pos = N / 2 - M / 2; b.straight = 1;
    b.h_out = p->hpix; b.h_row = p->hpix; b.row_off = N / 2 - M / 2;
    TraceScope ts("fft_rows_inverse_correct_crop", s);
    LMG_HIP(launch_fft_pass(f64, b, s));
    return LMG_OK;
}

lmg_status lmg_predict_visibilities_planned(const lmg_plan* p, const void* image, void* vis_out, void* scratch,
                                            size_t scratch_bytes, void* stream) {
    if (!p || !image || (p->nvis > 0 && !vis_out)) return LMG_EINVAL;
    if (p->nchan != 1) return LMG_ENOTSUP;
    if (!scratch_ok(p, LMG_OP_PREDICT, scratch, scratch_bytes)) return LMG_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (wait_plan(p, s) != LMG_OK) return LMG_EHIP;
    {
        const lmg_status st = ensure_flags(p);     // the occupied band prunes the transforms
        if (st != LMG_OK) return st;
    }
    const int N = p->g.N, M = p->M;
    const Scratch L = plan_scratch(p, LMG_OP_PREDICT);
    char* sc = static_cast<char*>(scratch);
    void* grid = sc + L.grid;
    void* tmp = sc + L.tmp;
    int* counters = reinterpret_cast<int*>(sc + L.counters);
    const bool f64 = p->prec == LMG_F64;
    const size_t cs = cplx_size(p->prec);
    const int r0 = p->band_r0, nr = p->band_r1 - p->band_r0, c0 = p->band_c0, nc = p->band_c1 - p->band_c0;
    if (nr > 0) {
        // Rows q of the image: correct by h(x_p) h(y_q), zero-pad to N, transform over p, keep the outputs n in
        // the occupied column band, write transposed (tmp: nc rows n, M columns q).
        FftArgs a = fft_args(N, -1, p->twiddle);
        a.nrows = M; a.src = image; a.src_pitch = M; a.in_count = M; a.in_pos = N / 2 - M / 2;
        a.dst = tmp; a.dst_pitch = M; a.dst_blocked = 1; a.out_count = nc; a.out_pos = c0;
        a.h_in = p->hpix; a.h_row = p->hpix; a.row_off = N / 2 - M / 2;
        {
            TraceScope ts("fft_rows_forward_correct_pad", s);
            LMG_HIP(launch_fft_pass(f64, a, s));
        }
        // Rows n of tmp: zero-pad to N, transform over q, write the occupied band of the grid, stored transposed
        // (rows n).
        FftArgs b = fft_args(N, -1, p->twiddle);
        b.nrows = nc; b.src = tmp; b.src_pitch = M; b.src_blocked = 1; b.in_count = M; b.in_pos = N / 2 - M / 2;
        b.dst = static_cast<char*>(grid) + (static_cast<size_t>(c0) * N + r0) * cs; b.dst_pitch = N; b.straight = 1;
        b.out_count = nr; b.out_pos = r0;
        b.zero = counters + 1;
        {
            TraceScope ts("fft_cols_forward", s);
            LMG_HIP(launch_fft_pass(f64, b, s));
        }
    }
    return run_degrid(p, grid, true, vis_out, sc + L.vs, counters, nr > 0, s);
}

lmg_status lmg_workspace_size(int N, int W, double x0, int64_t nvis, lmg_precision prec, int op, size_t* bytes) {
    int M = 0;
    if (!bytes || W < 1 || W > kMaxW || nvis < 0 || nvis > INT32_MAX || prec < LMG_F32 || prec > LMG_F64 ||
        op < LMG_OP_GRID || op > LMG_OP_PREDICT || !valid_grid(N, W, x0, &M))
        return LMG_EINVAL;
    const Layout L = plan_layout(N, nvis, prec, choose_cap());
    size_t sc = 0;
    for (int T = 8; T <= 128; T *= 2)          // any tile the plan may settle on
        if (T <= N && N / T <= 128) sc = std::max(sc, scratch_for(N, W, T, M, L.max_items, nvis, prec, op));
    *bytes = L.total + sc;
    return LMG_OK;
}

}  // extern "C"

namespace {
// Largest grid on which a one-shot image call transforms the whole grid rather than wait for the band its
// visibilities occupy: that wait, in the middle of the call, drains the queue; the wait for the plan at the call's end
// finds the rest queued (dirty image and prediction, waiting against whole: 2,000 visibilities on 128^2 123 and 108 us,
// 201,600 on 512^2 203 and 194; on 1024^2 2,000 130 and 124, in FP64 136 and 131, 201,600 210 and 208, in FP64 263 and
// 265, 1.0M 259 and 255, in FP64 323 and 323; on 2048^2 2,000 174 and 180, 1.0M 298 and 310, in FP64 383 and 416).
constexpr int kWholeImageN = 1024;

template <typename F>
lmg_status one_shot(const lmg_table* t, int N, lmg_precision prec, int64_t nvis, const double* uv, void* ws,
                    size_t ws_bytes, void* stream, int op, F&& body) {
    if (!t) return LMG_EINVAL;
    size_t need = 0;
    lmg_status st = lmg_workspace_size(N, t->W, t->x0, nvis, prec, op, &need);
    if (st != LMG_OK) return st;
    if (!ws || ws_bytes < need) return LMG_EWORKSPACE;
    size_t pbytes = 0;
    lmg_plan_workspace_size(N, t->W, nvis, prec, &pbytes);
    lmg_plan* p = nullptr;
    const int64_t offsets[2] = {0, nvis};
    bool counts = false;
    if (op == LMG_OP_DIRTY || op == LMG_OP_PREDICT) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;       // a capture still meets the wait, which refuses it
        if (hipStreamIsCapturing(static_cast<hipStream_t>(stream), &cap) != hipSuccess) {
            (void)hipGetLastError();
            cap = hipStreamCaptureStatusActive;
        }
        counts = N > kWholeImageN || cap != hipStreamCaptureStatusNone;
    }
    st = create_plan(t, N, prec, 1, offsets, uv, 0, ws, pbytes, stream, &p, counts);
    if (st != LMG_OK) return st;
    st = body(p, static_cast<char*>(ws) + pbytes, ws_bytes - pbytes);
    lmg_plan_destroy(p);
    return st;
}

// Batched one-shot calls use the default tile edge for N (not shrunk to the
// table: fewer waves per workgroup instead), so that the size query is exact.
template <typename F>
lmg_status one_shot_batched(const lmg_table* t, int N, lmg_precision prec, int nchan, const int64_t* offsets,
                            const double* uv, void* ws, size_t ws_bytes, void* stream, int op, F&& body) {
    if (!t || !offsets || nchan < 1) return LMG_EINVAL;
    size_t need = 0;
    lmg_status st = lmg_workspace_size_batched(N, t->W, nchan, offsets[nchan], prec, op, &need);
    if (st != LMG_OK) return st;
    if (!ws || ws_bytes < need) return LMG_EWORKSPACE;
    size_t pbytes = 0;
    lmg_batch_workspace_size(N, t->W, nchan, offsets[nchan], prec, &pbytes);
    lmg_plan* p = nullptr;
    st = create_plan(t, N, prec, nchan, offsets, uv, choose_tile(N, t->W), ws, pbytes, stream, &p, false);
    if (st != LMG_OK) return st;
    st = body(p, static_cast<char*>(ws) + pbytes, ws_bytes - pbytes);
    lmg_plan_destroy(p);
    return st;
}
}  // namespace

extern "C" {

lmg_status lmg_grid(const lmg_table* t, int N, lmg_precision prec, int64_t nvis, const double* uv, const void* vis,
                    const float* w, void* grid, void* ws, size_t ws_bytes, void* stream) {
    return one_shot(t, N, prec, nvis, uv, ws, ws_bytes, stream, LMG_OP_GRID, [&](lmg_plan* p, void* sc, size_t sb) {
        return lmg_grid_planned(p, vis, w, grid, 1, sc, sb, stream);
    });
}

lmg_status lmg_degrid(const lmg_table* t, int N, lmg_precision prec, int64_t nvis, const double* uv, const void* grid,
                      void* vis_out, void* ws, size_t ws_bytes, void* stream) {
    return one_shot(t, N, prec, nvis, uv, ws, ws_bytes, stream, LMG_OP_DEGRID, [&](lmg_plan* p, void* sc, size_t sb) {
        return lmg_degrid_planned(p, grid, vis_out, sc, sb, stream);
    });
}

lmg_status lmg_make_dirty_image(const lmg_table* t, int N, lmg_precision prec, int64_t nvis, const double* uv,
                                const void* vis, const float* w, void* image, void* ws, size_t ws_bytes, void* stream) {
    return one_shot(t, N, prec, nvis, uv, ws, ws_bytes, stream, LMG_OP_DIRTY, [&](lmg_plan* p, void* sc, size_t sb) {
        return lmg_make_dirty_image_planned(p, vis, w, image, sc, sb, stream);
    });
}

lmg_status lmg_predict_visibilities(const lmg_table* t, int N, lmg_precision prec, int64_t nvis, const double* uv,
                                    const void* image, void* vis_out, void* ws, size_t ws_bytes, void* stream) {
    return one_shot(t, N, prec, nvis, uv, ws, ws_bytes, stream, LMG_OP_PREDICT,
                    [&](lmg_plan* p, void* sc, size_t sb) {
                        return lmg_predict_visibilities_planned(p, image, vis_out, sc, sb, stream);
                    });
}

lmg_status lmg_workspace_size_batched(int N, int W, int nchan, int64_t nvis, lmg_precision prec, int op,
                                      size_t* bytes) {
    size_t plan = 0;
    if (op != LMG_OP_GRID && op != LMG_OP_DEGRID) return LMG_EINVAL;
    lmg_status st = lmg_batch_workspace_size(N, W, nchan, nvis, prec, &plan);
    if (st != LMG_OK) return st;
    const int T = choose_tile(N, W);
    const Layout L = plan_layout(N, nvis, prec, choose_cap(), nchan);
    *bytes = plan + scratch_for(N, W, T, 0, L.max_items, nvis, prec, op);
    return LMG_OK;
}

lmg_status lmg_grid_batched(const lmg_table* t, int N, lmg_precision prec, int nchan, const int64_t* offsets,
                            const double* uv, const void* vis, const float* w, void* grids, void* ws,
                            size_t ws_bytes, void* stream) {
    return one_shot_batched(t, N, prec, nchan, offsets, uv, ws, ws_bytes, stream, LMG_OP_GRID,
                            [&](lmg_plan* p, void* sc, size_t sb) {
                                return lmg_grid_planned(p, vis, w, grids, 1, sc, sb, stream);
                            });
}

lmg_status lmg_degrid_batched(const lmg_table* t, int N, lmg_precision prec, int nchan, const int64_t* offsets,
                              const double* uv, const void* grids, void* vis_out, void* ws, size_t ws_bytes,
                              void* stream) {
    return one_shot_batched(t, N, prec, nchan, offsets, uv, ws, ws_bytes, stream, LMG_OP_DEGRID,
                            [&](lmg_plan* p, void* sc, size_t sb) {
                                return lmg_degrid_planned(p, grids, vis_out, sc, sb, stream);
                            });
}

lmg_status lmg_fft2_centred(int N, lmg_precision prec, int sign, void* data, void* scratch, void* stream) {
    if (!is_pow2(N) || N < 4 || N > 8192 || (sign != 1 && sign != -1) || !data || !scratch || prec < LMG_F32 ||
        prec > LMG_F64)
        return LMG_EINVAL;
    if (ensure_attributes() != hipSuccess) return LMG_EHIP;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool f64 = prec == LMG_F64;
    const void* host = f64 ? static_cast<const void*>(twiddles_f64(N).data()) : twiddles_f32(N).data();
    void* tw = nullptr;
    LMG_HIP(fft2_twiddles(f64, N, host, &tw, s));
    FftArgs a = fft_args(N, sign, tw);
    a.nrows = N; a.src = data; a.src_pitch = N; a.in_count = N; a.in_pos = 0;
    a.dst = scratch; a.dst_pitch = N; a.dst_blocked = 1; a.out_count = N; a.out_pos = 0;
    LMG_HIP(launch_fft_pass(f64, a, s));
    FftArgs b = a;
    b.src = scratch; b.src_blocked = 1; b.dst = data; b.dst_blocked = 0;
    LMG_HIP(launch_fft_pass(f64, b, s));
    return LMG_OK;
}

}  // extern "C"

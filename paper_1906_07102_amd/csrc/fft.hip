// Centred 2D FFT passes (Stockham radix 8, LDS-resident rows) with the correction,
// crop and zero pad fused into their loads and stores.
#include <mutex>

#include "dev_common.h"

namespace lmg {
namespace dev {

// Twiddles of the transform that a caller runs by itself (fft2_twiddles): its scratch holds the N x N intermediate and
// nothing else. N elements from element N on for each N = 4 .. 8192.
__device__ float2 g_twiddles32[2 * 8192];
__device__ double2 g_twiddles64[2 * 8192];

// ------------------------------------------------------------------ FFT
// One pass of the centred 2D transform: ROWS rows of `src` (`in_count` values
// placed from position `in_pos`, zeros elsewhere) are transformed with
// Stockham stages (radix 8, plus one of radix 4 or 2 when log2 N is not a
// multiple of 3) of sign SIGN, and the outputs at positions [out_pos, out_pos
// + out_count) are written into `dst`: transposed (dst row = output position,
// dst column = source row), or straight (kStraight: dst row = source row). A
// transform over both axes takes one transposed pass and one straight one, so
// one side of it is stored transposed: the image calls keep their internal
// grid so. A transposed store leaves in pieces of two values and is bound by
// the number of write requests (without its store a pass on 8192^2 took 110
// us instead of 169 in FP32, 181 instead of 326 in FP64); a straight one
// leaves in whole lines, from the last stage's registers. Optional real factors: h_in[s] on inputs,
// h_out[r] on outputs, h_row[row + row_off] on a whole row.
//
// Centring: positions are indices shifted by N / 2, so position s enters the
// plain transform at s - N / 2 mod N and its output q leaves as position
// q + N / 2 mod N. The core has exponent sign -1; for SIGN = +1 the real and
// imaginary parts are exchanged on the way in and out.
//
// The first stage works on the loaded values in registers (its butterfly j
// takes N / 8 j's neighbours in memory from all lanes, so the loads are
// coalesced); rows pass through LDS between stages and once more before the
// transposed store, so that a row block's values leave side by side.
//
// What bounds it: VALU issue. A pass over the 2,048 occupied rows of a 4096^2
// FP32 image took 29 us with 12.1M VALU instructions, most of them around the
// butterflies: quadrant selection of looked-up twiddles, sign products,
// checkerboard products and LDS slots. Here a stage's twiddles are read in the
// order its lanes use them (stage tables, see twiddle layout below), the sign
// and the checkerboard are index and register names, and slots are constants.
template <int N, int ROWS>
struct FftShape {
    static constexpr int kRad0 = N >= 8 ? 8 : 4;                        // radix of the first stage
    static constexpr int kThreads = (ROWS * N / 8) < 1024 ? (ROWS * N / 8 > 0 ? ROWS * N / 8 : 1) : 1024;
};

// Rows in LDS hold one pad element after every 16: the first radix-8 stage
// stores each thread's eight outputs to consecutive positions, so the lanes of
// a wave store 8 elements apart, into few LDS banks, and the pad spreads them
// (four passes of a 4096^2 image about 145 us against 153 us unpadded, before
// the later changes).
template <typename R, int N, int ROWS>
struct FftLds {
    static constexpr size_t kEl = sizeof(typename C2<R>::T);
    static constexpr bool kRowPad = N >= 16 && static_cast<size_t>(ROWS) * (N + N / 16) * kEl <= kMaxLds;
    static constexpr int kPitch = kRowPad ? N + N / 16 : N;      // elements from one row to the next
    static constexpr size_t kBytes = static_cast<size_t>(ROWS) * kPitch * kEl;
};

// LDS slot of row position s.
template <bool PAD>
__device__ __forceinline__ int row_slot(int s) { return PAD ? s + (s >> 4) : s; }
// Slot of position base + r STEP, r < 8, given pbase = row_slot(base): a step
// that is a multiple of 16 carries whole pad elements along; with STEP = 8 or
// 1 (second and first radix-8 stage) base mod 16 is below 8, or a multiple of
// 8, so the pads before base + r STEP are those of base and r / 2 or none.
template <bool PAD, int STEP>
__device__ __forceinline__ int row_slot_step(int base, int pbase, int r) {
    if constexpr (!PAD) return base + r * STEP;
    else if constexpr (STEP % 16 == 0) return pbase + r * (STEP + STEP / 16);
    else if constexpr (STEP == 8) return pbase + r * 8 + r / 2;
    else if constexpr (STEP == 1) return pbase + r;
    else return row_slot<true>(base + r * STEP);
}

template <typename VT>
__device__ __forceinline__ VT cadd(VT a, VT b) {
    VT o;
    o.x = a.x + b.x;
    o.y = a.y + b.y;
    return o;
}
template <typename VT>
__device__ __forceinline__ VT csub(VT a, VT b) {
    VT o;
    o.x = a.x - b.x;
    o.y = a.y - b.y;
    return o;
}
// a - i b and a + i b
template <typename VT>
__device__ __forceinline__ VT csub_i(VT a, VT b) {
    VT o;
    o.x = a.x + b.y;
    o.y = a.y - b.x;
    return o;
}
template <typename VT>
__device__ __forceinline__ VT cadd_i(VT a, VT b) {
    VT o;
    o.x = a.x - b.y;
    o.y = a.y + b.x;
    return o;
}

// Joins the 4-point DFTs e and o of the even and the odd inputs of 8 points: v[k] = e[k] + e^{-2 pi i k / 8} o[k]. The
// products by cos(pi / 4) go into the sums unrounded (with products of their own a 4096^2 transform in FP32 was off by
// 1.739e-7, with these by 1.729e-7).
template <typename R>
__device__ __forceinline__ void join8(const typename C2<R>::T* e, const typename C2<R>::T* o, typename C2<R>::T* v) {
    using VT = typename C2<R>::T;
    const R h = static_cast<R>(0.70710678118654752440);   // cos(pi / 4)
    VT o1, o3;
    o1.x = o[1].x + o[1].y;                               // o1 (1 - i)
    o1.y = o[1].y - o[1].x;
    o3.x = o[3].y - o[3].x;                               // o3 (-1 - i)
    o3.y = -o[3].x - o[3].y;
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1].x = fma(h, o1.x, e[1].x);
    v[1].y = fma(h, o1.y, e[1].y);
    v[5].x = fma(-h, o1.x, e[1].x);
    v[5].y = fma(-h, o1.y, e[1].y);
    v[2] = csub_i(e[2], o[2]);
    v[6] = cadd_i(e[2], o[2]);
    v[3].x = fma(h, o3.x, e[3].x);
    v[3].y = fma(h, o3.y, e[3].y);
    v[7].x = fma(-h, o3.x, e[3].x);
    v[7].y = fma(-h, o3.y, e[3].y);
}

// In-place DFT of RAD = 2, 4 or 8 points with exponent sign -1.
template <typename R, int RAD>
__device__ __forceinline__ void small_dft(typename C2<R>::T* v) {
    using VT = typename C2<R>::T;
    if constexpr (RAD == 2) {
        const VT a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (RAD == 4) {
        const VT t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]), t2 = cadd(v[1], v[3]), t3 = csub(v[1], v[3]);
        v[0] = cadd(t0, t2);
        v[1] = csub_i(t1, t3);
        v[2] = csub(t0, t2);
        v[3] = cadd_i(t1, t3);
    } else {
        static_assert(RAD == 8, "radix 2, 4 or 8");
        VT e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        small_dft<R, 4>(e);
        small_dft<R, 4>(o);
        join8<R>(e, o, v);
    }
}
// The 8-point DFT of inputs of which 2 .. 5 are zero.
template <typename R>
__device__ __forceinline__ void outer_dft8(typename C2<R>::T* v) {
    using VT = typename C2<R>::T;
    const VT e[4] = {cadd(v[0], v[6]), cadd_i(v[0], v[6]), csub(v[0], v[6]), csub_i(v[0], v[6])};
    const VT o[4] = {cadd(v[1], v[7]), cadd_i(v[1], v[7]), csub(v[1], v[7]), csub_i(v[1], v[7])};
    join8<R>(e, o, v);
}

// Barrier of the workgroup that orders LDS accesses alone: nothing else is shared, and loads in flight stay so.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One Stockham stage of radix RAD on every row of the workgroup, after stages
// that have combined Ns = 2^LNS points: butterfly j of a row reads positions
// j + r N / RAD, twists them by e^{-2 pi i r (j mod Ns) / (RAD Ns)}, and
// after a barrier stores its outputs to positions
// (j - j mod Ns) RAD + j mod Ns + r Ns. In the last stage (outputs j + r N /
// RAD) with `outer` only the outputs in the first and last quarter of the row
// are stored: the central half of the positions.
//
// Twiddle layout: the table holds, for the stages after the first in turn,
// e^{-2 pi i r k / (RAD Ns)} at [(r - 1) Ns + k], r = 1 .. RAD - 1, k < Ns; the
// stage tables of Ns = 8, 64, ... start at Ns - 8 and end before N.
//
// Up to 4096 points a stage's twiddles are loaded into registers a stage
// ahead, so that their latency is spent in the barriers and the LDS traffic
// between (four passes 4096^2 FP32 141 -> 136 us, 2048^2 FP64 71 -> 69); rows
// of 8192 points, which leave one workgroup on a compute unit, load them where
// they are used (FP32 644 us against 720, FP64 1213 against 1398).
template <typename R, int N, int ROWS, int LNS>
struct FftStage {
    static constexpr int Ns = 1 << LNS;
    static constexpr bool kNone = Ns >= N;               // past the last stage
    static constexpr int RAD = kNone ? 1 : (N / Ns >= 8 ? 8 : N / Ns);
    static constexpr int nb = N / RAD;
    static constexpr int KB = kNone ? 1 : ROWS * nb / FftShape<N, ROWS>::kThreads;   // butterflies per thread
    static constexpr int kTw = kNone ? 1 : KB * (RAD - 1);
    static constexpr bool kAhead = N <= 4096;
    using VT = typename C2<R>::T;
    // the twiddles of this thread's butterflies; each from the table (deriving the others as powers of one is
    // faster but doubles the rounding floor of an FP32 4096-point transform)
    __device__ static __forceinline__ void load(const VT* __restrict__ tw, VT* w) {
        if constexpr (!kNone) {
#pragma unroll
            for (int q = 0; q < KB; ++q) {
                const int j = (threadIdx.x + q * FftShape<N, ROWS>::kThreads) % nb;
                const VT* t = tw + (Ns - 8) + (j & (Ns - 1));
#pragma unroll
                for (int r = 1; r < RAD; ++r) w[q * (RAD - 1) + r - 1] = t[(r - 1) * Ns];
            }
        }
    }
};

// The stages from Ns = 2^LNS points on. `w`: this stage's twiddles if kAhead. With kStraight the last stage's outputs
// are handed to `store` (row of the workgroup, output, value) from registers instead of staying in LDS.
template <typename R, int N, int ROWS, int LNS, bool kStraight, typename Store>
__device__ __forceinline__ void stockham_stages(typename C2<R>::T* buf, const typename C2<R>::T* __restrict__ tw,
                                                typename C2<R>::T* w, bool outer, const Store& store) {
    using VT = typename C2<R>::T;
    using L = FftLds<R, N, ROWS>;
    using St = FftStage<R, N, ROWS, LNS>;
    if constexpr (!St::kNone) {
        using Next = FftStage<R, N, ROWS, LNS + 3>;
        constexpr int NT = FftShape<N, ROWS>::kThreads;
        constexpr bool PR = L::kRowPad;
        constexpr int Ns = St::Ns, RAD = St::RAD, nb = St::nb, KB = St::KB;
        static_assert(KB >= 1 && KB * NT == ROWS * nb, "butterflies per thread");
        if constexpr (!St::kAhead) St::load(tw, w);
        VT hold[RAD * KB];
#pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int b = threadIdx.x + q * NT;
            const int rr = b / nb, j = b % nb;
            const VT* row = buf + rr * L::kPitch;
            const int pj = row_slot<PR>(j);
            VT* v = hold + RAD * q;
            v[0] = row[pj];
#pragma unroll
            for (int r = 1; r < RAD; ++r) {
                const VT x = row[row_slot_step<PR, nb>(j, pj, r)];
                const VT t = w[q * (RAD - 1) + r - 1];
                v[r].x = x.x * t.x - x.y * t.y;
                v[r].y = x.x * t.y + x.y * t.x;
            }
            small_dft<R, RAD>(v);
        }
        if constexpr (Next::kNone && kStraight) {
#pragma unroll
            for (int q = 0; q < KB; ++q) {
                const int b = threadIdx.x + q * NT;
#pragma unroll
                for (int r = 0; r < RAD; ++r) {
                    if (RAD >= 4 && outer && r >= RAD / 4 && r < RAD - RAD / 4) continue;    // uniform
                    store(b / nb, b % nb + r * nb, hold[RAD * q + r]);
                }
            }
            return;
        }
        VT wn[Next::kTw];
        if constexpr (Next::kAhead) Next::load(tw, wn);
        lds_barrier();
#pragma unroll
        for (int q = 0; q < KB; ++q) {
            const int b = threadIdx.x + q * NT;
            const int rr = b / nb, j = b % nb;
            const int jm = j & (Ns - 1);
            VT* row = buf + rr * L::kPitch;
            const int d = (j - jm) * RAD + jm;
            const int pd = row_slot<PR>(d);
#pragma unroll
            for (int r = 0; r < RAD; ++r) {
                if (Next::kNone && RAD >= 4 && outer && r >= RAD / 4 && r < RAD - RAD / 4) continue;    // uniform
                row[row_slot_step<PR, Ns>(d, pd, r)] = hold[RAD * q + r];
            }
        }
        lds_barrier();
        stockham_stages<R, N, ROWS, LNS + 3, kStraight>(buf, tw, wn, outer, store);
    }
}

template <typename R, int N, int ROWS, int SIGN, bool kStraight>
__global__ __launch_bounds__((FftShape<N, ROWS>::kThreads)) void k_fft_pass(FftArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    using VT = typename C2<R>::T;
    using S = FftShape<N, ROWS>;
    using L = FftLds<R, N, ROWS>;
    constexpr int NT = S::kThreads;
    constexpr int RAD = S::kRad0;
    constexpr int nb = N / RAD;
    constexpr int KB = ROWS * nb / NT;
    static_assert(KB >= 1 && KB * NT == ROWS * nb, "butterflies per thread");
    VT* buf = reinterpret_cast<VT*>(smem);
    if (a.zero && blockIdx.x == 0 && threadIdx.x == 0) *a.zero = 0;
    // Consecutive row blocks go to one XCD, so that its L2 gathers the narrow transposed writes of
    // neighbouring blocks into whole lines.
    const int row0 = xcd_chunk(blockIdx.x, gridDim.x) * ROWS;
    const VT* src = reinterpret_cast<const VT*>(a.src);
    const VT* tw = reinterpret_cast<const VT*>(a.twiddle);
    // Blocked intermediate: element (output o, source row r) of a transposed pass in a block of kBO outputs by ROWS
    // rows.
    constexpr int kBO = ROWS * sizeof(VT) < 64 ? 64 / (ROWS * sizeof(VT)) : 1;
    auto blocked = [&](int o, int r, int pitch) {
        return ((static_cast<size_t>(o / kBO) * (pitch / ROWS) + r / ROWS) * kBO + o % kBO) * ROWS + r % ROWS;
    };
    const R* h_in = reinterpret_cast<const R*>(a.h_in);
    const R* h_out = reinterpret_cast<const R*>(a.h_out);
    const R* h_row = reinterpret_cast<const R*>(a.h_row);
    // Inputs confined to the central half of the positions are the transform's first and last quarter.
    const bool outer_in = N >= 8 && a.in_pos >= N / 4 && a.in_pos + a.in_count <= N - N / 4;
    const bool outer_out = N >= 8 && a.out_pos >= N / 4 && a.out_pos + a.out_count <= N - N / 4;
    // First stage: a thread's values are j + r N / RAD of a row. All guarded loads (values and factors) are issued
    // before any is used, so a thread waits on memory once.
    using First = FftStage<R, N, ROWS, 3>;
    VT w[First::kTw];
    VT v[KB * RAD];
    R hin[KB * RAD], hrow[KB];
#pragma unroll
    for (int q = 0; q < KB; ++q) {
        const int b = threadIdx.x + q * NT;
        const int rr = b / nb, j = b % nb;
        const int row = row0 + rr;
        hrow[q] = 1;
        if (h_row && row < a.nrows) hrow[q] = h_row[row + a.row_off];
#pragma unroll
        for (int r = 0; r < RAD; ++r) {
            const int i = q * RAD + r;
            v[i].x = 0;
            v[i].y = 0;
            hin[i] = 1;
            if (outer_in && r >= RAD / 4 && r < RAD - RAD / 4) continue;      // uniform
            const int s = (j + r * nb + N / 2) & (N - 1);                     // position
            const int c = s - a.in_pos;
            if (row < a.nrows && c >= 0 && c < a.in_count) {
                v[i] = src[a.src_blocked ? blocked(row, c + a.src_col, a.src_pitch) : static_cast<size_t>(row) * a.src_pitch + c];
                if (h_in) hin[i] = h_in[s];
            }
        }
    }
    if constexpr (First::kAhead) First::load(tw, w);
#pragma unroll
    for (int q = 0; q < KB; ++q) {
        const int b = threadIdx.x + q * NT;
        const int rr = b / nb, j = b % nb;
        VT* x = v + q * RAD;
        if (h_in || h_row) {                                                  // uniform
#pragma unroll
            for (int r = 0; r < RAD; ++r) {
                const R f = hin[q * RAD + r] * hrow[q];
                x[r].x *= f;
                x[r].y *= f;
            }
        }
        if constexpr (SIGN > 0) {
#pragma unroll
            for (int r = 0; r < RAD; ++r) {
                const R t = x[r].x;
                x[r].x = x[r].y;
                x[r].y = t;
            }
        }
        if constexpr (RAD == 8) {
            if (outer_in) outer_dft8<R>(x);
            else small_dft<R, 8>(x);
        } else {
            small_dft<R, RAD>(x);
        }
        VT* row = buf + rr * L::kPitch;
        const int pd = row_slot<L::kRowPad>(j * RAD);
#pragma unroll
        for (int r = 0; r < RAD; ++r) row[row_slot_step<L::kRowPad, 1>(j * RAD, pd, r)] = x[r];
    }
    lds_barrier();
    VT* dst = reinterpret_cast<VT*>(a.dst);
    auto emit = [&](VT* to, VT x, R f) {
        if constexpr (SIGN > 0) {
            const R t = x.x;
            x.x = x.y;
            x.y = t;
        }
        if (h_out) {                                                          // uniform
            x.x *= f;
            x.y *= f;
        }
        *to = x;
    };
    // Straight: output q of row rr, from the last stage's registers; neighbouring lanes hold neighbouring outputs.
    auto store = [&](int rr, int q, VT x) {
        const int row = row0 + rr, r = (q + N / 2) & (N - 1), o = r - a.out_pos;
        if (row < a.nrows && o >= 0 && o < a.out_count)
            emit(dst + static_cast<size_t>(row) * a.dst_pitch + o, x, h_out ? h_out[r] : R(1));
    };
    stockham_stages<R, N, ROWS, 3, kStraight>(buf, tw, w, outer_out, store);
    if constexpr (kStraight) return;
    // Transposed: from LDS, the rows of the workgroup side by side. out_count * ROWS <=
    // kPer * NT outputs; the factors' loads issued first.
    constexpr int kPer = ROWS * N / NT;
    const int nout = a.out_count * ROWS;
    R hout[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int idx = threadIdx.x + q * NT;
        hout[q] = 1;
        if (h_out && idx < nout) hout[q] = h_out[a.out_pos + idx / ROWS];
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int idx = threadIdx.x + q * NT;
        const int o = idx / ROWS, rr = idx % ROWS;
        const int row = row0 + rr;
        if (idx >= nout || row >= a.nrows) continue;
        const VT x = buf[rr * L::kPitch + row_slot<L::kRowPad>((a.out_pos + o + N / 2) & (N - 1))];
        const size_t at = a.dst_blocked ? blocked(o, row + a.dst_col, a.dst_pitch) : static_cast<size_t>(o) * a.dst_pitch + row;
        emit(dst + at, x, hout[q]);
    }
}

}  // namespace dev

namespace {
template <typename R, int N, int ROWS, int SIGN, bool kStraight>
hipError_t launch_fft_sign(const FftArgs& a, hipStream_t s) {
    using S = dev::FftShape<N, ROWS>;
    static const hipError_t attr =
        hipFuncSetAttribute(reinterpret_cast<const void*>(&dev::k_fft_pass<R, N, ROWS, SIGN, kStraight>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    const unsigned nb = static_cast<unsigned>((a.nrows + ROWS - 1) / ROWS);
    const size_t shm = dev::FftLds<R, N, ROWS>::kBytes;
    hipLaunchKernelGGL((dev::k_fft_pass<R, N, ROWS, SIGN, kStraight>), dim3(nb), dim3(S::kThreads), shm, s, a);
    return hipGetLastError();
}
template <typename R, int N>
hipError_t launch_fft_n(const FftArgs& a, hipStream_t s) {
    constexpr size_t row_bytes = static_cast<size_t>(N) * 2 * sizeof(R);
    // two rows per workgroup: two workgroups share a compute unit, one loading while the other transforms
    constexpr int rows = (2 * row_bytes <= 131072) ? 2 : 1;
    if (a.straight) {
        // the image calls' last passes, on grids of at least 64 cells (the straight store takes the last of several stages)
        if constexpr (N < 64) return hipErrorInvalidValue;
        else return a.sign > 0 ? launch_fft_sign<R, N, rows, 1, true>(a, s) : launch_fft_sign<R, N, rows, -1, true>(a, s);
    }
    return a.sign > 0 ? launch_fft_sign<R, N, rows, 1, false>(a, s) : launch_fft_sign<R, N, rows, -1, false>(a, s);
}
template <typename R>
hipError_t launch_fft_t(const FftArgs& a, hipStream_t s) {
    switch (a.N) {
        case 4: return launch_fft_n<R, 4>(a, s);
        case 8: return launch_fft_n<R, 8>(a, s);
        case 16: return launch_fft_n<R, 16>(a, s);
        case 32: return launch_fft_n<R, 32>(a, s);
        case 64: return launch_fft_n<R, 64>(a, s);
        case 128: return launch_fft_n<R, 128>(a, s);
        case 256: return launch_fft_n<R, 256>(a, s);
        case 512: return launch_fft_n<R, 512>(a, s);
        case 1024: return launch_fft_n<R, 1024>(a, s);
        case 2048: return launch_fft_n<R, 2048>(a, s);
        case 4096: return launch_fft_n<R, 4096>(a, s);
        case 8192: return launch_fft_n<R, 8192>(a, s);
    }
    return hipErrorInvalidValue;
}
}  // namespace

hipError_t fft2_twiddles(bool f64, int N, const void* host, void** out, hipStream_t s) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* base[kMaxDevices][2] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    {
        std::lock_guard<std::mutex> lk(mu);
        void*& p = base[dev][f64 ? 1 : 0];
        if (!p) e = f64 ? hipGetSymbolAddress(&p, HIP_SYMBOL(dev::g_twiddles64)) : hipGetSymbolAddress(&p, HIP_SYMBOL(dev::g_twiddles32));
        if (e != hipSuccess) return e;
        *out = static_cast<char*>(p) + static_cast<size_t>(N) * (f64 ? sizeof(double2) : sizeof(float2));
    }
    return hipMemcpyAsync(*out, host, static_cast<size_t>(N) * (f64 ? sizeof(double2) : sizeof(float2)),
                          hipMemcpyHostToDevice, s);
}

hipError_t launch_fft_pass(bool f64, const FftArgs& a, hipStream_t s) {
    if (a.nrows == 0) return hipSuccess;
    return f64 ? launch_fft_t<double>(a, s) : launch_fft_t<float>(a, s);
}

}  // namespace lmg

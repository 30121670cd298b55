// MPA long step on windows larger than one workgroup's transform
// (8192 <= N <= 2^22 points per window): either one full periodic window (no
// taper, halo or roll-off), or the time blocks of a blocked plan with
// B > 4096, every window gathered with its halos and tapered, run side by side
// (grid dimension y = window), its spectrum rolled off at reconstruction and
// its core stitched back.  Every transform of Eqs. 2 and 6 is an N-point
// transform done as a four-step FFT over N = N1 N2 (row-major matrix
// x[n1][n2], n = N2 n1 + n2):
//   forward   column pass  Y[k1][n2] = w_N^{n2 k1} sum_{n1} x[n1][n2] w_N1^{n1 k1}
//             row pass     X[k1][k2] = sum_{n2} Y[k1][n2] w_N2^{n2 k2}
//   inverse   row pass     Y[k1][n2] = w_N^{-n2 k1} sum_{k2} X[k1][k2] w_N2^{-n2 k2}
//             column pass  x[n1][n2] = sum_{k1} Y[k1][n2] w_N1^{-n1 k1}
// with w = exp(+2 pi i / .) (the paper's transform).  Spectra stay in the
// row-pass order: position k1 N2 + k2 holds frequency k = k1 + N1 k2, and the
// phase tables are built in that order.
//
// Per long step, in the node order of the fused kernel (nodes l = 1..M, all
// sweeps at each node) with the same precision split (node evaluations in T,
// psi_0, the trapezoid sums and the reconstruction in FP64):
//   init    columns(+) and rows(+) of |A|^2 A in T -> U_0 / 2; columns(+) of A
//           in FP64, then one row pass: rows(+) -> psi_0, psi_0 e^{i beta_1},
//           rows(-) in T
//   (l, s)  columns: inverse column pass, A = e^{Gamma_l} ., sigma dz e^{-Gamma_l}
//           |A|^2 A, forward column pass;
//           rows: forward row pass, U = i sigma dz e^{-Gamma_l} e^{-i beta_l} .,
//           psi^(s+1)_l = psi_0 + S^(s) + U / 2, S^(s) += U, and at once the
//           next evaluation's psi e^{i beta} and inverse row pass (the last
//           evaluation: psi_M e^{i beta_M + Gamma_M} and its inverse row pass
//           in FP64)
//   final   columns(-) in FP64.
// Blocked plans add a gather (taper, FP64) before init and a stitch of the
// cores after final.  This path measures the blocking error of the
// time-blocked plans at full size and gives the autotuner blocks above 4096;
// it makes 2 n_iter M + 5 passes over the windows per long step, bound by their
// memory traffic: up to 2^20 modes the state stays in the 256 MiB last-level
// cache, at 2^22 (FP64 psi_0 and sums, 200 MiB) it does not.  Long step, M = 4, two
// sweeps, FP32, against row passes in and out of their own (3 n_iter M + 6), two
// FP32 table gathers a point for w_N and column groups dealt round the XCDs:
// 2^22 modes 1645 -> 825 us, 2^20 511 -> 246, 2^16 176 -> 103, 2^13 140 -> 89.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "block_fft.hpp"
#include "launch.hpp"

namespace mpa {

namespace {

constexpr int WP = 8;          // points per thread
constexpr int ROW_THREADS = 256;

template <typename T>
__device__ __forceinline__ cx<double> widen(cx<T> a) { return {double(a.re), double(a.im)}; }

template <typename T>
__device__ __forceinline__ cx<T> narrow(cx<double> a) { return {T(a.re), T(a.im)}; }

// FP32 transforms take seven twiddles a pass, from a pass table, whose rows a wave
// reads contiguously.  With four (three rounded twiddles in a row) the error of a
// field was 0.5 % larger after a few long steps (2^13 to 2^16 modes) and 7 to 12 % after
// a strongly nonlinear one than with products of seven; now it is as with those.  Four
// long steps of 2^20 modes 1003 us (978 with four; 1039 with seven gathered from the
// N-point table, 1020 loaded at the start of each pass).
template <typename T>
constexpr int win_rounding() { return sizeof(T) == 4 ? SEVEN : W8_TABLE; }

// w_N^{j} = twh[j >> split] twl[j mod 2^split], j = n2 k1 < N
template <typename T>
__device__ __forceinline__ cx<T> wN(const cx<T>* __restrict__ twl, const cx<T>* __restrict__ twh, int split,
                                    long long j) {
    return cmul(twh[j >> split], twl[j & ((1LL << split) - 1)]);
}

// w_N^{a (i0 + m di)}, m = 0..7, one call per m in turn: FP32 transforms take the
// powers from two FP64 lookups and a recurrence in FP64 (rounded once each;
// two FP32 gathers a point cost more than the transform's own loads), FP64
// ones look every power up.
template <typename T>
struct Powers {
    const cx<double>* __restrict__ twl;
    const cx<double>* __restrict__ twh;
    int split;
    long long j, dj;
    cx<double> w, step;
    __device__ __forceinline__ Powers(const cx<double>* __restrict__ l, const cx<double>* __restrict__ h, int sp,
                                      long long a, long long i0, long long di)
        : twl(l), twh(h), split(sp), j(a * i0), dj(a * di) {
        if constexpr (sizeof(T) == 4) {
            w = wN(twl, twh, split, j);
            step = wN(twl, twh, split, dj);
        }
    }
    __device__ __forceinline__ cx<T> next() {
        if constexpr (sizeof(T) == 4) {
            const cx<T> r = narrow<T>(w);
            w = cmul(w, step);
            return r;
        } else {
            const cx<T> r = wN(twl, twh, split, j);
            j += dj;
            return r;
        }
    }
};

}  // namespace

enum WinColMode { WC_FWD = 0, WC_FWD_CUBE = 1, WC_NODE = 2, WC_INV = 3 };

// TC columns of N1 points per workgroup (thread t TC + c: consecutive lanes
// read consecutive columns of one row).  Loads TIN, computes in TK, stores TOUT.
//   WC_FWD       forward column pass
//   WC_FWD_CUBE  |x|^2 x in FP64, rounded to TK, then the forward column pass
//   WC_NODE      inverse column pass, A = c a, d |A|^2 A, forward column pass
//   WC_INV       inverse column pass
// Column groups go to the XCDs in contiguous runs (workgroup b runs on XCD
// b mod 8), so that the groups that share a cache line of a row share that
// XCD's L2; the columns' exchange buffers are offset so that the lanes the LDS
// serves together (16 of 8 bytes, 8 of 16 bytes) meet distinct banks.
// `dst` may be `src` (no restrict qualifier on either): a thread writes the
// elements that it alone read.
template <typename TIN, typename TK, typename TOUT, int N1, int TC, int MODE>
__global__ void __launch_bounds__(TC * N1 / WP)
win_cols_kernel(const cx<TIN>* src, cx<TOUT>* dst, int n2,
                const cx<TK>* __restrict__ tw1, const cx<double>* __restrict__ twl,
                const cx<double>* __restrict__ twh, int split, TK cnode, TK dnode) {
    constexpr int R = WP, NT = N1 / R;
    constexpr int group = sizeof(TK) == 4 ? 16 : 8;
    constexpr int stride = N1 + (group > TC ? group / TC : 1);
    constexpr bool DBUF = sizeof(TK) == 4;
    __shared__ cx<TK> lds[(DBUF ? 2 : 1) * TC * stride];
    const int groups = gridDim.x, b = blockIdx.x;
    const int grp = groups % 8 == 0 ? (b % 8) * (groups / 8) + b / 8 : b;
    const int c = threadIdx.x % TC, t = threadIdx.x / TC;
    const int col = grp * TC + c;
    const size_t woff = (size_t)blockIdx.y * N1 * n2;      // window of a blocked plan
    src += woff;
    dst += woff;
    cx<TK>* my = lds + c * stride;
    cx<TK>* my1 = my + (DBUF ? TC * stride : 0);
    cx<TK> v[R];
#pragma unroll
    for (int m = 0; m < R; ++m) {
        const cx<TIN> x = src[(size_t)(t + NT * m) * n2 + col];
        if constexpr (MODE == WC_FWD_CUBE) {
            const cx<double> a = widen(x);
            v[m] = narrow<TK>(scale(a, norm2(a)));
        } else {
            v[m] = cx<TK>{TK(x.re), TK(x.im)};
        }
    }
    if constexpr (MODE == WC_NODE || MODE == WC_INV) block_fft<TK, N1, -1, DBUF, TW_AHEAD, false, win_rounding<TK>()>(v, my, my1, tw1, t);
    if constexpr (MODE != WC_INV) {
        if constexpr (MODE == WC_NODE) {
            TK f[R];
#pragma unroll
            for (int m = 0; m < R; ++m) {
                v[m] = scale(v[m], cnode);
                f[m] = cube_factor(v[m], dnode);
            }
            block_fft_scaled<TK, N1, +1, DBUF, TW_AHEAD, false, win_rounding<TK>()>(v, f, my, my1, tw1, t);
        } else {
            block_fft<TK, N1, +1, DBUF, TW_AHEAD, false, win_rounding<TK>()>(v, my, my1, tw1, t);
        }
        Powers<TK> w(twl, twh, split, col, t, NT);
#pragma unroll
        for (int m = 0; m < R; ++m) v[m] = cmul(v[m], w.next());
    }
#pragma unroll
    for (int m = 0; m < R; ++m) dst[(size_t)(t + NT * m) * n2 + col] = cx<TOUT>{TOUT(v[m].re), TOUT(v[m].im)};
}

enum WinRowMode { WR_FIRST = 0, WR_U0 = 1, WR_NODE = 2, WR_LAST = 3 };

struct WinRowArgs {
    const void* src;          // row-pass input (T, or FP64 for WR_FIRST)
    void* dst;                // WR_FIRST / WR_NODE output (T), WR_LAST (FP64)
    double* psi0;             // N FP64 complex
    double* S;                // FP64 complex running sums of this sweep
    void* u0;                 // N complex (T): U_0 / 2, every sweep's sum before node 1
    const void* ph;           // this node's phasors (T), spectral order
    const void* ph_next;      // the next evaluation's
    const void* ph_last;      // node-M phasors (FP64), spectral order
    double half_d0, out_scale;
    int first_node, last_node, last_sweep;
};

// TR rows of N2 points per workgroup.
//   WR_U0     forward row pass (T) -> U_0 / 2 = i d0 / 2 .
//   WR_FIRST  forward row pass (FP64) -> psi_0; psi_0 e^{i beta_1}, inverse row pass,
//             w_N^{-n2 k1} -> dst (T)
//   WR_NODE   forward row pass, U, Eq. 6 update of S^(s); the next evaluation's
//             psi e^{i beta}, inverse row pass, w_N^{-n2 k1} -> dst (T)
//   WR_LAST   forward row pass, U, psi_M; psi_M e^{i beta_M} e^{Gamma_M}, inverse row
//             pass, w_N^{-n2 k1} in FP64 -> dst
template <typename T, int N2, int TR, int MODE>
__global__ void __launch_bounds__(TR * N2 / WP) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2)))
win_rows_kernel(WinRowArgs a, const cx<T>* __restrict__ tw2, const cx<double>* __restrict__ tw2_64,
                const cx<double>* __restrict__ twl64, const cx<double>* __restrict__ twh64, int split, long long N) {
    constexpr int R = WP, NT = N2 / R;
    constexpr bool WIDE = MODE == WR_FIRST || MODE == WR_LAST || sizeof(T) == 8;   // an FP64 transform among them
    constexpr bool DBUF = !WIDE;
    __shared__ cx<double> lds[TR * N2];          // FP64: one buffer; FP32: two
    const int r = threadIdx.x / NT, t = threadIdx.x - r * NT;
    const long long k1 = (long long)blockIdx.x * TR + r;
    const size_t base = (size_t)k1 * N2 + t;
    const size_t woff = (size_t)blockIdx.y * N;            // window of a blocked plan (tables: no offset)
    cx<double>* d0 = lds + r * N2;
    cx<double>* d1 = d0;
    cx<T>* b0 = reinterpret_cast<cx<T>*>(d0);
    cx<T>* b1 = b0 + (DBUF ? N2 : 0);
    cx<double>* psi0 = reinterpret_cast<cx<double>*>(a.psi0) + woff + base;
    cx<T> v[R];
    cx<double> z[R];
    if constexpr (MODE == WR_FIRST) {
        const cx<double>* src = static_cast<const cx<double>*>(a.src) + woff + base;
#pragma unroll
        for (int m = 0; m < R; ++m) z[m] = src[NT * m];
        block_fft<double, N2, +1, false, TW_AHEAD, false, W8_TABLE>(z, d0, d1, tw2_64, t);
#pragma unroll
        for (int m = 0; m < R; ++m) {
            psi0[NT * m] = z[m];
            v[m] = narrow<T>(z[m]);
        }
    } else {
        const cx<T>* src = static_cast<const cx<T>*>(a.src) + woff + base;
#pragma unroll
        for (int m = 0; m < R; ++m) v[m] = src[NT * m];
        block_fft<T, N2, +1, DBUF, TW_AHEAD, false, win_rounding<T>()>(v, b0, b1, tw2, t);
    }
    cx<T>* u0 = static_cast<cx<T>*>(a.u0) + woff + base;
    if constexpr (MODE == WR_U0) {
#pragma unroll
        for (int m = 0; m < R; ++m) u0[NT * m] = rot<+1>(scale(v[m], T(a.half_d0)));
        return;
    }
    if constexpr (MODE == WR_NODE || MODE == WR_LAST) {
#pragma clang fp contract(off)
        cx<double>* S = reinterpret_cast<cx<double>*>(a.S) + woff + base;
        const cx<T>* ph = static_cast<const cx<T>*>(a.ph) + base;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            const cx<double> u = widen(rot<+1>(cmulc(v[m], ph[NT * m])));
            const cx<double> s = a.first_node ? widen(u0[NT * m]) : S[NT * m];
            const cx<double> p0 = psi0[NT * m];
            const cx<double> nxt = p0 + mad(u, 0.5, s);
            if constexpr (MODE == WR_LAST) {
                z[m] = nxt;
            } else {
                // the last sweep's psi is needed at node M only (WR_LAST)
                v[m] = a.last_sweep ? narrow<T>(p0) : narrow<T>(nxt);
                if (!a.last_node) S[NT * m] = s + u;
            }
        }
    }
    if constexpr (MODE == WR_LAST) {
        const cx<double>* pl = static_cast<const cx<double>*>(a.ph_last) + base;
#pragma unroll
        for (int m = 0; m < R; ++m) z[m] = cmul(z[m], pl[NT * m]);
        block_fft_scaled<double, N2, -1, false, TW_AHEAD, false, W8_TABLE>(z, a.out_scale, d0, d1, tw2_64, t);
        cx<double>* dst = static_cast<cx<double>*>(a.dst) + woff + base;
        Powers<double> w(twl64, twh64, split, k1, t, NT);
#pragma unroll
        for (int m = 0; m < R; ++m) dst[NT * m] = cmulc(z[m], w.next());
    } else {
        const cx<T>* ph = static_cast<const cx<T>*>(a.ph_next) + base;
#pragma unroll
        for (int m = 0; m < R; ++m) v[m] = cmul(v[m], ph[NT * m]);
        block_fft<T, N2, -1, DBUF, TW_AHEAD, false, win_rounding<T>()>(v, b0, b1, tw2, t);
        cx<T>* dst = static_cast<cx<T>*>(a.dst) + woff + base;
        Powers<T> w(twl64, twh64, split, k1, t, NT);
#pragma unroll
        for (int m = 0; m < R; ++m) dst[NT * m] = cmulc(v[m], w.next());
    }
}

// Blocked plans: window w of B samples starts at w C - lead (mod n) and is
// multiplied by the taper, in FP64 (out[w][t]).
template <typename T>
__global__ void win_gather_kernel(const cx<T>* __restrict__ in, cx<double>* __restrict__ out, long long n, int B,
                                  int core, int lead, const double* __restrict__ taper, long long total) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        const long long w = i / B;
        const int t = (int)(i - w * B);
        long long j = (w * core - lead + t) % n;
        if (j < 0) j += n;
        const cx<T> x = in[j];
        out[i] = scale(cx<double>{double(x.re), double(x.im)}, taper[t]);
    }
}

// Sample i of the field is sample lead + (i - w C) of window w = i / C (the
// cores partition the field; the last one may be shorter).
template <typename T>
__global__ void win_stitch_kernel(const cx<double>* __restrict__ win, cx<T>* __restrict__ out, long long n, int B,
                                  int core, int lead) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const long long w = i / core;
        const cx<double> x = win[w * B + lead + (i - w * core)];
        out[i] = cx<T>{T(x.re), T(x.im)};
    }
}

// ---- launchers -------------------------------------------------------------------

// Columns per workgroup: 2048 points, or 4096 (32-byte row segments) for FP32
// columns of 1024.  Long step at 2^22 modes, M = 4, two sweeps, 2048 / 4096 / 8192
// points: FP32 859 / 803 / 824 us, FP64 1275 / 1315 / 1317; 2^18 modes (512-point
// columns) FP32 131 / 139 / 162, FP64 164 / 187 / 231.
template <typename TK, int N1>
constexpr int col_tile() {
    constexpr int points = sizeof(TK) == 4 && N1 >= 1024 ? 4096 : 2048;
    return points / N1 > 16 ? 16 : points / N1;
}

template <int N2>
constexpr int row_tile() { return (ROW_THREADS * WP / N2) > 1 ? (ROW_THREADS * WP / N2) : 1; }

template <typename TIN, typename TK, typename TOUT, int MODE, int N1>
static hipError_t cols_n1(const WindowStepArgs& w, const void* src, void* dst, const void* tw1, double cnode,
                          double dnode) {
    constexpr int TC = col_tile<TK, N1>();
    if (w.n2 % TC) return hipErrorInvalidValue;
    hipLaunchKernelGGL((win_cols_kernel<TIN, TK, TOUT, N1, TC, MODE>), dim3(w.n2 / TC, w.windows), dim3(TC * N1 / WP), 0,
                       w.stream, static_cast<const cx<TIN>*>(src), static_cast<cx<TOUT>*>(dst), w.n2,
                       static_cast<const cx<TK>*>(tw1), static_cast<const cx<double>*>(w.twl),
                       static_cast<const cx<double>*>(w.twh), w.split, TK(cnode), TK(dnode));
    return hipGetLastError();
}

template <typename TIN, typename TK, typename TOUT, int MODE>
static hipError_t cols(const WindowStepArgs& w, const void* src, void* dst, double cnode = 1.0,
                       double dnode = 1.0) {
    const void* tw1 = sizeof(TK) == 8 ? w.tw1_64 : w.tw1;
    switch (w.n1) {
        case 64: return cols_n1<TIN, TK, TOUT, MODE, 64>(w, src, dst, tw1, cnode, dnode);
        case 128: return cols_n1<TIN, TK, TOUT, MODE, 128>(w, src, dst, tw1, cnode, dnode);
        case 256: return cols_n1<TIN, TK, TOUT, MODE, 256>(w, src, dst, tw1, cnode, dnode);
        case 512: return cols_n1<TIN, TK, TOUT, MODE, 512>(w, src, dst, tw1, cnode, dnode);
        case 1024: return cols_n1<TIN, TK, TOUT, MODE, 1024>(w, src, dst, tw1, cnode, dnode);
        default: return hipErrorInvalidValue;
    }
}

template <typename T, int MODE, int N2>
static hipError_t rows_n2(const WindowStepArgs& w, const WinRowArgs& a) {
    constexpr int TR = row_tile<N2>();
    if (w.n1 % TR) return hipErrorInvalidValue;
    hipLaunchKernelGGL((win_rows_kernel<T, N2, TR, MODE>), dim3(w.n1 / TR, w.windows), dim3(TR * N2 / WP), 0, w.stream, a,
                       static_cast<const cx<T>*>(w.tw2), static_cast<const cx<double>*>(w.tw2_64),
                       static_cast<const cx<double>*>(w.twl), static_cast<const cx<double>*>(w.twh), w.split,
                       (long long)w.n);
    return hipGetLastError();
}

template <typename T, int MODE>
static hipError_t rows(const WindowStepArgs& w, const WinRowArgs& a) {
    switch (w.n2) {
        case 128: return rows_n2<T, MODE, 128>(w, a);
        case 256: return rows_n2<T, MODE, 256>(w, a);
        case 512: return rows_n2<T, MODE, 512>(w, a);
        case 1024: return rows_n2<T, MODE, 1024>(w, a);
        case 2048: return rows_n2<T, MODE, 2048>(w, a);
        case 4096: return rows_n2<T, MODE, 4096>(w, a);
        default: return hipErrorInvalidValue;
    }
}

template <typename T>
static hipError_t window_step_t(const WindowStepArgs& w) {
    const size_t N = (size_t)w.n;
    hipError_t e;
    // one full window reads and writes the field itself: exactly one window
    if (w.windows < 1 || (!w.blocked && (w.windows != 1 || w.n_field != w.n))) return hipErrorInvalidValue;
    WinRowArgs a{};
    a.psi0 = static_cast<double*>(w.psi0);
    a.u0 = w.cur;
    const double* ns = w.node_scale_host;           // c_j, e_j as built (FP64), rounded to T below
    const auto phase = [&](int l) { return static_cast<const char*>(w.phase) + (size_t)l * N * sizeof(cx<T>); };
    // init: U_0 / 2 = i sigma dz / 2 F[|A|^2 A], psi_0 = F[A] (FP64)
    if (w.blocked) {
        // the tapered windows in FP64; the cube's column pass reads them before the
        // forward column pass overwrites them in place
        const long long total = (long long)w.n * w.windows;
        const unsigned grid = (unsigned)std::min<long long>((total + 255) / 256, 8192);
        hipLaunchKernelGGL(win_gather_kernel<T>, dim3(grid), dim3(256), 0, w.stream, static_cast<const cx<T>*>(w.in),
                           static_cast<cx<double>*>(w.work64), (long long)w.n_field, (int)w.n, w.core, w.lead,
                           w.taper, total);
        if ((e = hipGetLastError())) return e;
        if ((e = cols<double, T, T, WC_FWD_CUBE>(w, w.work64, w.work))) return e;
        if ((e = cols<double, double, double, WC_FWD>(w, w.work64, w.work64))) return e;
    } else {
        if ((e = cols<T, T, T, WC_FWD_CUBE>(w, w.in, w.work))) return e;
        if ((e = cols<T, double, double, WC_FWD>(w, w.in, w.work64))) return e;
    }
    a.src = w.work;
    a.half_d0 = double(T(T(w.sigma) * T(ns[1])) * T(0.5));
    if ((e = rows<T, WR_U0>(w, a))) return e;
    a.src = w.work64;
    a.dst = w.work;
    a.ph_next = phase(1);
    if ((e = rows<T, WR_FIRST>(w, a))) return e;
    a.src = w.work;
    for (int l = 1; l <= w.M; ++l) {
        const double cl = T(ns[2 * l]), dl = T(w.sigma) * T(ns[2 * l + 1]);
        a.ph = phase(l);
        a.first_node = l == 1;
        a.last_node = l == w.M;
        for (int s = 0; s < w.n_iter; ++s) {
            if ((e = cols<T, T, T, WC_NODE>(w, w.work, w.work, cl, dl))) return e;
            a.S = static_cast<double*>(w.sums) + (size_t)s * 2 * N * w.windows;
            a.last_sweep = s == w.n_iter - 1;
            if (a.last_sweep && a.last_node) break;
            a.ph_next = phase(a.last_sweep ? l + 1 : l);
            if ((e = rows<T, WR_NODE>(w, a))) return e;
        }
    }
    // final: A(z0 + L) from psi_M (FP64)
    a.ph_last = w.phase_last;
    a.out_scale = w.out_scale;
    a.dst = w.work64;
    if ((e = rows<T, WR_LAST>(w, a))) return e;
    if (!w.blocked) return cols<double, double, T, WC_INV>(w, w.work64, w.out);
    if ((e = cols<double, double, double, WC_INV>(w, w.work64, w.work64))) return e;
    const unsigned grid = (unsigned)std::min<long long>((w.n_field + 255) / 256, 8192);
    hipLaunchKernelGGL(win_stitch_kernel<T>, dim3(grid), dim3(256), 0, w.stream,
                       static_cast<const cx<double>*>(w.work64), static_cast<cx<T>*>(w.out), (long long)w.n_field,
                       (int)w.n, w.core, w.lead);
    return hipGetLastError();
}

std::vector<double> pass_table(int n) {
    std::vector<double> t(2 * (size_t)product_elems(n));
    for (int s = 1; s < n_passes(n); ++s) {
        const int p = pass_span(n, s);
        for (int q = 1; q < 8; ++q)
            for (int k = 0; k < p; ++k) {
                const double a = 2.0 * 3.14159265358979323846 * (double(q * k) / (8 * p));
                const size_t i = (size_t)product_offset(n, s) + (size_t)(q - 1) * p + k;
                t[2 * i] = std::cos(a);
                t[2 * i + 1] = std::sin(a);
            }
    }
    return t;
}

hipError_t launch_window_step(const WindowStepArgs& w) {
    return w.precision == 0 ? window_step_t<float>(w) : window_step_t<double>(w);
}

}  // namespace mpa

// Workgroup-wide power-of-two FFT held in registers, exchanged through LDS.
//
// A workgroup of NT = B / 8 threads transforms B points; thread `tid` holds
// the 8 points with index tid + NT * m (m = 0..7) in registers, both before
// and after the transform.  Every array indexed by frequency (spectra,
// running sums, phase factors) can therefore stay in the registers of the
// thread that owns those frequencies for the whole long step.
//
// The passes follow the Stockham autosort formulation: pass s with radix r
// and span p (product of the earlier radices) reads x[i + q B / r] for
// butterfly i (q = 0..r-1), multiplies by w^(q k), k = i mod p,
// w = exp(SIGN 2 pi i / (p r)), takes an r-point DFT and writes
// y[(i - k) r + k + q p].  The first pass (radix 8, or the remainder
// 2^(log2 B mod 3)) has no twiddles and reads registers, the others are
// radix 8 with one butterfly per thread, the last writes registers (its
// output index set is again tid + NT m), the passes in between exchange
// through LDS.  Results come out in natural order.
//
// A radix-8 pass with twiddles is three levels of radix-2 butterflies
// a +- t b, the twiddle inside the butterfly: s = a + t b is four fused
// multiply-adds, a - t b = 2 a - s two more.  With w = w^k of the pass the
// levels use t = w^4; w^2 and i w^2; w, e^{i pi/4} w, i w and e^{3 i pi/4} w
// (conjugated for SIGN = -1), so a pass takes 72 operations and four stored
// twiddles (w, w^2, w^4, e^{i pi/4} w) where seven complex products in front
// of an 8-point DFT take 80 and seven.
// Rounding, 4096 points, rms relative error against long double: 1.34e-7 in
// FP32 (1.19e-7 with products of table twiddles), 2.7e-16 in FP64, 2.4e-16 with
// W8_TABLE (2.3e-16; 4.0e-16 with the seven twiddles formed from one table load).
// SEVEN takes 72 operations too, with seven stored twiddles: x_1, x_2, x_3 times
// theirs, the first level's butterflies with w^4 .. w^7, two levels without: every
// point meets one rounded twiddle a pass instead of three, 1.21e-7.
//
// SIGN = +1 is the transform with kernel exp(+i omega t) (the paper's F),
// SIGN = -1 its unnormalised inverse.
#pragma once

#include <type_traits>

#include "cx.hpp"

namespace mpa {

constexpr int ilog2(int x) { return x <= 1 ? 0 : 1 + ilog2(x / 2); }

// LDS slot of element j of a transform's exchange buffer: a permutation of
// j inside aligned groups, so that the lanes the LDS serves together (16
// lanes of 8-byte FP32 elements, 8 lanes of 16-byte FP64 elements, over 32
// banks of 4 bytes) meet distinct banks both in the contiguous reads and in
// the strided writes of the passes, for B = 512 .. 4096.  FP32:
// j ^ h(t), t = j >> 4, with h's bits (t0, t0 ^ t1, t1 ^ t2, t2): its low
// bits separate the stride-8, -4 and -2 writes of a radix-8, -4 or -2 first
// pass, its high bits the 64-, 32- and 16-element runs of the pass after it.
// FP64: j ^ ((j >> 3) & 7).  (A pad slot every 8 elements, the simpler
// layout, leaves a 2-way conflict in most FP32 accesses of 16 lanes.)
template <typename T>
__device__ __forceinline__ int lds_slot(int j) {
    if constexpr (sizeof(T) == 4) {
        const int t = j >> 4;
        const int h = (t & 1) | ((t ^ (t << 1)) & 6) | ((t << 1) & 8);
        return j ^ h;
    } else {
        return j ^ ((j >> 3) & 7);
    }
}

// The slot is linear over exclusive or and changes only the low bits of j, so
// for elements a | c with a of the thread and c known at compile time (no
// common bits) it is (slot(a) ^ low bits of slot(c)) + the rest of c: at most
// one operation per access, the rest in the access's offset.  `a`: slot(a) in
// bytes.
template <typename T>
__device__ __forceinline__ cx<T>& lds_at(cx<T>* buf, int a, int c) {
    constexpr int low = sizeof(T) == 4 ? 15 : 7;
    const int s = lds_slot<T>(c);
    return *reinterpret_cast<cx<T>*>(reinterpret_cast<char*>(buf) + (a ^ ((s & low) * (int)sizeof(cx<T>))) +
                                     (s & ~low) * (int)sizeof(cx<T>));
}

template <typename T, bool LEAN>
__device__ __forceinline__ int lds_base(int j) {
    int a = lds_slot<T>(j) * (int)sizeof(cx<T>);
    if constexpr (LEAN) asm volatile("" : "+v"(a));
    return a;
}

// ---- small DFTs in registers (output in natural order, in place) ----------

template <int SIGN, typename T>
__device__ __forceinline__ void dft2(cx<T>& a, cx<T>& b) {
    cx<T> t = a;
    a = t + b;
    b = t - b;
}

template <int SIGN, typename T>
__device__ __forceinline__ void dft4(cx<T>& x0, cx<T>& x1, cx<T>& x2, cx<T>& x3) {
    cx<T> t0 = x0 + x2, t1 = x0 - x2, t2 = x1 + x3, t3 = rot<SIGN>(x1 - x3);
    x0 = t0 + t2;
    x2 = t0 - t2;
    x1 = t1 + t3;
    x3 = t1 - t3;
}

// The same of x_q f_q.  The product of the second input of each first
// butterfly is rounded, the first one's is fused into the sum and the
// difference, by the source and not as the compiler happens to (which fused
// it for one kernel's inputs and not for another's: schedules that are to
// agree bitwise did not in FP64).
template <typename T>
__device__ __forceinline__ void dft2_scaled(cx<T>& a, cx<T>& b, T fa, T fb) {
    const cx<T> p = scale(b, fb), t = a;
    a = mad(t, fa, p);
    b = {fma(t.re, fa, -p.re), fma(t.im, fa, -p.im)};
}

// the second level of dft4, of first-level sums and differences t0 = x0 + x2, t1 = x0 - x2,
// t2 = x1 + x3, t3 = x1 - x3
template <int SIGN, typename T>
__device__ __forceinline__ void dft4_second(cx<T>& t0, cx<T>& t2, cx<T>& t1, cx<T>& t3) {
    const cx<T> a = t0, b = t2, c = t1, d = rot<SIGN>(t3);
    t0 = a + b;
    t1 = a - b;
    t2 = c + d;
    t3 = c - d;
}

template <int SIGN, typename T>
__device__ __forceinline__ void dft4_scaled(cx<T>& x0, cx<T>& x1, cx<T>& x2, cx<T>& x3, T f0, T f1, T f2, T f3) {
    dft2_scaled(x0, x2, f0, f2);
    dft2_scaled(x1, x3, f1, f3);
    dft4_second<SIGN>(x0, x1, x2, x3);
}

template <int SIGN, typename T>
__device__ __forceinline__ void dft8_last(cx<T> (&x)[8]);

// 8-point DFT as two 4-point DFTs of the even and odd samples:
// X_k = E_k + w^k O_k, X_{k+4} = E_k - w^k O_k, w = exp(SIGN 2 pi i / 8).
template <int SIGN, typename T>
__device__ __forceinline__ void dft8(cx<T> (&x)[8]) {
    dft4<SIGN>(x[0], x[2], x[4], x[6]);
    dft4<SIGN>(x[1], x[3], x[5], x[7]);
    dft8_last<SIGN>(x);
}

template <int SIGN, typename T>
__device__ __forceinline__ void dft8_scaled(cx<T> (&x)[8], const T (&f)[8]) {
    dft4_scaled<SIGN>(x[0], x[2], x[4], x[6], f[0], f[2], f[4], f[6]);
    dft4_scaled<SIGN>(x[1], x[3], x[5], x[7], f[1], f[3], f[5], f[7]);
    dft8_last<SIGN>(x);
}

template <int SIGN, typename T>
__device__ __forceinline__ void dft8_last(cx<T> (&x)[8]) {
    const T h = T(0.70710678118654752440084436210484903928);
    // twiddle the odd half: O_1 *= w, O_2 *= w^2 = SIGN i, O_3 *= w^3
    // w O_1 = h (O_1 + SIGN i O_1) and w^3 O_3 = h (-O_3 + SIGN i O_3): the sums
    // are exact up to one rounding, the factor h is applied inside an
    // explicit fused multiply-add with E_k
    cx<T> o1 = x[3], o2 = x[5], o3 = x[7];
    const T s = T(SIGN);
    const cx<T> t1 = {o1.re - s * o1.im, o1.im + s * o1.re};
    const cx<T> t3 = {-o3.re - s * o3.im, -o3.im + s * o3.re};
    o2 = rot<SIGN>(o2);
    cx<T> e0 = x[0], e1 = x[2], e2 = x[4], e3 = x[6], o0 = x[1];
    x[0] = e0 + o0;
    x[4] = e0 - o0;
    x[1] = {fma(t1.re, h, e1.re), fma(t1.im, h, e1.im)};
    x[5] = {fma(-t1.re, h, e1.re), fma(-t1.im, h, e1.im)};
    x[2] = e2 + o2;
    x[6] = e2 - o2;
    x[3] = {fma(t3.re, h, e3.re), fma(t3.im, h, e3.im)};
    x[7] = {fma(-t3.re, h, e3.re), fma(-t3.im, h, e3.im)};
}

template <int SIGN, int r, typename T>
__device__ __forceinline__ void dft(cx<T> (&x)[r]) {
    if constexpr (r == 2) {
        dft2<SIGN>(x[0], x[1]);
    } else if constexpr (r == 4) {
        dft4<SIGN>(x[0], x[1], x[2], x[3]);
    } else {
        static_assert(r == 8, "radix");
        dft8<SIGN>(x);
    }
}

template <int SIGN, int r, typename T>
__device__ __forceinline__ void dft_scaled(cx<T> (&x)[r], const T (&f)[r]) {
    if constexpr (r == 2) {
        dft2_scaled(x[0], x[1], f[0], f[1]);
    } else if constexpr (r == 4) {
        dft4_scaled<SIGN>(x[0], x[1], x[2], x[3], f[0], f[1], f[2], f[3]);
    } else {
        static_assert(r == 8, "radix");
        dft8_scaled<SIGN>(x, f);
    }
}

// a, b = a + t b, a - t b with t = w (SIGN = +1) or conj(w) (SIGN = -1)
template <int SIGN, typename T>
__device__ __forceinline__ void bfly(cx<T>& a, cx<T>& b, cx<T> w) {
    const T wi = SIGN > 0 ? w.im : -w.im;
    const cx<T> s = {fma(-wi, b.im, fma(w.re, b.re, a.re)), fma(wi, b.re, fma(w.re, b.im, a.im))};
    b = {fma(T(2), a.re, -s.re), fma(T(2), a.im, -s.im)};
    a = s;
}

// Twiddles of one radix-8 pass for one thread: w = exp(2 pi i k / (8 p)),
// w^2, w^4 and e^{i pi/4} w.
template <typename T>
struct PassTw {
    cx<T> w1, w2, w4, w8;
};

// w .. w^7 (SEVEN)
template <typename T>
struct PassTw7 {
    cx<T> w[7];
};

// Rounding of a transform (file comment):
//   W8_FORMED  e^{i pi/4} w formed from w
//   W8_TABLE   ... from the table
//   SEVEN      w .. w^7, loaded from a pass table (pass_table in launch.hpp)
enum Rounding { W8_FORMED = 0, W8_TABLE = 1, SEVEN = 2 };

template <typename T>
constexpr int rounding() { return sizeof(T) == 4 ? W8_TABLE : W8_FORMED; }

template <typename T, int RND>
using TwOf = std::conditional_t<RND == SEVEN, PassTw7<T>, PassTw<T>>;

// 8-point DFT of x_q w^q (see the file comment), output in natural order.
template <int SIGN, typename T>
__device__ __forceinline__ void dft8_tw(cx<T> (&x)[8], const PassTw<T>& w) {
    const cx<T> iw2 = {-w.w2.im, w.w2.re}, iw1 = {-w.w1.im, w.w1.re}, iw8 = {-w.w8.im, w.w8.re};
    bfly<SIGN>(x[0], x[4], w.w4);
    bfly<SIGN>(x[2], x[6], w.w4);
    bfly<SIGN>(x[1], x[5], w.w4);
    bfly<SIGN>(x[3], x[7], w.w4);
    bfly<SIGN>(x[0], x[2], w.w2);
    bfly<SIGN>(x[4], x[6], iw2);
    bfly<SIGN>(x[1], x[3], w.w2);
    bfly<SIGN>(x[5], x[7], iw2);
    bfly<SIGN>(x[0], x[1], w.w1);      // X_0, X_4
    bfly<SIGN>(x[4], x[5], w.w8);      // X_1, X_5
    bfly<SIGN>(x[2], x[3], iw1);       // X_2, X_6
    bfly<SIGN>(x[6], x[7], iw8);       // X_3, X_7
    const cx<T> x1 = x[4], x3 = x[6], x4 = x[1], x6 = x[3];
    x[1] = x1;
    x[3] = x3;
    x[4] = x4;
    x[6] = x6;
}

template <int SIGN, typename T>
__device__ __forceinline__ void dft8_tw(cx<T> (&x)[8], const PassTw7<T>& t) {
    const auto times = [](cx<T>& a, cx<T> w) {
        if constexpr (SIGN < 0) w.im = -w.im;
        a = cmul(a, w);
    };
    times(x[2], t.w[1]);
    times(x[1], t.w[0]);
    times(x[3], t.w[2]);
    bfly<SIGN>(x[0], x[4], t.w[3]);
    bfly<SIGN>(x[2], x[6], t.w[5]);
    bfly<SIGN>(x[1], x[5], t.w[4]);
    bfly<SIGN>(x[3], x[7], t.w[6]);
    dft4_second<SIGN>(x[0], x[2], x[4], x[6]);
    dft4_second<SIGN>(x[1], x[3], x[5], x[7]);
    dft8_last<SIGN>(x);
}

// ---- passes --------------------------------------------------------------------

constexpr int first_radix(int B) { return ilog2(B) % 3 == 0 ? 8 : (1 << (ilog2(B) % 3)); }

constexpr int n_passes(int B) {
    int n = 0;
    for (int p = 1; p < B; p *= (n == 0 ? first_radix(B) : 8), ++n) {
    }
    return n;
}

// span of pass s (s = 0: the first)
constexpr int pass_span(int B, int s) { return s == 0 ? 1 : first_radix(B) * (1 << (3 * (s - 1))); }

// Where the twiddles of the passes come from; the values are the same.
//   TW_REGS   the caller's registers (load_twiddles once per kernel): node
//             transforms, whose loop has the registers (24 at 4096 points, FP32)
//   TW_AHEAD  loads from the B-point table two passes ahead of their use:
//             transforms outside the node loop (all of them loaded when the call
//             begins, FP64, cost 40 spilled registers there)
//   TW_PASS   loads at the start of each pass (fewer registers)
//   TW_TABLE  a table in LDS (fill_twiddle_table), read at the start of each
//             pass: transforms inside a loop whose registers cannot hold them
//   TW_PRODUCTS  a table in LDS of w .. w^7 (fill_product_table), each input
//             multiplied by its own in front of an 8-point DFT: 80 operations
//             instead of 72, and less rounding (1.19e-7 against 1.34e-7 in
//             FP32): transforms whose FP32 rounding reaches a result unscaled
enum TwiddleSource { TW_REGS = 0, TW_AHEAD = 1, TW_PASS = 2, TW_TABLE = 3, TW_PRODUCTS = 4 };

// e^{i pi/4} w: from the table in FP32, formed from w in FP64 (three 16-byte
// loads per pass instead of four, 4 % of a 2^22-mode split-step, and an LDS
// table that fits beside two 4096-point exchange buffers), or from the table
// there too where the caller asks for it (W8_TABLE).
template <typename T>
constexpr int tl_rows() { return sizeof(T) == 4 ? 4 : 3; }

template <typename T>
__device__ __forceinline__ cx<T> eighth(cx<T> w) {
    const T h = T(0.70710678118654752440084436210484903928);
    return {h * (w.re - w.im), h * (w.re + w.im)};
}

// pass S (S >= 1) of a B-point transform, from the B-point table `tw`
constexpr int product_offset(int B, int s);

template <typename T, int B, int S, int RND>
__device__ __forceinline__ void pass_twiddles(TwOf<T, RND>& w, const cx<T>* __restrict__ tw, int tid) {
    constexpr int p = pass_span(B, S);
    if constexpr (RND == SEVEN) {
        const cx<T>* __restrict__ row = tw + product_offset(B, S) + (tid & (p - 1));
#pragma unroll
        for (int q = 0; q < 7; ++q) w.w[q] = row[q * p];
        return;
    } else {
    constexpr int stride = B / (p * 8);
    const int k = tid & (p - 1);
    w.w1 = tw[k * stride];
    w.w2 = tw[2 * k * stride];
    w.w4 = tw[4 * k * stride];
    if constexpr (RND != W8_FORMED) w.w8 = tw[(k + p) * stride];
    else w.w8 = eighth(w.w1);
    }
}

// LDS twiddle table: pass s >= 1 (span p) holds w, w^2, w^4 and, in FP32,
// e^{i pi/4} w, p entries each, at tl_offset(s), so that the lanes of a pass,
// whose k are consecutive, read consecutive entries.
template <typename T>
constexpr int tl_offset(int B, int s) {
    int o = 0;
    for (int t = 1; t < s; ++t) o += tl_rows<T>() * pass_span(B, t);
    return o;
}

template <typename T>
constexpr int tl_elems(int B) { return tl_offset<T>(B, n_passes(B)); }

// Fills the table from the B-point table `tw`, `nthreads` threads striding
// over it; the caller puts a barrier between this and the first transform.
template <typename T, int B>
__device__ __forceinline__ void fill_twiddle_table(cx<T>* tl, const cx<T>* __restrict__ tw, int tid, int nthreads) {
    constexpr int NP = n_passes(B);
    for (int e = tid; e < tl_elems<T>(B); e += nthreads) {
        int s = 1;
        while (s + 1 < NP && e >= tl_offset<T>(B, s + 1)) ++s;
        const int p = pass_span(B, s);
        const int r = e - tl_offset<T>(B, s);
        const int q = r / p, k = r - q * p;
        tl[e] = tw[(q == 3 ? k + p : (k << q)) * (B / (8 * p))];
    }
}

// The table of TW_PRODUCTS, and a pass table: pass s >= 1 holds w^q, q = 1..7, in seven rows of p.
constexpr int product_offset(int B, int s) {
    int o = 0;
    for (int t = 1; t < s; ++t) o += 7 * pass_span(B, t);
    return o;
}

constexpr int product_elems(int B) { return product_offset(B, n_passes(B)); }

template <typename T, int B>
__device__ __forceinline__ void fill_product_table(cx<T>* tl, const cx<T>* __restrict__ tw, int tid, int nthreads) {
    constexpr int NP = n_passes(B);
    for (int e = tid; e < product_elems(B); e += nthreads) {
        int s = 1;
        while (s + 1 < NP && e >= product_offset(B, s + 1)) ++s;
        const int p = pass_span(B, s);
        const int r = e - product_offset(B, s);
        const int q = r / p + 1, k = r - (q - 1) * p;
        tl[e] = tw[q * k * (B / (8 * p))];
    }
}

template <typename T, int B, int S, int NP>
__device__ __forceinline__ void all_twiddles(PassTw<T> (&w)[NP - 1], const cx<T>* __restrict__ tw, int tid) {
    if constexpr (S < NP) {
        pass_twiddles<T, B, S, W8_TABLE>(w[S - 1], tw, tid);
        all_twiddles<T, B, S + 1, NP>(w, tw, tid);
    }
}

// twiddles of every pass for TW_REGS, all from the table
template <typename T, int B>
struct Twiddles {
    PassTw<T> w[n_passes(B) - 1];
};

template <typename T, int B>
__device__ __forceinline__ void load_twiddles(Twiddles<T, B>& t, const cx<T>* __restrict__ tw, int tid) {
    all_twiddles<T, B, 1, n_passes(B)>(t.w, tw, tid);
}

// The pieces of a pass.  Reads are issued in the order the butterflies take
// them.  FP32 reads of 2048 points or more form their addresses separately:
// with common ones the compiler pairs neighbouring reads, and the first
// butterflies wait for more of them (292 against 287 us a long step at 2^22
// modes; at 1024 points the paired form is the faster one by 0.7 %).
template <typename T, int B, bool LEAN>
__device__ __forceinline__ void pass_read(cx<T> (&v)[8], cx<T>* in, int tid) {
    constexpr int NT = B / 8;
    constexpr int order[8] = {0, 4, 2, 6, 1, 5, 3, 7};
    const int a = lds_base<T, LEAN>(tid);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int m = order[q];
        if constexpr (sizeof(T) == 4 && B >= 2048 && !LEAN) v[m] = in[lds_slot<T>(tid + NT * m)];
        else v[m] = lds_at<T>(in, a, NT * m);
    }
}

template <typename T, int B, int S, bool LEAN>
__device__ __forceinline__ void pass_write(const cx<T> (&v)[8], cx<T>* out, int tid) {
    constexpr int p = pass_span(B, S);
    const int k = tid & (p - 1);
    const int a = lds_base<T, LEAN>((tid - k) * 8 + k);
#pragma unroll
    for (int q = 0; q < 8; ++q) lds_at<T>(out, a, q * p) = v[q];
}

// the first pass: no twiddles, 8 / r butterflies of radix r; SC: of v_m f_m
template <typename T, int B, int SIGN, bool LEAN, bool SC = false>
__device__ __forceinline__ void pass_first(const cx<T> (&v)[8], cx<T>* out, int tid, const T* f = nullptr) {
    constexpr int NT = B / 8, r = first_radix(B), NB = 8 / r;
    const int a = lds_base<T, LEAN>(tid * r);
#pragma unroll
    for (int u = 0; u < NB; ++u) {
        cx<T> x[r];
#pragma unroll
        for (int q = 0; q < r; ++q) x[q] = v[u + q * NB];
        if constexpr (SC) {
            T fx[r];
#pragma unroll
            for (int q = 0; q < r; ++q) fx[q] = f[u + q * NB];
            dft_scaled<SIGN, r>(x, fx);
        } else {
            dft<SIGN, r>(x);
        }
#pragma unroll
        for (int q = 0; q < r; ++q) lds_at<T>(out, a, u * NT * r + q) = x[q];
    }
}

template <typename T, int B, int SIGN, int S, int NP, bool DBUF, int TWS, bool LEAN, int RND, bool SC>
__device__ __forceinline__ void passes(cx<T> (&v)[8], cx<T>* buf0, cx<T>* buf1, TwOf<T, RND> (&wall)[NP - 1],
                                       const cx<T>* __restrict__ tw, const cx<T>* tl, int tid, const T* f) {
    if constexpr (TWS == TW_AHEAD) {
        int t = tid;
        asm volatile("" : "+v"(t));          // loaded here, not earlier
        if constexpr (S == 0) pass_twiddles<T, B, 1, RND>(wall[0], tw, t);
        if constexpr (S + 2 < NP) pass_twiddles<T, B, S + 2, RND>(wall[S + 1], tw, t);
    }
    constexpr int p = pass_span(B, S);
    constexpr bool first = (S == 0), last = (S == NP - 1);
    // exchange buffers: alternating (DBUF, pass S reads buf[(S - 1) % 2] and
    // writes buf[S % 2]) or one
    cx<T>* in = DBUF ? ((S % 2) ? buf0 : buf1) : buf0;
    cx<T>* out = DBUF ? ((S % 2) ? buf1 : buf0) : buf0;
    if constexpr (first) {
        pass_first<T, B, SIGN, LEAN, SC>(v, out, tid, f);
    } else {
        __syncthreads();        // the previous pass's writes are visible
        pass_read<T, B, LEAN>(v, in, tid);
        if constexpr (!DBUF) {
            // every read done before this pass overwrites.  The values are pinned in front
            // of the barrier: with a branch after the transform the compiler sank the last
            // pass's reads into it, below the barrier, where other waves already write
#pragma unroll
            for (int m = 0; m < 8; ++m) asm volatile("" : "+v"(v[m].re), "+v"(v[m].im));
            __syncthreads();
        }
        TwOf<T, RND> w;
        if constexpr (TWS == TW_PRODUCTS) {
            int k = tid & (p - 1);
            asm volatile("" : "+v"(k));      // read here, not hoisted out of the caller's loops
            const cx<T>* row = tl + product_offset(B, S) + k;
#pragma unroll
            for (int q = 1; q < 8; ++q) {
                cx<T> t = row[(q - 1) * p];
                if constexpr (SIGN < 0) t.im = -t.im;
                v[q] = cmul(v[q], t);
            }
        } else if constexpr (TWS == TW_REGS || TWS == TW_AHEAD) {
            w = wall[S - 1];
        } else if constexpr (TWS == TW_PASS) {
            int t = tid;
            asm volatile("" : "+v"(t));      // loaded here, not earlier
            pass_twiddles<T, B, S, RND>(w, tw, t);
        } else if constexpr (RND != SEVEN) {
            int k = tid & (p - 1);
            asm volatile("" : "+v"(k));      // read here, not hoisted out of the caller's loops
            const cx<T>* row = tl + tl_offset<T>(B, S) + k;
            w.w1 = row[0];
            w.w2 = row[p];
            w.w4 = row[2 * p];
            if constexpr (tl_rows<T>() == 4) w.w8 = row[3 * p];
            else w.w8 = eighth(w.w1);
        }
        if constexpr (TWS == TW_PRODUCTS) dft8<SIGN>(v);
        else dft8_tw<SIGN>(v, w);
        if constexpr (!last) pass_write<T, B, S, LEAN>(v, out, tid);
    }
    if constexpr (!last) passes<T, B, SIGN, S + 1, NP, DBUF, TWS, LEAN, RND, SC>(v, buf0, buf1, wall, tw, tl, tid, f);
}

// B-point transform of the workgroup's registers (see the file comment); must
// be called by every thread of the workgroup (it contains barriers).
//   DBUF = false: one exchange buffer of B elements (buf1 unused), two
//     barriers per exchange.
//   DBUF = true: passes alternate between two buffers: pass s writes
//     buf[s % 2] and pass s + 1 reads it after one barrier; the barrier after
//     the reads is not needed, since the next write goes to the other buffer,
//     whose last readers passed the barrier before this read.  A call ends
//     having read buf[(E - 1) % 2] (E exchanges); the next call must start by
//     writing the other buffer, so for odd E the two pointers are swapped on
//     return.  LDS accesses made otherwise to either buffer must be separated
//     from the call by a barrier.
// `tw` holds exp(+2 pi i j / B), j = 0..B-1; `regs` for TW_REGS, `tl` for
// TW_TABLE and TW_PRODUCTS.  LEAN: every access forms its LDS address (one operation) instead of
// the caller's loop keeping it in a register, for callers that spill otherwise.
template <typename T, int B, int SIGN, bool DBUF, int TWS, bool LEAN = false, int RND = rounding<T>(),
          bool SC = false>
__device__ __forceinline__ void block_fft(cx<T> (&v)[8], cx<T>*& buf0, cx<T>*& buf1, const cx<T>* __restrict__ tw,
                                          int tid, const Twiddles<T, B>* regs = nullptr, const cx<T>* tl = nullptr,
                                          const T* f = nullptr) {
    static_assert((B & (B - 1)) == 0 && B >= 64, "power-of-two block of at least 64 points");
    constexpr int NP = n_passes(B);
    static_assert(RND != SEVEN || TWS == TW_AHEAD || TWS == TW_PASS, "seven twiddles are loaded");
    TwOf<T, RND> w[NP - 1];
    if constexpr (TWS == TW_REGS) {
#pragma unroll
        for (int i = 0; i < NP - 1; ++i) w[i] = regs->w[i];
    }
    passes<T, B, SIGN, 0, NP, DBUF, TWS, LEAN, RND, SC>(v, buf0, buf1, w, tw, tl, tid, f);
    if constexpr (DBUF && (NP - 1) % 2 == 1) {
        cx<T>* s = buf0;
        buf0 = buf1;
        buf1 = s;
    }
}

// The transform of v_m f_m (f real, one factor a point): half of the products
// are fused into the first pass's additions (dft2_scaled).
template <typename T, int B, int SIGN, bool DBUF, int TWS, bool LEAN = false, int RND = rounding<T>()>
__device__ __forceinline__ void block_fft_scaled(cx<T> (&v)[8], const T (&f)[8], cx<T>*& buf0, cx<T>*& buf1,
                                                 const cx<T>* __restrict__ tw, int tid,
                                                 const Twiddles<T, B>* regs = nullptr, const cx<T>* tl = nullptr) {
    block_fft<T, B, SIGN, DBUF, TWS, LEAN, RND, true>(v, buf0, buf1, tw, tid, regs, tl, f);
}

// ... with the same factor at every point
template <typename T, int B, int SIGN, bool DBUF, int TWS, bool LEAN = false, int RND = rounding<T>()>
__device__ __forceinline__ void block_fft_scaled(cx<T> (&v)[8], T s, cx<T>*& buf0, cx<T>*& buf1,
                                                 const cx<T>* __restrict__ tw, int tid,
                                                 const Twiddles<T, B>* regs = nullptr, const cx<T>* tl = nullptr) {
    const T f[8] = {s, s, s, s, s, s, s, s};
    block_fft<T, B, SIGN, DBUF, TWS, LEAN, RND, true>(v, buf0, buf1, tw, tid, regs, tl, f);
}

// ---- two transforms side by side --------------------------------------------------
// Two independent B-point transforms of one workgroup, pass by pass with one
// barrier for both, each between two buffers of its own (as DBUF): the second
// one's reads are in flight under the first one's butterflies, and the first
// one's writes under the second's.
template <typename T, int B, int SA, int SB, int S, int NP, bool SC>
__device__ __forceinline__ void pair_passes(cx<T> (&va)[8], cx<T> (&vb)[8], cx<T>* a0, cx<T>* a1, cx<T>* b0, cx<T>* b1,
                                            const PassTw<T> (&w)[NP - 1], int tid, const T* fa, const T* fb) {
    constexpr bool last = (S == NP - 1);
    // at 4096 points the reads share one address: the separate ones spill (272 against
    // 265 us a long step at 2^22 modes; 13.5 against 13.7 at 2^15, 1024 points)
    constexpr bool SHARED = B >= 4096;
    if constexpr (S == 0) {
        pass_first<T, B, SA, false, SC>(va, a0, tid, fa);
        pass_first<T, B, SB, false, SC>(vb, b0, tid, fb);
    } else {
        __syncthreads();
        pass_read<T, B, SHARED>(va, (S % 2) ? a0 : a1, tid);
        pass_read<T, B, SHARED>(vb, (S % 2) ? b0 : b1, tid);
        dft8_tw<SA>(va, w[S - 1]);
        if constexpr (!last) pass_write<T, B, S, false>(va, (S % 2) ? a1 : a0, tid);
        dft8_tw<SB>(vb, w[S - 1]);
        if constexpr (!last) pass_write<T, B, S, false>(vb, (S % 2) ? b1 : b0, tid);
    }
    if constexpr (!last) pair_passes<T, B, SA, SB, S + 1, NP, SC>(va, vb, a0, a1, b0, b1, w, tid, fa, fb);
}

// The buffers of both are swapped on return as block_fft's are.  SC: the
// transforms of va_m fa_m and vb_m fb_m, as block_fft_scaled.
template <typename T, int B, int SA, int SB, bool SC = false>
__device__ __forceinline__ void block_fft_pair(cx<T> (&va)[8], cx<T> (&vb)[8], cx<T>*& a0, cx<T>*& a1, cx<T>*& b0,
                                               cx<T>*& b1, const Twiddles<T, B>& regs, int tid, const T* fa = nullptr,
                                               const T* fb = nullptr) {
    constexpr int NP = n_passes(B);
    pair_passes<T, B, SA, SB, 0, NP, SC>(va, vb, a0, a1, b0, b1, regs.w, tid, fa, fb);
    if constexpr ((NP - 1) % 2 == 1) {
        cx<T>* s = a0;
        a0 = a1;
        a1 = s;
        s = b0;
        b0 = b1;
        b1 = s;
    }
}

}  // namespace mpa

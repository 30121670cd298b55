// Node-parallel (Jacobi) schedule of one MPA long step: the order of the
// paper's steps 2-6, sweep by sweep, with the z-nodes of every block as
// independent workgroups.
//
// Per long step:
//   init    one workgroup per block: gather the tapered window, psi_0 = F[A_0]
//           (FP64)
//   sweep s one workgroup per (block, node l): steps 2-4 for node l = 1..M from
//           psi^(s)_l (psi^(0)_l = psi_0), storing U^(s)_l; in sweep 0 one more
//           per block computes U_0 / 2 = i sigma dz F[|A_0|^2 A_0] / 2, which
//           only the sums need (many blocks: init does)
//   final   one workgroup per block: step 7 from psi^(n_iter)_M, scatter of the core
//           (a march of one full window: and the next step's init).
// psi^(s+1)_l = psi_0 + U_0/2 + sum_{0<j<l} U_j + U_l/2 (Eq. 6, FP64, left to
// right) is added up by the workgroup that needs it (NP_OWN), or, where those
// sums are long and CUs idle, by a launch of its own after each sweep, one
// thread per (block, frequency) (NP_SUMMED; see sums_apart).
// Every operation, and the order of every sum, is that of the fused
// wavefront kernel, so both schedules give bitwise the same field (which
// products are fused into additions is written out, see cx.hpp and
// dft2_scaled; left to the compiler it differed between the two in FP64);
// this one exposes M times more workgroups for the node work, at the price of keeping
// psi_0, the increments and the nodes' spectra in device memory (L2/MALL-
// resident at the sizes used here) instead of registers.
//
// Workgroup placement: consecutive workgroup ids go to different XCDs
// (id mod 8).  Node workgroup id = xcd + 8 k with k = (l - 1) + M kk and
// block b = 8 kk + xcd, so the M node workgroups of one block share an XCD
// and its L2, where psi_0 and the increments of that block are read.
#include <type_traits>

#include "block_fft.hpp"
#include "launch.hpp"

namespace mpa {

namespace {

constexpr int PTS = 8;
constexpr int XCDS = 8;

template <typename T>
__device__ __forceinline__ cx<double> widen(cx<T> a) { return {double(a.re), double(a.im)}; }

template <typename T>
__device__ __forceinline__ cx<T> narrow(cx<double> a) { return {T(a.re), T(a.im)}; }

__device__ __forceinline__ long long wrap(long long g, long long n) {
    if (g < 0) g += n;
    if (g >= n) g -= n;
    return g;
}

}  // namespace

// the tapered window's sample t
template <typename T>
__device__ __forceinline__ cx<double> window_sample(const cx<T>* __restrict__ in, const double* __restrict__ taper,
                                                    long long w0, int t, long long n) {
    return scale(widen(in[wrap(w0 + t, n)]), taper[t]);
}

// FEW (a CU for every block): psi_0 alone, two exchange buffers; else U_0 / 2 too and one
// buffer (two workgroups of 4096 points per CU instead of one).
template <typename T, int B, bool FEW>
__global__ void __launch_bounds__(B / PTS)
np_init_kernel(const cx<T>* __restrict__ in, cx<double>* __restrict__ psi0_buf, cx<T>* __restrict__ h0_buf,
               long long n, int core, int lead, const T* __restrict__ node_scale, const cx<T>* __restrict__ tw,
               const cx<double>* __restrict__ tw64, const double* __restrict__ taper, T sigma) {
    constexpr int R = PTS;
    constexpr int NT = B / R;
    __shared__ cx<double> lds64[(FEW ? 2 : 1) * B];
    const int tid = threadIdx.x;
    const long long w0 = (long long)blockIdx.x * core - lead;
    cx<double> psi0[R];
    cx<T> cur[R];
#pragma unroll
    for (int m = 0; m < R; ++m) {
        psi0[m] = window_sample(in, taper, w0, tid + NT * m, n);
        if constexpr (!FEW) cur[m] = narrow<T>(scale(psi0[m], norm2(psi0[m])));
    }
    cx<double>* e0 = lds64;
    cx<double>* e1 = lds64 + (FEW ? B : 0);
    block_fft<double, B, +1, FEW, TW_AHEAD>(psi0, e0, e1, tw64, tid);
    const size_t base = (size_t)blockIdx.x * B;
#pragma unroll
    for (int m = 0; m < R; ++m) psi0_buf[base + tid + NT * m] = psi0[m];
    if constexpr (!FEW) {
        cx<T>* l0 = reinterpret_cast<cx<T>*>(lds64);
        cx<T>* l1 = l0;
        block_fft<T, B, +1, false, TW_AHEAD>(cur, l0, l1, tw, tid);
        const T d0 = sigma * node_scale[1];
#pragma unroll
        for (int m = 0; m < R; ++m) h0_buf[base + tid + NT * m] = rot<+1>(scale(cur[m], d0 * T(0.5)));
    }
}

// psi_0 + (U_0/2 + U_1 + ... + U_{l-1} + U_l/2), summed left to right in FP64; the
// increments outside, the points inside, so that the loads of all points of one
// increment are in flight together.  `u`: node 1's row.
template <typename T, int B>
__device__ __forceinline__ void trapezoid(cx<double> (&v)[PTS], const cx<double>* __restrict__ psi0,
                                          const cx<T>* __restrict__ h0, const cx<T>* __restrict__ u, int l, int tid) {
#pragma clang fp contract(off)
    constexpr int NT = B / PTS;
#pragma unroll
    for (int m = 0; m < PTS; ++m) v[m] = widen(h0[tid + NT * m]);
#pragma unroll 2
    for (int j = 1; j < l; ++j) {
        const cx<T>* __restrict__ uj = u + (size_t)(j - 1) * B;
#pragma unroll
        for (int m = 0; m < PTS; ++m) v[m] = v[m] + widen(uj[tid + NT * m]);
    }
#pragma unroll
    for (int m = 0; m < PTS; ++m) {
        const int t = tid + NT * m;
        v[m] = psi0[t] + mad(widen(u[(size_t)(l - 1) * B + t]), 0.5, v[m]);
    }
}

// NP_FIRST (sweep 0): nodes first..M, psi^(0)_l = psi_0, node 0 computes U_0 / 2 into
// h0_buf (first = 1: np_init_kernel has); else nodes 1..M, psi^(s)_l from the last sweep's increments `prev` (NP_OWN) or from
// `prev` itself (NP_SUMMED).  Two exchange buffers (one barrier per exchange) when DBUF,
// else one (three workgroups of 4096 FP32 points per CU instead of one).
enum NodeMode { NP_FIRST = 0, NP_OWN = 1, NP_SUMMED = 2 };

template <typename T, int B, int MODE, bool DBUF>
__global__ void __launch_bounds__(B / PTS)
np_node_kernel(const cx<T>* __restrict__ in, const cx<double>* __restrict__ psi0_buf, cx<T>* __restrict__ h0_buf,
               const cx<T>* __restrict__ prev, cx<T>* __restrict__ u_buf, int n_blocks, long long n, int core,
               int lead, const cx<T>* __restrict__ phase, const T* __restrict__ node_scale,
               const cx<T>* __restrict__ tw, const double* __restrict__ taper, int M, int first, T sigma) {
    constexpr int R = PTS;
    constexpr int NT = B / R;
    constexpr bool FIRST = MODE == NP_FIRST;
    const int xcd = blockIdx.x % XCDS;
    const int k = blockIdx.x / XCDS;
    const int nodes = M + 1 - first;              // nodes first..M (first = 1 after sweep 0)
    const int l = k % nodes + first;
    const int b = (k / nodes) * XCDS + xcd;
    if (b >= n_blocks) return;                    // the whole workgroup leaves together
    __shared__ cx<T> lds[(DBUF ? 2 : 1) * B];
    // the transforms' twiddles from an LDS table, filled while the spectrum loads
    __shared__ cx<T> twl[tl_elems<T>(B)];
    fill_twiddle_table<T, B>(twl, tw, threadIdx.x, B / PTS);
    const int tid = threadIdx.x;
    const size_t base = (size_t)b * B;
    const size_t row1 = (size_t)b * M * B;               // node 1's row of u_buf and prev
    const size_t row = row1 + (size_t)(l - 1) * B;
    cx<T>* l0 = lds;
    cx<T>* l1 = lds + (DBUF ? B : 0);
    cx<T> cur[R], ph[R];
    if (FIRST && l == 0) {
        const long long w0 = (long long)b * core - lead;
#pragma unroll
        for (int m = 0; m < R; ++m) {
            const cx<double> a = window_sample(in, taper, w0, tid + NT * m, n);
            cur[m] = narrow<T>(scale(a, norm2(a)));
        }
        __syncthreads();                          // the twiddle table is complete
        block_fft<T, B, +1, DBUF, TW_TABLE>(cur, l0, l1, tw, tid, nullptr, twl);
        const T d0 = sigma * node_scale[1];
#pragma unroll
        for (int m = 0; m < R; ++m) h0_buf[base + tid + NT * m] = rot<+1>(scale(cur[m], d0 * T(0.5)));
        return;
    }
    if constexpr (MODE == NP_OWN) {
        cx<double> v[R];
        trapezoid<T, B>(v, psi0_buf + base, h0_buf + base, prev + row1, l, tid);
#pragma unroll
        for (int m = 0; m < R; ++m) cur[m] = narrow<T>(v[m]);
    }
#pragma unroll
    for (int m = 0; m < R; ++m) {
        const int t = tid + NT * m;
        if constexpr (FIRST) cur[m] = narrow<T>(psi0_buf[base + t]);
        if constexpr (MODE == NP_SUMMED) cur[m] = prev[row + t];
        ph[m] = phase[(size_t)l * B + t];
    }
    const T c3 = cube_scale<T>(node_scale[2 * l], sigma * node_scale[2 * l + 1]);
    // steps 2-3: A = e^{Gamma_l} F^-1[psi e^{i beta_l}]
#pragma unroll
    for (int m = 0; m < R; ++m) cur[m] = cmul(cur[m], ph[m]);
    __syncthreads();                              // the twiddle table is complete
    block_fft<T, B, -1, DBUF, TW_TABLE>(cur, l0, l1, tw, tid, nullptr, twl);
    T f[R];
#pragma unroll
    for (int m = 0; m < R; ++m) f[m] = cube_factor(cur[m], c3);
    // step 4: U_l = i sigma dz e^{-Gamma_l} e^{-i beta_l} F[|A|^2 A]
    block_fft_scaled<T, B, +1, DBUF, TW_TABLE>(cur, f, l0, l1, tw, tid, nullptr, twl);
#pragma unroll
    for (int m = 0; m < R; ++m) u_buf[row + tid + NT * m] = rot<+1>(cmulc(cur[m], ph[m]));
}

constexpr int SUM_TPB = 64;      // 64 workgroups already at one 4096-point window

// Eq. 6 at every node from the increments of a sweep: psi_buf row l - 1 receives
// psi^(s+1)_l; LAST: psi0_buf receives psi^(n_iter)_M (FP64) instead.
template <typename T, bool LAST>
__global__ void __launch_bounds__(SUM_TPB)
np_sum_kernel(cx<double>* __restrict__ psi0_buf, const cx<T>* __restrict__ h0_buf, const cx<T>* __restrict__ u_buf,
              cx<T>* __restrict__ psi_buf, int B, int M, long long total) {
    const long long i = (long long)blockIdx.x * SUM_TPB + threadIdx.x;
    if (i >= total) return;
    const size_t row = (size_t)(i / B) * M * B + (size_t)(i % B);   // node 1 of this block and frequency
    const cx<double> psi0 = psi0_buf[i];
    cx<double> S = widen(h0_buf[i]);
    constexpr int AHEAD = 8;                      // loads in flight per thread
    for (int j0 = 0; j0 < M; j0 += AHEAD) {
#pragma clang fp contract(off)
        cx<T> u[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q)
            if (j0 + q < M) u[q] = u_buf[row + (size_t)(j0 + q) * B];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) {
            if (j0 + q >= M) break;
            const cx<double> ud = widen(u[q]);
            const bool last = j0 + q == M - 1;
            if (!LAST || last) {
                const cx<double> nxt = psi0 + mad(ud, 0.5, S);
                if constexpr (LAST) psi0_buf[i] = nxt;
                else psi_buf[row + (size_t)(j0 + q) * B] = narrow<T>(nxt);
            }
            S = S + ud;
        }
    }
}

// OWN: psi^(n_iter)_M from the last sweep's increments u_buf, else in psi0_buf (np_sum_kernel).
// NEXT (one full window): the stored field is the next long step's input, so the workgroup
// goes on to its psi_0, as np_init_kernel computes it (4096 points, FP64, M = 16, three
// sweeps: 52 to 51 us a long step; a launch and its first loads).
template <typename T, int B, bool OWN, bool FEW, bool NEXT>
__global__ void __launch_bounds__(B / PTS)
np_final_kernel(cx<double>* __restrict__ psi0_buf, const cx<T>* __restrict__ h0_buf,
                const cx<T>* __restrict__ u_buf, cx<T>* __restrict__ out, long long n, int core, int lead,
                const cx<double>* __restrict__ phase_last, const cx<double>* __restrict__ tw64,
                const double* __restrict__ taper, int M, double out_scale) {
    constexpr int R = PTS;
    constexpr int NT = B / R;
    __shared__ cx<double> lds64[(FEW ? 2 : 1) * B];
    const int tid = threadIdx.x;
    const int b = blockIdx.x;
    const size_t base = (size_t)b * B;
    cx<double> v[R];
    if constexpr (OWN) {
        trapezoid<T, B>(v, psi0_buf + base, h0_buf + base, u_buf + base * M, M, tid);
    } else {
#pragma unroll
        for (int m = 0; m < R; ++m) v[m] = psi0_buf[base + tid + NT * m];
    }
    // step 7: A(z0 + L) = e^{Gamma_M} F^-1[psi_M e^{i beta_M}] (times the roll-off and gain)
#pragma unroll
    for (int m = 0; m < R; ++m) v[m] = cmul(v[m], phase_last[tid + NT * m]);
    cx<double>* e0 = lds64;
    cx<double>* e1 = lds64 + (FEW ? B : 0);
    block_fft_scaled<double, B, -1, FEW, TW_AHEAD>(v, out_scale, e0, e1, tw64, tid);
    const long long c0 = (long long)b * core;
    const long long rest = n - c0;
    const int clen = rest < core ? (int)rest : core;
#pragma unroll
    for (int m = 0; m < R; ++m) {
        const int t = tid + NT * m;
        if (t >= lead && t < lead + clen) out[c0 + (t - lead)] = narrow<T>(v[m]);
        if constexpr (NEXT) v[m] = scale(widen(narrow<T>(v[m])), taper[t]);
    }
    if constexpr (NEXT) {
        block_fft<double, B, +1, FEW, TW_AHEAD>(v, e0, e1, tw64, tid);
#pragma unroll
        for (int m = 0; m < R; ++m) psi0_buf[base + tid + NT * m] = v[m];
    }
}

template <typename T, int B, int MODE, bool DBUF>
static void launch_sweep(const BlockStepArgs& a, const NodeBuffers& nb, const void* prev, void* u, int first) {
    const unsigned groups = (unsigned)(XCDS * (a.M + 1 - first) * ((a.n_blocks + XCDS - 1) / XCDS));
    hipLaunchKernelGGL((np_node_kernel<T, B, MODE, DBUF>), dim3(groups), dim3(B / PTS), 0, a.stream,
                       static_cast<const cx<T>*>(a.in), static_cast<const cx<double>*>(nb.psi0),
                       static_cast<cx<T>*>(nb.half_u0), static_cast<const cx<T>*>(prev), static_cast<cx<T>*>(u),
                       a.n_blocks, (long long)a.n, a.core, a.lead, static_cast<const cx<T>*>(a.phase),
                       static_cast<const T*>(a.node_scale), static_cast<const cx<T>*>(a.twiddle),
                       static_cast<const double*>(a.taper), a.M, first, T(a.sigma));
}

// Whether Eq. 6's sums get a launch of their own.  A node's workgroup that adds
// up its own prefix reads up to M rows through one CU's path to L2, which a
// launch of one thread per frequency spreads over the chip.  Measured per long
// step, own against apart, B = 512 .. 4096, M = 4 .. 128, 1 to 16 blocks, one and
// three sweeps, both precisions: where the rule takes the sums apart that is 0.985 to
// 3.4 times as fast (1.41 on the average; one block of 4096, M = 16, three sweeps, FP32
// 55.8 / 43.9 us, FP64 59.1 / 51.9; four blocks 58.2 / 49.6, 62.0 / 61.9; 512 points, M = 128
// 78.2 / 58.6, 75.2 / 62.4).  The product M B stands for the bytes that one CU reads, and the
// line is where no plan loses: at half of it FP64 loses up to 15 % (2048 points, M = 16,
// eight blocks 40.7 / 47.0) and FP32 gains up to 13 % or loses up to 8 % (512 points, M = 64
// 44.7 / 39.9; 4096, M = 8 43.6 / 40.3; 1024, M = 32, eight blocks 38.6 / 42.0); sixteen blocks of
// 4096 lose at M = 16 (64.3 / 71.4) and would gain at M = 32 (121 / 88).
static bool sums_apart(const BlockStepArgs& a) {
    const long long longest = (long long)a.M * a.block;
    return longest >= 65536 && a.n_blocks <= longest / 16384;
}

template <typename T, int B>
static hipError_t node_step_typed(const BlockStepArgs& a) {
    const NodeBuffers& nb = *a.nodes;
    const dim3 threads(B / PTS);
    auto* psi0 = static_cast<cx<double>*>(nb.psi0);
    const auto* h0 = static_cast<const cx<T>*>(nb.half_u0);
    const auto* tw64 = static_cast<const cx<double>*>(a.twiddle64);
    // with a CU for every block, U_0 is node 0 of the first sweep, beside the others; with
    // more it is computed with psi_0 (2^19 modes, 1024 blocks of 2048, M = 1, two sweeps:
    // 66.7 us a long step as node 0, where every workgroup fills its twiddle table first,
    // 59 with psi_0)
    const bool few = a.n_blocks <= a.cus;
    const int first = few ? 0 : 1;
    const auto init = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(a.n_blocks), threads, 0, a.stream, static_cast<const cx<T>*>(a.in), psi0,
                           static_cast<cx<T>*>(nb.half_u0), (long long)a.n, a.core, a.lead,
                           static_cast<const T*>(a.node_scale), static_cast<const cx<T>*>(a.twiddle), tw64,
                           static_cast<const double*>(a.taper), T(a.sigma));
    };
    if (!a.psi0_ready) {
        if (few) init(np_init_kernel<T, B, true>);
        else init(np_init_kernel<T, B, false>);
    }
    const long long total = (long long)a.n_blocks * B;
    const dim3 sum_groups((unsigned)((total + SUM_TPB - 1) / SUM_TPB));
    const bool dbuf = (long long)a.n_blocks * (a.M + 1) <= a.cus;
    const bool apart = sums_apart(a);
    for (int s = 0; s < a.n_iter; ++s) {
        // increments alternate between the two buffers, or (sums apart) the first holds
        // the increments and the second the spectra
        const void* prev = apart ? nb.u[1] : nb.u[(s + 1) & 1];
        void* u = apart ? nb.u[0] : nb.u[s & 1];
        const auto sweep = [&](auto db) {
            constexpr bool D = decltype(db)::value;
            if (s == 0) launch_sweep<T, B, NP_FIRST, D>(a, nb, prev, u, first);
            else if (apart) launch_sweep<T, B, NP_SUMMED, D>(a, nb, prev, u, 1);
            else launch_sweep<T, B, NP_OWN, D>(a, nb, prev, u, 1);
        };
        if (dbuf) sweep(std::true_type{});
        else sweep(std::false_type{});
        if (!apart) continue;
        const auto sum = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, sum_groups, dim3(SUM_TPB), 0, a.stream, psi0, h0,
                               static_cast<const cx<T>*>(nb.u[0]), static_cast<cx<T>*>(nb.u[1]), B, a.M, total);
        };
        if (s + 1 < a.n_iter) sum(np_sum_kernel<T, false>);
        else sum(np_sum_kernel<T, true>);
    }
    const auto final = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(a.n_blocks), threads, 0, a.stream, psi0, h0,
                           static_cast<const cx<T>*>(nb.u[(a.n_iter - 1) & 1]), static_cast<cx<T>*>(a.out),
                           (long long)a.n, a.core, a.lead, static_cast<const cx<double>*>(a.phase_last), tw64,
                           static_cast<const double*>(a.taper), a.M, a.out_scale);
    };
    if (a.next_psi0) {
        if (a.n_blocks != 1 || a.n != B || a.lead != 0) return hipErrorInvalidValue;
        if (apart) final(np_final_kernel<T, B, false, true, true>);
        else final(np_final_kernel<T, B, true, true, true>);
    } else if (apart) {
        final(np_final_kernel<T, B, false, true, false>);
    } else if (few) {
        final(np_final_kernel<T, B, true, true, false>);
    } else {
        final(np_final_kernel<T, B, true, false, false>);
    }
    return hipGetLastError();
}

template <typename T>
static hipError_t node_step_b(const BlockStepArgs& a) {
    switch (a.block) {
        case 512: return node_step_typed<T, 512>(a);
        case 1024: return node_step_typed<T, 1024>(a);
        case 2048: return node_step_typed<T, 2048>(a);
        case 4096: return node_step_typed<T, 4096>(a);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_node_parallel_step(const BlockStepArgs& a) {
    if (!a.nodes || a.batch || !block_step_supported(a.precision, a.block, a.n_iter)) return hipErrorInvalidValue;
    return a.precision == 0 ? node_step_b<float>(a) : node_step_b<double>(a);
}

}  // namespace mpa

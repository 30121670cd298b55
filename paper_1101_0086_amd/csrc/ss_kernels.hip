// Split-step comparator (Eq. 4) for gfx950.
//
// Small windows (N <= 4096): one workgroup holds the whole field in
// registers for a run of split-steps; each step is FFT -> spectral phase
// (merged half steps) -> inverse FFT -> exact nonlinear kick
// A exp(i sigma |A|^2 dz), with no HBM traffic inside the run.  The field is
// read and written in its storage type ST (float or double); the arithmetic,
// twiddles, phase tables and scales are FP64 for both, so no constant is
// rounded the same way every step (an FP32 twiddle, phasor or scale would
// bias every step alike and the error would grow linearly with the number
// of steps).
#include "block_fft.hpp"
#include "ss.hpp"
#include "ss_kick.hpp"

namespace mpa {

constexpr int SS_PTS = 8;

// One workgroup, a chain of 2 steps + 2 transforms: bound by their exchange
// latency.  The transforms are double-buffered (128 KB of LDS at 4096 points,
// one workgroup on the chip) and keep their twiddles and the full step's
// phasors in registers (two waves per SIMD may hold 256); the half step's
// phasors are loaded at the run's ends.  4096 modes, 320 split-steps: 4.5 us a
// step, 10.7 us with one buffer, twiddles gathered in each pass, 320 bytes
// spilled and the kick's divisions (see ss_kick.hpp).
template <typename ST, int B>
__global__ void __launch_bounds__(B / SS_PTS) __attribute__((amdgpu_waves_per_eu(2)))
ss_run_small_kernel(cx<ST>* __restrict__ field, const cx<double>* __restrict__ half_ph,
                    const cx<double>* __restrict__ full_ph, const cx<double>* __restrict__ tw, int steps,
                    double sdz, double half_scale, double full_scale, double end_scale) {
    constexpr int R = SS_PTS, NT = B / R;
    __shared__ cx<double> lds[2 * B];
    const int tid = threadIdx.x;
    cx<double>* l0 = lds;
    cx<double>* l1 = lds + B;
    Twiddles<double, B> rt;
    load_twiddles<double, B>(rt, tw, tid);
    cx<double> v[R], fp[R];
#pragma unroll
    for (int m = 0; m < R; ++m) {
        const int k = tid + NT * m;
        const cx<ST> f = field[k];
        v[m] = cx<double>{double(f.re), double(f.im)};
        fp[m] = full_ph[k];
    }
    // L dz/2
    block_fft<double, B, +1, true, TW_REGS>(v, l0, l1, tw, tid, &rt);
#pragma unroll
    for (int m = 0; m < R; ++m) v[m] = cmul(v[m], half_ph[tid + NT * m]);
    block_fft_scaled<double, B, -1, true, TW_REGS>(v, half_scale, l0, l1, tw, tid, &rt);
    for (int j = 1; j <= steps; ++j) {
        kick<false>(v, sdz);
        block_fft<double, B, +1, true, TW_REGS>(v, l0, l1, tw, tid, &rt);
        if (j < steps) {
#pragma unroll
            for (int m = 0; m < R; ++m) v[m] = cmul(v[m], fp[m]);
        } else {
#pragma unroll
            for (int m = 0; m < R; ++m) v[m] = cmul(v[m], half_ph[tid + NT * m]);
        }
        block_fft_scaled<double, B, -1, true, TW_REGS>(v, j < steps ? full_scale : end_scale, l0, l1, tw, tid, &rt);
    }
#pragma unroll
    for (int m = 0; m < R; ++m) field[tid + NT * m] = cx<ST>{ST(v[m].re), ST(v[m].im)};
}

template <typename ST, int B>
static hipError_t launch_small_typed(const SSRunArgs& a) {
    hipLaunchKernelGGL((ss_run_small_kernel<ST, B>), dim3(1), dim3(B / SS_PTS), 0, a.stream,
                       static_cast<cx<ST>*>(a.field), static_cast<const cx<double>*>(a.half_ph),
                       static_cast<const cx<double>*>(a.full_ph), static_cast<const cx<double>*>(a.twiddle),
                       a.steps, a.sigma_dz, a.half_scale, a.full_scale, a.end_scale);
    return hipGetLastError();
}

template <typename ST>
static hipError_t launch_small_n(const SSRunArgs& a) {
    switch (a.n) {
        case 512: return launch_small_typed<ST, 512>(a);
        case 1024: return launch_small_typed<ST, 1024>(a);
        case 2048: return launch_small_typed<ST, 2048>(a);
        case 4096: return launch_small_typed<ST, 4096>(a);
        default: return hipErrorInvalidValue;
    }
}

bool ss_small_supported(int precision, int64_t n) {
    return (precision == 0 || precision == 1) && (n == 512 || n == 1024 || n == 2048 || n == 4096);
}

hipError_t launch_ss_run_small(const SSRunArgs& a) {
    if (!ss_small_supported(a.precision, a.n)) return hipErrorInvalidValue;
    return a.precision == 0 ? launch_small_n<float>(a) : launch_small_n<double>(a);
}

}  // namespace mpa

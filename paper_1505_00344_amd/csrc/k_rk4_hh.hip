// Fused RK4 instantiations: Hodgkin-Huxley rings of 1 and 3 neurons.
#include "ff_ring.h"
#include "ff_rk4.h"

namespace ff {

template <typename R> using HH1 = HHRing<R, 1>;
template <typename R> using HH3 = HHRing<R, 3>;

// Single precision is held to 64 VGPRs, eight waves per SIMD: left alone it
// takes 65-72, six or seven waves, and 1-2 % longer.
template <typename R, int N, bool KAHAN>
__global__ void __launch_bounds__(256, sizeof(R) == 4 ? 8 : 1) k_ring(RK4Args a) {
    ring_tile<R, N, KAHAN>(a, (int64_t)blockIdx.x * ring_per_block<N>(blockDim.x));
}

namespace {

template <typename R, bool KAHAN>
hipError_t launch_ring3(const RK4Launch& L) {
    const int per = ring_per_block<3>(L.block);
    const int64_t grid = (L.n + per - 1) / per;
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_ring<R, 3, KAHAN>), dim3((unsigned)grid), dim3(L.block), 0, L.stream, make_args(L));
    return hipGetLastError();
}

// Whether a lane per neuron is the faster split of n particles.  Measured on
// 200 steps (one thread per particle, blocks of 128 -> one lane per neuron):
//   20,011 particles    FP32 0.371 -> 0.146 ms, FP32-Kahan 0.378 -> 0.157, FP64 1.039 -> 0.383
//   140,001             FP32 1.046 -> 0.767 ms, FP32-Kahan 1.075 -> 0.804, FP64 3.18 -> 2.45
//   1,048,576           FP32 5.41 -> 4.81 ms, FP32-Kahan 5.53 -> 5.08, FP64 16.1 -> 16.6
// Both splits are bound by VALU issue, and take whole rounds of one block of
// 256 threads per CU: 65,536 particles with a thread each, 21,504 with three
// lanes each (3.05 of these to one of those).  Lanes need the fewer rounds
// of a part-filled chip; on a full one single precision gains from its eight
// waves per SIMD (two to four with a thread per particle), which it needs to
// issue two instructions at a time, and double precision, which issues one
// at a time anyway, pays for the idle lane and the exchange.  A round of
// lanes costs 0.29-0.31 of a round of threads in single precision and 0.337
// in double.  A launch of a few steps is bound by HBM instead, where the
// lanes' rows of 21 particles are read less well (1M particles, one step,
// FP32: 38 -> 56 us); the steps win that back from the sixth on (65,536
// particles or fewer: the second).
bool lane_per_neuron(const RK4Launch& L) {
    // two particles per thread are what the caller's tuning asks for
    if (L.ppt > 1 || L.reset || L.record || L.n > (int64_t)1 << 30) return false;
    if (L.steps < (L.n <= 65536 ? 2 : 8)) return false;
    const int64_t threads = (L.n + 65535) / 65536, lanes = (L.n + 21503) / 21504;
    return (double)lanes * (L.prec == FF_FP64 ? 0.337 : 0.31) < (double)threads;
}

}  // namespace

// Three neurons: a lane per neuron (ff_ring.h).  The reset rule and recording
// treat a particle as a whole and keep one thread per particle, as do tunings
// of two particles per thread and ensembles whose lanes would pass the launch
// limit of 2^32 threads.
hipError_t launch_rk4_hh(int neurons, const RK4Launch& L) {
    switch (neurons) {
        case 1: return dispatch_rk4<HH1, 2>(L);
        case 3:
            if (!lane_per_neuron(L)) return dispatch_rk4<HH3, 2>(L);
            switch (L.prec) {
                case FF_FP64: return launch_ring3<double, false>(L);
                case FF_FP32: return launch_ring3<float, false>(L);
                case FF_FP32_KAHAN: return launch_ring3<float, true>(L);
            }
    }
    return hipErrorInvalidValue;
}

}  // namespace ff

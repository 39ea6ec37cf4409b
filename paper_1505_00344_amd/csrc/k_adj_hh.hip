// Discrete-adjoint instantiations: Hodgkin-Huxley rings.  No register tape
// (every state of a segment is a sub-checkpoint in HBM: 5 doubles per neuron
// and step next to ~4 RK4 steps of exp-heavy arithmetic).
#include "ff_adjoint.h"
#include "ff_ring.h"

namespace ff {

template <typename R> using HH1 = HHRing<R, 1>;

// One neuron in double precision: two waves per SIMD (256 VGPRs, a few
// spilled) take 76.6 ms for 4M particles x 200 steps, one wave 82.3; below
// about 65,536 particles, where there is one wave anyway, 4 % more.
template <> struct AdjMinBlocks<HHRing<double, 1>> {
    static constexpr int value = 2;
};

namespace {

// Three neurons: a lane per neuron (ff_ring.h) at every size.  VALU issue
// bounds it, with 240 VGPRs in single precision (two waves per SIMD) and more
// than 256 in double (one).  200 steps, K = 50, one thread per particle -> a
// lane per neuron -> psi' shared, loads ahead and the parameter adjoints that are
// wanted: 20,011 particles FP64 4.34 -> 1.20 -> 1.01 ms, FP32-Kahan 1.84 ->
// 0.57 -> 0.49; 524,288 particles FP64 35.6 -> 30.7 -> 25.5 ms, FP32-Kahan 12.4
// -> 10.1 -> 8.1.  Parking the stage points in LDS (LOWREG), which one thread
// per particle needs, and caps at 256, 168 and 128 VGPRs (spills) are slower:
// 10.1-11.2 ms in single precision, 32-54 in double.
template <typename R, bool KAHAN>
hipError_t launch_ring3_adj(const AdjLaunch& A) {
    const int per = ring_per_block<3>(kAdjBlock);
    const int64_t grid = (A.f.n + per - 1) / per;
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_adj<RingLane<R, 3>, R, KAHAN, 1, false, false, RingMap<3>>), dim3((unsigned)grid),
                       dim3(kAdjBlock), 0, A.f.stream, make_adj_args(A));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_adj_hh(int neurons, const AdjLaunch& A) {
    switch (neurons) {
        case 1: return dispatch_adj<HH1, 1, true>(A);
        case 3:
            switch (A.f.prec) {
                case FF_FP64: return launch_ring3_adj<double, false>(A);
                case FF_FP32: return launch_ring3_adj<float, false>(A);
                case FF_FP32_KAHAN: return launch_ring3_adj<float, true>(A);
            }
    }
    return hipErrorInvalidValue;
}

}  // namespace ff

// ff_ring.h — the Hodgkin-Huxley ring with one neuron per lane.
//
// A particle of an N-neuron ring (N = 3: 15 state variables) occupies N
// neighbouring lanes of a wavefront, lane j of them holding neuron j's
// [V, m, h, n, s]; a wavefront carries 64 / N particles (21 for N = 3, one
// lane idle).  The neurons meet only in the synapse (neuron j reads the s of
// neuron (j + N - 1) % N), one ds_bpermute per right-hand side.  Each neuron
// runs the operations of HHRing in their order (hh_neuron), so the results
// are those of one thread per particle bit for bit.
//
// What bounds it: VALU issue.  One thread per particle holds 240 VGPRs (two
// waves per SIMD, too few to pair single-precision instructions), and an
// ensemble needs 65,536 particles to give every SIMD one wave; a lane per
// neuron needs a third of the registers and of the particles.
#pragma once
#include "ff_kernel.h"
#include "ff_rhs.h"

namespace ff {

template <int N> struct RingWave {
    static constexpr int kPerWave = 64 / N;  // particles per wavefront
    int slot, j, prev, next;                 // particle in the wave, neuron, byte addresses of the ring neighbours
    __device__ __forceinline__ RingWave() {
        const int lane = threadIdx.x & 63;
        slot = lane / N;
        j = lane - N * slot;
        // a lane beyond the last whole particle addresses a lane of the next
        // wave's numbering; ds_bpermute takes the address modulo the wave
        prev = 4 * (j == 0 ? lane + N - 1 : lane - 1);
        next = 4 * (j == N - 1 ? lane - N + 1 : lane + 1);
    }
    __device__ __forceinline__ bool whole() const { return slot < kPerWave; }
};

__device__ __forceinline__ float lane_read(int addr, float v) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}
__device__ __forceinline__ double lane_read(int addr, double v) {
    const int lo = __builtin_amdgcn_ds_bpermute(addr, __double2loint(v));
    const int hi = __builtin_amdgcn_ds_bpermute(addr, __double2hiint(v));
    return __hiloint2double(hi, lo);
}

// The system one lane integrates: one neuron of the ring.
template <typename R, int N> struct RingLane {
    static constexpr int D = 5, NP = 14, NQ = 1, UNROLL = 1, FUSED_INC = M<R>::kFast;
    static __device__ __forceinline__ void derive(const R (&p)[NP], R (&q)[NQ]) { HHRing<R, N>::derive(p, q); }
    static __device__ __forceinline__ void f(const R (&p)[NP], const R (&q)[NQ], const R (&x)[D], R (&o)[D]) {
        hh_neuron<R>(p, q[0], M<R>::rcp_(p[6]), x, lane_read(RingWave<N>().prev, x[4]), o);
    }
    static __device__ __forceinline__ void vjp(const R (&p)[NP], const R (&q)[NQ], const R (&x)[D], const R (&a)[D],
                                               uint32_t need, R (&gx)[D], R (&gp)[NP]) {
        const RingWave<N> w;
        const R gpre = hh_neuron_vjp<R>(p, q[0], M<R>::rcp_(p[6]), x, lane_read(w.prev, x[4]), a, need, gx,
                                        gp);
        gx[4] += lane_read(w.next, gpre);
    }
};

// Particles a block of `block` threads advances.
template <int N> __host__ __device__ constexpr int ring_per_block(int block) { return block / 64 * (64 / N); }

// Advance ring_per_block(blockDim) particles starting at `first`; the
// counterpart of rk4_tile.  Lanes without a particle of their own shadow the
// last one, all neurons of it, so that every lane reads live neighbours.
template <typename R, int N, bool KAHAN>
__device__ __forceinline__ void ring_tile(const RK4Args& a, int64_t first) {
    using S = RingLane<R, N>;
    const RingWave<N> w;
    const int64_t i0 = first + (int64_t)(threadIdx.x >> 6) * RingWave<N>::kPerWave + w.slot;
    const bool act = w.whole() && i0 < a.n;
    const int64_t i = act ? i0 : a.n - 1;
    R* st = static_cast<R*>(a.state);
    R* cp = static_cast<R*>(a.comp);
    R p[S::NP], q[S::NQ], x[5], c[5];
    load_params<S, R>(a, i, p);
    S::derive(p, q);
#pragma unroll
    for (int d = 0; d < 5; ++d) {
        x[d] = st[(5 * w.j + d) * a.ld + i];
        c[d] = KAHAN ? cp[(5 * w.j + d) * a.ld + i] : R(0);
    }
    if (a.ckpt && act) {  // checkpointed forward: keep the starting state of this launch
        R* ck = static_cast<R*>(a.ckpt);
        R* ckc = static_cast<R*>(a.ckpt_c);
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            ck[(5 * w.j + d) * a.ckpt_ld + i] = x[d];
            if (KAHAN) ckc[(5 * w.j + d) * a.ckpt_ld + i] = c[d];
        }
    }
    const R h = R(a.h), h2 = R(a.h2), h6 = R(a.h6);
#pragma unroll 1
    for (int64_t s = 0; s < a.steps; ++s) rk4_step<S, R, KAHAN>(p, q, x, c, h, h2, h6);
#pragma unroll
    for (int d = 0; d < 5; ++d) {
        if (!act) continue;
        st[(5 * w.j + d) * a.ld + i] = x[d];
        if (KAHAN) cp[(5 * w.j + d) * a.ld + i] = c[d];
    }
}

// The adjoint kernel's view of the same split (ThreadMap is its counterpart
// for one thread per particle).
template <int N> struct RingMap {
    static constexpr int DT = 5 * N;
    RingWave<N> w;
    int64_t i;
    bool act;
    __device__ __forceinline__ explicit RingMap(int64_t n) {
        const int64_t i0 = (int64_t)blockIdx.x * ring_per_block<N>(blockDim.x) +
                           (int64_t)(threadIdx.x >> 6) * RingWave<N>::kPerWave + w.slot;
        act = w.whole() && i0 < n;
        i = act ? i0 : n - 1;
    }
    __device__ __forceinline__ int row(int d) const { return 5 * w.j + d; }
    // neuron 0's, then 1's, ... in every lane of the particle
    template <typename R> __device__ __forceinline__ R total(R v) const {
        const int first = 4 * ((threadIdx.x & 63) - w.j);
        R s = lane_read(first, v);
#pragma unroll
        for (int k = 1; k < N; ++k) s = s + lane_read(first + 4 * k, v);
        return s;
    }
    __device__ __forceinline__ bool leader() const { return act && w.j == 0; }
};

}  // namespace ff

"""Who writes what in the adjoint kernel, on the CPU: the kernel's own text
(ff_adjoint_kernel.h) is compiled for the host and run one thread at a time.

The sub-checkpoint slots are used again by every checkpoint segment and the
waves of a block are not synchronised, so a slot, an entry of lambda or of mu
may be stored by one thread only: the one whose particle it is.  Threads past
the last particle shadow it; they may store nothing, whatever they read."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_1505_00344_amd", "csrc")

MATH = r"""
#pragma once
#include <cmath>
#include <cstdint>
#define __device__
#define __global__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
struct Dim { unsigned x; };
static Dim threadIdx, blockIdx, blockDim;
static inline double __shfl_xor(double v, int, int) { return v; }
static inline uint64_t __ballot(bool b) { return b; }
static inline void __syncthreads() {}
namespace ff {
template <typename R> struct M {
    static constexpr bool kFast = false;
    static R fma_(R a, R b, R c) { return std::fma(a, b, c); }
};
}
"""
RNG = r"""
#pragma once
#include <cstdint>
namespace ff { inline uint32_t draw_word(uint64_t, uint64_t, uint32_t, int) { return 0; } }
"""
SRC = r"""
#include "ff_math.h"
#include "ff_adjoint_kernel.h"
using namespace ff;
struct Decay {  // x0' = -p x0, x1' = x0 - x1
    static constexpr int D = 2, NP = 1, NQ = 1, UNROLL = 1, FUSED_INC = 0;
    static void derive(const double (&)[1], double (&q)[1]) { q[0] = 0; }
    static void f(const double (&p)[1], const double (&)[1], const double (&x)[2], double (&o)[2]) {
        o[0] = -p[0] * x[0];
        o[1] = x[0] - x[1];
    }
    static void vjp(const double (&p)[1], const double (&)[1], const double (&x)[2], const double (&a)[2], uint32_t,
                    double (&gx)[2], double (&gp)[1]) {
        gx[0] += a[1] - p[0] * a[0];
        gx[1] -= a[1];
        gp[0] -= x[0] * a[0];
    }
};
template <int T, bool LOWREG, bool CAPTURE> static void thread(unsigned b, unsigned t, const AdjArgs& a) {
    blockDim.x = kAdjBlock;
    blockIdx.x = b;
    threadIdx.x = t;
    k_adj<Decay, double, true, T, LOWREG, CAPTURE>(a);
}
extern "C" int block_size() { return kAdjBlock; }
extern "C" void run_thread(int variant, unsigned b, unsigned t, int64_t n, int64_t nsteps, int64_t K, double h,
                           const double* pp, const double* ckpt, const double* ckpt_c, double* sub, double* sub_c,
                           double* lam, double* mu) {
    AdjArgs a{};
    a.pp = pp;
    a.n = a.ld = n;
    a.n_pp = 1;
    a.h = h;
    a.h2 = h * 0.5;
    a.h6 = h / 6;
    a.h3 = h / 3;
    a.ckpt = ckpt;
    a.ckpt_c = ckpt_c;
    a.sub = sub;
    a.sub_c = sub_c;
    a.lam = lam;
    a.mu = mu;
    a.nsteps = nsteps;
    a.K = K;
    a.need = 1;
    switch (variant) {
        case 0: return thread<1, false, false>(b, t, a);
        case 1: return thread<1, true, false>(b, t, a);
        case 2: return thread<4, false, false>(b, t, a);
        case 3: return thread<4, false, true>(b, t, a);
    }
}
"""
TAPE = [1, 1, 4, 4]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("adjoint_host")
    for name in ("ff_kernel.h", "ff_adjoint_kernel.h"):
        shutil.copy(os.path.join(CSRC, name), d)
    (d / "ff_math.h").write_text(MATH)
    (d / "ff_rng.h").write_text(RNG)
    (d / "host.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-w", "-shared", "-fPIC", "-D__HIPCC_RTC__",
                    "host.cpp", "-o", "host.so"], cwd=d, check=True)
    return ctypes.CDLL(str(d / "host.so"))


@pytest.mark.parametrize("variant", range(4))
@pytest.mark.parametrize("n", [1, 65, 257, 300])
def test_only_the_owner_stores(lib, variant, n):
    nsteps, K, block = 14, 6, lib.block_size()
    rng = np.random.default_rng(n)
    nseg, nsub = -(-nsteps // K), -(-K // TAPE[variant])
    pp, ckpt = rng.uniform(1, 2, (1, n)), rng.normal(size=(nseg, 2, n))
    ckpt_c, lam0 = np.zeros_like(ckpt), rng.normal(size=(2, n))
    untouched = -123.25
    lam, mu = lam0.copy(), np.full((1, n), untouched)
    sub, subc = np.full((2, nsub, 2, n), untouched)

    def ptr(a):
        return a.ctypes.data_as(ctypes.c_void_p)

    def run(t):
        lib.run_thread(variant, t // block, t % block, ctypes.c_int64(n), ctypes.c_int64(nsteps), ctypes.c_int64(K),
                       ctypes.c_double(0.01), ptr(pp), ptr(ckpt), ptr(ckpt_c), ptr(sub), ptr(subc), ptr(lam), ptr(mu))

    for t in range(n):
        for a in (sub, subc):
            a[:] = untouched
        run(t)
        own = np.arange(n) == t
        assert np.all(sub[:, :, own] != untouched)
        for a in (sub, subc):
            assert np.all(a[:, :, ~own] == untouched), t
    assert np.all(lam != lam0) and np.all(mu != untouched)
    before = lam.copy(), mu.copy()
    for a in (sub, subc):
        a[:] = untouched
    for t in range(n, -(-n // block) * block):  # the shadows of the last block
        run(t)
        for a in (sub, subc):
            assert np.all(a == untouched), t
    assert np.array_equal(lam, before[0]) and np.array_equal(mu, before[1])

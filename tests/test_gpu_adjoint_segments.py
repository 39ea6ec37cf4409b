"""The one-launch adjoint over many checkpoint segments, with last blocks that
hold whole waves without particles: gradients of K = nsteps (one segment),
K = 1 and K = 7 (hundreds of them) are the same bits, the last particle's too."""
import numpy as np
import pytest

from helpers import api, to_dev, to_host
from paper_1505_00344_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIX = ["x1 - x0", "x0*x2 - p0*x1", "sin(x3) - x2", "x4 - p1*x3", "tanh(x5) - x4", "x0 - x5"]


def system(A, name):
    """The system, its initial state per component and a per-particle parameter's slot and value."""
    if name == "lorenz":
        return A.System(name, 3, I.LORENZ_PARAMS), [1.0, 2.0, 20.0], 1, 28.0
    if name == "wilson_cowan":
        return A.System(name, 2, I.WC_PARAMS), [0.4, 0.3], 8, 1.0
    if name == "linear":
        return A.System(name, 1, [-0.3]), [1.0], 0, -0.4
    if name == "hh1":
        return A.System("hh_ring", 5, I.HH_PARAMS), [-60.0, 0.1, 0.5, 0.4, 0.2], 7, 9.0
    if name == "expr3":
        return A.System.from_exprs(["exp(-x0)", "x0 - p0*x1", "x1*x0 - x2"], [0.7]), [0.1, 0.2, 0.3], 0, 0.7
    return A.System.from_exprs(SIX, [0.5, 0.8]), [0.1, 0.2, 0.3, 0.4, 0.5, 0.6], 1, 0.8


def gradients(A, sys_, x0, pp0, slot, lamT, steps, K, kahan):
    dtype = torch.float32 if kahan else torch.float64
    x, pp, lam = to_dev(x0, dtype), to_dev(pp0, dtype), to_dev(lamT, dtype)
    kw = dict(pparams=pp, pp_slot=[slot], prec="fp32_kahan" if kahan else "fp64")
    comp = torch.zeros_like(x) if kahan else None
    ws = torch.empty(A.adjoint_workspace_size(sys_, x, steps, K, comp=comp, **kw), dtype=torch.uint8, device="cuda:0")
    A.integrate_checkpointed(sys_, x, 0.003, steps, K, ws, comp=comp, **kw)
    mu = torch.empty_like(pp)
    mug = torch.empty(sys_.n_params, dtype=torch.float64, device="cuda:0")
    A.adjoint(sys_, x, 0.003, steps, K, ws, lam, mu=mu, mu_global=mug, **kw)
    torch.cuda.synchronize()
    return [to_host(v) for v in (lam, mu, mug)]


@pytest.mark.parametrize("kahan", [False, True])
@pytest.mark.parametrize("name", ["lorenz", "wilson_cowan", "linear", "hh1", "expr3", "expr6"])
def test_bitwise_independent_of_K_with_empty_waves(name, kahan):
    A = api()
    sys_, x1, slot, p1 = system(A, name)
    for n in (1, 64, 65, 257, 300, 256 * 128 + 1):
        rng = np.random.default_rng(n)
        x0 = np.array(x1)[:, None] * rng.uniform(0.9, 1.1, (len(x1), n))
        pp0, lamT = p1 * rng.uniform(0.9, 1.1, (1, n)), rng.normal(size=x0.shape)
        one, *rest = [gradients(A, sys_, x0, pp0, slot, lamT, 301, K, kahan) for K in (301, 1, 7, 301, 1, 7)]
        assert all(np.all(np.isfinite(v)) for v in one)
        for other in rest:
            for a, b in zip(one, other):
                assert np.array_equal(a, b), n

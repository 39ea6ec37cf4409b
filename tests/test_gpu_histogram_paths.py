"""Every route of the density projection at its edges, against the oracle:
direct atomics (up to 8192 particles), one LDS grid (up to 16384 bins), and
the two passes over tiles (32, 64 and 128 bins a side, runs of 16384 for
degenerate shapes; 1024, 4096 and 16384 particles per block; tiles that hold
most of the ensemble)."""
import ctypes

import numpy as np
import pytest

from helpers import api, to_dev, to_host
from paper_1505_00344_amd import _ffi
from paper_1505_00344_amd import inputs as I

torch = pytest.importorskip("torch")

GRIDS = [(128, 128), (129, 128), (512, 511), (1024, 1024), (1025, 1030), (2100, 2000), (5000, 3000), (33, 4097),
         (1, 70001), (70001, 1), (3, 2000003)]


def ensemble(kind, n):
    rng = np.random.default_rng(n)
    x = rng.uniform(-0.05, 1.05, (3, n))
    if kind == "one_bin":
        x[:2] = 0.51
    elif kind == "two_bins":
        x[:2] = np.where(np.arange(n) % 2, 0.25, 0.75)
    elif kind == "line":
        x[1] = 0.3
    elif kind == "mostly_one":
        x[:2, rng.uniform(size=n) < 0.9] = 0.123
    x[0, ::97] = np.nan
    return x


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 8192, 8193, 262144, 262145, 1048577])
@pytest.mark.parametrize("kind", ["uniform", "one_bin", "two_bins", "line", "mostly_one"])
def test_every_route_is_exact(ora, n, kind):
    A = api()
    sys_ = A.System("lorenz", 3, I.LORENZ_PARAMS)
    x = ensemble(kind, n)
    grids = GRIDS if n < 300000 else GRIDS[1:7:2]
    for nx, ny in grids:
        st = to_dev(x, torch.float64)
        # a workspace at an odd address, and a grid that is added to
        ws = torch.empty(A.histogram_workspace_size(n, nx, ny) + 4, dtype=torch.uint8, device="cuda:0")[4:]
        want, wd = ora.histogram(x, 0, 1, (0.0, 1.0), (0.0, 1.0), nx, ny)
        h, d = A.project_histogram(sys_, st, 0, 1, (0.0, 1.0), (0.0, 1.0), nx, ny, workspace=ws)
        assert np.array_equal(to_host(h).view(np.uint32), want), (nx, ny)
        assert int(d.item()) == wd
        A.project_histogram(sys_, st, 0, 1, (0.0, 1.0), (0.0, 1.0), nx, ny, hist=h, n_dropped=d, accumulate=True,
                            workspace=ws)
        assert np.array_equal(to_host(h).view(np.uint32), 2 * want), (nx, ny)
        assert int(d.item()) == 2 * wd


@pytest.mark.gpu
def test_few_particles_clear_a_large_grid(ora):
    """More of the grid than the particles' blocks clear, held by something else before."""
    A = api()
    x = ensemble("uniform", 8193)
    want, _ = ora.histogram(x, 0, 1, (0.0, 1.0), (0.0, 1.0), 5000, 3000)
    h = torch.full((3000, 5000), -1, dtype=torch.int32, device="cuda:0")
    A.project_histogram(A.System("lorenz", 3, I.LORENZ_PARAMS), to_dev(x, torch.float64), 0, 1, (0.0, 1.0),
                        (0.0, 1.0), 5000, 3000, hist=h)
    assert np.array_equal(to_host(h).view(np.uint32), want)


def test_workspace_size_is_unchanged():
    """6 bytes per particle, 4 per 16384-bin tile and 4096 particles, and the
    tile totals: callers may have sized their workspaces with it."""
    L = _ffi.lib()
    al = lambda v: (v + 255) // 256 * 256  # noqa: E731
    out = ctypes.c_size_t()
    for n in (0, 1, 8193, 262145, 5_000_000):
        for nx, ny in GRIDS:
            assert L.ff_histogram_workspace_size(n, nx, ny, ctypes.byref(out)) == 0
            nt, nb = -(-nx * ny // 16384), -(-n // 4096)
            want = al(4 * n) + al(2 * n) + al(4 * nt * nb) + al(4 * nt) + 2 * al(4 * (nt + 1))
            assert out.value == (want if nx * ny > 16384 else 0), (n, nx, ny)

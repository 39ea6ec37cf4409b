"""Calls that overlap on two streams, each with its own workspace, may add to
one grid, one image and one counter: every route's adds are atomic."""
import numpy as np
import pytest

from helpers import api, to_dev, to_host
from paper_1505_00344_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MVP = np.diag([1.0, 1.0, 1.0, 1.0])
CALLS = 24


def overlapping(shape, add, workspace):
    """(target, count) after CALLS calls on each of two streams into one pair, and after the same calls in a row."""
    out = []
    for streams in ([torch.cuda.Stream(), torch.cuda.Stream()], [torch.cuda.current_stream()] * 2):
        target = torch.zeros(shape, dtype=torch.int32, device="cuda:0")
        count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
        ws = [torch.empty(max(workspace, 1), dtype=torch.uint8, device="cuda:0") for _ in streams]
        torch.cuda.synchronize()
        for _ in range(CALLS):
            for k, s in enumerate(streams):
                add(k, target, count, ws[k], s)
        torch.cuda.synchronize()
        out.append((to_host(target), int(count.item())))
    return out


def particles(n):
    rng = np.random.default_rng(n)
    return [to_dev(rng.uniform(-1.1, 1.1, (3, n)), torch.float32) for _ in range(2)]


@pytest.mark.parametrize("n,nx,ny", [(5000, 512, 512), (200003, 100, 100), (200003, 512, 512), (200003, 3000, 2000)])
def test_grid(n, nx, ny):
    A = api()
    sys_ = A.System("lorenz", 3, I.LORENZ_PARAMS)
    x = particles(n)

    def add(k, h, d, ws, s):
        A.project_histogram(sys_, x[k], 0, 1, (-1.0, 1.0), (-1.0, 1.0), nx, ny, hist=h, n_dropped=d, accumulate=True,
                            workspace=ws, stream=s)

    (a, ad), (b, bd) = overlapping((ny, nx), add, A.histogram_workspace_size(n, nx, ny))
    assert np.array_equal(a, b) and ad == bd
    assert int(a.sum()) + ad == 2 * CALLS * n


@pytest.mark.parametrize("n,radius,weight", [(5000, 0, 0.1), (200003, 0, 0.1), (200003, 0, 1.0), (200003, 0, 600.0),
                                             (20011, 2, 0.3), (3000, 9, 0.3)])
def test_image(n, radius, weight):
    A = api()
    sys_ = A.System("lorenz", 3, I.LORENZ_PARAMS)
    x = particles(n)
    w, h = 333, 201

    def add(k, img, cu, ws, s):
        A.render_image(sys_, x[k], (0, 1, 2), MVP, w, h, base=(0.2, 0.5, 1.0), weight=weight, radius=radius, img=img,
                       n_culled=cu, accumulate=True, workspace=ws, stream=s)

    (a, ac), (b, bc) = overlapping((h, w, 3), add, A.render_workspace_size(n, w, h, radius))
    assert np.array_equal(a, b) and ac == bc and a.any()

"""A tuning's particles per thread select the kernel of the three-neuron ring:
a lane per neuron (ring_tile) belongs to one particle per thread only."""
import pytest

from helpers import api
from paper_1505_00344_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
profiler = pytest.importorskip("torch.profiler")


def kernels(run):
    run()
    torch.cuda.synchronize()
    with profiler.profile(activities=[profiler.ProfilerActivity.CUDA, profiler.ProfilerActivity.CPU]) as p:
        run()
        torch.cuda.synchronize()
    return [e.name for e in p.events() if "ff::" in e.name]


@pytest.mark.parametrize("ppt,kernel", [(1, "k_ring<float, 3, false>"), (2, "float, false, 2>"),
                                        (4, "float, false, 2>")])  # rings are limited to two per thread
def test_integrate(ppt, kernel):
    A = api()
    x = torch.rand((15, 500), dtype=torch.float32, device="cuda:0")
    sys_ = A.System("hh_ring", 15, I.HH_PARAMS)
    got = kernels(lambda: A.integrate(sys_, x, 0.01, 20, tuning=(20, ppt, 256)))
    assert len(got) == 1 and kernel in got[0], got


@pytest.mark.parametrize("ppt,lanes", [(1, "true"), (2, "false"), (4, "false")])
def test_groups(ppt, lanes):
    A = api()
    x = torch.rand((15, 500), dtype=torch.float32, device="cuda:0")
    sys_ = A.System("hh_ring", 15, I.HH_PARAMS)
    g = A.make_groups([(sys_, A.make_batch(x, None, None, (), None, "fp32", 0), 0.01)])
    ws = torch.empty(A.groups_workspace_size(1), dtype=torch.uint8, device="cuda:0")
    got = kernels(lambda: A.integrate_groups(g, 20, tuning=(20, ppt, 256), workspace=ws))
    assert any(f"k_groups<float, false, {ppt}, {lanes}>" in k for k in got), got


@pytest.mark.parametrize("prec,rings,others,steps,lanes", [
    ("fp32_kahan", 43008, 0, 8, True), ("fp32_kahan", 43008, 0, 7, False),  # two whole rounds of lanes
    ("fp32_kahan", 43009, 0, 31, False), ("fp32_kahan", 43009, 0, 32, True),
    ("fp32_kahan", 64512, 0, 32, True), ("fp32_kahan", 64513, 0, 32, False),  # three rounds of lanes, four
    ("fp32", 65536, 0, 32, False), ("fp32", 65536, 1, 32, True),  # one round of threads, two
    ("fp32_kahan", 131072, 1, 32, False), ("fp32", 131072, 1, 32, True),
    ("fp32", 5000, 262144, 8, True), ("fp32", 5000, 262145, 31, False), ("fp32", 5000, 262145, 32, True),
    ("fp64", 43009, 0, 32, False), ("fp64", 200000, 0, 32, True), ("fp64", 262144, 0, 32, False),
    ("fp64", 5000, 1966079, 8, True), ("fp64", 5000, 1966080, 8, False)])
def test_rings_of_a_batch_take_lanes_where_their_rounds_cost_less(prec, rings, others, steps, lanes):
    A = api()
    dtype = torch.float64 if prec == "fp64" else torch.float32
    r, t = ("double", "false") if prec == "fp64" else ("float", "true" if prec == "fp32_kahan" else "false")
    specs = []
    for name, dim, params, n in (("hh_ring", 15, I.HH_PARAMS, rings), ("lorenz", 3, I.LORENZ_PARAMS, others)):
        x = torch.zeros((dim, n), dtype=dtype, device="cuda:0")
        comp = torch.zeros_like(x) if prec == "fp32_kahan" else None
        specs.append((A.System(name, dim, params), A.make_batch(x, None, None, (), comp, prec, 0), 0.01))
    g = A.make_groups(specs)
    ws = torch.empty(A.groups_workspace_size(2), dtype=torch.uint8, device="cuda:0")
    got = kernels(lambda: A.integrate_groups(g, steps, workspace=ws))
    want = f"k_groups<{r}, {t}, 1, {'true' if lanes else 'false'}>"
    assert any(want in k for k in got), (want, got)

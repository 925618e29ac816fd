"""Landscape scans larger than one launch of a sphere-sum kernel can be: more instances times gammas
than 2^32 threads, and ground states spread over several launches."""
import sys

import numpy as np
import pytest

from paper_2104_03293_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2104_03293_amd import sv as m

    return m


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu] {request.node.nodeid}", flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("count,ng", [(17000, 1024), (4200, 16384)])  # 256 threads for each of 2^24 (instance, gamma[s])
def test_scan_of_more_points_than_one_launch(sv, count, ng):
    """The same two instances over and over: every copy has the values of a scan of the two alone."""
    two = [sv.Ising.from_instance(I.ring(4)), sv.Ising.from_instance(I.degree4_int2(5, 1))]
    g, b = np.linspace(-3.0, 3.0, ng), np.array([0.7])
    e0, p0 = sv.batch_p1_scan(two, g, b, dtype="c64")
    e, p = sv.batch_p1_scan([two[k & 1] for k in range(count)], g, b, dtype="c64")
    for k in range(2):
        assert np.array_equal(e[k::2], np.broadcast_to(e0[k], e[k::2].shape))
        assert np.array_equal(p[k::2], np.broadcast_to(p0[k], p[k::2].shape))


def one_field(n):
    """One field: half of all states are ground states."""
    h = np.zeros(n)
    h[3] = 1.0
    return I.make_instance(n, np.zeros((0, 2)), h, np.zeros(0))


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("ng", [1024, 1100])
def test_ground_states_over_several_launches(sv, ng, dtype):
    """Sphere sums of 1024 gammas fit a launch for 204 ground states: the 512 of an instance are spread
    over several, and launches end inside instances and between them."""
    assert (64 << 20) // (1024 * 20 * 16) == 204
    insts = [one_field(10), I.ring(10), one_field(10), I.regular3_pm1(10, 5), I.fields_only(10, 3), one_field(9)]
    insts += [I.make_instance(8, np.array([[0, 1]]), np.zeros(8), np.ones(1))]  # 128 ground states
    Hs = [sv.Ising.from_instance(x) for x in insts]
    g, b = np.linspace(-3.0, 3.0, ng), np.array([0.4, -1.0])
    out = []
    for spheres in (1, 0):
        old = sv.tune_get("batchsphere")
        sv.tune_set("batchsphere", spheres)
        try:
            out.append(sv.batch_p1_scan(Hs, g, b, dtype=dtype))
        finally:
            sv.tune_set("batchsphere", old)
    tol = 1e-10 if dtype == "c128" else 1e-5  # the direct scan's amplitudes
    for x, y in zip(*out):
        assert np.max(np.abs(x - y)) <= tol

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

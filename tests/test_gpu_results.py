"""Results read from pinned memory as they arrive: never those of an earlier call, on any thread,
and NaN results come back as NaN."""
import threading

import numpy as np
import pytest

from paper_2104_03293_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sv():
    from paper_2104_03293_amd import sv as m

    return m


@pytest.mark.parametrize("dtype,n", [("c128", 14), ("c64", 16), ("c64", 20), ("c128", 22)])
def test_results_belong_to_their_call(sv, dtype, n):
    H = sv.Ising.from_instance(I.degree4_int2(n, n))
    angles = [I.uniform_params(1 + k % 3, k) for k in range(6)]
    s = sv.State(n, dtype)
    # the reference: the observables of the state each call leaves, from a program of its own
    want = []
    for g, b in angles:
        sv.qaoa_forward(s, H, g, b)
        want.append(sv.expect(s, H))
    tol = 1e-9 if dtype == "c128" else 2e-5
    bad = []

    def work():
        st = sv.State(n, dtype, owner="lib")
        for k in list(range(6)) * 5:
            e, p, nrm = sv.qaoa_energy(st, H, *angles[k])
            for x, y in zip((e, p, nrm), want[k]):
                if not abs(x - y) <= tol * max(1.0, abs(y)):
                    bad.append((k, x, y))
            if k == 3:
                ps, es, sz = sv.aqa_run_observe(st, H, *angles[k])
                if not abs(es[-1] - want[k][0]) <= tol * max(1.0, abs(want[k][0])):
                    bad.append(("observe", es[-1]))

    threads = [threading.Thread(target=work) for _ in range(2)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not bad


@pytest.mark.parametrize("n", [14, 20])
def test_nan_results(sv, n):
    H = sv.Ising.from_instance(I.degree4_int2(n, n))
    s = sv.State(n, "c128")
    a = np.full(1 << n, np.nan, dtype=np.complex128)
    a.view(np.uint64)[:] = 0x7FF8A1D25EC0DE01  # the payload that marks a result still to come
    s.from_numpy(a)
    assert all(np.isnan(x) for x in sv.expect(s, H)[:1])

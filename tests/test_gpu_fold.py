"""Eq. AQA4 steps whose last layer is unit-diagonal, its diagonal applied by the phase before it,
against the general form of every layer."""
import numpy as np
import pytest

from paper_2104_03293_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [1, 2, 5])
@pytest.mark.parametrize("dtype,n", [("c128", 5), ("c64", 13), ("c128", 15), ("c128", 22), ("c64", 23), ("c128", 24)])
@pytest.mark.parametrize("kind", ["int", "real"])
def test_folded_last_layer(dtype, n, steps, kind):
    from paper_2104_03293_amd import sv

    inst = I.degree4_int2(n, 7 + n) if kind == "int" else I.random_real(n, 2 * n, 9 + n)
    H = sv.Ising.from_instance(inst)
    rng = np.random.default_rng(n + steps)
    A, B = rng.uniform(0.2, 1.0, steps), rng.uniform(0.2, 1.0, steps)
    s = sv.State(n, dtype)
    old = sv.tune_get("genunit"), sv.tune_get("tile")
    out = []
    try:
        sv.tune_set("tile", 0)
        for unit in (1, 0):
            sv.tune_set("genunit", unit)
            sv.qsds_run(s, H, 0.7, A, B)
            psi = s.to_numpy()
            obs = sv.qsds_run(s, H, 0.7, A, B, observe=True)
            out.append([psi, *[np.asarray(o) for o in obs], s.to_numpy()])
    finally:
        sv.tune_set("genunit", old[0])
        sv.tune_set("tile", old[1])
    tol = 1e-11 if dtype == "c128" else 2e-5
    for x, y in zip(*out):
        assert np.max(np.abs(x - y)) <= tol * max(1.0, float(np.max(np.abs(y))))
    # the global phase too (summed in double precision: vdot of complex64 loses 2e-4 over 2^23 terms)
    assert abs(np.vdot(*[o[0].astype(np.complex128) for o in out]) - 1.0) <= tol

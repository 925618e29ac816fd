"""Landscape scan by sphere sums against the direct scan and the oracle: sizes from one qubit up,
uneven lists, half-integer grids, instances with more ground states than grid points, real-valued
ones among them, and grids of more gammas than one launch takes."""
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


def scan(sv, Hs, g, b, dtype, spheres):
    old = sv.tune_get("batchsphere")
    sv.tune_set("batchsphere", spheres)
    try:
        return sv.batch_p1_scan(Hs, g, b, dtype=dtype)
    finally:
        sv.tune_set("batchsphere", old)


def instances():
    out = [I.fields_only(1, 3), I.fields_only(2, 4), I.ring(3), I.ring(6, J=0.5, h=0.5)]
    out += [I.regular3_pm1(n, 70 + n) for n in (5, 9, 12, 14, 17)]
    out += [I.degree4_int2(n, 80 + n) for n in (7, 13, 16)]
    out.append(I.random_real(8, 14, 5))  # off the grid: direct scan
    out.append(I.make_instance(7, np.zeros((0, 2)), np.zeros(7), np.zeros(0)))  # every state is a ground state
    half = I.degree4_int2(10, 91)
    out.append(I.make_instance(10, np.stack([half["ei"], half["ej"]], 1), half["h"] * 0.25, half["J"] * 0.5))
    return out


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_sphere_scan_matches_oracle_and_direct_scan(sv, orc, dtype):
    insts = instances()
    Hs = [sv.Ising.from_instance(x) for x in insts]
    g = np.array([0.0, 0.3, -1.1, 2.9, 7.5])
    b = np.array([0.0, 0.2, np.pi / 4, -np.pi / 4, 1.4, np.pi / 2, -2.6, 9.0])
    e, p = scan(sv, Hs, g, b, dtype, 1)
    e0, p0 = scan(sv, Hs, g, b, dtype, 0)
    tol = 1e-6 if dtype == "c64" else 1e-11  # energy bar of the library / its double-precision amplitudes
    for k, inst in enumerate(insts):
        scale = max(1.0, orc.coeff_scale(inst))
        assert np.max(np.abs(e[k] - e0[k])) <= tol * scale, k
        assert np.max(np.abs(p[k] - p0[k])) <= tol, k
        if inst["n"] > 12:
            continue
        for i in range(len(g)):
            for j in range(len(b)):
                psi = orc.qaoa_state(inst, [g[i]], [b[j]])
                _, re, rp = orc.observables(inst, psi)
                assert abs(e[k, i, j] - re) <= tol * scale and abs(p[k, i, j] - rp) <= tol, (k, i, j)


def test_many_gammas_and_many_ground_states(sv):
    """More gammas than one launch takes, and ground states spread over several launches."""
    insts = [I.make_instance(10, I.regular3_edges(10, np.random.default_rng(1)), np.zeros(10), np.ones(15)),
             I.regular3_pm1(8, 5)]
    Hs = [sv.Ising.from_instance(x) for x in insts]
    g = np.linspace(-3.0, 3.0, 2100)
    b = np.array([0.4, -1.0])
    e, p = scan(sv, Hs, g, b, "c128", 1)
    e0, p0 = scan(sv, Hs, g, b, "c128", 0)
    assert np.max(np.abs(e - e0)) <= 1e-10 and np.max(np.abs(p - p0)) <= 1e-11

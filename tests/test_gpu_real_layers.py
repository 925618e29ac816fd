"""Real general single-qubit layers on small tiles (a kernel variant of their own, chosen launch by
launch) against the oracle: tile edges, lists with complex layers among the real ones, and more layers
than one launch holds."""
import sys

import numpy as np
import pytest

from paper_2104_03293_amd import inputs as I

pytestmark = pytest.mark.gpu
AMP_TOL = {"c128": 1e-11, "c64": 2e-5}  # parity bars of the whole library


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


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,layers,mixed",
                         [(n, k, m) for n in (1, 9, 10, 11, 13, 14, 17, 18) for k, m in ((1, False), (5, False), (6, True))] +
                         [(n, 110, m) for n in (1, 9, 10, 11, 13) for m in (False, True)])  # states of one tile
def test_real_and_mixed_layers(sv, orc, n, layers, mixed, dtype):
    rng = np.random.default_rng(1000 * n + layers)
    U = np.linalg.qr(rng.normal(size=(layers, n, 2, 2)))[0].astype(np.complex128)
    if mixed:  # every third layer complex, one matrix of another one
        U[::3] = np.linalg.qr(rng.normal(size=U[::3].shape) + 1j * rng.normal(size=U[::3].shape))[0]
        U[1, n // 2] *= 1j
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi /= np.linalg.norm(psi)
    s = sv.State(n, dtype)
    s.from_numpy(psi)
    sv.gate_layers(s, U)
    assert np.max(np.abs(s.to_numpy() - orc.gate_layers(n, psi, U))) <= AMP_TOL[dtype]


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("tile", [-1, 0])
@pytest.mark.parametrize("n,kind", [(15, "real"), (16, "int"), (22, "real")])
def test_real_layers_beside_phases(sv, orc, n, kind, tile, dtype):
    """Eq. AQA4 steps without fields have identity layers, real ones, beside the phases of couplings on
    and off the energy grid; with an x field in some steps, complex ones in other passes."""
    inst = I.random_real(n, 2 * n, n) if kind == "real" else I.degree4_int2(n, n)
    inst = I.make_instance(n, np.stack([inst["ei"], inst["ej"]], 1), np.zeros(n), inst["J"])
    H = sv.Ising.from_instance(inst)
    s = sv.State(n, dtype)
    old = sv.tune_get("tile")
    sv.tune_set("tile", tile)
    try:
        for A in ([0.0, 0.0, 0.0], [0.0, 0.9, 0.0], [0.7, 0.0, 0.0]):
            B = [0.3, 1.0, 0.6]
            sv.qsds_run(s, H, 0.8, A, B)
            psi = orc.qsds_run(inst, 0.8, A, B)
            assert np.max(np.abs(s.to_numpy() - psi)) <= AMP_TOL[dtype]
    finally:
        sv.tune_set("tile", old)

"""Deep circuits on small tiles: gradients whose reverse sweep runs in launches of many layers,
against the oracle."""
import sys

import numpy as np
import pytest

from paper_2104_03293_amd import inputs as I

pytestmark = pytest.mark.gpu
EPS = {"c128": 2.0 ** -53, "c64": 2.0 ** -24}


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


class knob:
    def __init__(self, sv, name, value):
        self.sv, self.name, self.value = sv, name, value

    def __enter__(self):
        self.old = self.sv.tune_get(self.name)
        self.sv.tune_set(self.name, self.value)

    def __exit__(self, *a):
        self.sv.tune_set(self.name, self.old)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("kind", ["deg4", "real"])
@pytest.mark.parametrize("p", [30, 60])
@pytest.mark.parametrize("n", [8, 10, 13])
def test_deep_gradients_of_one_tile_states(sv, orc, n, p, kind, dtype):
    """Mixer angles that leave cos(beta)^n per layer: uniform in [-pi, pi), constant 0.6 and pi/2 - 0.1,
    by both adjoint schemes, from |+> and from the forward state.

    Each of the 4 p n butterfly rounds adds a relative rounding of eps to the vectors, at random:
    2 eps sqrt(4 p n); a derivative is a form of at most n terms between psi and lambda,
    |lambda| <= sum|h| + sum|J|, which doubles it."""
    inst = I.degree4_int2(n, 5 * n) if kind == "deg4" else I.random_real(n, 2 * n, 5 * n)
    H = sv.Ising.from_instance(inst)
    rng = np.random.default_rng(100 * n + p)
    scale = orc.coeff_scale(inst)
    tol = 4.0 * n * scale * EPS[dtype] * np.sqrt(4.0 * p * n)
    psi, lam = sv.State(n, dtype), sv.State(n, dtype)
    for b in (rng.uniform(-np.pi, np.pi, p), np.full(p, 0.6), np.full(p, np.pi / 2 - 0.1)):
        g = rng.uniform(-1.0, 1.0, p)
        f, rg, rb = orc.grad_tangent(inst, g, b)
        for zeta in (-1, 0):
            with knob(sv, "adjzeta", zeta):
                for fwd in (False, True):
                    if fwd:
                        sv.qaoa_forward(psi, H, g, b)
                    e, dg, db = sv.grad(psi, lam, H, g, b, psi_is_forward=fwd)
                    assert abs(e - f) <= tol, (zeta, fwd, e, f)
                    assert np.max(np.abs(dg - rg)) <= tol and np.max(np.abs(db - rb)) <= tol, (zeta, fwd)

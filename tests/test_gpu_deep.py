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


RUN_TOL = {"c128": 1e-10, "c64": 2e-4}  # ten times the parity bars of amplitudes: thousands of layers


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [8, 14])
def test_runs_of_more_steps_than_the_small_tiles_take(sv, orc, n, dtype):
    """Annealing and Eq. AQA4 runs with more results than the small tiles' ops can name: accepted, and
    equal to the shorter run of the same steps at every step that both have."""
    inst = I.degree4_int2(n, n)
    H = sv.Ising.from_instance(inst)
    tol = RUN_TOL[dtype] * max(1.0, orc.coeff_scale(inst))
    s = sv.State(n, dtype)
    rng = np.random.default_rng(n)
    for steps, short, observe in ((3000, 1900, True), (11000, 10800, False)):
        g, b = rng.uniform(0.0, 0.5, steps), rng.uniform(-0.5, 0.5, steps)
        run = (lambda k: sv.aqa_run_observe(s, H, g[:k], b[:k])) if observe else (
            lambda k: sv.aqa_run(s, H, g[:k], b[:k], per_step=True))
        for x, y in zip(run(steps), run(short)):
            assert x.shape[0] == steps and np.max(np.abs(x[:short] - y)) <= tol
    g, b = rng.uniform(0.0, 1.0, 3000), rng.uniform(0.0, 1.0, 3000)
    for x, y in zip(sv.qsds_run(s, H, 0.3, g, b, observe=True), sv.qsds_run(s, H, 0.3, g[:1900], b[:1900], observe=True)):
        assert np.max(np.abs(x[:1900] - y)) <= tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n", [9, 14])
def test_gradients_of_more_layers_than_the_small_tiles_take(sv, orc, n, dtype):
    """A circuit followed by thousands of identity layers has the circuit's energy and derivatives."""
    inst = I.degree4_int2(n, n)
    H = sv.Ising.from_instance(inst)
    p = 16400 if n == 9 else 11000
    g, b = np.zeros(p), np.zeros(p)
    g[:3], b[:3] = I.uniform_params(3, n)
    f, rg, rb = orc.grad_tangent(inst, g[:3], b[:3])
    e, dg, db = sv.grad(sv.State(n, dtype), sv.State(n, dtype), H, g, b)
    tol = RUN_TOL[dtype] * max(1.0, orc.coeff_scale(inst))
    assert abs(e - f) <= tol
    assert np.max(np.abs(dg[:3] - rg)) <= tol and np.max(np.abs(db[:3] - rb)) <= tol

"""Small-tile programs (states of up to 21 qubits) against the oracle and against the large tiles:
the sizes at the edges of the tile rule (one partly filled tile, whole tiles of every width, two
groups with the shortest and longest second group), op lists longer than one launch holds, and
phase angles beyond the small tiles' range."""
import numpy as np
import pytest

from paper_2104_03293_amd import inputs as I

pytestmark = pytest.mark.gpu

AMP_TOL = {"c128": 1e-11, "c64": 2e-5}  # parity bars of the whole library
ENERGY_TOL = 1e-6
GRAD_TOL = {"c128": 1e-6, "c64": 5e-6}


@pytest.fixture(scope="module")
def sv():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from paper_2104_03293_amd import sv as m

    return m


class knob:
    def __init__(self, sv, name, value):
        self.sv, self.name, self.value = sv, name, value

    def __enter__(self):
        self.old = self.sv.tune_get(self.name)
        self.sv.tune_set(self.name, self.value)

    def __exit__(self, *a):
        self.sv.tune_set(self.name, self.old)


def instance(n, kind, seed):
    m = min(2 * n, n * (n - 1) // 2)
    if n == 1:
        return I.fields_only(1, seed)
    return I.random_real(n, m, seed) if kind == "real" else I.make_instance(
        n, I.gnm_edges(n, m, np.random.default_rng(seed)), np.random.default_rng(seed + 1).integers(-1, 2, n),
        np.random.default_rng(seed + 2).integers(-2, 3, m).astype(float))


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("kind", ["int", "real"])
@pytest.mark.parametrize("n", [1, 3, 9, 10, 11, 13, 14, 17, 18, 19, 21])
def test_energy_state_and_gradient(sv, orc, n, kind, dtype):
    inst = instance(n, kind, 40 + n)
    scale = orc.coeff_scale(inst)
    H = sv.Ising.from_instance(inst)
    g, b = I.uniform_params(3, n)  # angles beyond pi/4 take two mixer ops
    s, lam = sv.State(n, dtype), sv.State(n, dtype)
    e, p, nrm = sv.qaoa_energy(s, H, g, b)
    ref = orc.qaoa_state(inst, g, b)
    _, re, rp = orc.observables(inst, ref)
    assert np.max(np.abs(s.to_numpy() - ref)) <= AMP_TOL[dtype]
    assert abs(e - re) <= ENERGY_TOL * max(abs(re), scale)
    assert abs(p - rp) <= AMP_TOL[dtype] and abs(nrm - 1.0) <= AMP_TOL[dtype]
    assert np.max(np.abs(sv.spin_z(s) - orc.spin_z(n, ref))) <= 10 * AMP_TOL[dtype]
    f, rg, rb = orc.grad_tangent(inst, g, b)
    tol = GRAD_TOL[dtype] * max(scale, float(np.max(np.abs(np.concatenate([rg, rb])))))
    for fwd in (True, False):  # from the state just computed, then from |+>
        e2, dg, db = sv.grad(s, lam, H, g, b, psi_is_forward=fwd)
        assert abs(e2 - f) <= ENERGY_TOL * max(abs(f), scale)
        assert np.max(np.abs(dg - rg)) <= tol and np.max(np.abs(db - rb)) <= tol


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n,steps", [(8, 70), (13, 40), (18, 30)])
def test_long_programs_and_large_tiles_agree(sv, n, steps, dtype):
    """More ops than one launch holds (one-tile states), and many columns: observables, general
    layers and the gradient of deep circuits on small and on large tiles."""
    inst = instance(n, "int", 60 + n)
    H = sv.Ising.from_instance(inst)
    g, b = sv.schedule_linear(steps, 0.7)
    A, B = 1.0 - np.arange(steps) / steps, np.arange(steps) / steps
    s, lam = sv.State(n, dtype), sv.State(n, dtype)
    out = []
    for tile in (-1, 0):
        with knob(sv, "tile", tile):
            obs = sv.aqa_run_observe(s, H, g, b)
            psi = s.to_numpy()
            q = sv.qsds_run(s, H, 0.5, A, B, observe=True)
            grad = sv.grad(s, lam, H, g, b)
            out.append((*obs, psi, *q, np.array(grad[0]), grad[1], grad[2]))
    tol = (1e-11 if dtype == "c128" else 2e-5) * 10
    for x, y in zip(*out):
        assert np.max(np.abs(x - y)) <= tol * max(1.0, float(np.max(np.abs(y))))


@pytest.mark.parametrize("n", [12, 16])
def test_phase_angles_beyond_the_small_tiles(sv, orc, n):
    """|gamma| sum|J| past the range of the small tiles' phase factors takes the large tiles."""
    inst = instance(n, "int", 80 + n)
    H = sv.Ising.from_instance(inst)
    s = sv.State(n, "c128")
    for gam in (1.0e3, 1.0e6):
        sv.qaoa_forward(s, H, [gam], [0.4])
        assert np.max(np.abs(s.to_numpy() - orc.qaoa_state(inst, [gam], [0.4]))) <= 1e-9  # angle rounding: eps * 1e7


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("gam", [300.0, 4.0e4])
def test_real_couplings_on_the_large_tiles(sv, orc, gam, dtype):
    """Real-valued couplings on full large tiles, with phase angles inside and beyond the range of the
    in-place phase factors (beyond it the library's sincos kernels run)."""
    n = 22
    inst = I.random_real(n, 2 * n, 7)
    H = sv.Ising.from_instance(inst)
    s, lam = sv.State(n, dtype), sv.State(n, dtype)
    sv.qaoa_forward(s, H, [gam, 0.3], [0.4, -0.2])
    ref = orc.qaoa_state(inst, [gam, 0.3], [0.4, -0.2])
    # the angle itself is known to eps * gamma * sum(|h| + |J|); amplitudes are about 2^-11
    tol = AMP_TOL[dtype] + 2.0 ** -50 * gam * orc.coeff_scale(inst)
    assert np.max(np.abs(s.to_numpy() - ref)) <= tol


@pytest.mark.parametrize("dtype,n,total,q", [("c128", 5, 511, 1), ("c128", 5, 512, 1), ("c128", 12, 255.5, 2),
                                             ("c64", 12, 127.75, 4), ("c64", 14, 511, 1), ("c128", 16, 300, 1)])
def test_phase_table_edges(sv, dtype, n, total, q):
    """Grid-valued instances whose phase table is full, one entry too long, and on the finer grids."""
    rng = np.random.default_rng(n)
    inst = I.degree4_int2(n, n)
    h = np.array(inst["h"], dtype=float) / q
    J = np.array(inst["J"], dtype=float) / q
    h[0] = 0.0
    h[0] = total - np.abs(h).sum() - np.abs(J).sum()
    assert h[0] > 0
    ei, ej = np.array(inst["ei"]), np.array(inst["ej"])
    H = sv.Ising(n, h, ei, ej, J)
    z = np.arange(1 << n)
    sp = np.where((z[:, None] >> np.arange(n)) & 1, 1.0, -1.0)
    E = sp @ h + (sp[:, ei] * sp[:, ej]) @ J
    g, b = rng.uniform(0.1, 1.0, 3), rng.uniform(0.1, 1.0, 3)
    psi = np.full(1 << n, 2.0 ** (-n / 2), dtype=np.complex128)
    for gg, bb in zip(g, b):
        psi *= np.exp(-1j * gg * E)
        for i in range(n):
            v = psi.reshape(-1, 2, 1 << i)
            psi = (np.cos(bb) * v - 1j * np.sin(bb) * v[:, ::-1]).reshape(-1)
    s = sv.State(n, dtype)
    e, p, nrm = sv.qaoa_energy(s, H, g, b)
    tol = 1e-11 if dtype == "c128" else 2e-5
    want = float((np.abs(psi) ** 2 * E).sum())
    assert abs(e - want) <= tol * max(1.0, float(np.abs(E).max()))
    assert abs(nrm - 1.0) <= tol
    assert np.max(np.abs(s.to_numpy() - psi)) <= tol


@pytest.mark.parametrize("n", [20, 21])
def test_gradients_and_spins_up_to_and_above_256_tiles(sv, n):
    """Register budgets of the double-precision variants: one wave per SIMD up to 256 tiles, two above."""
    H = sv.Ising.from_instance(I.degree4_int2(n, n))
    g, b = I.uniform_params(2, n)
    s, lam = sv.State(n, "c128"), sv.State(n, "c128")
    out = []
    for tile in (-1, 0):
        with knob(sv, "tile", tile):
            gr = sv.grad(s, lam, H, g, b)
            out.append([gr[-2], gr[-1], *sv.aqa_run_observe(s, H, g, b), *sv.qsds_run(s, H, 0.5, g, b, observe=True)])
    for x, y in zip(*out):
        assert np.max(np.abs(np.asarray(x) - y)) <= 1e-11 * max(1.0, float(np.max(np.abs(y))))

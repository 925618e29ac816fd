"""Performance cases: the calls that a user of the engine makes, through the public binding.

Each case names an entry point ("kind"), a size (n qubits), an amplitude type and the options of the call:

  energy    one objective evaluation of a QAOA optimiser: (<H_C>, P_gs, norm) and the final state
  noalloc   the same for serving loops: results stay in a device array, nothing is allocated, no synchronisation
  grad      objective and adjoint gradient (one step of a gradient-based optimiser)
  forward   the QAOA state alone, then its observables as separate calls (expect, spin_z)
  aqa       coarse annealing with per-step <H_C> and P_gs; "observe" also records every <sigma^z_i> per step
  qsds      second-order time stepping of the annealing Hamiltonian (general single-qubit layers + cost phase)
  layers    layers of single-qubit gates (the Hadamard benchmark circuit, or arbitrary unitaries)
  batch     p = 1 landscape scan over many small instances of uneven n
  ground    a new instance and its brute-force ground state

Instances: "reg3" 3-regular +-1 couplings, "deg4" average degree 4 with integer couplings, "real" real-valued
couplings, "cover" dense half-integer exact-cover couplings.

Results computed from complex64 amplitudes are returned in single precision, the precision that they have.
"""
import math

import numpy as np
import torch

from paper_2104_03293_amd import inputs as I
from paper_2104_03293_amd import sv


def listed():
    return [
        # the smallest calls: one evaluation of a 14-qubit 3-regular instance (latency of a whole call) ...
        {"name": "energy_n14_c128_p1", "kind": "energy", "n": 14, "dtype": "c128", "p": 1, "inst": "reg3"},
        # ... and a serving loop over a 12-qubit one, enqueued without allocation or synchronisation
        {"name": "noalloc_n12_c64_p4", "kind": "noalloc", "n": 12, "dtype": "c64", "p": 4, "inst": "reg3"},
        # the inner loop of an optimiser at a size where it runs hundreds of calls; odd n
        {"name": "grad_n17_c128_p4", "kind": "grad", "n": 17, "dtype": "c128", "p": 4, "inst": "deg4"},
        # a deep circuit on an ordinary state in single precision
        {"name": "energy_n20_c64_p8", "kind": "energy", "n": 20, "dtype": "c64", "p": 8, "inst": "deg4"},
        # real-valued couplings: no phase tables
        {"name": "energy_n21_real_c128_p3", "kind": "energy", "n": 21, "dtype": "c128", "p": 3, "inst": "real"},
        # deep-circuit adjoint gradient in single precision (16 parameters)
        {"name": "grad_n30_c64_p8", "kind": "grad", "n": 30, "dtype": "c64", "p": 8, "inst": "deg4"},
        # coarse annealing: 20 steps with the success probability after each
        {"name": "aqa_n26_c128_s20", "kind": "aqa", "n": 26, "dtype": "c128", "p": 20, "inst": "deg4", "observe": False},
        # annealing trajectory with every spin expectation recorded; odd n
        {"name": "aqa_obs_n23_c64_s12", "kind": "aqa", "n": 23, "dtype": "c64", "p": 12, "inst": "deg4",
         "observe": True},
        # time stepping of the annealing Hamiltonian
        {"name": "qsds_n24_c128_s10", "kind": "qsds", "n": 24, "dtype": "c128", "p": 10, "inst": "deg4",
         "observe": False},
        # landscape scan: 128 instances of 10 to 18 qubits on a 32 x 32 grid
        {"name": "batch_128x32x32_c64", "kind": "batch", "dtype": "c64", "count": 128, "nmin": 10, "nmax": 18, "ng": 32,
         "nb": 32},
        # a new instance and its full enumeration; odd n
        {"name": "ground_n31", "kind": "ground", "n": 31, "inst": "deg4"},
        # the largest: one evaluation of a 64 GiB state
        {"name": "energy_n32_c128_p4", "kind": "energy", "n": 32, "dtype": "c128", "p": 4, "inst": "deg4"},
    ]


def draw(rng):
    """A case of the same ranges: every entry point, from a few qubits to the sizes of the large listed cases."""
    kind = rng.choice(["energy", "energy", "noalloc", "grad", "grad", "forward", "aqa", "aqa", "qsds", "layers", "batch",
                       "ground"])
    dtype = rng.choice(["c128", "c64"])
    inst = rng.choice(["reg3", "deg4", "deg4", "deg4", "real", "cover"])
    if kind == "batch":
        nmin = rng.randint(4, 14)
        return {"kind": kind, "dtype": dtype, "count": int(round(math.exp(rng.uniform(math.log(4), math.log(128))))),
                "nmin": nmin, "nmax": rng.randint(nmin, 18), "ng": rng.randint(3, 32), "nb": rng.randint(3, 32)}
    if kind == "ground":
        return {"kind": kind, "n": rng.randint(10, 31), "inst": inst}
    top = {"energy": 30, "noalloc": 24, "grad": 28, "forward": 28, "aqa": 27, "qsds": 26, "layers": 28}[kind]
    n = rng.randint(8, top)
    case = {"kind": kind, "n": n, "dtype": dtype, "inst": inst}
    if kind == "layers":
        del case["inst"]
        case["p"] = rng.randint(1, 12)
        case["gates"] = rng.choice(["hadamard", "unitary"])
    elif kind in ("aqa", "qsds"):
        case["p"] = rng.randint(3, 24)
        case["observe"] = rng.random() < 0.5
    else:
        case["p"] = rng.randint(1, 10)
    return case


# ---------------------------------------------------------------------------------------------- inputs
def _instance(kind, n, seed):
    seed = int(seed) % (1 << 31)
    if kind == "reg3":
        return I.regular3_pm1(n, seed)
    if kind == "real":
        return I.random_real(n, min(2 * n, n * (n - 1) // 2), seed)
    if kind == "cover":
        a = I.exact_cover_matrix(n, 4 * n, seed).astype(np.float64)  # Eqs. HChi, HCJij as a plain instance
        ov = a @ a.T
        ei, ej = np.nonzero(np.triu(ov, 1))
        h = 0.5 * ov.sum(axis=1) - a.sum(axis=1)
        scale = 2.0 ** -math.ceil(math.log2(max(1.0, float(ov[ei, ej].max(initial=1.0)) / 2.0)))
        return I.make_instance(n, np.stack([ei, ej], axis=1), np.round(2.0 * h * scale) / 2.0,
                               np.round(ov[ei, ej] * scale) / 2.0)
    return I.degree4_int2(n, seed)


def _ramp(p, seed):
    """An annealing-like ramp with some spread, as an optimiser visits it."""
    g = np.random.default_rng([7, int(seed)])
    gam, bet = I.linear_ramp_params(p)
    return gam * g.uniform(0.9, 1.1, p), (bet - 0.02) * g.uniform(0.9, 1.1, p)


def _schedule(steps, seed):
    """(tau, A, B) of a linear annealing schedule."""
    s = np.arange(steps) / steps
    return 0.4 + 0.2 * np.random.default_rng([9, int(seed)]).random(), 1.0 - s, s


def _gates(kind, layers, n, seed):
    if kind == "hadamard":
        # the Hadamard circuit acts on what the register holds: the state is seeded instead
        u = np.array([[1, 1], [1, -1]], dtype=np.complex128) / math.sqrt(2.0)
        return np.broadcast_to(u, (layers, n, 2, 2)).copy()
    g = np.random.default_rng([11, int(seed)])
    m = g.normal(size=(layers, n, 2, 2)) + 1j * g.normal(size=(layers, n, 2, 2))
    return np.linalg.qr(m)[0]


def _batch_instances(case, seed):
    g = np.random.default_rng([13, int(seed)])
    out = []
    for _ in range(case["count"]):
        out.append(I.regular3_pm1(int(g.integers(case["nmin"], case["nmax"] + 1)), int(g.integers(1 << 31))))
    return out


def _tdtype(case):
    return torch.complex128 if case["dtype"] == "c128" else torch.complex64


def _random_state(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 31))
    real = torch.float64 if case["dtype"] == "c128" else torch.float32
    v = torch.randn((1 << case["n"], 2), generator=g, device="cuda", dtype=real)
    v = v / torch.sqrt((v.double() ** 2).sum()).to(real)
    return torch.view_as_complex(v)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        insts = _batch_instances(case, seed)
        gam, bet = I.batch_grid(case["ng"], case["nb"])
        return {"case": case, "H": [sv.Ising.from_instance(x) for x in insts], "gam": gam, "bet": bet}
    if kind == "ground":
        return {"case": case, "inst": _instance(case["inst"], case["n"], seed)}
    st = {"case": case, "s": sv.State(case["n"], case["dtype"])}
    if kind == "layers":
        st["U"] = _gates(case["gates"], case["p"], case["n"], seed)
        st["psi0"] = _random_state(case, seed)
        return st
    st["H"] = sv.Ising.from_instance(_instance(case["inst"], case["n"], seed))
    sv.ground(st["H"])
    if kind == "qsds":
        st["tau"], st["A"], st["B"] = _schedule(case["p"], seed)
        return st
    if kind == "aqa":
        tau = 0.5 + 0.2 * np.random.default_rng([9, int(seed)]).random()
        st["gam"], st["bet"] = sv.schedule_linear(case["p"], tau)
        return st
    st["gam"], st["bet"] = _ramp(case["p"], seed)
    if kind == "grad":
        st["lam"] = sv.State(case["n"], case["dtype"])
    if kind == "noalloc":
        st["out"] = torch.zeros(3, dtype=torch.float64, device="cuda")
        sv.qaoa_energy(st["s"], st["H"], st["gam"], st["bet"])  # builds the instance's tables, as the call asks for
    return st


# ---------------------------------------------------------------------------------------------- the calls
#: states up to this size are returned whole
_PSI_MAX = 26


def _num(case, x):
    """Numbers in the precision of the amplitudes they come from."""
    return np.asarray(x, dtype=np.float64 if case["dtype"] == "c128" else np.float32)


def _with_state(case, s, out):
    if case["n"] <= _PSI_MAX:
        out["psi"] = s.tensor
    return out


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        e, p = sv.batch_p1_scan(state["H"], state["gam"], state["bet"], case["dtype"])
        return {"energy": _num(case, e), "p_gs": _num(case, p)}
    if kind == "ground":
        H = sv.Ising.from_instance(state["inst"])
        e, deg, arg = sv.ground(H)
        H.close()
        return {"e_min": np.float64(e), "degeneracy": deg, "argmin": arg}
    s = state["s"]
    if kind == "layers":
        s.tensor.copy_(state["psi0"])
        sv.gate_layers(s, state["U"])
        return {"psi": s.tensor}
    H = state["H"]
    if kind == "energy":
        e, p, nrm = sv.qaoa_energy(s, H, state["gam"], state["bet"])
        return _with_state(case, s, {"energy": _num(case, e), "p_gs": _num(case, p), "norm": _num(case, nrm)})
    if kind == "noalloc":
        sv.qaoa_energy_noalloc(s, H, state["gam"], state["bet"], state["out"])
        out = state["out"] if case["dtype"] == "c128" else state["out"].float()
        return _with_state(case, s, {"norm_energy_pgs": out})
    if kind == "grad":
        e, p, dg, db = sv.grad(s, state["lam"], H, state["gam"], state["bet"], with_pgs=True)
        return {"energy": _num(case, e), "p_gs": _num(case, p), "dgamma": _num(case, dg), "dbeta": _num(case, db)}
    if kind == "forward":
        sv.qaoa_forward(s, H, state["gam"], state["bet"])
        e, p, nrm = sv.expect(s, H)
        return _with_state(case, s, {"energy": _num(case, e), "p_gs": _num(case, p), "norm": _num(case, nrm),
                                     "spin_z": _num(case, sv.spin_z(s))})
    if kind == "aqa":
        if case["observe"]:
            p, e, z = sv.aqa_run_observe(s, H, state["gam"], state["bet"])
            return _with_state(case, s, {"p_gs": _num(case, p), "energy": _num(case, e), "spin_z": _num(case, z)})
        p, e = sv.aqa_run(s, H, state["gam"], state["bet"], per_step=True)
        return _with_state(case, s, {"p_gs": _num(case, p), "energy": _num(case, e)})
    if case["observe"]:
        e, p, z = sv.qsds_run(s, H, state["tau"], state["A"], state["B"], observe=True)
        return _with_state(case, s, {"energy": _num(case, e), "p_gs": _num(case, p), "spin_z": _num(case, z)})
    sv.qsds_run(s, H, state["tau"], state["A"], state["B"])
    return _with_state(case, s, {})


# ---------------------------------------------------------------------------------------------- work
def work(case):
    """The final state written once (a landscape scan: its outputs) and the arithmetic of the circuit: 6 operations per
    amplitude for a phase, 4 per qubit for a mixer (14 for general gates)."""
    kind = case["kind"]
    if kind == "batch":
        amps = case["count"] * float(np.mean([2.0 ** n for n in range(case["nmin"], case["nmax"] + 1)]))
        pts = case["ng"] * case["nb"]
        return {"bytes": 16.0 * case["count"] * pts, "flops": amps * pts * (11 + 4 * 0.5 * (case["nmin"] + case["nmax"]))}
    n = case["n"]
    N = 2.0 ** n
    if kind == "ground":
        return {"bytes": 16.0 * 3 * n, "flops": 2.0 * N}
    size = N * (16 if case["dtype"] == "c128" else 8)
    per = (14 * n) if kind == "layers" else (14 * n + 6) if kind == "qsds" else (4 * n + 6)
    if kind == "grad":
        return {"bytes": size, "flops": 3 * case["p"] * N * per}
    return {"bytes": size * (2 if kind == "layers" else 1), "flops": case["p"] * N * per + 5 * N}


# ---------------------------------------------------------------------------------------------- 64-bit values
_DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _spin(z, i):
    return ((z >> i) & 1).to(torch.float64) * 2.0 - 1.0


def _energies(inst, lo, hi):
    z = torch.arange(lo, hi, device=_DEV)
    e = torch.zeros(hi - lo, dtype=torch.float64, device=_DEV)
    spins = [_spin(z, i) for i in range(inst["n"])] if hi - lo <= 1 << 22 else None
    get = (lambda i: spins[i]) if spins is not None else (lambda i: _spin(z, i))
    for i in range(inst["n"]):
        e += float(inst["h"][i]) * get(i)
    for i, j, J in zip(inst["ei"], inst["ej"], inst["J"]):
        e += float(J) * get(int(i)) * get(int(j))
    return e


def _all_energies(inst):
    n = inst["n"]
    step = 1 << min(n, 22)
    return torch.cat([_energies(inst, a, a + step) for a in range(0, 1 << n, step)])


def _gate(psi, q, u):
    """psi <- the 2x2 matrix u on qubit q, in place (psi: [..., 2^n])."""
    v = psi.view(-1, 2, 1 << q)
    a, b = v[:, 0, :].clone(), v[:, 1, :]
    v[:, 0, :] = u[0][0] * a + u[0][1] * b
    v[:, 1, :] = u[1][0] * a + u[1][1] * b


def _mix(psi, n, beta):
    c, s = math.cos(beta), -1j * math.sin(beta)
    for q in range(n):
        _gate(psi, q, ((c, s), (s, c)))


def _plus(n):
    return torch.full((1 << n,), 2.0 ** (-0.5 * n), dtype=torch.complex128, device=_DEV)


def _observables(E, emin, tol, psi):
    w = psi.real ** 2 + psi.imag ** 2
    return float((E * w).sum()), float(w[(E - emin).abs() <= tol].sum()), float(w.sum())


def _spin_sums(psi, n):
    w = psi.real ** 2 + psi.imag ** 2
    return np.array([float((w.view(-1, 2, 1 << q)[:, 1] - w.view(-1, 2, 1 << q)[:, 0]).sum()) for q in range(n)])


def _x_form(lam, psi, n):
    """Im <lam| sum_q sigma^x_q |psi>"""
    t = 0.0
    for q in range(n):
        a, b = lam.view(-1, 2, 1 << q), psi.view(-1, 2, 1 << q)
        t += float((a[:, 0].conj() * b[:, 1]).imag.sum() + (a[:, 1].conj() * b[:, 0]).imag.sum())
    return t


def _host(psi, case):
    return {"psi": psi} if case["n"] <= _PSI_MAX else {}


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        if case["count"] * case["ng"] * case["nb"] > 140000:
            return None
        en, pg = [], []
        gam, bet = I.batch_grid(case["ng"], case["nb"])
        for inst in _batch_instances(case, seed):
            n = inst["n"]
            E = _all_energies(inst)
            gs = (E == E.min()).to(torch.float64)
            # the mixer is diagonal after a Hadamard transform of the phase state
            wt = torch.zeros(1 << n, dtype=torch.float64, device=_DEV)
            z = torch.arange(1 << n, device=_DEV)
            for q in range(n):
                wt += _spin(z, q)
            rb = torch.exp(1j * torch.as_tensor(bet, device=_DEV).view(-1, 1) * wt.view(1, -1))
            r = math.sqrt(0.5)
            for g in gam:
                phi = torch.exp(-1j * float(g) * E) * 2.0 ** (-0.5 * n)
                for q in range(n):
                    _gate(phi, q, ((r, r), (r, -r)))
                v = (rb * phi.view(1, -1)).contiguous()
                for q in range(n):
                    _gate(v, q, ((r, r), (r, -r)))
                w = v.real ** 2 + v.imag ** 2
                en.append((w @ E).cpu().numpy())
                pg.append((w @ gs).cpu().numpy())
        shape = (case["count"], case["ng"], case["nb"])
        return {"energy": np.stack(en).reshape(shape), "p_gs": np.stack(pg).reshape(shape)}
    n, p = case["n"], case.get("p", 1)
    if kind == "ground":
        inst = _instance(case["inst"], n, seed)
        step = 1 << min(n, 25)
        return {"e_min": np.float64(min(float(_energies(inst, a, a + step).min()) for a in range(0, 1 << n, step)))}
    if p * n * 2.0 ** n * {"grad": 4, "qsds": 2}.get(kind, 1) > 4e10:
        return None
    if kind == "layers":
        psi = _random_state(case, seed).to(torch.complex128)
        U = _gates(case["gates"], p, n, seed)
        for k in range(p):
            for q in range(n):
                _gate(psi, q, U[k, q].tolist())
        return {"psi": psi}
    inst = _instance(case["inst"], n, seed)
    E = _all_energies(inst)
    emin = float(E.min())
    tol = 1e-9 * max(1.0, float(np.abs(inst["h"]).sum() + np.abs(inst["J"]).sum()))
    psi = _plus(n)
    if kind == "qsds":
        tau, A, B = _schedule(p, seed)
        Ez = torch.zeros_like(E)
        z = torch.arange(1 << n, device=_DEV)
        for i in range(n):
            Ez += float(inst["h"][i]) * _spin(z, i)
        EJ = E - Ez
        en, pg, sz = [], [], []

        def half(l):
            for i in range(n):
                a, c = float(A[l]), -float(B[l]) * float(inst["h"][i])
                r = math.hypot(a, c)
                cs, sr = math.cos(0.5 * tau * r), (math.sin(0.5 * tau * r) / r if r > 0 else 0.5 * tau)
                _gate(psi, i, ((cs - 1j * sr * c, 1j * sr * a), (1j * sr * a, cs + 1j * sr * c)))

        for l in range(p):
            half(l)
            psi *= torch.exp(-1j * tau * float(B[l]) * EJ)
            half(l)
            if case["observe"]:
                e, g, _ = _observables(E, emin, tol, psi)
                en.append(e)
                pg.append(g)
                sz.append(_spin_sums(psi, n))
        out = {"energy": np.array(en), "p_gs": np.array(pg), "spin_z": np.array(sz)} if case["observe"] else {}
        return {**out, **_host(psi, case)}
    if kind == "aqa":
        tau = 0.5 + 0.2 * np.random.default_rng([9, int(seed)]).random()
        k = np.arange(1, p + 1) / p
        en, pg, sz = [], [], []
        for g, b in zip(tau * k, -tau * (1.0 - k)):
            psi *= torch.exp(-1j * float(g) * E)
            _mix(psi, n, float(b))
            e, gs, _ = _observables(E, emin, tol, psi)
            en.append(e)
            pg.append(gs)
            if case["observe"]:
                sz.append(_spin_sums(psi, n))
        out = {"p_gs": np.array(pg), "energy": np.array(en)}
        if case["observe"]:
            out["spin_z"] = np.array(sz)
        return {**out, **_host(psi, case)}
    gam, bet = _ramp(p, seed)
    for g, b in zip(gam, bet):
        psi *= torch.exp(-1j * float(g) * E)
        _mix(psi, n, float(b))
    e, pg, nrm = _observables(E, emin, tol, psi)
    if kind == "energy":
        return {"energy": np.float64(e), "p_gs": np.float64(pg), "norm": np.float64(nrm), **_host(psi, case)}
    if kind == "noalloc":
        return {"norm_energy_pgs": np.array([nrm, e, pg]), **_host(psi, case)}
    if kind == "forward":
        return {"energy": np.float64(e), "p_gs": np.float64(pg), "norm": np.float64(nrm), "spin_z": _spin_sums(psi, n),
                **_host(psi, case)}
    lam = E * psi
    dg, db = np.zeros(p), np.zeros(p)
    for k in range(p - 1, -1, -1):
        db[k] = 2.0 * _x_form(lam, psi, n)
        for v in (psi, lam):
            _mix(v, n, -float(bet[k]))
        dg[k] = 2.0 * float((E * (lam.conj() * psi).imag).sum())
        ph = torch.exp(1j * float(gam[k]) * E)
        psi *= ph
        lam *= ph
    return {"energy": np.float64(e), "p_gs": np.float64(pg), "dgamma": dg, "dbeta": db}

"""Plans with two tile groups (64-byte runs or 14-bit complex128 tiles) and small-tile plans: every
layout covers every amplitude and every qubit once (on the CPU), and on the GPU the same results as
the three-group plans."""
import numpy as np
import pytest

from paper_2104_03293_amd import inputs as I

TWO = [("c128", 24), ("c128", 25), ("c128", 26), ("c64", 25)]


@pytest.fixture(scope="module")
def sv():
    from paper_2104_03293_amd import sv as m

    return m


@pytest.mark.parametrize("dtype,n", TWO + [(d, n) for d in ("c128", "c64") for n in (1, 6, 10, 13, 14, 17, 19, 21)])
def test_plans_cover_every_qubit_and_amplitude(sv, dtype, n):
    plans = sv.describe(n, dtype)["plans"]
    groups = plans["two_groups" if (dtype, n) in TWO else "small_tiles"]
    assert len(groups) == (1 if n <= 13 else 2)
    covered = []
    for gi, g in enumerate(groups):
        T, R, c, lo, gb = g["T"], g["R"], g["c"], g["lo"], g["g"]
        active = list(range(min(n, T))) if gi == 0 else list(range(c, T))
        covered += [l if gi == 0 or l < c else lo + l - c for l in active]
        assert g["ntiles"] << T >= 1 << n and len(g["blocks"]) <= 4
        for direction in ("fwd", "bwd"):
            seen = []
            for blk in g["blocks"]:
                assert len(set(blk["bits"])) == R and max(blk["bits"]) < T
                seen += [blk["bits"][k] for k in range(R) if blk[direction] >> k & 1]
                tb = [l for l in range(T) if l not in blk["bits"]]
                if "pair" in blk:  # small tiles: lane bits 4 and 5 hold pair and pair + 1
                    p = blk["pair"]
                    tb = [l for l in tb if l not in (p, p + 1)]
                    assert len(tb) == T - R - 2 and p + 1 < T
                    tb[4:4] = [p, p + 1]
                    # 16 lanes of an exchange reach 16 different LDS slots (either form of the layout)
                    slot = lambda l: 1 << l | (1 << (l & 3) if l >= 4 else 0)
                    low = {0}
                    for l in tb[:4]:
                        low |= {x ^ (slot(l) & 15) for x in low}
                    assert len(low) == 16
                    assert blk["dpp"] & ~0x30 == 0 and (not blk["dpp"] or blk in (g["blocks"][0], g["blocks"][-1]))
                seen += [tb[q] for q in range(6) if blk["dpp"] >> q & 1]
            assert sorted(seen) == active
        if n > T:  # tile index and tile bits together address every amplitude once
            assert c + gb == T and c <= lo and lo + gb <= n and (lo - c) + (n - lo - gb) == n - T
    assert sorted(covered) == list(range(n))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,n", TWO)
def test_two_groups_match_three(sv, dtype, n):
    out = []
    for kind in ("int", "real"):
        inst = I.degree4_int2(n, 7 + n) if kind == "int" else I.random_real(n, 2 * n, 9 + n)
        H = sv.Ising.from_instance(inst)
        g, b = I.uniform_params(3, n)
        A, B = 1.0 - np.arange(3) / 3, np.arange(3) / 3
        s = sv.State(n, dtype)
        for two in (1, 0):
            old = sv.tune_get("twogroup")
            sv.tune_set("twogroup", two)
            try:
                e = sv.qaoa_energy(s, H, g, b)
                psi = s.to_numpy()
                obs = sv.aqa_run_observe(s, H, g, b)
                q = sv.qsds_run(s, H, 0.5, A, B, observe=True)
                sv.mixer(s, 0.3)
                out.append((np.array(e), psi, *obs, *q, s.to_numpy()))
            finally:
                sv.tune_set("twogroup", old)
        tol = 1e-11 if dtype == "c128" else 2e-5  # the library's amplitude bars; sums on the scale of <H_C>
        for x, y in zip(*out[-2:]):
            assert np.max(np.abs(x - y)) <= tol * max(1.0, float(np.max(np.abs(y))))


@pytest.mark.gpu
@pytest.mark.parametrize("first", ["energy", "grad", "qsds"])
@pytest.mark.parametrize("n", [24, 25, 26])
def test_noalloc_follows_calls_with_other_plans(sv, n, first):
    """Calls whose own plan has three groups leave what a non-allocating evaluation looks up."""
    import torch

    H = sv.Ising.from_instance(I.degree4_int2(n, 3 + n))
    s = sv.State(n, "c128")
    g, b = I.uniform_params(3, n)
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    with pytest.raises(sv.SVError):
        sv.qaoa_energy_noalloc(s, H, g, b, out)
    if first == "energy":
        sv.qaoa_energy(s, H, g, b)
    elif first == "grad":
        sv.grad(s, sv.State(n, "c128"), H, g, b)
    else:
        sv.qsds_run(s, H, 0.5, [1.0, 0.5, 0.2], [0.1, 0.5, 0.9])
    sv.ground(H)
    sv.qaoa_energy_noalloc(s, H, g, b, out)
    torch.cuda.synchronize()
    ref = sv.qaoa_energy(s, H, g, b)
    got = out.cpu().numpy()
    assert abs(got[1] - ref[0]) <= 1e-9 * max(1.0, abs(ref[0]))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [5, 13, 14])
def test_noalloc_c64_follows_ground_alone(sv, n):
    import torch

    H = sv.Ising.from_instance(I.degree4_int2(n, 3 + n))
    s = sv.State(n, "c64")
    g, b = I.uniform_params(3, n)
    out = torch.zeros(3, dtype=torch.float64, device="cuda")
    sv.ground(H)
    sv.qaoa_energy_noalloc(s, H, g, b, out)
    torch.cuda.synchronize()
    assert abs(out.cpu().numpy()[1] - sv.qaoa_energy(s, H, g, b)[0]) <= 2e-5 * n

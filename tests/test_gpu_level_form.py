"""GPU: complex128 evolutions from |s> in the level form (counts of the cost
table, a recursion over the occupied levels, one write of the state) against
the oracle's statevector, at the edges of its pieces: one launch up to n = 15
and three beyond; levels held 64, 128 and 256 to the wave (synthetic tables
with that many levels); chunks of 16, 8 and 4 rounds and their remainders;
angles as kernel arguments up to 112 rounds and from memory beyond; p = 0; a
cost table at an odd address. Bars: the complex128 ones of the statevector
tests, 1e-12 on P_sol, the norm and every amplitude, 1e-12 m on E.

Gradients in the level form against the oracle's statevector sweep at the same
edges, batched (each instance its own table, m and target): 1e-12 on P and
dP/dbeta, 1e-12 m on dP/dgamma."""
import numpy as np
import pytest

from gpu_common import log, need_gpu
from oracle.evolve import evolve_sv
from oracle.grad import grad_sv
from paper_2402_02585_amd import gqaoa as g

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels,p,odd", [
    (3, 3, 1, False), (4, 2, 0, False), (6, 1, 5, True), (8, 64, 16, False), (8, 65, 17, False), (10, 128, 9, False),
    (11, 129, 5, True), (12, 256, 4, False), (12, 30, 112, False), (12, 30, 113, False), (15, 40, 33, False),
    (16, 40, 15, False), (16, 255, 3, True), (17, 100, 40, False), (20, 50, 2, False)])
def test_level_form_matches_statevector_oracle(n, levels, p, odd):
    torch = need_gpu()
    rng = np.random.Generator(np.random.PCG64(600 + 7 * n + levels))
    m = max(levels - 1, 1)
    cost = rng.integers(0, levels, 2 ** n).astype(np.uint8)
    cost[:levels] = np.arange(levels)[:2 ** n]           # every level occupied
    buf = torch.zeros(2 ** n + 16, dtype=torch.uint8, device="cuda")
    dev = buf[1:2 ** n + 1] if odd else buf[:2 ** n]
    dev.copy_(torch.from_numpy(cost))
    b, gm = rng.uniform(0, 2 * np.pi, p), rng.uniform(0, np.pi, p)
    target = int(rng.integers(0, levels))
    log(f"level form n={n} levels={levels} p={p} odd={odd}")
    for rep in range(2):                                 # the second call finds the first one's scratch
        psi, ps, en, no = g.gqaoa_evolve(n, m, dev, b, gm, dtype=g.C128, target_level=target)
    rpsi, rp, re, rn = evolve_sv(n, cost, b, gm, target=target)
    assert np.abs(ps - rp).max() < 1e-12 and np.abs(no - rn).max() < 1e-12
    assert np.abs(en - re).max() < 1e-12 * m
    assert np.abs(psi.cpu().numpy() - rpsi).max() < 1e-12
    if p:
        plan = g.EvolvePlan(n, m, dev, p, dtype=g.C128, target_level=target)
        try:
            for rep in range(2):
                plan.psi.fill_(0)
                got = plan.run(b, gm)
                assert all(np.array_equal(x, y) for x, y in zip(got, (ps, en, no))), rep
                assert torch.equal(plan.psi, psi), rep
                torch.cuda.synchronize()
        finally:
            plan.close()
    absent = m if levels == 1 else None                  # an unoccupied target level
    if absent is not None:
        assert g.gqaoa_evolve(n, m, dev, b, gm, dtype=g.C128, target_level=absent)[1].max() == 0.0


@pytest.mark.parametrize("n,I,levels,p,odd", [
    (3, 5, 3, 1, False), (7, 3, 64, 16, True), (7, 2, 65, 17, False), (9, 3, 129, 5, False), (10, 2, 256, 9, False),
    (12, 4, 30, 33, False), (15, 2, 40, 2, False), (16, 3, 40, 15, False), (16, 2, 200, 5, True), (17, 1, 30, 1, False)])
def test_level_gradient_matches_statevector_oracle(n, I, levels, p, odd):
    torch = need_gpu()
    rng = np.random.Generator(np.random.PCG64(700 + 7 * n + levels))
    cost = rng.integers(0, levels, (I, 2 ** n)).astype(np.uint8)
    cost[:, :levels] = np.arange(levels)[:2 ** n]
    buf = torch.zeros(I * 2 ** n + 16, dtype=torch.uint8, device="cuda")
    dev = buf[1:I * 2 ** n + 1] if odd else buf[:I * 2 ** n]
    dev.copy_(torch.from_numpy(cost.reshape(-1)))
    ms = np.minimum(levels - 1 + np.arange(I), 255).astype(np.int32)
    tg = rng.integers(0, levels, I).astype(np.int32)
    b, gm = rng.uniform(0, 2 * np.pi, (I, p)), rng.uniform(0, np.pi, (I, p))
    log(f"level gradient n={n} I={I} levels={levels} p={p} odd={odd}")
    for ckpt in (0, 3):
        P, db, dg = g.gqaoa_grad_batched(n, ms, dev, b, gm, dtype=g.C128, targets=tg, ckpt_every=ckpt)
    for i in range(I):
        rP, rb, rg = grad_sv(n, cost[i], b[i], gm[i], target=int(tg[i]))
        assert abs(P[i] - rP) < 1e-12 and np.abs(db[i] - rb).max() < 1e-12, i
        assert np.abs(dg[i] - rg).max() < 1e-12 * levels, i


@pytest.mark.parametrize("n,m,p,odd", [
    (3, 2, 1, False), (5, 7, 3, True), (8, 97, 16, False), (9, 98, 17, False), (9, 188, 5, False), (10, 189, 4, True),
    (11, 254, 6, False), (13, 50, 113, False), (16, 40, 15, True), (17, 67, 9, False), (20, 84, 3, False)])
def test_given_state_in_level_form(n, m, p, odd):
    """From a random state that is not constant on the levels: the level sums'
    column counts (16, 8 and 4 columns: up to 98, 189 and 255 levels), blocks of
    a few amplitudes and of several tiles, a plan's runs chained from psi's own
    contents, and reruns with the same bits."""
    torch = need_gpu()
    rng = np.random.Generator(np.random.PCG64(800 + 7 * n + m))
    cost = rng.integers(0, m + 1, 2 ** n).astype(np.uint8)
    v = rng.normal(size=2 ** n) + 1j * rng.normal(size=2 ** n)
    v /= np.linalg.norm(v)
    buf = torch.zeros(2 ** n + 16, dtype=torch.uint8, device="cuda")
    dev = buf[1:2 ** n + 1] if odd else buf[:2 ** n]
    dev.copy_(torch.from_numpy(cost))
    b, gm = rng.uniform(0, 2 * np.pi, p), rng.uniform(0, np.pi, p)
    target = int(cost[0])
    log(f"given state n={n} m={m} p={p} odd={odd}")
    runs = [g.gqaoa_evolve(n, m, dev, b, gm, dtype=g.C128, psi=torch.tensor(v, device="cuda"), init_uniform=False,
                           target_level=target) for _ in range(3)]
    psi, ps, en, no = runs[0]
    for r in runs[1:]:
        assert torch.equal(r[0], psi) and all(np.array_equal(x, y) for x, y in zip(r[1:], runs[0][1:]))
    rpsi, rp, re, rn = evolve_sv(n, cost, b, gm, psi0=v, target=target)
    assert np.abs(ps - rp).max() < 1e-12 and np.abs(no - rn).max() < 1e-12
    assert np.abs(en - re).max() < 1e-12 * m
    assert np.abs(psi.cpu().numpy() - rpsi).max() < 1e-12
    plan = g.EvolvePlan(n, m, dev, p, dtype=g.C128, init_uniform=False, target_level=target,
                        psi=torch.tensor(v, device="cuda"))
    try:
        got = plan.run(b, gm)
        assert all(np.array_equal(x, y) for x, y in zip(got, (ps, en, no))) and torch.equal(plan.psi, psi)
        got = plan.run(b, gm)
        rpsi, rp, _, _ = evolve_sv(n, cost, b, gm, psi0=rpsi, target=target)
        assert np.abs(got[0] - rp).max() < 1e-12 and np.abs(plan.psi.cpu().numpy() - rpsi).max() < 1e-12
    finally:
        plan.close()


@pytest.mark.parametrize("uniform", [False, True])
@pytest.mark.parametrize("n,m,p", [(4, 3, 1), (8, 97, 2), (8, 98, 17), (10, 188, 1), (10, 189, 3), (12, 254, 2),
                                   (16, 40, 15), (16, 5, 113)])
def test_costs_above_m_get_the_phase_factor_zero(n, m, p, uniform, monkeypatch):
    """A cost table with entries above m (m the level sums' column counts on
    either side, and 254, where one level is above): the level form gives what
    the round passes give, whose phase tables hold 0 there. 1e-12 on the
    probabilities, the norm and every amplitude, 255e-12 on E."""
    torch = need_gpu()
    rng = np.random.Generator(np.random.PCG64(850 + 7 * n + m))
    cost = rng.integers(0, m + 1, 2 ** n).astype(np.uint8)
    above = rng.random(2 ** n) < 0.1
    above[1] = True
    cost[above] = rng.integers(m + 1, 256, int(above.sum()))
    v = rng.normal(size=2 ** n) + 1j * rng.normal(size=2 ** n)
    v /= np.linalg.norm(v)
    dev = torch.from_numpy(cost).cuda()
    b, gm = rng.uniform(0, 2 * np.pi, p), rng.uniform(0, np.pi, p)
    target = int(cost[~above][0])
    log(f"costs above m n={n} m={m} p={p} uniform={uniform}")
    call = lambda: g.gqaoa_evolve(n, m, dev, b, gm, dtype=g.C128, psi=torch.tensor(v, device="cuda"),
                                  init_uniform=uniform, target_level=target)
    psi, ps, en, no = call()
    monkeypatch.setenv("GQAOA_SV_RESIDENT", "0")
    rpsi, rp, re, rn = call()
    assert np.abs(ps - rp).max() < 1e-12 and np.abs(no - rn).max() < 1e-12
    assert np.abs(en - re).max() < 255e-12
    assert (psi - rpsi).abs().max().item() < 1e-12


@pytest.mark.parametrize("n,m,p,uniform,passes", [
    (23, 189, 1, False, 1), (23, 255, 1, False, 1), (23, 188, 1, False, 0), (22, 255, 1, False, 0),
    (23, 255, 2, False, 0), (23, 255, 1, True, 0), (24, 50, 0, True, 0), (25, 50, 0, True, 0), (25, 50, 1, True, 0)])
def test_the_faster_form_of_few_rounds(n, m, p, uniform, passes):
    """One round from a given large state with many levels goes through a round
    pass (`passes` of them timed under their name), its neighbours and calls
    from |s> take the level form, and p = 0 from |s> writes |s> either way.
    Readouts and sampled amplitudes from level sums in float64: 1e-12, E 1e-12 m."""
    torch = need_gpu()
    rng = np.random.Generator(np.random.PCG64(900 + 7 * n + m + p))
    N = 2 ** n
    cost = torch.from_numpy(rng.integers(0, m + 1, N).astype(np.uint8)).cuda()
    b, gm = rng.uniform(0, 2 * np.pi, p), rng.uniform(0, np.pi, p)
    psi0 = torch.full((N,), 2.0 ** (-n / 2), dtype=torch.complex128, device="cuda")
    if not uniform:
        psi0 *= torch.polar(torch.ones(N, dtype=torch.float64, device="cuda"),
                            torch.linspace(0, 2, N, dtype=torch.float64, device="cuda"))
    log(f"few rounds n={n} m={m} p={p} uniform={uniform}")
    want = psi0.clone()
    E, P = [], []
    lev = cost.double()
    for j in range(p + 1):
        if j:
            want *= torch.polar(torch.ones_like(lev), -gm[j - 1] * lev)
            want += complex(np.exp(-1j * b[j - 1]) - 1) * want.mean()
        q = want.real ** 2 + want.imag ** 2
        E.append((q * lev).sum().item())
        P.append(q[cost == 7].sum().item())
    g.gqaoa_profile_reset()
    g.gqaoa_profile_enable(1)
    try:
        psi, ps, en, no = g.gqaoa_evolve(n, m, cost, b, gm, dtype=g.C128, psi=psi0, init_uniform=uniform, target_level=7)
        assert g.gqaoa_profile_read("sv_round_c128")[1] == passes
    finally:
        g.gqaoa_profile_enable(0)
        g.gqaoa_profile_reset()
    assert np.abs(ps - P).max() < 1e-12 and np.abs(en - E).max() < 1e-12 * m and np.abs(no - 1).max() < 1e-12
    assert (psi - want).abs().max().item() < 1e-12


def test_profile_names_of_the_level_form_and_the_crossing_scan():
    """A profiled call reads back under its name: evolutions of several launches
    (from |s> and from a given state), of one launch, gradients, and a crossing
    scan whose buckets run side by side, timed once and not longer than the call."""
    import time
    torch = need_gpu()
    rng = np.random.Generator(np.random.PCG64(950))
    n, m, p = 16, 40, 5
    cost = torch.from_numpy(rng.integers(0, m + 1, 2 ** n).astype(np.uint8)).cuda()
    b, gm = rng.uniform(0, 6, p), rng.uniform(0, 3, p)
    psi = torch.full((2 ** n,), 2.0 ** -8, dtype=torch.complex128, device="cuda")
    h = np.zeros((9, 41), dtype=np.uint64)
    for i, K in enumerate(range(2, 38, 4)):
        h[i, :K] = rng.multinomial((1 << 16) - K, np.ones(K) / K) + 1
    calls = {
        "level_evolve": [lambda: g.gqaoa_evolve(n, m, cost, b, gm, dtype=g.C128),
                         lambda: g.gqaoa_evolve(n, m, cost, b, gm, dtype=g.C128, psi=psi, init_uniform=False)],
        "sv_resident_c128": [lambda: g.gqaoa_evolve(10, m, cost, b, gm, dtype=g.C128)],
        "level_grad": [lambda: g.gqaoa_grad(n, m, cost, b, gm, dtype=g.C128)],
        "scan": [lambda: g.gqaoa_scan_crossing([16] * 9, [40] * 9, h, np.linspace(0, 6, 90), np.linspace(0, 3, 45), 400, 0.9)],
    }
    for name, fs in calls.items():
        for f in fs:
            f()
            torch.cuda.synchronize()
            log(f"profile {name}")
            g.gqaoa_profile_reset()
            g.gqaoa_profile_enable(1)
            try:
                t0 = time.perf_counter()
                f()
                torch.cuda.synchronize()
                wall = (time.perf_counter() - t0) * 1e3
            finally:
                g.gqaoa_profile_enable(0)
            ms, count = g.gqaoa_profile_read(name)
            g.gqaoa_profile_reset()
            assert count == 1 and 0 < ms < wall, (name, ms, count, wall)

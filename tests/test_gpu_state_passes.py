"""GPU: the round and reverse passes over the state where a call would take the
level form by itself (complex128, through GQAOA_SV_RESIDENT=0), and complex64
gradients whose passes fold their partial rows. Each complex128 test reads the
launch counts back, so that a call which runs no pass fails it.

Bars: those of the statevector tests, 1e-12 on probabilities, the norm and
amplitudes, 1e-12 m on E and dP/dgamma (complex128), 2e-5 and 2e-5 m on complex64
gradients; the same bits where the same launches run on the same inputs."""
import numpy as np
import pytest

from gpu_common import log, need_gpu, rand_lits, rand_state
from oracle.cost import cost_table, level_histogram
from oracle.evolve import evolve_sv
from oracle.grad import grad_hist, grad_sv
from paper_2402_02585_amd import gqaoa as g
from paper_2402_02585_amd import instances as inst

pytestmark = pytest.mark.gpu


@pytest.fixture
def passes(monkeypatch):
    """Calls by passes over the state; yields a function that returns how often
    the named pass ran since the last one."""
    need_gpu()
    monkeypatch.setenv("GQAOA_SV_RESIDENT", "0")
    g.gqaoa_profile_reset()
    g.gqaoa_profile_enable(1)

    def ran(name):
        n = g.gqaoa_profile_read(name)[1]
        g.gqaoa_profile_reset()
        return n

    yield ran
    g.gqaoa_profile_enable(0)
    g.gqaoa_profile_reset()


def _instance(n, m, seed):
    lits = rand_lits(n, m, seed)
    return g.gqaoa_cost_table(n, lits)[0], cost_table(n, lits)


def test_checkpoint_intervals_complex128(passes):
    """Every interval recomputes the same rounds: the oracle's gradient, the same
    bits for all of them, and forward passes beyond the first p (the states of the
    segments but the last) where there are segments."""
    n, m, p = 11, 47, 7
    cost, ref = _instance(n, m, 9)
    beta, gamma = inst.uniform_angles(19, p)
    rP, rdb, rdg = grad_sv(n, ref, beta, gamma)
    first = None
    for ckpt in (0, 1, 2, 3, 7, 50):
        log(f"checkpoint interval {ckpt}")
        P, db, dg = g.gqaoa_grad(n, m, cost, beta, gamma, dtype=g.C128, ckpt_every=ckpt)
        forward = g.gqaoa_profile_read("sv_round_c128")[1]
        assert passes("sv_reverse_c128") == p
        assert forward > p if 0 < ckpt < p else forward == p
        assert abs(P - rP) < 1e-12 and np.abs(db - rdb).max() < 1e-12 and np.abs(dg - rdg).max() < 1e-12 * m
        first = first or (P, db, dg)
        assert P == first[0] and (db == first[1]).all() and (dg == first[2]).all()


def test_chosen_checkpoint_interval_complex128(passes):
    """ckpt_every=None in a workspace one byte short of all states recomputes
    segments, to the bits of the sweep that keeps them."""
    torch = need_gpu()
    n, m, p, I = 14, 59, 12, 3
    costs = torch.stack([_instance(n, m, 400 + i)[0] for i in range(I)])
    rng = np.random.Generator(np.random.PCG64(401))
    betas, gammas = rng.uniform(0, np.pi, (I, p)), rng.uniform(0, np.pi, (I, p))
    ref = g.gqaoa_grad_batched(n, [m] * I, costs, betas, gammas, ckpt_every=0)
    assert passes("sv_round_c128") == p
    ws = torch.empty(g.gqaoa_grad_workspace_bytes(I, n, p, g.C128, 0) - 1, dtype=torch.uint8, device="cuda")
    small = g.gqaoa_grad_batched(n, [m] * I, costs, betas, gammas, workspace=ws)
    assert passes("sv_round_c128") > p
    assert all(np.array_equal(a, b) for a, b in zip(ref, small))


@pytest.mark.parametrize("ckpt", [0, 2])
def test_folded_gradients_complex128(passes, ckpt):
    """Two instances of n = 22: 4,096 blocks each, folded in the forward and the
    reverse passes."""
    torch = need_gpu()
    n, p = 22, 4
    m = inst.m_from_density(n, 4.2)
    made = [_instance(n, m, 310 + k) for k in range(2)]
    rng = np.random.Generator(np.random.PCG64(311))
    betas, gammas = rng.uniform(0, np.pi, (2, p)), rng.uniform(0, np.pi, (2, p))
    log(f"folded gradients complex128 ckpt={ckpt}")
    P, db, dg = g.gqaoa_grad_batched(n, [m, m], torch.stack([c for c, _ in made]), betas, gammas, dtype=g.C128,
                                     ckpt_every=ckpt)
    assert passes("sv_reverse_c128") == p
    for k in range(2):
        rP, rdb, rdg = grad_hist(level_histogram(made[k][1], m), betas[k], gammas[k])
        assert abs(P[k] - rP) < 1e-12 and np.abs(db[k] - rdb).max() < 1e-10 and np.abs(dg[k] - rdg).max() < 1e-10


@pytest.mark.parametrize("I", [1, 5])
def test_folded_gradients_complex64(I):
    """complex64 at n = 22: one instance chains its passes behind the folds, five
    finalize separately; each against the oracle."""
    torch = need_gpu()
    n, p = 22, 3
    m = inst.m_from_density(n, 4.2)
    made = [_instance(n, m, 330 + k) for k in range(min(I, 2))]
    rng = np.random.Generator(np.random.PCG64(331))
    betas, gammas = rng.uniform(0, np.pi, (I, p)), rng.uniform(0, np.pi, (I, p))
    log(f"folded gradients complex64 I={I}")
    costs = torch.stack([made[k % 2][0] for k in range(I)])
    for ckpt in (0, 1):
        P, db, dg = g.gqaoa_grad_batched(n, [m] * I, costs, betas, gammas, dtype=g.C64, ckpt_every=ckpt)
        for k in range(I):
            rP, rdb, rdg = grad_hist(level_histogram(made[k % 2][1], m), betas[k], gammas[k])
            assert abs(P[k] - rP) < 2e-5, (ckpt, k)
            assert np.abs(db[k] - rdb).max() < 2e-5 and np.abs(dg[k] - rdg).max() < 2e-5 * m, (ckpt, k)


@pytest.mark.parametrize("n,p", [(10, 7), (15, 12), (22, 4)])
def test_rounds_and_plans_complex128(passes, n, p):
    """Evolutions from |s> and from a given state, and the captured plan of either,
    in streamed rounds (n = 22: with folds) against the oracle; a plan gives the
    bits of the eager call, with eager work between its runs."""
    torch = need_gpu()
    m = 4 * n
    cost, ref = _instance(n, m, 70 + n)
    psi0 = rand_state(n, n)
    for uniform in (True, False):
        state = lambda: None if uniform else torch.tensor(psi0, device="cuda")
        plan = g.EvolvePlan(n, m, cost, p, dtype=g.C128, init_uniform=uniform, psi=state())
        try:
            for rep in range(3):
                beta, gamma = inst.uniform_angles(80 + rep, p)
                log(f"rounds complex128 n={n} uniform={uniform} run {rep}")
                psi, ps, en, no = g.gqaoa_evolve(n, m, cost, beta, gamma, dtype=g.C128, psi=state(), init_uniform=uniform)
                assert passes("sv_round_c128") == p
                if not uniform:
                    plan.psi.copy_(state())
                got = plan.run(beta, gamma)
                assert all(np.array_equal(x, y) for x, y in zip(got, (ps, en, no))) and torch.equal(plan.psi, psi)
                if rep == 0:
                    rpsi, rp, re, rn = evolve_sv(n, ref, beta, gamma, psi0=None if uniform else psi0)
                    assert np.abs(ps - rp).max() < 1e-12 and np.abs(no - rn).max() < 1e-12
                    assert np.abs(en - re).max() < 1e-12 * m
                    assert np.abs(psi.cpu().numpy() - rpsi).max() < 1e-12
        finally:
            plan.close()


@pytest.mark.parametrize("n", [15, 19, 21, 22])
def test_plans_are_the_eager_calls_complex64(n):
    """Chained, separate and folded passes alike: a complex64 plan gives the bits
    of the eager call, replay after replay."""
    torch = need_gpu()
    m, p = 60, 4
    cost, _ = _instance(n, m, 500 + n)
    plan = g.EvolvePlan(n, m, cost, p, dtype=g.C64, target_level=3)
    try:
        for rep in range(3):
            beta, gamma = inst.uniform_angles(90 + rep, p)
            log(f"plan and eager complex64 n={n} run {rep}")
            psi, *want = g.gqaoa_evolve(n, m, cost, beta, gamma, dtype=g.C64, target_level=3)
            torch.cuda.synchronize()
            plan.psi.fill_(0)
            got = plan.run(beta, gamma)
            assert all(np.array_equal(x, y) for x, y in zip(got, want)) and torch.equal(plan.psi, psi)
    finally:
        plan.close()


def test_level_space_gradient_against_the_sweep(passes):
    """The level-space gradient of a histogram against the statevector sweep of
    its cost table: two programs that share no kernel."""
    n, m, p = 10, 44, 9
    cost, ref = _instance(n, m, 731)
    beta, gamma = inst.uniform_angles(732, p)
    P, db, dg = g.gqaoa_hist_grad_batched([n], [m], level_histogram(ref, m)[None, :], beta[None, :], gamma[None, :])
    Ps, dbs, dgs = g.gqaoa_grad(n, m, cost, beta, gamma, dtype=g.C128, ckpt_every=0)
    assert passes("sv_reverse_c128") == p
    assert abs(P[0] - Ps) < 1e-12 and np.abs(db[0] - dbs).max() < 1e-12 and np.abs(dg[0] - dgs).max() < 1e-12 * m


def test_checkpointed_batch_of_gradients_complex128(passes):
    """64 gradients of n = 20, p = 32, checkpoints every 8 rounds: the sweep over
    13 states an instance against the oracle's level-space sweep."""
    torch = need_gpu()
    n, m, p, I = 20, 85, 32, 64
    made = [_instance(n, m, 600 + k) for k in range(4)]
    costs = torch.stack([made[k % 4][0] for k in range(I)])
    betas = np.stack([inst.uniform_angles(100 + i, p)[0] for i in range(I)])
    gammas = np.stack([inst.uniform_angles(100 + i, p)[1] for i in range(I)])
    log(f"checkpointed batch I={I} n={n} p={p}")
    P, db, dg = g.gqaoa_grad_batched(n, [m] * I, costs, betas, gammas, dtype=g.C128, ckpt_every=8)
    assert passes("sv_reverse_c128") == p
    torch.cuda.empty_cache()
    for i in (0, 1, 31, 63):
        rP, rdb, rdg = grad_hist(level_histogram(made[i % 4][1], m), betas[i], gammas[i])
        assert abs(P[i] - rP) < 1e-12 and np.abs(db[i] - rdb).max() < 1e-11 and np.abs(dg[i] - rdg).max() < 1e-10

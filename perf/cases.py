"""The work that users of this framework have it do, as measurable cases.

Each case is one pass through the public entry points of
``paper_2402_02585_amd.gqaoa``: statevector evolution (from |s> and from a
given state, eager and as a captured plan), adjoint gradients on the
statevector and in the level space, the batched single-pair scan and the
first-crossing scan, cost tables and batched level histograms, the
transverse-field comparator and a training step of the angle network.

``exact`` gives the same outputs in 64 bits from the definitions, in plain
torch (on the GPU when there is one) and numpy.
"""
import math

import numpy as np
import torch

from paper_2402_02585_amd import gqaoa as g

DEV = "cuda"


# ---- instances and angles ---------------------------------------------------------------
def _clauses(rng, n, m):
    """m random clauses: three distinct variables each, every literal negated
    with probability 1/2 (lit = 2 var + neg)."""
    var = np.argsort(rng.random((m, n)), axis=1)[:, :3]
    return (2 * var + rng.integers(0, 2, (m, 3))).astype(np.int32)


def _instance(case, rng):
    return _clauses(rng, case["n"], case["m"])


def _batch(case, rng):
    """Instances of uneven size: n uniform in [n_lo, n_hi], m = round(n d),
    d one of the scan workload's densities or, for "max-sat", in (4.6, 8)."""
    ns = rng.integers(case["n_lo"], case["n_hi"] + 1, case["instances"]).astype(np.int32)
    if case["density"] == "max-sat":
        d = rng.uniform(4.6, 8.0, case["instances"])
    else:
        d = rng.choice([3.0, 4.2, 5.0], case["instances"])
    ms = np.floor(ns * d + 0.5).astype(np.int32)
    lits = [_clauses(rng, int(n), int(m)) for n, m in zip(ns, ms)]
    return ns, ms, lits


def _angles(rng, *shape):
    return rng.uniform(0.0, math.pi, shape), rng.uniform(0.0, math.pi, shape)


def _dtype(case):
    return g.C64 if case["dtype"] == "complex64" else g.C128


def _lowest(hists):
    """Target level: the lowest occupied one (level 0 when satisfiable)."""
    return (np.asarray(hists) > 0).argmax(axis=-1).astype(np.int32)


def _grids(case):
    if case["grid"] == "box":            # [0, pi]^2, endpoints included
        return np.linspace(0.0, math.pi, case["nb"]), np.linspace(0.0, math.pi, case["ng"])
    return (np.linspace(0.0, 2 * math.pi, case["nb"], endpoint=False),   # the fundamental domain
            np.linspace(0.0, math.pi, case["ng"]))


def _gauss_state(rng, n, dtype):
    v = rng.standard_normal((1 << n, 2))
    v /= np.sqrt((v * v).sum())
    return torch.view_as_complex(torch.from_numpy(v)).to(dtype)


# ---- cases ------------------------------------------------------------------------------
def listed():
    return [
        # one small instance in double precision, 20 rounds: parity checks and
        # angle searches at n = 10, where a call is all latency
        {"name": "evolve_n10_c128", "kind": "evolve", "n": 10, "m": 42, "p": 20, "dtype": "complex128"},
        # the headline run: n = 28, m = 118, 64 rounds from |s>
        {"name": "evolve_n28_c64", "kind": "evolve", "n": 28, "m": 118, "p": 64, "dtype": "complex64"},
        # one mid-size instance evolved again and again with new angles
        {"name": "plan_n18_c64", "kind": "plan", "n": 18, "m": 76, "p": 32, "dtype": "complex64"},
        # rounds from a given, unstructured state
        {"name": "evolve_from_n22_c128", "kind": "evolve_from", "n": 22, "m": 92, "p": 16, "dtype": "complex128"},
        # adjoint gradients of a batch of n = 20 instances, all 2p angles,
        # checkpoints every 8 rounds
        {"name": "grad_64x_n20_c128", "kind": "grad", "instances": 64, "n": 20, "m": 85, "p": 32,
         "dtype": "complex128", "ckpt": 8},
        # the batched angle scan: 64 x 64 pairs, four readouts, n = 8..20
        {"name": "scan_1024x_64x64", "kind": "scan", "instances": 1024, "n_lo": 8, "n_hi": 20, "density": "scan",
         "nb": 64, "ng": 64, "grid": "box", "p_list": "1,4,16,64", "energy": True},
        # rounds to reach 50%: pi/180 grid over the fundamental domain
        {"name": "crossing_128x_360x181", "kind": "crossing", "instances": 128, "n_lo": 12, "n_hi": 20,
         "density": "max-sat", "nb": 360, "ng": 181, "grid": "domain", "threshold": 0.5},
        # one evaluation of the lockstep optimizer of all 2p angles
        {"name": "level_grad_200x_p100", "kind": "level_grad", "instances": 200, "n_lo": 10, "n_hi": 20,
         "density": "max-sat", "p": 100},
        # level histograms of thousands of instances
        {"name": "hists_4096x", "kind": "hists", "instances": 4096, "n_lo": 8, "n_hi": 20, "density": "scan"},
        # the headline instance's cost table and histogram
        {"name": "cost_table_n28", "kind": "cost_table", "n": 28, "m": 118},
        # the transverse-field comparator, 16 rounds
        {"name": "evolve_x_n26_c64", "kind": "evolve_x", "n": 26, "m": 109, "p": 16, "dtype": "complex64"},
        # one optimizer step of the angle network
        {"name": "train_b512", "kind": "train", "batch": 512, "step": 200},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _density_m(rng, n):
    return max(3, min(255, int(n * rng.uniform(2.0, 8.0) + 0.5)))


def draw(rng):
    kind = rng.choice([c["kind"] for c in listed()])
    dtype = rng.choice(["complex64", "complex128"])
    if kind in ("evolve", "plan", "evolve_from", "evolve_x"):
        top = {"evolve": 27, "plan": 22, "evolve_from": 24, "evolve_x": 25}[kind]
        n = rng.randint(6, top)
        p = _log_int(rng, 1, {"evolve": 64, "plan": 64, "evolve_from": 32, "evolve_x": 16}[kind])
        return {"kind": kind, "n": n, "m": _density_m(rng, n), "p": p, "dtype": dtype}
    if kind == "grad":
        n = rng.randint(8, 20)
        p = _log_int(rng, 1, 32)
        return {"kind": kind, "instances": _log_int(rng, 1, 64), "n": n, "m": _density_m(rng, n), "p": p,
                "dtype": dtype, "ckpt": rng.choice([0, 1, 3, 8])}
    dens = rng.choice(["scan", "max-sat"])
    n_lo = rng.randint(8, 14)
    n_hi = rng.randint(n_lo, 20)
    if kind == "scan":
        return {"kind": kind, "instances": _log_int(rng, 8, 1024), "n_lo": n_lo, "n_hi": n_hi, "density": dens,
                "nb": rng.randint(5, 64), "ng": rng.randint(5, 64), "grid": rng.choice(["box", "domain"]),
                "p_list": rng.choice(["1,4,16,64", "16", "64", "3,17", "1,2,5,11,33"]),
                "energy": rng.random() < 0.5}
    if kind == "crossing":
        # the good pairs lie outside [0, pi]^2, so the search takes the whole domain
        return {"kind": kind, "instances": _log_int(rng, 8, 128), "n_lo": n_lo, "n_hi": n_hi, "density": dens,
                "nb": rng.randint(90, 360), "ng": rng.randint(45, 181), "grid": "domain",
                "threshold": rng.choice([0.25, 0.5, 0.75])}
    if kind == "level_grad":
        return {"kind": kind, "instances": _log_int(rng, 1, 400), "n_lo": n_lo, "n_hi": n_hi, "density": dens,
                "p": _log_int(rng, 1, 150)}
    if kind == "hists":
        return {"kind": kind, "instances": _log_int(rng, 4, 4096), "n_lo": n_lo, "n_hi": n_hi, "density": dens}
    if kind == "cost_table":
        n = rng.randint(6, 28)
        return {"kind": kind, "n": n, "m": min(_density_m(rng, n), 200)}
    return {"kind": "train", "batch": _log_int(rng, 16, 1024), "step": rng.randint(1, 4000)}


# ---- preparation and passes ---------------------------------------------------------------
def _train_inputs(case, rng):
    """Features of the learned form's inputs (a normalized histogram, n, d, p),
    angle labels, and a network some steps into its training."""
    B = case["batch"]
    k = np.arange(128)
    n = rng.integers(12, 21, B)
    d = rng.choice([3.0, 4.2, 5.0], B)
    m = n * d
    w = np.exp(-0.5 * (k[None, :] - m[:, None] / 8) ** 2 / (7 * m[:, None] / 64)) * rng.uniform(0.8, 1.2, (B, 128))
    w *= k[None, :] <= m[:, None]
    w /= w.sum(axis=1, keepdims=True)
    x = np.concatenate([w, n[:, None] / 24, d[:, None] / 8, rng.choice([0, 2, 4, 6], (B, 1)) / 6], axis=1)
    y = np.stack([rng.uniform(3.4, 6.1, B), rng.uniform(0.07, 0.67, B)], axis=1)
    prm = np.zeros(g.MLP_NPARAMS)
    for key, fan_in in (("W1", 131), ("W2", 256), ("W3", 256)):
        off, shape = g.MLP_OFFSETS[key]
        a = np.zeros(shape)
        a[:fan_in] = rng.uniform(-1, 1, (fan_in, shape[1])) / math.sqrt(fan_in)
        prm[off:off + a.size] = a.ravel()
    for key in ("b1", "b2", "b3"):
        off, shape = g.MLP_OFFSETS[key]
        prm[off:off + shape[0]] = rng.uniform(-0.05, 0.05, shape[0])
    m1 = rng.standard_normal(g.MLP_NPARAMS) * 1e-4
    v1 = (1e-4 * rng.uniform(0.3, 3.0, g.MLP_NPARAMS)) ** 2
    off, shape = g.MLP_OFFSETS["W1"]
    m1[off + 131 * 256:off + 160 * 256] = 0.0
    v1[off + 131 * 256:off + 160 * 256] = 0.0
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)
    return f32(x), f32(y), f32(prm), f32(np.concatenate([m1, v1]))


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    s = {"case": case}
    if kind in ("evolve", "plan", "evolve_from", "evolve_x"):
        n, p, dt = case["n"], case["p"], _dtype(case)
        s["lits"] = _instance(case, rng)
        s["beta"], s["gamma"] = _angles(rng, p)
        s["cost"], hist = g.gqaoa_cost_table(n, s["lits"])
        s["target"] = int(_lowest(hist.cpu().numpy()))
        cdt = torch.complex64 if dt == g.C64 else torch.complex128
        s["psi"] = torch.empty(1 << n, dtype=cdt, device=DEV)
        if kind == "evolve_x":
            s["ws"] = torch.empty(g.gqaoa_x_workspace_bytes(n, p, dt), dtype=torch.uint8, device=DEV)
        elif kind == "plan":
            s["plan"] = g.EvolvePlan(n, case["m"], s["cost"], p, dtype=dt, target_level=s["target"], psi=s["psi"])
        else:
            s["ws"] = torch.empty(g.gqaoa_workspace_bytes(n, p, dt), dtype=torch.uint8, device=DEV)
        if kind == "evolve_from":
            s["psi0"] = _gauss_state(rng, n, cdt).to(DEV)
        return s
    if kind == "grad":
        n, m, I, p = case["n"], case["m"], case["instances"], case["p"]
        ns, ms = [n] * I, [m] * I
        lits = [_clauses(rng, n, m) for _ in range(I)]
        costs, off, hists = g.gqaoa_cost_batched(ns, ms, lits)
        s["costs"] = costs[:I << n].view(I, 1 << n) if n >= 6 else costs
        s["ms"], s["targets"] = np.array(ms, dtype=np.int32), _lowest(hists.cpu().numpy())
        s["beta"], s["gamma"] = _angles(rng, I, p)
        s["ws"] = torch.empty(g.gqaoa_grad_workspace_bytes(I, n, p, _dtype(case), case["ckpt"]), dtype=torch.uint8,
                              device=DEV)
        return s
    if kind in ("scan", "crossing", "level_grad", "hists"):
        ns, ms, lits = _batch(case, rng)
        flat = np.concatenate([l.reshape(-1) for l in lits])
        s.update(ns=ns, ms=ms, flat=flat)
        if kind == "hists":
            return s
        s["hists"] = g.gqaoa_hist_batched(ns, ms, flat).cpu().numpy()
        s["targets"] = _lowest(s["hists"])
        if kind == "level_grad":
            s["beta"], s["gamma"] = _angles(rng, case["instances"], case["p"])
            return s
        s["b"], s["g"] = _grids(case)
        if kind == "scan":
            s["plan"] = g.ScanPlan(ns, ms, s["hists"], s["b"], s["g"], _p_list(case), targets=s["targets"],
                                   with_energy=case["energy"])
        else:
            s["caps"] = _caps(ns, s["hists"], s["targets"], case["threshold"])
        return s
    if kind == "cost_table":
        s["lits"] = _instance(case, rng)
        return s
    x, y, prm, st = _train_inputs(case, rng)
    s.update(x=torch.from_numpy(x).to(DEV), y=torch.from_numpy(y).to(DEV), prm=torch.from_numpy(prm).to(DEV),
             st=torch.from_numpy(st).to(DEV), step=case["step"],
             grads=torch.empty(g.MLP_NPARAMS, dtype=torch.float32, device=DEV))
    return s


def _p_list(case):
    return [int(v) for v in case["p_list"].split(",")]


def _caps(ns, hists, targets, threshold):
    """Round caps of the search: 3 / sqrt(P) (9 / sqrt(P) for S = 75%)."""
    P = hists[np.arange(len(ns)), targets] / np.exp2(ns.astype(np.float64))
    return np.ceil((9.0 if threshold > 0.6 else 3.0) / np.sqrt(P)).clip(1, 400).astype(np.int32)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "evolve":
        return g.gqaoa_evolve(case["n"], case["m"], s["cost"], s["beta"], s["gamma"], dtype=_dtype(case),
                              psi=s["psi"], target_level=s["target"], workspace=s["ws"])
    if kind == "plan":
        return (s["psi"],) + s["plan"].run(s["beta"], s["gamma"])
    if kind == "evolve_from":
        s["psi"].copy_(s["psi0"])
        return g.gqaoa_evolve(case["n"], case["m"], s["cost"], s["beta"], s["gamma"], dtype=_dtype(case),
                              psi=s["psi"], init_uniform=False, target_level=s["target"], workspace=s["ws"])
    if kind == "evolve_x":
        return g.gqaoa_evolve_x(case["n"], case["m"], s["cost"], s["beta"], s["gamma"], dtype=_dtype(case),
                                psi=s["psi"], target_level=s["target"], workspace=s["ws"])
    if kind == "grad":
        return g.gqaoa_grad_batched(case["n"], s["ms"], s["costs"], s["beta"], s["gamma"], dtype=_dtype(case),
                                    targets=s["targets"], ckpt_every=case["ckpt"], workspace=s["ws"])
    if kind == "scan":
        psol, energy = s["plan"].run(s["b"], s["g"])
        return (psol, energy) if case["energy"] else psol
    if kind == "crossing":
        return g.gqaoa_scan_crossing(s["ns"], s["ms"], s["hists"], s["b"], s["g"], s["caps"], case["threshold"],
                                     targets=s["targets"])
    if kind == "level_grad":
        return g.gqaoa_hist_grad_batched(s["ns"], s["ms"], s["hists"], s["beta"], s["gamma"], targets=s["targets"])
    if kind == "hists":
        return g.gqaoa_hist_batched(s["ns"], s["ms"], s["flat"])
    if kind == "cost_table":
        return g.gqaoa_cost_table(case["n"], s["lits"])
    # one step of AngleMLP.train on a gathered batch
    out, act = g.gqaoa_mlp_forward(s["prm"], s["x"])
    dout, loss = g.gqaoa_mlp_loss(out, s["y"])
    g.gqaoa_mlp_backward(s["prm"], act, dout, grads=s["grads"])
    g.gqaoa_mlp_adam(s["prm"], s["grads"], s["st"], s["step"])
    return {"out": out, "dout": dout, "loss": loss, "grads": s["grads"], "params": s["prm"], "state": s["st"]}


# ---- algorithmic work ---------------------------------------------------------------------
def _levels(m):
    """Typical number of occupied levels of a random instance."""
    return min(m + 1.0, 6.5 * math.sqrt(7.0 * m / 64.0) + 1.0)


def _batch_m(case):
    n = 0.5 * (case["n_lo"] + case["n_hi"])
    return n * (6.3 if case["density"] == "max-sat" else 4.07)


def work(case):
    kind = case["kind"]
    cs = 16 if case.get("dtype") == "complex128" else 8
    if kind in ("evolve", "plan", "evolve_from"):
        # from |s> the state is one amplitude per level; from any state the
        # deviations from the level means only rotate
        N = 1 << case["n"]
        given = kind == "evolve_from"
        return {"bytes": N * (1 + cs * (2 if given else 1)),
                "flops": 12.0 * case["p"] * _levels(case["m"]) + (16.0 * N if given else 0.0)}
    if kind == "evolve_x":
        N = 1 << case["n"]
        return {"bytes": N * (1 + cs) * case["p"], "flops": N * case["p"] * (6.0 * case["n"] + 6.0)}
    if kind == "grad":
        return {"bytes": case["instances"] << case["n"],
                "flops": 40.0 * case["instances"] * case["p"] * _levels(case["m"])}
    if kind == "cost_table":
        N = 1 << case["n"]
        return {"bytes": N + 8 * (case["m"] + 1), "flops": 0.3 * N * case["m"]}
    if kind == "train":
        B = case["batch"]
        return {"bytes": 4.0 * (B * (131 + 2 + 4) + 7 * g.MLP_NPARAMS),
                "flops": 3.0 * 2.0 * B * (131 * 256 + 256 * 256 + 256 * 2)}
    I, m = case["instances"], _batch_m(case)
    K = _levels(m)
    if kind == "hists":
        N = (2.0 ** (case["n_hi"] + 1) - 2.0 ** case["n_lo"]) / (case["n_hi"] - case["n_lo"] + 1)
        return {"bytes": I * (12.0 * m + 8.0 * (m + 1)), "flops": 0.3 * N * m * I}
    if kind == "level_grad":
        return {"bytes": I * (12.0 * K + 32.0 * case["p"]), "flops": 40.0 * I * K * case["p"]}
    cells = float(I) * case["nb"] * case["ng"]
    if kind == "scan":
        pl = _p_list(case)
        return {"bytes": cells * 4 * len(pl) * (2 if case["energy"] else 1), "flops": cells * 12.0 * K * pl[-1]}
    return {"bytes": cells * 4, "flops": cells * 12.0 * K * 30}


# ---- the same outputs in 64 bits -------------------------------------------------------------
def _costs64(n, lits):
    z = torch.arange(1 << n, dtype=torch.int32, device=DEV)
    cost = torch.zeros(1 << n, dtype=torch.uint8, device=DEV)
    for clause in lits.reshape(-1, 3):
        f = None
        for lit in clause.tolist():
            hit = ((z >> (lit >> 1)) & 1) == (lit & 1)
            f = hit if f is None else f.logical_and_(hit)
        cost += f
    return cost


def _hist64(n, m, lits):
    return torch.bincount(_costs64(n, lits).int(), minlength=m + 1)[:m + 1].double()


def _phase64(gamma, m):
    a = torch.arange(m + 1, dtype=torch.float64, device=DEV) * float(gamma)
    return torch.polar(torch.ones_like(a), -a)


def _mix64(beta):
    return complex(math.cos(beta) - 1.0, -math.sin(beta))


def _evolve64(case, s, x_mixer):
    n, m, t = case["n"], case["m"], s["target"]
    cost = _costs64(n, s["lits"]).int()
    cf = cost.double()
    psi = (s["psi0"].to(torch.complex128) if "psi0" in s
           else torch.full((1 << n,), 2.0 ** (-n / 2), dtype=torch.complex128, device=DEV))
    ro = []

    def readout():
        pr = psi.real ** 2 + psi.imag ** 2
        ro.append([float(pr[cost == t].sum()), float((cf * pr).sum()), float(pr.sum())])

    readout()
    for b, gm in zip(s["beta"], s["gamma"]):
        psi = psi * _phase64(gm, m)[cost]
        if x_mixer:
            c, sn = math.cos(b), math.sin(b)
            for q in range(n):
                v = psi.view(-1, 2, 1 << q)
                psi = (c * v - 1j * sn * v.flip(1)).reshape(-1)
        else:
            psi = psi + _mix64(b) * psi.sum() / (1 << n)
        readout()
    r = np.array(ro)
    return psi, r[:, 0].copy(), r[:, 1].copy(), r[:, 2].copy()


def _grad64(case, s):
    n, p, I = case["n"], case["p"], case["instances"]
    N = 1 << n
    P, db, dg = np.empty(I), np.empty((I, p)), np.empty((I, p))
    for i in range(I):
        cost = s["costs"].reshape(I, N)[i].int()
        cf = cost.double()
        psi = torch.full((N,), 2.0 ** (-n / 2), dtype=torch.complex128, device=DEV)
        phis, sums = [], []
        for k in range(p):
            phi = psi * _phase64(s["gamma"][i, k], case["m"])[cost]
            S = phi.sum()
            psi = phi + _mix64(s["beta"][i, k]) * S / N
            phis.append(phi)
            sums.append(S)
        lam = torch.where(cost == int(s["targets"][i]), psi, torch.zeros_like(psi))
        P[i] = float((lam.real ** 2 + lam.imag ** 2).sum())
        for k in range(p - 1, -1, -1):
            b = s["beta"][i, k]
            L = lam.sum()
            mu = lam + _mix64(-b) * L / N
            db[i, k] = 2 * float((L.conj() * sums[k] * complex(math.cos(b), -math.sin(b)) * -1j).real) / N
            dg[i, k] = 2 * float((mu.conj() * phis[k] * cf).sum().imag)
            lam = mu * _phase64(s["gamma"][i, k], case["m"])[cost].conj()
    return P, db, dg


def _level_batch64(s):
    """Weights [I, L] of every level, occupied or not, and the levels."""
    w = torch.from_numpy(s["hists"].astype(np.float64)).to(DEV) / torch.exp2(
        torch.from_numpy(s["ns"].astype(np.float64)).to(DEV))[:, None]
    return w, torch.arange(w.shape[1], dtype=torch.float64, device=DEV)


def _scan64(case, s):
    w, lev = _level_batch64(s)
    I, L = w.shape
    pl = _p_list(case)
    nb, ng = case["nb"], case["ng"]
    psol = torch.empty((I, len(pl), ng, nb), dtype=torch.float64, device=DEV)
    energy = torch.empty_like(psol) if case["energy"] else None
    a = lev[:, None] * torch.from_numpy(s["g"]).to(DEV)[None, :]                     # [L, ng]
    ph = torch.polar(torch.ones_like(a), -a).repeat_interleave(nb, dim=1)            # [L, ng nb]
    bb = torch.from_numpy(s["b"]).to(DEV)
    mix = (torch.polar(torch.ones_like(bb), -bb) - 1.0).repeat(ng)                   # [ng nb]
    for i in range(I):
        k = torch.nonzero(w[i] > 0).flatten()
        wi, phi = w[i, k], ph[k]
        wc = wi.to(torch.complex128)
        b = torch.ones((k.numel(), ng * nb), dtype=torch.complex128, device=DEV)
        t = int(s["targets"][i])
        for j in range(1, pl[-1] + 1):
            b = b * phi
            b = b + mix * torch.mv(b.t(), wc)
            if j in pl:
                q = pl.index(j)
                pr = wi[:, None] * (b.real ** 2 + b.imag ** 2)
                psol[i, q] = pr[k == t].sum(0).view(ng, nb)
                if energy is not None:
                    energy[i, q] = (lev[k][:, None] * pr).sum(0).view(ng, nb)
    return (psol, energy) if energy is not None else psol


def _level_grad64(case, s):
    w, lev = _level_batch64(s)
    I, L = w.shape
    p = case["p"]
    wc = w.to(torch.complex128)
    bt, gm = torch.from_numpy(s["beta"]).to(DEV), torch.from_numpy(s["gamma"]).to(DEV)
    e = lambda x: torch.polar(torch.ones_like(x), x)
    psi = torch.ones((I, L), dtype=torch.complex128, device=DEV)
    phis, sums = [], []
    for k in range(p):
        phi = psi * e(-gm[:, k, None] * lev)
        S = (wc * phi).sum(1)
        psi = phi + ((e(-bt[:, k]) - 1.0) * S)[:, None]
        phis.append(phi)
        sums.append(S)
    hit = torch.zeros_like(w)
    hit[torch.arange(I), torch.from_numpy(s["targets"]).long()] = 1.0
    lam = psi * hit
    P = (w * (lam.real ** 2 + lam.imag ** 2)).sum(1)
    db, dg = np.empty((I, p)), np.empty((I, p))
    for k in range(p - 1, -1, -1):
        Ls = (wc * lam).sum(1)
        mu = lam + ((e(bt[:, k]) - 1.0) * Ls)[:, None]
        db[:, k] = 2 * (-1j * e(-bt[:, k]) * Ls.conj() * sums[k]).real.cpu().numpy()
        dg[:, k] = 2 * (w * lev * (mu.conj() * phis[k]).imag).sum(1).cpu().numpy()
        lam = mu * e(gm[:, k, None] * lev)
    return P.cpu().numpy(), db, dg


def _train64(case, seed):
    """The step in float64; the network's storage points (inputs, weights,
    hidden activations, pre-activation gradients) are bfloat16."""
    x, y, prm, st = (torch.from_numpy(a).double() for a in _train_inputs(case, np.random.default_rng(seed)))
    B = case["batch"]
    bf = lambda t: t.float().bfloat16().double()
    par = {k: prm[o:o + int(np.prod(sh))].view(sh) for k, (o, sh) in g.MLP_OFFSETS.items()}
    cdf = lambda z: 0.5 * (1.0 + torch.erf(z / math.sqrt(2.0)))
    dgelu = lambda z: cdf(z) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)
    xb = torch.zeros((B, 160), dtype=torch.float64)
    xb[:, :131] = bf(x)
    W1, W2, W3 = bf(par["W1"]), bf(par["W2"]), bf(par["W3"])
    z1 = xb @ W1 + par["b1"]
    h1 = bf(z1 * cdf(z1))
    z2 = h1 @ W2 + par["b2"]
    h2 = bf(z2 * cdf(z2))
    out = h2 @ W3 + par["b3"]
    sg = torch.sigmoid(out)
    r = sg - y / torch.tensor([2.0 * math.pi, math.pi], dtype=torch.float64)
    loss = (r * r).sum() / B
    dout = 2.0 * r * sg * (1.0 - sg) / B
    dz2 = bf((dout @ W3.t()) * dgelu(z2))
    dz1 = bf((dz2 @ W2.t()) * dgelu(z1))
    gr = {"W3": h2.t() @ dout, "b3": dout.sum(0), "W2": h1.t() @ dz2, "b2": dz2.sum(0), "W1": xb.t() @ dz1,
          "b1": dz1.sum(0)}
    grads = torch.zeros(g.MLP_NPARAMS, dtype=torch.float64)
    for k, (o, sh) in g.MLP_OFFSETS.items():
        grads[o:o + int(np.prod(sh))] = gr[k].reshape(-1)
    m1, v1 = st[:g.MLP_NPARAMS], st[g.MLP_NPARAMS:]
    m1 = 0.9 * m1 + 0.1 * grads
    v1 = 0.999 * v1 + 0.001 * grads * grads
    c1, c2 = 1.0 - 0.9 ** case["step"], 1.0 - 0.999 ** case["step"]
    new = prm - 1e-3 * (m1 / c1) / (torch.sqrt(v1 / c2) + 1e-8)
    return {"out": out, "dout": dout, "loss": loss.reshape(1), "grads": grads, "params": new,
            "state": torch.cat([m1, v1])}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("crossing", "hists", "cost_table"):   # whole numbers
        return None
    if kind == "train":
        return _train64(case, seed)
    s = prepare(case, seed)
    if kind in ("evolve", "plan", "evolve_from", "evolve_x"):
        return _evolve64(case, s, kind == "evolve_x")
    if kind == "grad":
        return _grad64(case, s)
    if kind == "scan":
        return _scan64(case, s)
    return _level_grad64(case, s)

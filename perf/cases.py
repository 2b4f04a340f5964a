"""The work that the library's speed is measured on: what a user has it do, through its public
entry points, over the range of sizes, precisions and options it is used with.

A case is a dict of plain values.  `kind` says which path it takes:

  md        blocks of 100 MD steps and one double-bridging sweep at the paper's attempt rate
            (bench.py's production step), then the state is read out, as for a trajectory frame
            or a checkpoint; one melt, or a batch of uneven ones
  ramp      the n-ramp protocol driver over some of its stages, then the state
  learned   md with the learned proposal (a network set beforehand)
  log       MD and a logged sweep: the training records of the learned proposal
  train     one full-batch Adam step of the proposal's network
  readings  what is read at the end of a protocol stage: R^2(n)/n, energies, g(r), S(q)

Melts start as the library makes them (seeded random walks and the 1000-step warm-up), so the
inputs of a case are a melt under its own distribution of positions, velocities and bonds.
"""
import math

import numpy as np
import torch

import paper_2109_11001_amd as kg

RHO = 0.85
BLOCK = 100  # MD steps between sweeps
PREC = {"fp64": kg.PREC_FP64, "mixed": kg.PREC_MIXED}
# the uneven batch: melt i has (chains / CHAIN_DIV[i mod 4]) chains of beads * BEAD_MUL[i mod 4]
# beads and kappa = KAPPAS[i mod 6]
CHAIN_DIV = (1.0, 1.8, 3.0, 4.5)
BEAD_MUL = (1, 2, 4, 8)
KAPPAS = (0.0, 0.5, 1.0, 1.5, 2.0, 2.5)


def listed():
    return [
        # the smallest melt in use (20 chains of 50 beads, plain FP64 path): latency and launches
        {"name": "md-1k-fp64", "kind": "md", "M": 20, "N": 50, "kappa": 1.5, "n": 2.0, "dt": 0.01,
         "precision": "fp64", "melts": 1, "blocks": 2},
        # short chains that equilibrate within a run; many chains, so the sweep's list is long
        {"name": "md-50k-short-chains", "kind": "md", "M": 2000, "N": 25, "kappa": 2.0, "n": 2.0, "dt": 0.01,
         "precision": "mixed", "melts": 1, "blocks": 10},
        # the benchmark's melt, mixed precision
        {"name": "md-200k-mixed", "kind": "md", "M": 200, "N": 1000, "kappa": 2.0, "n": 2.0, "dt": 0.01,
         "precision": "mixed", "melts": 1, "blocks": 10},
        # the same melt on the plain FP64 path
        {"name": "md-200k-fp64", "kind": "md", "M": 200, "N": 1000, "kappa": 2.0, "n": 2.0, "dt": 0.01,
         "precision": "fp64", "melts": 1, "blocks": 2},
        # stiff long chains with the hard core of the standard model (n = 12)
        {"name": "md-200k-stiff-n12", "kind": "md", "M": 100, "N": 2000, "kappa": 3.0, "n": 12.0, "dt": 0.01,
         "precision": "mixed", "melts": 1, "blocks": 5},
        # the batched form: uneven melts of different stiffness in one batch
        {"name": "md-470k-batch16", "kind": "md", "M": 225, "N": 100, "kappa": 0.0, "n": 2.0, "dt": 0.01,
         "precision": "mixed", "melts": 16, "blocks": 4},
        # a melt whose state leaves the last-level cache
        {"name": "md-1M-mixed", "kind": "md", "M": 1000, "N": 1000, "kappa": 2.0, "n": 2.0, "dt": 0.01,
         "precision": "mixed", "melts": 1, "blocks": 4},
        # the paper's melt (1000 chains of 400 beads, dt = tau / 125) through three stages of the
        # n-ramp, whose exponents take the general form of the pair potential
        {"name": "ramp-400k", "kind": "ramp", "M": 1000, "N": 400, "kappa": 2.0, "n": 3.0, "dt": 0.008,
         "precision": "mixed", "stages": 3, "steps": 300},
        # the learned proposal on the 200 x 1000 melt
        {"name": "learned-200k", "kind": "learned", "M": 200, "N": 1000, "kappa": 2.5, "n": 2.0, "dt": 0.01,
         "precision": "mixed", "blocks": 3},
        # training records from six melts of different stiffness
        {"name": "log-6x25k", "kind": "log", "M": 125, "N": 200, "melts": 6, "attempts": 300},
        # a training step on the records of a whole run (full batch)
        {"name": "train-46000", "kind": "train", "rows": 46000},
        # the readings at the end of a stage of the paper's melt
        {"name": "readings-400k", "kind": "readings", "M": 1000, "N": 400, "kappa": 2.0, "n": 3.0, "nq": 5600},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _melt_shape(rng, lo, hi, n_lo=20, n_hi=2000):
    """Chains and beads of a melt of lo to hi monomers.  At most 1000 chains (2000 short ones): the
    sweep refuses a list that grows past 3072 candidates, which more chains than that come near."""
    nm = _log_uniform(rng, lo, hi)
    n = _log_uniform(rng, n_lo, min(n_hi, max(n_lo, nm // 8)))
    most = 2000 if n <= 40 else 1000
    return max(4, min(most, nm // n)), max(n, nm // most if n > 40 else n)


def draw(rng):
    kind = rng.choice(("md", "md", "md", "md", "batch", "ramp", "learned", "log", "train", "readings"))
    kappa = rng.choice((0.0, 0.5, 1.0, 1.5, 2.0, 2.5, 3.0, 5.5))
    if kind == "train":
        return {"kind": "train", "rows": _log_uniform(rng, 64, 46000)}
    if kind == "log":
        M, N = _melt_shape(rng, 1000, 40000, 20, 400)
        return {"kind": "log", "M": M, "N": N, "melts": rng.randint(1, 6), "attempts": _log_uniform(rng, 50, 1000)}
    if kind == "readings":
        M, N = _melt_shape(rng, 2000, 400000)
        return {"kind": "readings", "M": M, "N": N, "kappa": kappa, "n": rng.choice(kg.XI),
                "nq": _log_uniform(rng, 100, 5600)}
    if kind == "ramp":
        M, N = _melt_shape(rng, 2000, 400000)
        return {"kind": "ramp", "M": M, "N": N, "kappa": kappa, "n": rng.choice(kg.XI[1:9]), "dt": 0.008,
                "precision": "mixed", "stages": rng.randint(1, 3), "steps": rng.randint(100, 300)}
    if kind == "learned":
        M, N = _melt_shape(rng, 2000, 200000, 50, 2000)
        return {"kind": "learned", "M": M, "N": N, "kappa": kappa, "n": 2.0, "dt": 0.01,
                "precision": rng.choice(("mixed", "fp64")), "blocks": 2}
    if kind == "batch":
        M, N = _melt_shape(rng, 1000, 22000, 20, 200)
        return {"kind": "md", "M": max(M, 20), "N": N, "kappa": 0.0, "n": rng.choice((2.0, 5.0, 12.0)), "dt": 0.01,
                "precision": rng.choice(("mixed", "fp64")), "melts": rng.randint(2, 16), "blocks": 2}
    M, N = _melt_shape(rng, 1000, 700000)
    return {"kind": "md", "M": M, "N": N, "kappa": kappa, "n": rng.choice((2.0, 2.0, 5.75, 12.0)), "dt": 0.01,
            "precision": rng.choice(("mixed", "fp64")), "melts": 1, "blocks": rng.randint(1, 2)}


def _melts(case, seed):
    """The parameters of a case's melts."""
    base = dict(rho=RHO, dt=case.get("dt", 0.01), n_exp=case.get("n", 2.0), seed=seed,
                precision=PREC[case.get("precision", "mixed")])
    if case["kind"] == "learned":
        base["proposal"] = kg.PROPOSAL_LEARNED
    if case["kind"] == "log":
        return [dict(base, M=case["M"], N=case["N"], kappa=KAPPAS[i % 6], melt_id=i) for i in range(case["melts"])]
    if case.get("melts", 1) > 1:
        return [dict(base, M=max(4, int(case["M"] / CHAIN_DIV[i % 4])), N=case["N"] * BEAD_MUL[i % 4],
                     kappa=KAPPAS[i % 6], melt_id=i) for i in range(case["melts"])]
    return [dict(base, M=case["M"], N=case["N"], kappa=case["kappa"])]


def _network(seed):
    """Seeded weights of the 25-128-128-128-1 proposal network."""
    rng = np.random.default_rng(seed)
    parts = []
    for rows, cols in ((128, 25), (128, 128), (128, 128), (1, 128)):
        parts += [rng.normal(0.0, 0.3, rows * cols), rng.normal(0.0, 0.3, rows)]
    return np.concatenate(parts).astype(np.float32)


def _q_vectors(L, nq, seed):
    """nq reciprocal-lattice vectors spread evenly over 0 < |q| < 12 / sigma."""
    rng = np.random.default_rng(seed)
    v = rng.normal(size=(nq, 3))
    v *= (12.0 * (np.arange(nq) + rng.random(nq)) / nq / np.linalg.norm(v, axis=1))[:, None]
    n = np.rint(v * L / (2 * math.pi)).astype(np.int32)
    n[(n == 0).all(axis=1), 0] = 1
    return n


def _train_inputs(case, seed):
    """Rows as logged sweeps give them: 24 coordinates of eight beads around two bonds and kappa."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = case["rows"]
    feat = torch.randn((n, 25), generator=g, device="cuda")
    feat[:, 24] = 0.5 * torch.randint(0, 7, (n,), generator=g, device="cuda").float()
    label = (torch.rand(n, generator=g, device="cuda") < 0.2).to(torch.int32)
    return feat, label


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        feat, label = _train_inputs(case, seed)
        return {"case": case, "feat": feat, "label": label,
                "trainer": kg.Trainer(_network(seed), max_batch=case["rows"], lr=3e-3)}
    batch = kg.Batch(_melts(case, seed))
    state = {"case": case, "batch": batch}
    if kind == "learned":
        batch.set_proposal_net(_network(seed), 0.1)
    if kind == "ramp":
        i = kg.XI.index(case["n"])
        state["stages"] = list(kg.XI[i : i + case["stages"]])
    if kind == "readings":
        state["q"] = _q_vectors(batch.geom[0]["L"], case["nq"], seed)
    return state


def _frame(batch, k):
    s = batch.get_state(k)
    return {"x": s["x"], "v": s["v"], "chains": s["chains"]}


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "train":
        t = state["trainer"]
        loss = t.step(state["feat"], state["label"])
        return {"params": t.params, "m": t.m, "v": t.v, "loss": loss}
    b = state["batch"]
    if kind == "readings":
        r2n, ell_k, bond = b.observables()
        counts, g = b.pair_correlation(3.0, 150) if b.geom[0]["L"] >= 8.0 else (np.zeros(1), np.zeros(1))
        return {"r2n": r2n, "ell_k": ell_k, "bond": bond, "energy": b.energy(), "counts": counts.astype(np.int64),
                "g": g, "S": b.structure_factor(state["q"])}
    if kind == "ramp":
        stages = b.run_protocol(state["stages"], [case["steps"]] * len(state["stages"]), sweep_every=BLOCK)
        swaps = np.array([[s["steps"], s["attempts"], s["no_candidate"], s["accepted"]] for s in stages])
        return {"frame": _frame(b, 0), "swaps": swaps}
    if kind == "log":
        b.md_steps(BLOCK)
        stats, feat, label, n = b.db_sweep_log(case["attempts"], cap=case["attempts"])
        return {"feat": torch.cat([feat[k, : n[k]] for k in range(b.nm)]),
                "label": torch.cat([label[k, : n[k]] for k in range(b.nm)]), "accepted": [s["accepted"] for s in stats]}
    swaps, dE = [], []
    for _ in range(case["blocks"]):
        b.md_steps(BLOCK)
        stats = b.db_sweep()
        swaps.append([[s["attempts"], s["accepted"], s["sum_ncand"]] for s in stats])
        dE.append([s["sum_dE_accepted"] for s in stats])
    return {"frames": [_frame(b, k) for k in range(b.nm)], "swaps": np.array(swaps), "dE": np.array(dE)}


# bytes a monomer's step cannot do without: neighbours' and chain partners' positions, the state
# read and written once (4-byte coordinates for the forces of the mixed path, 8-byte state)
STEP_BYTES = {"mixed": 168.0, "fp64": 196.0}
STEP_FLOPS = 500.0    # about 5 neighbours in range, two bonds, three angles, noise, update
FRAME_BYTES = 2 * 52  # x, v and the chain table, read and written once
NET_MAC = 25 * 128 + 2 * 128 * 128 + 128


def work(case):
    kind = case["kind"]
    if kind == "train":
        n = case["rows"]
        return {"bytes": 104.0 * n + 24.0 * (NET_MAC + 385), "flops": 6.0 * NET_MAC * n}
    if kind == "readings":
        nm = case["M"] * case["N"]
        pairs = nm * RHO * 4.0 / 3.0 * math.pi * 27.0
        return {"bytes": 3 * 24.0 * nm + 28.0 * nm, "flops": 9.0 * nm * case["N"] / 2 + 12.0 * pairs + 30.0 * nm * case["nq"]}
    if kind == "log":
        nm = case["M"] * case["N"] * case["melts"]
        return {"bytes": nm * (STEP_BYTES["mixed"] * BLOCK + 32.0) + 104.0 * case["melts"] * case["attempts"],
                "flops": nm * STEP_FLOPS * BLOCK}
    nm = sum(m["M"] * m["N"] for m in _melts(case, 0))
    steps = case["stages"] * case["steps"] if kind == "ramp" else case["blocks"] * BLOCK
    sweeps = steps // BLOCK
    return {"bytes": nm * (STEP_BYTES[case["precision"]] * steps + 32.0 * sweeps + FRAME_BYTES), "flops": nm * STEP_FLOPS * steps}


# ---- the same results in 64 bits, written with torch and numpy alone
def _exact_train(case, seed):
    feat, label = _train_inputs(case, seed)
    P = torch.as_tensor(_network(seed)).cuda().double()
    n, sizes, at, W = case["rows"], ((128, 25), (128, 128), (128, 128), (1, 128)), 0, []
    for rows, cols in sizes:
        W.append([P[at : at + rows * cols].view(rows, cols), P[at + rows * cols : at + rows * (cols + 1)]])
        at += rows * (cols + 1)
    code = lambda t, lo: (64.0 * t).round().clamp(lo, 255.0) / 64.0  # noqa: E731
    h, acts, masks = code(feat.double(), -255.0), [], []
    for k, (w, b) in enumerate(W):
        acts.append(h)
        z = (h @ code(w, -255.0).T).float() + b.float()  # the pre-activation is an FP32 value by definition
        if k == 3:
            break
        masks.append((z > 0) & (z < 255.0 / 16.0))
        h = (16.0 * z).round().clamp(0.0, 255.0).double() / 16.0
    z, y = z[:, 0].double(), label.double()
    loss = (torch.nn.functional.softplus(z) - y * z).mean()
    delta, grads = ((torch.sigmoid(z) - y) / n)[:, None], []
    for k in (3, 2, 1, 0):
        grads = [(delta.T @ acts[k]).reshape(-1), delta.sum(0)] + grads
        if k:
            delta = (delta @ code(W[k][0], -255.0)) * masks[k - 1]
    g = torch.cat(grads)
    b1, b2, eps, lr = 0.9, 0.999, 1e-8, 3e-3
    m, v = (1 - b1) * g, (1 - b2) * g * g
    new = P - lr * (m / (1 - b1)) / ((v / (1 - b2)).sqrt() + eps)
    weight, at = torch.zeros_like(P, dtype=torch.bool), 0
    for rows, cols in sizes:
        weight[at : at + rows * cols] = True
        at += rows * (cols + 1)
    new = torch.where(weight, new.clamp(-255.0 / 64.0, 255.0 / 64.0), new)
    return {"params": new, "m": m, "v": v, "loss": loss.reshape(1)}


def _pair_distances(x, L, reach):
    """Distances of all ordered pairs nearer than about `reach`, a batch of them at a time."""
    nc = max(3, int(L / reach))
    c = (x * (nc / L)).long().clamp(0, nc - 1)
    cell = (c[2] * nc + c[1]) * nc + c[0]
    order = torch.argsort(cell)
    count = torch.bincount(cell, minlength=nc**3)
    start = torch.cumsum(count, 0) - count
    cap = int(count.max())
    slot = torch.arange(cap, device=x.device)
    member = (start[:, None] + slot).clamp(max=x.shape[1] - 1)
    table = torch.where(slot < count[:, None], order[member], -1).view(nc, nc, nc, cap)
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                other = torch.roll(table, (-dz, -dy, -dx), (0, 1, 2))
                for z in range(nc):
                    i, j = table[z].unsqueeze(-1), other[z].unsqueeze(-2)
                    d = x[:, i.clamp(min=0)] - x[:, j.clamp(min=0)]
                    r = (d - L * torch.round(d / L)).square().sum(0).sqrt()
                    yield r[(i >= 0) & (j >= 0) & (i != j)]


def _fit_ell_k(r2n, N, l0):
    """l_K of the worm-like-chain form by least squares: the root of the derivative, by bisection."""
    n = np.arange((N + 3) // 4, N // 2 + 1)
    y = r2n[n - 1] / l0

    def slope(k):
        e = np.exp(-2 * n * l0 / k)
        f = k * (1 - k / (2 * n * l0) * (1 - e))
        return np.sum((f - y) * (1 + e - k / (n * l0) * (1 - e)))

    grid = np.exp(np.linspace(math.log(0.05), math.log(1e4), 257))
    sse = [np.sum((k * (1 - k / (2 * n * l0) * (1 - np.exp(-2 * n * l0 / k))) - y) ** 2) for k in grid]
    i = int(np.argmin(sse))
    lo, hi = grid[max(i - 1, 0)], grid[min(i + 1, 256)]
    for _ in range(100):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if slope(mid) < 0 else (lo, mid)
    return 0.5 * (lo + hi)


def _exact_readings(case, seed):
    state = prepare(case, seed)  # the melt in hand: only its positions, velocities and chains are taken
    b, q = state["batch"], state["q"]
    s, M, N, L = b.get_state(0), case["M"], case["N"], b.geom[0]["L"]
    x = torch.as_tensor(s["x"]).cuda()
    ch = torch.as_tensor(s["chains"].astype(np.int64)).cuda()
    image = lambda d: d - L * torch.round(d / L)  # noqa: E731
    bonds = image(x[:, ch[:, 1:]] - x[:, ch[:, :-1]])  # [3][M][N - 1]
    length = bonds.square().sum(0).sqrt()
    walk = torch.cat([torch.zeros_like(bonds[:, :, :1]), bonds.cumsum(2)], 2)
    r2n = np.array([float((walk[:, :, n:] - walk[:, :, :-n]).square().sum()) / (M * (N - n)) / n for n in range(1, N)])
    l0 = float(length.mean())
    # energies (Eqs. 3-6, 9-10, with the FENE argument continued below its floor)
    e, R0 = case["n"], 1.5
    ell, two = 0.960897, 2.0 ** (e / 6.0)
    k_fene = 6 * e * (R0**2 - ell**2) * (two * ell**-e - 2 * ell**-6) / ((e - 6) * R0**2 * ell**2)
    arg, floor = 1 - (length / R0) ** 2, 0.02
    logs = torch.where(arg < floor, math.log(floor) + (arg - floor) / floor, arg.clamp(min=floor).log())
    cosine = (bonds[:, :, 1:] * bonds[:, :, :-1]).sum(0) / (length[:, 1:] * length[:, :-1])
    u_pair, counts, far = 0.0, torch.zeros(150, dtype=torch.int64, device="cuda"), L >= 8.0
    for r in _pair_distances(x, L, 3.0 if far else 2.0 ** (1 / 6)):
        near = r[r < 2.0 ** (1 / 6)]
        u_pair += 0.5 * float((6 * two / (e - 6) * near**-e - 2 * e / (e - 6) * near**-6 + 1).sum())
        counts += torch.bincount((r[r < 3.0] / 0.02).long().clamp(max=149), minlength=150)
    energy = [u_pair, -0.5 * k_fene * R0**2 * float(logs.sum()), case["kappa"] * float((1 - cosine).sum()),
              0.5 * float(torch.as_tensor(s["v"]).square().sum())]
    i = np.arange(150.0)
    shell = 4.0 / 3.0 * math.pi * ((i + 1) ** 3 - i**3) * 0.02**3
    g = counts.cpu().numpy() / (M * N * RHO * shell) if far else np.zeros(1)
    S = np.empty(len(q))
    for at in range(0, len(q), 32):
        t = torch.as_tensor(q[at : at + 32].astype(np.float64)).cuda() @ (x / L)
        ph = 2 * math.pi * (t - t.round())
        S[at : at + 32] = ((ph.cos().sum(1).square() + ph.sin().sum(1).square()) / (M * N)).cpu().numpy()
    return {"r2n": r2n, "ell_k": _fit_ell_k(r2n, N, l0) if N >= 4 else None, "bond": l0, "energy": np.array(energy),
            "counts": None, "g": g, "S": S}


def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] == "readings":
        return _exact_readings(case, seed)
    return None  # a trajectory of hundreds of chaotic steps with sweeps has no independent 64-bit value

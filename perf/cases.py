"""What users of this framework have it compute, as measurable cases.

A case is a dict of plain values; `prepare` makes its inputs on the GPU from a
seed, `run` is one pass through the public entry points, `work` the bytes and
operations such a pass cannot do without and `exact` the same result by direct
summation in 64 bits, in plain torch.

Kinds of case:
  forces   one force evaluation, tree included (FMM.forces)
  frozen   a step that keeps the tree, replayed as a HIP graph (FMM.forces_frozen)
  batch    an ensemble of independent clusters in one pass (FMM.forces_batch)
  jerk     forces and their time derivative, for a Hermite integrator (FMM.jerk)
  rollout  a differentiable leapfrog, forward and backward (rollout.leapfrog)
  direct   the compensated direct sum that force errors are measured against (fmm.direct)
"""
import math

import numpy as np
import torch

from paper_2012_02207_amd import fmm, rollout, workloads

DEV = "cuda:0"
SOFT = 1e-5      # softening lengths in use, in Henon units: none, or this
DT = 1.0 / 1024  # leapfrog step of the rollouts


def listed():
    return [
        # a small cluster, stepped on its own: latency and launches
        dict(name="small_fp64", kind="forces", n=1000, p=6, err_tol=1e-6, precision="fp64", soft=0.0,
             model="plummer"),
        # the 4096-body configuration of the benchmark
        dict(name="plummer_4k_fp64", kind="forces", n=4096, p=6, err_tol=1e-6, precision="fp64", soft=0.0,
             model="plummer"),
        # one ordinary star cluster of the ensemble's upper sizes, softened
        dict(name="cluster_30k_mixed", kind="forces", n=30011, p=8, err_tol=1e-6, precision="mixed", soft=SOFT,
             model="plummer"),
        # the force evaluation of the 2^18-body rollout configuration
        dict(name="plummer_256k_fp64", kind="forces", n=1 << 18, p=10, err_tol=1e-7, precision="fp64", soft=0.0,
             model="plummer"),
        # the headline benchmark
        dict(name="plummer_1m_mixed", kind="forces", n=1 << 20, p=10, err_tol=1e-7, precision="mixed", soft=0.0,
             model="plummer"),
        # the largest configuration: Kroupa masses around a massive central body
        dict(name="kroupa_4m_mixed", kind="forces", n=1 << 22, p=12, err_tol=1e-7, precision="mixed", soft=0.0,
             model="kroupa"),
        # the paper's production parameters (section 4.1): N = 10^5, p = 20
        dict(name="plummer_100k_p20", kind="forces", n=100000, p=20, err_tol=1e-7, precision="fp64", soft=0.0,
             model="plummer"),
        # a step loop that rebuilds its tree only now and then
        dict(name="frozen_16k_mixed", kind="frozen", n=16384, p=8, err_tol=1e-6, precision="mixed", soft=SOFT,
             model="plummer"),
        # the ensemble benchmark: 256 clusters of 2^10 to 2^16 bodies
        dict(name="ensemble_256_mixed", kind="batch", count=256, lo_exp=10.0, hi_exp=16.0, p=8, err_tol=1e-6,
             precision="mixed", soft=0.0),
        # fourth-order Hermite integration
        dict(name="jerk_50k", kind="jerk", n=50021, p=10, err_tol=1e-7, soft=SOFT),
        # gradients of final states with respect to positions, velocities and masses
        dict(name="rollout_64k", kind="rollout", n=65537, p=10, err_tol=1e-7, soft=SOFT, steps=4),
        # the error check of the benchmark: 4096 sinks of the 2^20-body model
        dict(name="direct_4096_of_1m", kind="direct", n=1 << 20, nsink=4096, soft=0.0),
    ]


def _log(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi], odd as often as not."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _order(rng):
    """An expansion order and a tolerance that is used with it."""
    p = rng.randint(5, 12)
    return p, (1e-5 if p <= 5 else 1e-6 if p <= 8 else 1e-7)


def draw(rng):
    kind = rng.choice(["forces", "forces", "forces", "high", "frozen", "batch", "jerk", "rollout", "direct"])
    p, err_tol = _order(rng)
    soft = rng.choice([0.0, SOFT])
    precision = rng.choice(["fp64", "mixed"])
    if kind == "forces":
        n = _log(rng, 700, (1 << 20) if precision == "fp64" else (1 << 21))
        return dict(kind="forces", n=n, p=p, err_tol=err_tol, precision=precision, soft=soft,
                    model=rng.choice(["plummer", "plummer", "kroupa", "cube"]))
    if kind == "high":  # the orders of the paper's accuracy grid above the unrolled kernels
        return dict(kind="forces", n=_log(rng, 8000, 100000), p=rng.randint(13, 20), err_tol=1e-7,
                    precision="fp64", soft=soft, model="plummer")
    if kind == "frozen":
        return dict(kind="frozen", n=_log(rng, 1500, 150000), p=p, err_tol=err_tol, precision=precision,
                    soft=soft, model=rng.choice(["plummer", "kroupa"]))
    if kind == "batch":
        lo = rng.uniform(9.0, 11.0)
        return dict(kind="batch", count=rng.randint(5, 200), lo_exp=lo, hi_exp=rng.uniform(lo + 1.0, 15.0),
                    p=min(p, 10), err_tol=max(err_tol, 1e-6), precision=precision, soft=soft)
    if kind == "jerk":
        return dict(kind="jerk", n=_log(rng, 3000, 200000), p=p, err_tol=err_tol, soft=soft)
    if kind == "rollout":
        return dict(kind="rollout", n=_log(rng, 2000, 100000), p=p, err_tol=err_tol, soft=SOFT,
                    steps=rng.randint(2, 4))
    n = _log(rng, 10000, 1 << 20)
    return dict(kind="direct", n=n, nsink=_log(rng, 64, 4096), soft=soft)


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)
    return g


def _plummer_positions(n, g):
    """A Plummer sphere in Henon units, truncated at ten scale radii (the sampler of workloads.plummer)."""
    u = torch.rand((3, n), dtype=torch.float64, device=DEV, generator=g)
    x = torch.clamp(u[0] * (100.0 / 101.0) ** 1.5, min=1e-12)
    r = workloads.A_HENON / torch.sqrt(x ** (-2.0 / 3.0) - 1.0)
    z = 2.0 * u[1] - 1.0
    s = torch.sqrt(1.0 - z * z)
    phi = 2.0 * math.pi * u[2]
    return torch.stack([r * s * torch.cos(phi), r * s * torch.sin(phi), r * z], dim=1).contiguous()


def _bodies(case, seed):
    """Positions and masses of one system."""
    n, g = case["n"], _generator(seed)
    model = case.get("model", "plummer")
    if model == "cube":
        pos = 2.0 * torch.rand((n, 3), dtype=torch.float64, device=DEV, generator=g) - 1.0
        return pos, (0.5 + torch.rand(n, dtype=torch.float64, device=DEV, generator=g)) / n
    pos = _plummer_positions(n, g)
    if model == "plummer":
        return pos, torch.full((n,), 1.0 / n, dtype=torch.float64, device=DEV)
    m = torch.from_numpy(workloads.kroupa_masses(n, seed)).to(DEV)
    m[-1] = 0.0
    m *= 0.99 / m.sum()
    m[-1] = 0.01  # the central body, at rest in the middle
    pos[-1] = 0.0
    return pos, m


def _moving_bodies(case, seed):
    """Positions, velocities and masses of one Plummer sphere."""
    return [torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in workloads.plummer(case["n"], seed)]


def _cluster_offsets(case, seed):
    """Bounds of the clusters: log-uniform sizes, the same for every seed but in another order."""
    k = (np.arange(case["count"]) + 0.5) / case["count"]
    sizes = np.rint(2.0 ** (case["lo_exp"] + (case["hi_exp"] - case["lo_exp"]) * k)).astype(np.int64)
    sizes = np.random.Generator(np.random.PCG64(seed)).permutation(sizes)
    return np.concatenate([[0], np.cumsum(sizes)])


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("forces", "frozen"):
        s["pos"], s["mass"] = _bodies(case, seed)
        s["solver"] = fmm.FMM(p=case["p"], err_tol=case["err_tol"], precision=case["precision"])
        if kind == "frozen":  # the evaluation whose tree and lists the steps keep
            s["out"] = s["solver"].forces(s["pos"], s["mass"], eps_soft=case["soft"])
    elif kind == "batch":
        s["offsets"] = _cluster_offsets(case, seed)
        s["pos"] = _plummer_positions(int(s["offsets"][-1]), _generator(seed))
        n = torch.from_numpy(np.diff(s["offsets"])).to(DEV)
        s["mass"] = torch.repeat_interleave(1.0 / n.double(), n)
        s["solver"] = fmm.FMM(p=case["p"], err_tol=case["err_tol"], precision=case["precision"])
    elif kind == "jerk":
        s["pos"], s["vel"], s["mass"] = _moving_bodies(case, seed)
        s["solver"] = fmm.FMM(p=case["p"], err_tol=case["err_tol"])
    elif kind == "rollout":
        s["pos"], s["vel"], s["mass"] = (t.requires_grad_() for t in _moving_bodies(case, seed))
        s["wx"], s["wv"] = _loss_weights(case, seed)
        s["solver"] = [rollout.make_solver(p=case["p"], err_tol=case["err_tol"]) for _ in range(case["steps"] + 1)]
    else:
        s["pos"], s["mass"] = _bodies(case, seed)
        s["sinks"] = _sinks(case, seed)
    return s


def _loss_weights(case, seed):
    """dL/dx and dL/dv at the end of the rollout, for the linear loss L."""
    g = _generator(seed + 1)
    return [torch.randn((case["n"], 3), dtype=torch.float64, device=DEV, generator=g) for _ in range(2)]


def _sinks(case, seed):
    k = np.random.Generator(np.random.PCG64(seed + 3)).choice(case["n"], size=case["nsink"], replace=False)
    return torch.from_numpy(np.sort(k).astype(np.int32)).to(DEV)


# ------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind, soft = case["kind"], case["soft"]
    if kind == "forces":
        return s["solver"].forces(s["pos"], s["mass"], eps_soft=soft)
    if kind == "frozen":
        return s["solver"].forces_frozen(s["pos"], s["mass"], eps_soft=soft, out=s["out"], graph=True)
    if kind == "batch":
        return s["solver"].forces_batch(s["pos"], s["mass"], s["offsets"], eps_soft=soft)
    if kind == "jerk":
        return s["solver"].jerk(s["pos"], s["vel"], s["mass"], eps_soft=soft)
    if kind == "rollout":
        pos, vel, mass = s["pos"], s["vel"], s["mass"]
        x, v = rollout.leapfrog(pos, vel, mass, s["solver"], DT, case["steps"], eps_soft=soft, checkpoint_every=0)
        loss = (x * s["wx"]).sum() + (v * s["wv"]).sum()
        grads = torch.autograd.grad(loss, (pos, vel, mass))
        return (x.detach(), v.detach(), *grads)
    return fmm.direct(s["pos"], s["mass"], eps_soft=soft, sinks=s["sinks"])


# ------------------------------------------------------------------ work
def _swap_nonzeros(n):
    re = sum(1 for a in range(n + 1) for b in range(n + 1) if (a + b + n) % 2 == 0)
    im = sum(1 for a in range(1, n + 1) for b in range(1, n + 1) if (a + b + n) % 2 == 1)
    return re + im


def _m2l_flops(p):
    """One directed rotation-accelerated M2L: four swaps, four rotations about z, one translation along z."""
    f = 8 * sum(_swap_nonzeros(n) for n in range(p + 1)) + 24 * sum(range(p + 1))
    for n in range(p + 1):
        f += 2 * (p - n + 1) + sum(4 * (p - n - m + 1) for m in range(1, min(n, p - n) + 1))
    return f


PAIR = 20  # operations of one body pair: acceleration and potential


def _eval_flops(n, p):
    """One evaluation, from the pairs per body that the 2^20-body model has (about 3000 body pairs and 23
    M2L translations; a system of fewer bodies has no more than n partners for each)."""
    near = min(n, 3000)
    far = 23.0 * min(1.0, n / 20000.0)
    return n * (near * PAIR + far * _m2l_flops(p))


def work(case):
    kind = case["kind"]
    if kind == "batch":
        n = np.diff(_cluster_offsets(case, 0))
        return {"bytes": 64.0 * float(n.sum()), "flops": float(sum(_eval_flops(int(k), case["p"]) for k in n))}
    n = case["n"]
    if kind == "direct":
        return {"bytes": 32.0 * n + 36.0 * case["nsink"], "flops": float(PAIR) * n * case["nsink"]}
    f = _eval_flops(n, case["p"])
    if kind == "jerk":  # a second expansion pass and the derivative of every pair
        return {"bytes": 112.0 * n, "flops": 2.5 * f}
    if kind == "rollout":  # steps + 1 evaluations, and the gradient of each (twice an evaluation)
        k = case["steps"] + 1
        return {"bytes": 56.0 * n + 48.0 * n + 104.0 * n, "flops": (1.0 + 2.0) * k * f}
    return {"bytes": 64.0 * n, "flops": f}


# ------------------------------------------------------------------ direct sums in 64 bits
MOST_PAIRS = 1.5e11  # as many as fit in about twenty seconds


def _blocks(ni, nj):
    step = max(1, int(2e7) // max(nj, 1))
    return [(a, min(a + step, ni)) for a in range(0, ni, step)]


def _separations(pos, rows, soft):
    """Differences x_j - x_i of the listed rows, 1/s of each pair (0 for a pair of no extent)."""
    d = [pos[None, :, k] - pos[rows, k][:, None] for k in range(3)]
    s2 = d[0] * d[0]
    s2.addcmul_(d[1], d[1]).addcmul_(d[2], d[2]).add_(soft * soft)
    inv = s2.rsqrt_()
    inv[torch.arange(rows.numel(), device=pos.device), rows] = 0.0
    inv[torch.isinf(inv)] = 0.0
    return d, inv


def _direct(pos, mass, soft, rows=None):
    rows = torch.arange(pos.shape[0], device=pos.device) if rows is None else rows.long()
    acc = torch.empty((rows.numel(), 3), dtype=torch.float64, device=pos.device)
    pot = torch.empty(rows.numel(), dtype=torch.float64, device=pos.device)
    for a, b in _blocks(rows.numel(), pos.shape[0]):
        d, inv = _separations(pos, rows[a:b], soft)
        w = inv * mass
        pot[a:b] = -w.sum(1)
        w.mul_(inv).mul_(inv)
        for k in range(3):
            acc[a:b, k] = (w * d[k]).sum(1)
    return acc, pot


def _direct_jerk(pos, vel, mass, soft):
    n = pos.shape[0]
    jerk = torch.empty((n, 3), dtype=torch.float64, device=pos.device)
    every = torch.arange(n, device=pos.device)
    for a, b in _blocks(n, n):
        d, inv = _separations(pos, every[a:b], soft)
        w = [vel[None, :, k] - vel[a:b, k][:, None] for k in range(3)]
        uw = d[0] * w[0] + d[1] * w[1] + d[2] * w[2]
        m3 = mass * inv ** 3
        c = uw.mul_(3.0).mul_(inv).mul_(inv)
        for k in range(3):
            jerk[a:b, k] = (m3 * (w[k] - c * d[k])).sum(1)
    return jerk


def _direct_vjp(pos, mass, soft, gacc):
    """dL/dpos and dL/dmass of the direct sum's acceleration for dL/dacc = gacc."""
    n = pos.shape[0]
    gpos, gmass = torch.empty_like(pos), torch.empty_like(mass)
    every = torch.arange(n, device=pos.device)
    for a, b in _blocks(n, n):  # k: the rows a..b, j: every body; d = x_j - x_k
        d, inv = _separations(pos, every[a:b], soft)
        i3 = inv ** 3
        i2 = 3.0 * inv * inv
        gj = gacc.t()  # as a source, body k enters a_j with the separation -d
        gd = gj[0] * d[0] + gj[1] * d[1] + gj[2] * d[2]
        gmass[a:b] = -(gd * i3).sum(1)
        own = [gacc[a:b, k][:, None] for k in range(3)]
        od = own[0] * d[0] + own[1] * d[1] + own[2] * d[2]
        mk = mass[a:b][:, None]
        both = i2 * (mk * gd - mass * od)  # d/dx_k of m_j g_k.d/s^3 and of -m_k g_j.d/s^3
        for k in range(3):
            gpos[a:b, k] = (i3 * (mk * gj[k] - mass * own[k] - both * d[k])).sum(1)
    return gpos, gmass


def _direct_rollout(case, seed):
    pos, vel, mass = _moving_bodies(case, seed)
    soft, steps = case["soft"], case["steps"]
    xs, x, v = [pos], pos, vel
    a = _direct(x, mass, soft)[0]
    for _ in range(steps):
        v = v + 0.5 * DT * a
        x = x + DT * v
        a = _direct(x, mass, soft)[0]
        v = v + 0.5 * DT * a
        xs.append(x)
    gx, gv = _loss_weights(case, seed)
    gm = torch.zeros_like(mass)
    ga = torch.zeros_like(pos)  # dL/da of the evaluation at xs[t], from the step after it
    for t in range(steps, 0, -1):
        dp, dm = _direct_vjp(xs[t], mass, soft, ga + 0.5 * DT * gv)
        gx, gm = gx + dp, gm + dm
        gv = gv + DT * gx
        ga = 0.5 * DT * gv
    dp, dm = _direct_vjp(xs[0], mass, soft, ga)
    return x, v, gx + dp, gv, gm + dm


def exact(case, seed):
    kind, soft = case["kind"], case["soft"]
    if kind == "batch":
        off = _cluster_offsets(case, seed)
        n = np.diff(off)
        if float((n.astype(np.float64) ** 2).sum()) > MOST_PAIRS:
            return None
        pos = _plummer_positions(int(off[-1]), _generator(seed))
        parts = [_direct(pos[a:b], torch.full((int(b - a),), 1.0 / float(b - a), dtype=torch.float64, device=DEV),
                         soft) for a, b in zip(off[:-1], off[1:])]
        return torch.cat([q[0] for q in parts]), torch.cat([q[1] for q in parts])
    n = float(case["n"])
    pairs = {"direct": n * case.get("nsink", 0), "rollout": 8.0 * n * n, "jerk": 3.0 * n * n}.get(kind, n * n)
    if pairs > MOST_PAIRS:
        return None
    if kind == "jerk":
        pos, vel, mass = _moving_bodies(case, seed)
        return (*_direct(pos, mass, soft), _direct_jerk(pos, vel, mass, soft))
    if kind == "rollout":
        return _direct_rollout(case, seed)
    pos, mass = _bodies(case, seed)
    return _direct(pos, mass, soft, _sinks(case, seed) if kind == "direct" else None)

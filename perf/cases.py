"""The work this framework is used for, as cases that can be timed and compared.

A case names a path through the public entry points and its sizes:

  batch      fixed Hermite steps of a batch held in the caller's device tensors (hermite_steps_device)
  job        an ensemble from creation to its states and diagnostics, fixed Hermite steps, plain launches
  ragged     the same with mixed body counts on the persistent schedule
  lifetimes  adaptive steps with the stop rules on the persistent schedule, retired systems compacted away
  epochs     adaptive (Eq. 5) steps to observation epochs, the star's radial velocity recorded at each
  logged     fixed steps with an energy and angular momentum record every so many steps
  mvs        the mixed-variable symplectic integrator
  rkck       fixed Runge-Kutta Cash-Karp steps
  rkck_adaptive  Runge-Kutta Cash-Karp to a time under an error tolerance
  disk       planetesimal disks of more bodies than a lane or a wavefront holds (the large-n kernels)
  serve      a burst of requests to the integration server, every result read back

Initial conditions are the generators' own families (paper_1208_1157_amd.gen).
"""
import math

import numpy as np
import torch

from paper_1208_1157_amd import fewbody as fb
from paper_1208_1157_amd import gen

TWO_PI = 2.0 * math.pi
H = TWO_PI / 1000.0      # the benchmark's fixed step
H_FINE = TWO_PI / 2000.0  # ... of its ragged workload
ETA = 0.01               # pairwise step rule of the uneven-lifetimes workload
TAU = 0.017              # Eq. 5 step scale of Table 1
H_MVS = 1e-2             # the paper's MVS step
LOS = (0.6, 0.0, 0.8)
HOST_MOST = 15.0         # seconds that exact() may take


def listed():
    return [
        # the smallest call: a few steps of a few systems inside a torch program; launches and latency
        {"name": "batch_16x3_10", "kind": "batch", "systems": 16, "lo": 3, "hi": 3, "steps": 10},
        # an ordinary batch that cannot fill the device one system to a lane: the time of a step counts
        {"name": "batch_1000x6_1000", "kind": "batch", "systems": 1000, "lo": 6, "hi": 6, "steps": 1000},
        # the headline ensemble: 131072 three-body systems
        {"name": "job_131072x3_10000", "kind": "job", "systems": 131072, "lo": 3, "hi": 3, "steps": 10000},
        # mixed body counts in one launch
        {"name": "ragged_65536x3-15_500", "kind": "ragged", "systems": 65536, "lo": 3, "hi": 15, "steps": 500},
        # tightly packed systems, each followed until a close encounter, an ejection or the end
        {"name": "lifetimes_16384x4-8", "kind": "lifetimes", "systems": 16384, "lo": 4, "hi": 8, "orbits": 3.0},
        # trial systems of a radial-velocity fit, compared with 24 observations
        {"name": "epochs_2048x4_24", "kind": "epochs", "systems": 2048, "lo": 4, "hi": 4, "orbits": 4.0, "epochs": 24},
        # long stable integrations: the headline ensemble, and mid-size systems of mixed body counts
        {"name": "mvs_131072x3_4000", "kind": "mvs", "systems": 131072, "lo": 3, "hi": 3, "steps": 4000},
        {"name": "mvs_4099x5-12_500", "kind": "mvs", "systems": 4099, "lo": 5, "hi": 12, "steps": 500},
        # the high-order check of the other integrators: fixed steps, and steps under a tolerance
        {"name": "rkck_131072x3_1000", "kind": "rkck", "systems": 131072, "lo": 3, "hi": 3, "steps": 1000},
        {"name": "rkck_adaptive_9999x5", "kind": "rkck_adaptive", "systems": 9999, "lo": 5, "hi": 5, "orbits": 1.0,
         "eps": 1e-10},
        # planetesimal disks
        {"name": "disk_1024x64_400", "kind": "disk", "systems": 1024, "lo": 64, "hi": 64, "steps": 400},
        # a burst of small requests: their latency, and the mixing of their systems
        {"name": "serve_24", "kind": "serve", "requests": 24, "systems": 512, "lo": 3, "hi": 10, "orbits": 8.0},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["batch", "batch", "job", "job", "ragged", "lifetimes", "epochs", "logged", "mvs", "mvs", "rkck",
                       "rkck_adaptive", "disk", "serve"])
    c = {"kind": kind}
    if kind == "batch":
        c["lo"] = c["hi"] = rng.randint(2, 16)
        c["systems"], c["steps"] = _log(rng, 1, 20000), _log(rng, 10, 2000)
    elif kind == "job":
        c["lo"] = c["hi"] = rng.randint(2, 10)
        c["systems"], c["steps"] = _log(rng, 1, 131072), _log(rng, 1000, 10000)
    elif kind == "ragged":
        c["lo"], c["hi"] = rng.randint(2, 6), rng.randint(8, 16)
        c["systems"], c["steps"] = _log(rng, 64, 65536), _log(rng, 200, 2000)
    elif kind == "lifetimes":
        c["lo"], c["hi"] = rng.randint(3, 5), rng.randint(5, 8)
        c["systems"], c["orbits"] = _log(rng, 256, 16384), round(rng.uniform(1.0, 3.0), 2)
    elif kind == "epochs":
        c["lo"] = c["hi"] = rng.randint(3, 7)
        c["systems"], c["orbits"], c["epochs"] = _log(rng, 1, 4096), round(rng.uniform(1.0, 4.0), 2), _log(rng, 4, 40)
    elif kind == "logged":
        c["lo"] = c["hi"] = rng.randint(3, 5)
        c["systems"], c["steps"], c["every"] = _log(rng, 1000, 60000), _log(rng, 500, 2000), _log(rng, 50, 250)
    elif kind == "mvs":
        c["lo"] = rng.randint(2, 8)
        c["hi"] = c["lo"] if rng.random() < 0.5 else rng.randint(c["lo"], 14)
        c["systems"], c["steps"] = _log(rng, 1, 131072), _log(rng, 200, 4000)
    elif kind == "rkck":
        c["lo"] = c["hi"] = rng.randint(2, 12)
        c["systems"], c["steps"] = _log(rng, 1, 131072), _log(rng, 200, 1000)
    elif kind == "rkck_adaptive":
        c["lo"] = c["hi"] = rng.randint(3, 8)
        c["systems"], c["orbits"], c["eps"] = _log(rng, 1, 20000), round(rng.uniform(0.5, 1.0), 2), 10.0 ** -rng.randint(8, 10)
    elif kind == "disk":
        c["lo"] = c["hi"] = _log(rng, 17, 300)
        c["systems"], c["steps"] = _log(rng, 1, 2048), _log(rng, 50, 400)
    else:
        c["lo"], c["hi"] = 3, rng.randint(5, 12)
        c["requests"], c["systems"], c["orbits"] = rng.randint(2, 24), _log(rng, 4, 512), round(rng.uniform(2.0, 8.0), 2)
    # no drawn case costs more than the largest of its kind in listed()
    most = max([work(k)["flops"] for k in listed() if k["kind"] == kind] or [2e10])
    if kind in ("batch", "job"):
        most = {"batch": 2e10, "job": 9e11}[kind]
    while work(c)["flops"] > most:
        c["systems"] = max(1, c["systems"] // 2 + c["systems"] % 2)
        if "steps" in c:
            c["steps"] = max(10, int(c["steps"] * 0.8))
        elif c["systems"] == 1:
            break
    return c


def _ragged(counts, seed, **family):
    """The Hill-spaced family with these body counts, system by system."""
    ks = sorted(set(counts.tolist()))
    parts = [gen.ragged_hill(int((counts == n).sum()), seed + n, n_lo=n, n_hi=n, **family) for n in ks]
    e = gen.Ensemble(*(np.concatenate([getattr(p, k) for p in parts]) for k in ("n_body", "mass", "pos", "vel")))
    at = np.empty(len(counts), dtype=np.int64)
    at[np.argsort(counts, kind="stable")] = np.arange(len(counts))
    return e.subset(at) if len(ks) > 1 else e


def _ensemble(case, seed, systems=None):
    """Everything but the body counts comes from the seed; those belong to the sizes of the case."""
    n = case["systems"] if systems is None else systems
    if case["kind"] == "disk":
        return gen.planetesimal_disk(n, case["lo"], seed)
    if case["lo"] == case["hi"] == 3:
        return gen.three_body(n, seed)
    counts = np.random.default_rng(n).integers(case["lo"], case["hi"] + 1, n).astype(np.int32)
    tight = {"mlo": 1e-5, "mhi": 1e-3, "k_lo": 3.0, "k_hi": 6.0, "e_hi": 0.2} if case["kind"] == "lifetimes" else {}
    return _ragged(counts, seed, **tight)


def _requests(case, seed):
    """Sizes log-uniform up to the case's, lengths log-uniform from one orbit to the case's."""
    rng = np.random.default_rng(case["systems"])
    got = []
    for k in range(case["requests"]):
        n = int(min(case["systems"], math.floor(math.exp(rng.uniform(0.0, math.log(case["systems"] + 1))))))
        t_end = TWO_PI * math.exp(rng.uniform(0.0, math.log(case["orbits"])))
        got.append((_ensemble(case, seed + 100 * k, max(1, n)), t_end))
    return got


def prepare(case, seed):
    if case["kind"] == "serve":
        return {"case": case, "requests": _requests(case, seed),
                "server": fb.Server(budget_bytes=512 << 20, policy=fb.POLICY_SRPT, long_steps=300000)}
    e = _ensemble(case, seed)
    s = {"case": case, "n_body": e.n_body}
    for k in ("mass", "pos", "vel"):
        s[k] = torch.from_numpy(getattr(e, k)).cuda()
    if case["kind"] == "batch":
        s["status"] = torch.empty(e.n_sys, dtype=torch.int32, device="cuda")
        s["workspace"] = torch.empty(int(fb.lib().fb_hermite_steps_workspace_bytes(e.n_sys, case["lo"])) + 256,
                                     dtype=torch.uint8, device="cuda")
    return s


def _epochs(case):
    """Observation times, unevenly spaced."""
    k = np.arange(1, case["epochs"] + 1)
    return TWO_PI * case["orbits"] * (k / case["epochs"]) ** 1.3


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "batch":
        pos, vel = s["pos"].clone(), s["vel"].clone()
        fb.hermite_steps_device(c["lo"], s["mass"], pos, vel, c["steps"], H, status=s["status"],
                                workspace=s["workspace"])
        return {"pos": pos, "vel": vel, "status": s["status"]}
    if kind == "serve":
        ids = [s["server"].submit_gen(e, t_end, H) for e, t_end in s["requests"]]
        got = []
        for rid in ids:
            s["server"].wait(rid)
            got.append(s["server"].result(rid))
        return {k: np.concatenate([g[k] for g in got]) for k in ("pos", "vel", "t", "status", "steps")}
    with fb.Ensemble(s["n_body"], s["mass"], s["pos"], s["vel"]) as e:
        more = {}
        if kind in ("job", "disk"):
            e.integrate_steps(c["steps"], H)
        elif kind == "ragged":
            e.integrate_steps(c["steps"], H_FINE, fb.Opts(schedule=fb.SCHED_PERSISTENT))
        elif kind == "lifetimes":
            e.integrate(TWO_PI * c["orbits"], 0.0,
                        fb.Opts(adaptive=1, eta=ETA, stop_rules=fb.STOP_ENCOUNTER | fb.STOP_EJECT,
                                schedule=fb.SCHED_PERSISTENT, steps_per_quantum=500, compact=True))
        elif kind == "epochs":
            more["t_rv"], more["rv"] = e.integrate_to_times(_epochs(c), los=LOS, opts=fb.Opts(adaptive=2, eta=TAU))
        elif kind == "logged":
            more["t_rec"], more["E"], more["L"] = e.integrate_steps_logged(c["steps"], H, c["every"], kind=fb.LOG_ENERGY)
        elif kind == "mvs":
            e.integrate_mvs(c["steps"], H_MVS)
        elif kind == "rkck":
            e.integrate_rkck_steps(c["steps"], H)
        else:
            e.integrate_rkck(TWO_PI * c["orbits"], 0.01, c["eps"])
        if kind in ("job", "ragged", "mvs", "disk"):
            more["energy"], more["angmom"] = e.diagnostics()
        return {**e.state(), **more}


# -- what a pass cannot do without --------------------------------------------------------------------------------

def _per_step(kind, n):
    """Operations of one step of one n-body system (a fused multiply-add counts two; square root and division one)."""
    pairs = n * (n - 1) / 2
    if kind == "mvs":   # one pair acceleration, kicks and drifts, one Kepler drift of each planet
        return 36.0 * (n - 1) * (n - 2) / 2 + 30.0 * n + 160.0 * (n - 1)
    if kind.startswith("rkck"):   # six accelerations and the tableau's sums
        return 6 * 36.0 * pairs + 260.0 * n
    return 116.0 * pairs + 120.0 * n   # two accelerations with jerk, predictor, two corrections


# Steps an adaptive run takes per inner orbit, counted on these families.
STEPS_PER_ORBIT = {"lifetimes": 670, "epochs": 594, "rkck_adaptive": 162}


def work(case):
    kind = case["kind"]
    mean = np.mean([_per_step(kind, n) for n in range(case["lo"], case["hi"] + 1)])
    bodies = case["systems"] * 0.5 * (case["lo"] + case["hi"])
    steps = case.get("steps") or case["orbits"] * STEPS_PER_ORBIT.get(kind, 0)
    flops = case["systems"] * steps * mean
    bytes_ = bodies * (56 + 48) + case["systems"] * 20
    if kind == "serve":
        mean_sys = case["systems"] / math.log(case["systems"] + 1)
        mean_orbits = (case["orbits"] - 1) / math.log(case["orbits"])
        flops = case["requests"] * mean_sys * 1000 * mean_orbits * mean
        bytes_ = case["requests"] * mean_sys * (0.5 * (case["lo"] + case["hi"]) * 104 + 20)
    elif kind == "epochs":
        bytes_ += 16 * case["systems"] * case["epochs"]
    elif kind == "logged":
        bytes_ += 40 * case["systems"] * (2 + case["steps"] // case["every"])
    elif kind in ("job", "ragged", "mvs", "disk"):
        bytes_ += 32 * case["systems"]
    return {"bytes": float(bytes_), "flops": float(flops)}


# -- the same results from the equations, in plain torch ----------------------------------------------------------

def _padded(e, dev):
    """Masses, positions and velocities as [systems, most bodies(, 3)]; absent bodies are massless and far away."""
    n = int(e.n_body.max())
    here = np.arange(n)[None, :] < e.n_body[:, None]
    m = np.zeros((e.n_sys, n))
    x = np.zeros((e.n_sys, n, 3))
    v = np.zeros((e.n_sys, n, 3))
    x[:, :, 0] = 1e3 * (1.0 + np.arange(n))
    m[here], x[here], v[here] = e.mass, e.pos, e.vel
    return [torch.from_numpy(a).to(dev) for a in (m, x, v, here)]


class _Gravity:
    """Eq. 1, its time derivative, and the quantities of the step rules."""

    def __init__(self, m, here):
        self.m, self.here = m, here
        self.eye = torch.eye(m.shape[1], dtype=m.dtype, device=m.device)
        self.off = (1.0 - self.eye) * m[:, None, :]
        self.pair = here[:, :, None] & here[:, None, :] & (self.eye == 0)

    def acc(self, x):
        r = x[:, None, :, :] - x[:, :, None, :]
        r2 = (r * r).sum(3) + self.eye
        return ((self.off / (r2 * r2.sqrt()))[..., None] * r).sum(2)

    def acc_jerk(self, x, v, rule=False):
        r = x[:, None, :, :] - x[:, :, None, :]
        u = v[:, None, :, :] - v[:, :, None, :]
        r2 = (r * r).sum(3) + self.eye
        ru = (r * u).sum(3)
        w = (self.off / (r2 * r2.sqrt()))[..., None]
        jerk = (w * (u - (3.0 * ru / r2)[..., None] * r)).sum(2)
        q = None
        if rule:
            q = torch.where(self.pair, ((u * u).sum(3) + 3.0 * ru * ru / r2) / r2, 0.0).amax((1, 2))
        return (w * r).sum(2), jerk, q


def _hermite(g, x, v, a, j, h, rule=False):
    """One P(EC)^2 step of h [systems, 1, 1]: Eq. 3, and Eq. 4 twice."""
    xp = x + h * v + h * h / 2 * a + h ** 3 / 6 * j
    vp = v + h * a + h * h / 2 * j
    bx = xp - 3 / 20 * h * h * a - 7 / 60 * h ** 3 * j
    bv = vp - h / 2 * a - 5 / 12 * h * h * j
    x1, v1, q = xp, vp, None
    for k in range(2):
        a1, j1, q = g.acc_jerk(x1, v1, rule and k == 1)
        x1 = bx + 3 / 20 * h * h * a1 - h ** 3 / 30 * j1
        v1 = bv + h / 2 * a1 - h * h / 12 * j1
    return x1, v1, a1, j1, q


def _energy(m, x, v):
    r = x[:, None, :, :] - x[:, :, None, :]
    d = ((r * r).sum(3) + torch.eye(m.shape[1], dtype=m.dtype, device=m.device)).sqrt()
    pot = torch.triu(m[:, None, :] * m[:, :, None] / d, 1).sum((1, 2))
    return 0.5 * (m * (v * v).sum(2)).sum(1) - pot, (m[..., None] * torch.linalg.cross(x, v)).sum(1)


def _fixed(m, x, v, here, dt, steps, last=None):
    """`steps` [systems] steps of dt, then one of `last` [systems] where that is not zero."""
    g = _Gravity(m, here)
    a, j, _ = g.acc_jerk(x, v)
    n = torch.as_tensor(steps, device=x.device).expand(x.shape[0])
    most = int(n.max())
    same = last is None and int(n.min()) == most
    for k in range(most if last is None else most + 1):
        if same:
            x, v, a, j, _ = _hermite(g, x, v, a, j, torch.full((1, 1, 1), dt, dtype=x.dtype, device=x.device))
            continue
        h = torch.where(k < n, torch.full_like(m[:, 0], dt), 0.0)
        if last is not None:
            h = torch.where(k == n, last, h)
        y = _hermite(g, x, v, a, j, h[:, None, None])
        go = (h != 0.0)[:, None, None]
        x, v, a, j = (torch.where(go, p, q) for p, q in zip(y, (x, v, a, j)))
    return x, v


def _adaptive(m, x, v, here, times, rule, eta, stop):
    """Steps of the pairwise rule (1) or Eq. 5 (2) to each time; stop rules after every step. The states at each time."""
    g = _Gravity(m, here)
    live = torch.ones_like(m[:, 0], dtype=torch.bool)
    t = torch.zeros_like(m[:, 0])
    a, j, q = g.acc_jerk(x, v, True)
    here3 = here[..., None]
    far = torch.triu(here[:, 1:, None] & here[:, None, 1:], 1)
    got = []
    for t_end in times:
        for k in range(10 ** 6):
            go = live & (t < t_end)
            if k % 16 == 0 and not bool(go.any()):
                break
            if rule == 2:
                q = torch.where(here, (j * j).sum(2) / torch.where(here, (a * a).sum(2), 1.0), 0.0).sum(1)
            dt = eta / q.sqrt()
            end = t + dt >= t_end
            h = torch.where(end, t_end - t, dt)
            y = _hermite(g, x, v, a, j, h[:, None, None], rule == 1)
            w = go[:, None, None]
            x, v, a, j = (torch.where(w & here3, p, o) for p, o in zip(y, (x, v, a, j)))
            if rule == 1:
                q = torch.where(go, y[4], q)
            t = torch.where(go, torch.where(end, t_end, t + h), t)
            if stop:
                p = x[:, 1:] - x[:, :1]
                r = (p * p).sum(2).sqrt()
                d = p[:, :, None, :] - p[:, None, :, :]
                mm = m[:, 1:, None] + m[:, None, 1:]
                hill = (mm / (3.0 * m[:, :1, None])) ** (1 / 3) * (r[:, :, None] + r[:, None, :]) / 2
                hit = (far & ((d * d).sum(3).sqrt() < hill)).any(2).any(1) | (here[:, 1:] & (r > 100.0)).any(1)
                live = live & ~(go & hit)
        got.append((t.clone(), x.clone(), v.clone()))
    return got


def _mvs(m, x, v, here, dt, steps):
    """Democratic heliocentric splitting: drift, kick, Kepler drift, kick, drift."""
    M = m.sum(1)[:, None, None]
    X, Vc = (m[..., None] * x).sum(1, True) / M, (m[..., None] * v).sum(1, True) / M
    mp, m0, there = m[:, 1:], m[:, :1, None], here[:, 1:, None]
    Q, V = x[:, 1:] - x[:, :1], torch.where(there, v[:, 1:] - Vc, 0.0)
    Q = torch.where(there, Q, x[:, 1:])
    g = _Gravity(mp, here[:, 1:])
    acc = torch.where(there, g.acc(Q), 0.0)
    for _ in range(steps):
        Q = Q + torch.where(there, dt / 2 * (mp[..., None] * V).sum(1, True) / m0, 0.0)
        X = X + dt / 2 * Vc
        V = V + dt / 2 * acc
        r, v2, rv = (Q * Q).sum(2, True).sqrt(), (V * V).sum(2, True), (Q * V).sum(2, True)
        al = torch.where(there, 2.0 / r - v2 / m0, 1.0)
        sq = (m0 / al).sqrt()
        nm, ec, es = sq * al * al, 1.0 - r * al, rv / sq
        E = nm * dt
        for _ in range(5):
            s, c = torch.sin(E), torch.cos(E)
            E = E - (E - ec * s + es * (1 - c) - nm * dt) / (1 - ec * c + es * s)
        s, oc = torch.sin(E), 2 * torch.sin(E / 2) ** 2
        rn = (1 - ec * (1 - oc) + es * s) / al
        f, gg = 1 - oc / (al * r), dt - (E - s) / nm
        fd, gd = -sq * s / (rn * r), 1 - oc / (al * rn)
        Qn, Vn = f * Q + gg * V, fd * Q + gd * V
        Q, V = torch.where(there, Qn, Q), torch.where(there, Vn, V)
        acc = torch.where(there, g.acc(Q), 0.0)
        V = V + dt / 2 * acc
        Q = Q + torch.where(there, dt / 2 * (mp[..., None] * V).sum(1, True) / m0, 0.0)
        X = X + dt / 2 * Vc
    x0 = X - (mp[..., None] * Q).sum(1, True) / M
    v0 = Vc - (mp[..., None] * V).sum(1, True) / m0
    return torch.cat([x0, x0 + Q], 1), torch.cat([v0, Vc + V], 1)


# Cash and Karp's tableau: couplings, fifth- and fourth-order weights.
_A = [[], [1 / 5], [3 / 40, 9 / 40], [3 / 10, -9 / 10, 6 / 5], [-11 / 54, 5 / 2, -70 / 27, 35 / 27],
      [1631 / 55296, 175 / 512, 575 / 13824, 44275 / 110592, 253 / 4096]]
_B5 = [37 / 378, 0, 250 / 621, 125 / 594, 0, 512 / 1771]
_B4 = [2825 / 27648, 0, 18575 / 48384, 13525 / 55296, 277 / 14336, 1 / 4]


def _rkck_step(g, x, v, h):
    kx, kv = [], []
    for row in _A:
        kx.append(v + h * sum((c * k for c, k in zip(row, kv)), torch.zeros_like(v)))
        kv.append(g.acc(x + h * sum((c * k for c, k in zip(row, kx)), torch.zeros_like(x))))
    up = lambda w, k: h * sum(c * y for c, y in zip(w, k) if c)  # noqa: E731
    E = [b - a for b, a in zip(_B5, _B4)]
    return x + up(_B5, kx), v + up(_B5, kv), up(E, kx), up(E, kv)


def _rkck(m, x, v, here, dt, steps):
    g = _Gravity(m, here)
    h = torch.full((1, 1, 1), dt, dtype=x.dtype, device=x.device)
    for _ in range(steps):
        x, v, _, _ = _rkck_step(g, x, v, h)
    return x, v


def _rkck_adaptive(m, x, v, here, t_end, dt, eps):
    """Error norm and step control of the adaptive integrator."""
    g = _Gravity(m, here)
    t, dtn = torch.zeros_like(m[:, 0]), torch.full_like(m[:, 0], dt)
    top = lambda p: torch.where(here, p.norm(dim=2), 0.0).amax(1)  # noqa: E731
    for k in range(10 ** 6):
        go = t < t_end
        if k % 16 == 0 and not bool(go.any()):
            break
        last = t + dtn >= t_end
        h = torch.where(last, t_end - t, dtn)
        x5, v5, ex, ev = _rkck_step(g, x, v, h[:, None, None])
        E = torch.maximum(top(ex) / (eps * top(x)), top(ev) / (eps * top(v)))
        ok = go & (E <= 1.0)
        w = ok[:, None, None]
        x, v = torch.where(w, x5, x), torch.where(w, v5, v)
        t = torch.where(ok, torch.where(last, t_end, t + h), t)
        new = torch.where(last, dtn, h * (0.9 * E ** -0.2).clamp(0.2, 5.0))
        dtn = torch.where(ok, new, torch.where(go, h * (0.9 * E ** -0.25).clamp_min(0.1), dtn))
    return x, v


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    n, orbits = case["hi"], case.get("orbits", 0.0)
    iterations = case.get("steps") or orbits * {"serve": 1000, "lifetimes": 3000, "epochs": 800}.get(kind, 150)
    systems = case["systems"] if kind != "serve" else case["requests"] * case["systems"] / 3
    calls = {"mvs": 130, "rkck": 260, "rkck_adaptive": 300, "lifetimes": 130}.get(kind, 90)
    if iterations * calls * (5e-6 + systems * n * n * 24 / 6e12) > HOST_MOST:
        return None
    if kind == "serve":
        parts = [(gen.Request(0.0, e, t, H)) for e, t in _requests(case, seed)]
        e = gen.Ensemble(*(np.concatenate([getattr(p.ensemble, k) for p in parts]) for k in ("n_body", "mass", "pos", "vel")))
        t_end = np.concatenate([np.full(p.ensemble.n_sys, p.t_end) for p in parts])
    else:
        e = _ensemble(case, seed)
    m, x, v, here = _padded(e, dev)
    flat = lambda p: p[here]  # noqa: E731
    if kind in ("batch", "job", "disk", "ragged"):
        x, v = _fixed(m, x, v, here, H_FINE if kind == "ragged" else H, case["steps"])
        out = {"pos": flat(x), "vel": flat(v)}
    elif kind == "serve":
        t_end = torch.from_numpy(t_end).to(dev)
        whole = torch.floor(t_end / H)
        rest = t_end - whole * H
        x, v = _fixed(m, x, v, here, H, whole.long(), torch.where(rest > 1e-9 * H, rest, 0.0))
        return {"pos": flat(x), "vel": flat(v), "t": t_end}
    elif kind == "lifetimes":
        (t, x, v), = _adaptive(m, x, v, here, [TWO_PI * orbits], 1, ETA, True)
        return {"pos": flat(x), "vel": flat(v), "t": t}
    elif kind == "epochs":
        got = _adaptive(m, x, v, here, list(_epochs(case)), 2, TAU, False)
        los = torch.tensor(LOS, dtype=x.dtype, device=dev)
        rv = [((p[:, 0] - (m[..., None] * p).sum(1) / m.sum(1, True)) * los).sum(1) for _, _, p in got]
        return {"t_rv": torch.stack([t for t, _, _ in got], 1), "rv": torch.stack(rv, 1), "t": got[-1][0],
                "pos": flat(got[-1][1]), "vel": flat(got[-1][2])}
    elif kind == "logged":
        at = list(range(0, case["steps"], case["every"])) + [case["steps"]]
        g = _Gravity(m, here)
        a, j, _ = g.acc_jerk(x, v)
        h = torch.full((1, 1, 1), H, dtype=x.dtype, device=dev)
        E, L = [], []
        for k in range(case["steps"] + 1):
            if k:
                x, v, a, j, _ = _hermite(g, x, v, a, j, h)
            if k in at:
                p = _energy(m, x, v)
                E.append(p[0])
                L.append(p[1])
        t = torch.tensor([k * H for k in at], dtype=x.dtype, device=dev)
        return {"pos": flat(x), "vel": flat(v), "t_rec": t.expand(len(m), -1).contiguous(), "E": torch.stack(E, 1),
                "L": torch.stack(L, 1)}
    elif kind == "mvs":
        x, v = _mvs(m, x, v, here, H_MVS, case["steps"])
        out = {"pos": flat(x), "vel": flat(v)}
    elif kind == "rkck":
        x, v = _rkck(m, x, v, here, H, case["steps"])
        return {"pos": flat(x), "vel": flat(v)}
    else:
        x, v = _rkck_adaptive(m, x, v, here, TWO_PI * orbits, 0.01, case["eps"])
        return {"pos": flat(x), "vel": flat(v)}
    if kind != "batch":
        out["energy"], out["angmom"] = _energy(m, x, v)
    return out

"""Two and four lanes a body (fixed steps of ensembles that leave SIMDs free):
every body count, whole and partial tiles, against the same systems inside an
ensemble too large for these kernels.  All Hermite kernels add in one order,
so every comparison is bitwise."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen
from tests.helpers import per_system_rel_err, threads

pytestmark = pytest.mark.gpu
DT = 2 * math.pi / 1000
FULL = 12000   # more wavefronts than SIMDs, with two lanes a body, from 5 bodies up


def run(fb, ens, how, t0=None, opts=None):
    E = fb.Ensemble(ens.n_body, ens.mass, ens.pos, ens.vel, t0=t0)
    how(E, opts or fb.Opts())
    st, (acc, jerk, _) = E.state(), E.hermite_state()
    E.close()
    return {**st, "acc": acc, "jerk": jerk}


def same(a, b, n, k):
    for key in a:
        x, y = a[key], b[key]
        rows = k * n if key in ("pos", "vel", "acc", "jerk") else k
        assert np.array_equal(x[:rows], y[:rows], equal_nan=True), key


@pytest.mark.parametrize("n", range(5, 17))
@pytest.mark.parametrize("count", [1, 3, 700, 1500])   # 4 lanes a body, with 700 and 1500 (by n) 2, or 1
def test_equals_one_lane_a_body(plans, n, count):
    fb = plans
    fb.set_plan(n, fb.MAP_BPL, 1)
    big = gen.ragged_hill(FULL, 50 + n, n_lo=n, n_hi=n)
    ens = big.subset(range(count))
    t0 = np.random.default_rng(n).uniform(0.0, 20 * DT, FULL)   # uneven step counts in a tile, a shortened last step
    print("[case] split", n, count, flush=True)
    to_end = lambda E, o: E.integrate(31.3 * DT, DT, o)
    same(run(fb, ens, to_end, t0[:count]), run(fb, big, to_end, t0), n, count)
    steps = lambda E, o: E.integrate_steps(23, DT, o)
    want = run(fb, big, steps)
    same(run(fb, ens, steps), want, n, count)
    for opts in (fb.Opts(schedule=fb.SCHED_PERSISTENT), fb.Opts(steps_per_quantum=7),
                 fb.Opts(schedule=fb.SCHED_PERSISTENT, steps_per_quantum=9, compact=True)):
        same(run(fb, ens, steps, opts=opts), want, n, count)


def test_mixed_fused_launch_and_failing_systems(plans, ora):
    """Every body count in one fused launch, two systems that turn non-finite; the others against the oracle."""
    fb = plans
    ens = gen.ragged_hill(45, 90, n_lo=2, n_hi=16)
    off = ens.offsets
    bad = [int(np.argmax(ens.n_body)), int(np.flatnonzero(ens.n_body == 6)[0])]
    pos = ens.pos.copy()
    for s in bad:
        pos[off[s] + 2] = pos[off[s] + 1]
    e2 = gen.Ensemble(ens.n_body, ens.mass, pos, ens.vel)
    st = run(fb, e2, lambda E, o: E.integrate_steps(40, DT, o), opts=fb.Opts(schedule=fb.SCHED_PERSISTENT))
    plain = run(fb, e2, lambda E, o: E.integrate_steps(40, DT, o))
    for key in st:
        assert np.array_equal(st[key], plain[key], equal_nan=True), key
    ok = np.ones(ens.n_sys, dtype=bool)
    ok[bad] = False
    assert np.all(st["status"][bad] == fb.NONFINITE) and np.all(st["status"][ok] == fb.DONE)
    x, v, _, _ = ora.ensemble_fixed(ens.n_body, ens.mass, ens.pos, ens.vel, DT, 40, nthreads=threads())
    ex = per_system_rel_err(ens.n_body, st["pos"], x)[ok]
    ev = per_system_rel_err(ens.n_body, st["vel"], v)[ok]
    assert ex.max() <= 1e-10 and ev.max() <= 1e-10


@pytest.mark.parametrize("n", range(5, 17))
@pytest.mark.parametrize("count", [1, 3, 700, 1500])
def test_adaptive_equals_one_lane_a_body(plans, n, count):
    """Both step rules and the stop rules (tightly packed systems, so that some stop), and fixed steps with them."""
    fb = plans
    fb.set_plan(n, fb.MAP_BPL, 1)
    big = gen.ragged_hill(FULL // 2, 150 + n, n_lo=n, n_hi=n, mlo=1e-5, mhi=1e-3, k_lo=3.0, k_hi=6.0, e_hi=0.2)
    ens = big.subset(range(count))
    print("[case] split adaptive", n, count, flush=True)
    rules = fb.STOP_ENCOUNTER | fb.STOP_EJECT
    for kw in ({"adaptive": 1, "eta": 0.02, "stop_rules": rules}, {"adaptive": 1, "eta": 0.02},
               {"adaptive": 2, "eta": 0.03}, {"stop_rules": rules, "r_eject": 0.6}):
        go = lambda E, o: E.integrate(0.15, 0.0 if o.adaptive else 0.004, o)
        want = run(fb, big, go, opts=fb.Opts(**kw))
        same(run(fb, ens, go, opts=fb.Opts(**kw)), want, n, count)
        same(run(fb, ens, go, opts=fb.Opts(schedule=fb.SCHED_PERSISTENT, steps_per_quantum=5, compact=True, **kw)),
             want, n, count)


def test_compaction_through_every_mapping(plans):
    """One run whose survivors thin out from one lane a body to two and four, against plain launches."""
    fb = plans
    parts = [gen.ragged_hill(5000, 60 + n, n_lo=n, n_hi=n, mlo=1e-5, mhi=1e-3, k_lo=3.0, k_hi=4.0, e_hi=0.3)
             for n in (4, 6, 8)]
    ens = gen.Ensemble(*(np.concatenate([getattr(p, f) for p in parts]) for f in ("n_body", "mass", "pos", "vel")))
    t0 = np.random.default_rng(3).uniform(0.0, 2.0, ens.n_sys) ** 0.2   # few systems with a long way to go
    print("[case] split compaction", flush=True)
    got = {}
    for sched in (fb.SCHED_PLAIN, fb.SCHED_PERSISTENT):
        kw = {"steps_per_quantum": 10, "compact": True} if sched == fb.SCHED_PERSISTENT else {}
        E = fb.Ensemble(ens.n_body, ens.mass, ens.pos, ens.vel, t0=t0)
        E.integrate(1.2, 0.0, fb.Opts(adaptive=1, eta=0.02, stop_rules=3, schedule=sched, **kw))
        got[sched] = E.state()
        E.close()
    a, b = got[fb.SCHED_PLAIN], got[fb.SCHED_PERSISTENT]
    assert len(set(a["steps"].tolist())) > 20
    for key in a:
        assert np.array_equal(a[key], b[key], equal_nan=True), key


@pytest.mark.parametrize("per_n", [1, 40, 300, 900])
def test_server_and_fused_mixes(plans, per_n):
    """Groups of every body count get one, two or four lanes a body as SIMDs allow: a server's requests and a fused
    launch against plain launches, bitwise."""
    fb = plans
    ens = gen.ragged_hill(15 * per_n, 300, n_lo=2, n_hi=16)
    t_end = 60.4 * DT
    print("[case] split mixes", per_n, flush=True)
    want = run(fb, ens, lambda E, o: E.integrate(t_end, DT, o))
    fused = run(fb, ens, lambda E, o: E.integrate(t_end, DT, o), opts=fb.Opts(schedule=fb.SCHED_PERSISTENT))
    with fb.Server(budget_bytes=512 << 20, steps_per_quantum=25) as srv:
        ids = [srv.submit_gen(ens, t_end, DT), srv.submit_gen(ens.subset(range(0, ens.n_sys, 2)), t_end / 2, DT)]
        for rid in ids:
            assert srv.wait(rid, 60.0) == fb.REQ_DONE
        got = srv.result(ids[0])
    for key in ("pos", "vel", "t", "steps", "status"):
        assert np.array_equal(want[key], fused[key]), key
        assert np.array_equal(want[key], got[key]), key

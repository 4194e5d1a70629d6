"""The unrolled body-per-lane kernels where they can go wrong: every body count
(2..4 bodies exchange by lane permutes, the others through LDS), a wavefront
that is not full, systems of one wavefront that take different numbers of
steps, and every rule.  The arithmetic and its order are those of the other
Hermite kernels, so every comparison is bitwise."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu
TWO_PI = 2 * math.pi


def run(fb, ens, mode, t0=None, schedule=None, quantum=0):
    o = dict(steps_per_quantum=quantum)
    if schedule is not None:
        o["schedule"] = schedule
    E = fb.Ensemble(ens.n_body, ens.mass, ens.pos, ens.vel, t0=t0)
    if mode == "fixed":          # whole steps and a shortened last one
        E.integrate(0.9, TWO_PI / 300, fb.Opts(**o))
    elif mode == "fixed_stops":
        E.integrate(0.9, TWO_PI / 300, fb.Opts(stop_rules=3, r_eject=2.2, **o))
    elif mode == "pairwise_stops":
        E.integrate(0.9, 0.0, fb.Opts(adaptive=1, eta=0.02, stop_rules=3, r_eject=2.2, **o))
    else:
        E.integrate(0.9, 0.0, fb.Opts(adaptive=2, eta=0.02, **o))
    st = E.state()
    st["acc"], st["jerk"], st["dtn"] = E.hermite_state()
    E.close()
    return st


def same(a, b, keys=("pos", "vel", "acc", "jerk", "t", "status", "steps", "dtn")):
    for k in keys:
        assert np.array_equal(a[k], b[k]), k


def part(ens, st, s):
    off = ens.offsets
    sl = slice(off[s], off[s + 1])
    return {k: (st[k][sl] if k in ("pos", "vel", "acc", "jerk") else st[k][s:s + 1]) for k in st}


@pytest.mark.parametrize("mode", ["fixed", "fixed_stops", "pairwise_stops", "eq5"])
@pytest.mark.parametrize("n", range(2, 17))
def test_equals_the_other_kernels(plans, n, mode):
    fb = plans
    count = 2 * (16 if n <= 4 else 64 // n) + 3      # two full wavefronts and a remainder
    ens = gen.ragged_hill(count, seed=900 + n, n_lo=n, n_hi=n, mlo=1e-5, mhi=1e-3, k_lo=3.0, k_hi=6.0, e_hi=0.2)
    # different starting times: different numbers of steps side by side
    t0 = np.linspace(0.0, 0.6, count) if mode.startswith("fixed") else None
    got = run(fb, ens, mode, t0)
    fb.set_plan(0, fb.MAP_BPL, 2, 8)
    same(got, run(fb, ens, mode, t0, schedule=fb.SCHED_PERSISTENT))       # rolled tiles
    same(got, run(fb, ens, mode, t0, quantum=13))
    if n <= (10 if mode == "fixed" else 8):
        fb.set_plan(n, fb.MAP_SPL, 1)
        same(got, run(fb, ens, mode, t0))
        fb.set_plan(n, fb.MAP_AUTO, 1)
    for s in (0, count // 2, count - 1):                                  # and alone
        one = ens.subset([s])
        same(part(ens, got, s), run(fb, one, mode, None if t0 is None else t0[s:s + 1]))

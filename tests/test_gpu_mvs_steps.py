"""The MVS step kernels where their branches change: every body count of the
system-per-lane and the body-per-lane kernel, Kepler drifts on both sides of
one radian of eccentric anomaly (series and general solution), steps back in
time, and an unbound planet among systems that share its wavefront."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen
from tests.helpers import REL_TOL, per_system_rel_err

pytestmark = pytest.mark.gpu
TWO_PI = 2 * math.pi


def batch(n, count, seed):
    """Systems of n bodies, the second of them with a planet at up to 1.6 times its orbital speed
    (escaping in most)."""
    e = gen.ragged_hill(count, seed, n_lo=n, n_hi=n, e_hi=0.3)
    vel = e.vel.copy()
    vel[n + 1] *= 1.6
    return gen.Ensemble(e.n_body, e.mass, e.pos, vel)


def determined(ora, system, dt, nsteps, o, rng):
    """Whether the oracle's own result answers a change of the inputs by half
    a unit in the last place with less than the parity bar: over 40 steps of a
    quarter of a period a close pair's chaos can amplify that beyond it, and
    then the result says nothing about the arithmetic."""
    m, x, v = system
    for _ in range(4):
        p = ora.integrate_mvs(m, x * (1 + rng.uniform(-1, 1, x.shape) * 2.0 ** -53),
                              v * (1 + rng.uniform(-1, 1, v.shape) * 2.0 ** -53), dt, nsteps)
        if per_system_rel_err([len(m)], p["pos"], o["pos"])[0] > REL_TOL / 4:
            return False
    return True


# Each drift and kick is accurate to some units of 2^-53 and an error grows
# with the orbital phase, linearly over 40 steps: far inside the parity bar.
@pytest.mark.parametrize("dt_frac", [0.01, -0.02, 0.12, 0.23])
@pytest.mark.parametrize("n,mapping", [(2, "spl"), (3, "spl"), (8, "spl"), (2, "bpl"), (3, "bpl"), (7, "bpl"),
                                       (9, "bpl"), (13, "bpl"), (16, "bpl"), (17, "bpl")])
def test_steps_match_the_oracle(plans, ora, n, mapping, dt_frac):
    fb = plans
    ens = batch(n, 70, seed=700 + n)      # more than a wavefront's systems, with a remainder
    dt, nsteps = dt_frac * TWO_PI, 40
    if n <= fb.MAX_MVS_BODIES:
        fb.set_plan(n, fb.MAP_SPL if mapping == "spl" else fb.MAP_BPL, 2)
    E = fb.from_gen(ens)
    E.integrate_mvs(nsteps, dt, fb.Opts(steps_per_quantum=17))
    st = E.state()
    E.close()
    off = ens.offsets
    rng = np.random.default_rng(n)
    chaotic = 0
    for s in range(ens.n_sys):
        o = ora.integrate_mvs(*ens.system(s), dt, nsteps)
        assert st["status"][s] == (fb.UNBOUND if o["status"] == ora.UNBOUND else fb.DONE), (s, o["status"])
        assert st["steps"][s] == o["steps"]
        sl = slice(off[s], off[s + 1])
        near = (per_system_rel_err([n], st["pos"][sl], o["pos"])[0] <= REL_TOL
                and per_system_rel_err([n], st["vel"][sl], o["vel"])[0] <= REL_TOL)
        if not near:
            assert not determined(ora, ens.system(s), dt, nsteps, o, rng), s
            chaotic += 1
    assert chaotic <= 2

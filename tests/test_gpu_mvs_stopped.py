"""MVS systems that stop while others of their wavefront go on keep what they
stopped with, the last kick's accelerations included: step counts that differ
from system to system reach the cap apart, one system (with a massless star)
has reached it already, and the run goes on afterwards.  Every mapping and a
system alone do the same arithmetic, so the comparison is bitwise."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu
DT = 0.02 * 2 * math.pi
CAP = 41


def run(fb, ens, steps):
    with fb.from_gen(ens) as E:
        ck = E.checkpoint()
    with fb.Ensemble(ens.n_body, ens.mass, ck["pos"], ck["vel"], checkpoint={**ck, "steps": steps}) as E:
        E.integrate_mvs(60, DT, fb.Opts(max_steps=CAP))
        first = E.state()
        E.integrate_mvs(25, DT)
        return first, E.state()


@pytest.mark.parametrize("n", [3, 8])
def test_stopped_systems_keep_their_state(plans, n):
    fb = plans
    ens = gen.ragged_hill(75, seed=60 + n, n_lo=n, n_hi=n, e_hi=0.3)
    ens.mass[5 * n] = 0.0
    steps = np.arange(75) % 37
    steps[5] = CAP
    fb.set_plan(n, fb.MAP_BPL, 1)
    want = run(fb, ens, steps)
    assert np.all(want[0]["status"] == fb.MAXSTEPS) and np.all(want[0]["steps"] == CAP)
    fb.set_plan(n, fb.MAP_SPL, 1)
    got = run(fb, ens, steps)
    for w, g in zip(want, got):
        for k in w:
            assert np.array_equal(w[k], g[k], equal_nan=w[k].dtype.kind == "f"), k
    for s in (4, 40):
        alone = run(fb, ens.subset([s]), steps[s:s + 1])
        for w, g in zip(got, alone):
            assert np.array_equal(w["pos"][s * n:(s + 1) * n], g["pos"])
            assert np.array_equal(w["vel"][s * n:(s + 1) * n], g["vel"])

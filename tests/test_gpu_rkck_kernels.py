"""The Cash-Karp kernels where their branches change: fixed steps system per
lane and body per lane do the same arithmetic in the same order, so the
mapping never changes a result; wavefronts that are not full; several body
counts in one launch; and adaptive steps at the limits of the step factor."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen
from tests.helpers import REL_TOL, per_system_rel_err

pytestmark = pytest.mark.gpu
TWO_PI = 2 * math.pi


def fixed(fb, ens, steps, h, quantum=0):
    E = fb.from_gen(ens)
    E.integrate_rkck_steps(steps, h, fb.Opts(steps_per_quantum=quantum))
    st = E.state()
    E.close()
    return st


@pytest.mark.parametrize("n", range(2, 8))
@pytest.mark.parametrize("count", [1, 64, 131])
def test_mappings_agree_bitwise(plans, n, count):
    fb = plans
    ens = gen.ragged_hill(count, seed=800 + n, n_lo=n, n_hi=n)
    out = []
    for m in (fb.MAP_BPL, fb.MAP_SPL):      # above 6 bodies both run body per lane
        fb.set_plan(n, m, 1)
        out += [fixed(fb, ens, 50, TWO_PI / 500), fixed(fb, ens, 50, TWO_PI / 500, quantum=17)]
    for st in out[1:]:
        for k in out[0]:
            assert np.array_equal(st[k], out[0][k]), k


def test_body_counts_share_a_launch(fb):
    ens = gen.ragged_hill(300, seed=820, n_lo=2, n_hi=16)
    st = fixed(fb, ens, 40, TWO_PI / 500)
    off = ens.offsets
    for n in range(2, 17):
        idx = np.flatnonzero(ens.n_body == n)
        one = fixed(fb, ens.subset(idx), 40, TWO_PI / 500)
        rows = np.concatenate([np.arange(off[s], off[s + 1]) for s in idx])
        assert np.array_equal(one["pos"], st["pos"][rows]) and np.array_equal(one["vel"], st["vel"][rows])


# A first step far too long (factors at their lower limits, rejections) and far
# too short (the upper limit); both ends agree with the oracle to the parity bar.
@pytest.mark.parametrize("dt0", [3.0, 1e-6])
@pytest.mark.parametrize("n", [2, 5, 16])
def test_adaptive_step_limits(fb, ora, n, dt0):
    ens = gen.ragged_hill(9, seed=830 + n, n_lo=n, n_hi=n)
    E = fb.from_gen(ens)
    E.integrate_rkck(1.5, dt0, 1e-9)
    st = E.state()
    E.close()
    off = ens.offsets
    for s in range(ens.n_sys):
        o = ora.integrate_rkck_adaptive(*ens.system(s), 1.5, 1e-9, dt0)
        assert st["status"][s] == fb.DONE and st["steps"][s] == o["steps"], (s, st["steps"][s], o["steps"])
        sl = slice(off[s], off[s + 1])
        assert per_system_rel_err([n], st["pos"][sl], o["pos"])[0] <= REL_TOL
        assert per_system_rel_err([n], st["vel"][sl], o["vel"])[0] <= REL_TOL

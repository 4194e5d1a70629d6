"""Layouts of the large-n Hermite kernel: bodies per lane and lanes per body
are chosen from the body count and the number of systems, so each kernel is
run at sizes that reach it (whole and ragged divisions of the partners over
the lanes, a last workgroup that is not full, more workgroups than the
device holds) and compared with the oracle, fixed steps and both adaptive
rules."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen
from tests.helpers import REL_TOL, per_system_rel_err, threads

pytestmark = pytest.mark.gpu
DT = 2 * math.pi / 1000

# (bodies, systems): what the layout rule takes on 256 CUs
SIZES = [
    (17, 2),        # 1 body a lane, 8 lanes a body, a remainder of one partner
    (21, 3),        # 1 and 8, remainder 5
    (64, 5),        # 1 and 8, no remainder, a full workgroup
    (36, 2),        # 1 and 4
    (19, 1024),     # 1 and 2
    (17, 2050),     # 1 and 1, 3 systems a workgroup, the last one short
    (37, 4100),     # 1 and 1, 6 systems a workgroup, more than one round
    (17, 20001),    # 2 and 1, a lane's second body missing, several rounds
    (90, 901),      # 2 and 2, 4 systems a workgroup, the last one short
    (83, 301),      # 2 and 4, ragged, two systems a workgroup
    (201, 2),       # 2 and 4, one system
    (335, 2),       # 2 and 2
    (511, 2),       # 2 and 2, the widest workgroup, a lane's second body missing
    (512, 1),
]


@pytest.mark.parametrize("n,count", SIZES)
def test_layout_parity(fb, ora, n, count):
    ens = gen.planetesimal_disk(count, n, seed=1000 + n)
    pick = sorted({0, 1 % count, count // 2, count - 1})
    sub, off = ens.subset(pick), ens.offsets
    rows = np.concatenate([np.arange(off[s], off[s + 1]) for s in pick])
    print("[case] layout", n, count, flush=True)
    nsteps = 25
    E = fb.from_gen(ens)
    E.integrate_steps(nsteps, DT)
    st = E.state()
    E.close()
    assert np.all(st["steps"] == nsteps) and np.all(st["status"] == fb.DONE)
    x, v, _, _ = ora.ensemble_fixed(sub.n_body, sub.mass, sub.pos, sub.vel, DT, nsteps, nthreads=threads())
    assert per_system_rel_err(sub.n_body, st["pos"][rows], x).max() <= REL_TOL
    assert per_system_rel_err(sub.n_body, st["vel"][rows], v).max() <= REL_TOL
    for rule, eta in ((1, 0.01), (2, 1.7e-2)):
        t_end = 0.05
        E = fb.from_gen(ens)
        E.integrate(t_end, 0.0, fb.Opts(adaptive=rule, eta=eta))
        st = E.state()
        E.close()
        assert np.all(st["t"] == t_end) and np.all(st["status"] == fb.DONE)
        for s in pick:
            o = ora.integrate_adaptive(*ens.system(s), t_end, eta=eta, stop_rules=0, paper_rule=rule == 2)
            sl = slice(off[s], off[s + 1])
            assert o["steps"] == st["steps"][s], (rule, s)
            assert per_system_rel_err([n], st["pos"][sl], o["pos"])[0] <= REL_TOL, (rule, s)
            assert per_system_rel_err([n], st["vel"][sl], o["vel"])[0] <= REL_TOL, (rule, s)

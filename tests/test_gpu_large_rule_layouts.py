"""Layouts of the large-n Hermite kernel under rules (adaptive steps, stop
rules): they weigh the slowest system and the rules' own passes, so they differ
from those of fixed steps; each kernel is run at sizes that reach it and
compared with the oracle."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen
from tests.helpers import REL_TOL, per_system_rel_err, threads

pytestmark = pytest.mark.gpu
DT = 2 * math.pi / 1000

# (bodies, systems, adaptive rule, stop rules): what the layout rule takes on 256 CUs
SIZES = [
    (17, 3, 1, 3),       # 1 body a lane, 8 lanes a body, one system a workgroup
    (18, 700, 1, 3),     # 1 and 4
    (17, 1500, 2, 0),    # 1 and 4, three systems a workgroup
    (24, 1501, 1, 0),    # 1 and 2
    (17, 2999, 1, 3),    # 1 and 2, three systems a workgroup, the last one short
    (300, 3, 1, 3),      # 1 and 1
    (33, 3000, 0, 3),    # 1 and 1, seven systems a workgroup, the last one short
    (80, 3001, 0, 3),    # 2 and 1, six systems a workgroup
    (300, 41, 2, 0),     # 2 and 2
    (128, 1499, 1, 3),   # 2 and 4
    (128, 3, 1, 3),      # 2 and 8
]


@pytest.mark.parametrize("n,count,rule,stops", SIZES)
def test_rule_layout_parity(fb, ora, n, count, rule, stops):
    ens = gen.planetesimal_disk(count, n, seed=2000 + n)
    off = ens.offsets
    pick = sorted({0, 1 % count, count // 2, count - 1})
    print("[case] rule layout", n, count, rule, stops, flush=True)
    if rule == 0:
        with fb.from_gen(ens) as E:
            E.integrate_steps(20, DT, fb.Opts(stop_rules=stops))
            st = E.state()
        assert np.all(st["steps"][pick] == 20) and np.all(st["status"][pick] == fb.DONE)
        sub = ens.subset(pick)
        rows = np.concatenate([np.arange(off[s], off[s + 1]) for s in pick])
        x, v, _, _ = ora.ensemble_fixed(sub.n_body, sub.mass, sub.pos, sub.vel, DT, 20, nthreads=threads())
        assert per_system_rel_err(sub.n_body, st["pos"][rows], x).max() <= REL_TOL
        assert per_system_rel_err(sub.n_body, st["vel"][rows], v).max() <= REL_TOL
        return
    t_end, eta = 0.05, 0.01 if rule == 1 else 1.7e-2
    # the ejection radius that every other picked system's outermost planetesimal is beyond, and none
    r = [np.linalg.norm(ens.pos[off[s] + 1:off[s + 1]] - ens.pos[off[s]], axis=1).max() for s in pick]
    for r_eject in ((100.0, 0.5 * (min(r) + max(r))) if stops else (100.0,)):
        with fb.from_gen(ens) as E:
            E.integrate(t_end, 0.0, fb.Opts(adaptive=rule, eta=eta, stop_rules=stops, r_eject=r_eject))
            st = E.state()
        for s in pick:
            o = ora.integrate_adaptive(*ens.system(s), t_end, eta=eta, stop_rules=stops, r_eject=r_eject, paper_rule=rule == 2)
            sl = slice(off[s], off[s + 1])
            assert o["steps"] == st["steps"][s] and o["status"] == st["status"][s], s
            assert per_system_rel_err([n], st["pos"][sl], o["pos"])[0] <= REL_TOL, s
            assert per_system_rel_err([n], st["vel"][sl], o["vel"])[0] <= REL_TOL, s

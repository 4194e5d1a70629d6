"""The bound that lets a wavefront skip the Hill and ejection tests of a step
never skips one that triggers: runs with the stop rules against the system
per lane kernels, which test every pair at every step, bitwise; systems that
stop from the first step on and at every later time, ejection radii inside the
systems, planets as heavy as stars, massless ones, and planets that start on
the verge of a mutual Hill radius."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu


def tight(count, n, seed):
    return gen.ragged_hill(count, seed, n_lo=n, n_hi=n, mlo=1e-5, mhi=1e-3, k_lo=2.0, k_hi=6.0, e_hi=0.3)


def verge(count, n, seed):
    """Planets 1 and 2 apart by 0.9 to 1.1 of the separation that triggers."""
    ens = tight(count, n, seed)
    rng = np.random.default_rng(seed)
    pos, off = ens.pos.copy(), ens.offsets
    for s in range(count):
        m, o = ens.mass[off[s]:off[s + 1]], off[s]
        x0, x1 = pos[o], pos[o + 1]
        q = ((m[1] + m[2]) / (3 * m[0])) ** (1 / 3) / 2
        r = np.linalg.norm(x1 - x0)
        u = rng.normal(size=3)
        pos[o + 2] = x1 + u / np.linalg.norm(u) * q * 2 * r * rng.uniform(0.9, 1.1)
    return gen.Ensemble(ens.n_body, ens.mass, pos, ens.vel)


def heavy(count, n, seed):
    ens = tight(count, n, seed)
    mass = ens.mass.copy()
    rng = np.random.default_rng(seed)
    for s, o in enumerate(ens.offsets[:-1]):
        mass[o + 1] = mass[o] * rng.choice([0.0, 1e-14, 0.3, 11.9, 12.1, 40.0])
    return gen.Ensemble(ens.n_body, mass, ens.pos, ens.vel)


@pytest.mark.parametrize("n", [5, 6, 7, 8])
@pytest.mark.parametrize("family", [tight, verge, heavy])
@pytest.mark.parametrize("count", [200, 900, 9000])   # four, two and one lanes a body
def test_equals_every_pair_tested(plans, n, family, count):
    fb = plans
    ens = family(count, n, 60 + n)
    print("[case] stop bound", n, family.__name__, count, flush=True)
    for kw in ({"adaptive": 1, "eta": 0.02, "stop_rules": 3, "r_eject": 2.5},
               {"adaptive": 2, "eta": 0.03, "stop_rules": fb.STOP_EJECT, "r_eject": 1.7},
               {"stop_rules": fb.STOP_ENCOUNTER, "r_eject": 0.0}):
        out = []
        for mapping in (fb.MAP_SPL, fb.MAP_BPL):
            fb.set_plan(n, mapping, 1)
            E = fb.from_gen(ens)
            E.integrate(1.3, 0.0 if "adaptive" in kw else 0.004, fb.Opts(max_steps=400, **kw))
            out.append(E.state())
            E.close()
        for key in out[0]:
            assert np.array_equal(out[0][key], out[1][key], equal_nan=True), (key, kw)
        if family is verge and "adaptive" in kw and kw["adaptive"] == 1:
            assert 0.02 < np.mean(out[0]["status"] == fb.ENCOUNTER)

"""Launch forms chosen for runs with rules, around the sizes where the choice
changes: rolled and unrolled body-per-lane kernels for 9 and 10 bodies with stop
rules in fixed steps, fused launches that leave such buckets to plain launches, and
the lanes a body of a fused launch with rules.  All Hermite forms of up to 16 bodies do the same
arithmetic in the same order, so every comparison is bitwise, against the same
systems in small ensembles."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu
TWO_PI = 2 * math.pi


def outer(ens, n):
    """Median distance of the outermost body of the n-body systems: about half of them have it ejected."""
    at = ens.offsets[:-1][ens.n_body == n]
    return float(np.median(np.linalg.norm(ens.pos[at + n - 1] - ens.pos[at], axis=1)))


def run(fb, ens, kind, r_eject, **o):
    with fb.from_gen(ens) as E:
        if kind == "stops":
            E.integrate_steps(14, 0.004, fb.Opts(stop_rules=3, r_eject=r_eject, **o))
        else:
            E.integrate(0.05 * TWO_PI, 0.0, fb.Opts(adaptive=2, eta=0.03, **o))
        return E.state()


def check(fb, ens, kind, **o):
    r_eject = outer(ens, int(ens.n_body.max()))
    got = run(fb, ens, kind, r_eject, **o)
    off = ens.offsets
    print("[case]", kind, ens.n_sys, sorted(set(ens.n_body.tolist())), o, flush=True)
    if kind == "stops":
        assert np.any(got["status"] != fb.DONE) and np.any(got["status"] == fb.DONE)
    pick = np.unique(np.concatenate([np.arange(8), ens.n_sys - 1 - np.arange(8), ens.n_sys // 2 + np.arange(8)]))
    few = run(fb, ens.subset(pick), kind, r_eject)
    rows = np.concatenate([np.arange(off[s], off[s + 1]) for s in pick])
    for k in ("pos", "vel"):
        assert np.array_equal(got[k][rows], few[k]), k
    for k in ("t", "status", "steps"):
        assert np.array_equal(got[k][pick], few[k]), k


def family(count, n, seed):
    return gen.ragged_hill(count, seed=seed, n_lo=n, n_hi=n, mlo=1e-5, mhi=1e-3, k_lo=2.0, k_hi=6.0, e_hi=0.2)


# 2048 wavefronts are two a SIMD
@pytest.mark.parametrize("n,count", [(9, 7 * 2048), (9, 7 * 2048 + 1), (10, 6 * 2048), (10, 6 * 2048 + 5)])
def test_plain_stops(plans, n, count):
    check(plans, family(count, n, 70 + n), "stops")


@pytest.mark.parametrize("n", [10, 13, 16])
@pytest.mark.parametrize("quantum", [0, 5])
def test_fused_stops_with_plain_launches(plans, n, quantum):
    fb = plans
    big, small = family((64 // n) * 2048, n, 80 + n), family(50, 4, 81)
    ens = gen.Ensemble(*(np.concatenate([getattr(p, f) for p in (big, small)]) for f in ("n_body", "mass", "pos", "vel")))
    for compact in (False, True):
        check(fb, ens, "stops", schedule=fb.SCHED_PERSISTENT, steps_per_quantum=quantum, compact=compact)


# the systems that 1024 wavefronts hold with two lanes a body, and with four
@pytest.mark.parametrize("kind", ["stops", "eq5"])
@pytest.mark.parametrize("n", [11, 12, 13, 14, 16])
def test_fused_lanes_a_body(plans, n, kind):
    fb = plans
    for lanes in (2, 4):
        full = 1024 * (64 // (n * lanes))
        for count in (full, full + 1):
            check(fb, family(count, n, 90 + n), kind, schedule=fb.SCHED_PERSISTENT)

"""The unrolled body-per-lane kernels at the sizes that plain launches take them
at: from the first system that the launches with several lanes a body do not take
(their wavefronts past one a SIMD; 2..4 bodies have none) and, with rules and 11
bodies and more, to the last before the rolled kernels.  A last wavefront that is
not full, systems of one wavefront that take different numbers of steps.  The
arithmetic and its order are those of the other Hermite kernels, so every comparison
is bitwise: with a few of the same systems alone (several lanes a body), with the
system-per-lane and the fused kernels, and with twice the ensemble (rolled from 11
bodies on)."""
import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu
SIMDS = 1024
KEYS = ("pos", "vel", "acc", "jerk", "t", "status", "steps", "dtn")


def sizes(n, mode):
    if n <= 4:
        return [16 * 3 + 5, 16 * SIMDS - 3 if n < 4 else 16 * SIMDS + 3]
    first = SIMDS * (64 // (2 * n)) + 1
    return [first] if mode == "fixed" or n <= 10 else [first, SIMDS * (64 // n) - 1]


def run(fb, n, ens, mode, r_eject, t0, **o):
    with fb.Ensemble(ens.n_body, ens.mass, ens.pos, ens.vel, t0=t0) as E:
        if mode == "fixed":              # whole steps and a shortened last one
            E.integrate(0.21, 0.02, fb.Opts(**o))
        elif mode == "fixed_stops":
            E.integrate(0.21, 0.02, fb.Opts(stop_rules=3, r_eject=r_eject, **o))
        elif mode == "pairwise_stops":
            E.integrate(0.25, 0.0, fb.Opts(adaptive=1, eta=0.03, stop_rules=3, r_eject=r_eject, **o))
        else:
            E.integrate(0.25, 0.0, fb.Opts(adaptive=2, eta=0.03, **o))
        st = E.state()
        st["acc"], st["jerk"], st["dtn"] = E.hermite_state()
    return st


def rows(st, n, s):
    out = {}
    for k in KEYS:
        a = st[k].reshape(-1, n, 3) if k in ("pos", "vel", "acc", "jerk") else st[k]
        out[k] = a[s]
    return out


def same(a, b):
    for k in KEYS:
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("mode", ["fixed", "fixed_stops", "pairwise_stops", "eq5"])
@pytest.mark.parametrize("n", range(2, 17))
def test_equals_the_other_kernels(plans, n, mode):
    fb = plans
    for count in sizes(n, mode):
        print("[case]", n, mode, count, flush=True)
        ens = gen.ragged_hill(count, seed=700 + n, n_lo=n, n_hi=n, mlo=1e-5, mhi=1e-3, k_lo=2.5, k_hi=6.0, e_hi=0.2)
        x = ens.pos.reshape(count, n, 3)
        r_eject = float(np.median(np.linalg.norm(x[:, -1] - x[:, 0], axis=1)))
        t0 = np.linspace(0.0, 0.15, count)[np.argsort(np.arange(count) * 7919 % count)]
        fb.set_plan(n, fb.MAP_BPL, 1)    # also where 64-system wavefronts would fill the device
        got = run(fb, n, ens, mode, r_eject, t0)
        assert len(set(got["steps"][-(64 // n):])) > 1 or mode != "fixed"
        same(got, run(fb, n, ens, mode, r_eject, t0, steps_per_quantum=4))
        pick = np.r_[0:5, count // 2, count - 3:count]
        same(rows(got, n, pick), rows(run(fb, n, ens.subset(pick), mode, r_eject, t0[pick]), n, slice(None)))
        twice = np.r_[0:count, 0:count]
        both = run(fb, n, ens.subset(twice), mode, r_eject, t0[twice])
        same(rows(got, n, slice(None)), rows(both, n, slice(0, count)))
        same(rows(got, n, slice(None)), rows(both, n, slice(count, None)))
        fb.set_plan(n, fb.MAP_AUTO, 1)
        same(got, run(fb, n, ens, mode, r_eject, t0, schedule=fb.SCHED_PERSISTENT))
        if n <= (10 if mode == "fixed" else 8):
            fb.set_plan(n, fb.MAP_SPL, 1)
            same(got, run(fb, n, ens, mode, r_eject, t0))
            fb.set_plan(n, fb.MAP_AUTO, 1)

"""The fused launch of fixed steps with stop rules for 9..16 bodies (rolled tiles,
three wavefronts a SIMD), from the first size that takes it on, in one launch, in
quanta and compacted down to where the other class takes over.  All Hermite forms
of up to 16 bodies do the same arithmetic in the same order, so every comparison
is bitwise, against the plain schedule."""
import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu
TILES = 2048       # two wavefronts a SIMD


def family(parts):
    out = [gen.ragged_hill(c, seed=300 + n, n_lo=n, n_hi=n, mlo=1e-5, mhi=1e-3, k_lo=2.0, k_hi=6.0, e_hi=0.2) for n, c in parts]
    return gen.Ensemble(*(np.concatenate([getattr(p, f) for p in out]) for f in ("n_body", "mass", "pos", "vel")))


def run(fb, ens, r_eject, t_end=None, **o):
    opts = fb.Opts(stop_rules=3, r_eject=r_eject, **o)
    with fb.from_gen(ens) as E:
        E.integrate_steps(20, 0.01, opts) if t_end is None else E.integrate(t_end, 0.01, opts)
        st = E.state()
        st["acc"], st["jerk"], _ = E.hermite_state()
    return st


CASES = [[(n, TILES * (64 // n) + k)] for n in (10, 13, 16) for k in (0, 64 // n)] + [
    [(9, 7 * 900), (10, 6 * 700), (12, 5 * 600), (16, 4 * 300 + 1)],      # a quarter of 9 bodies
    [(9, 7 * 1500), (11, 5 * 700)],                                       # two thirds
    [(3, 40), (11, 5 * 1200), (16, 4 * 1300)]]                            # and beside smaller ones


@pytest.mark.parametrize("parts", CASES)
def test_equals_the_plain_schedule(plans, parts):
    fb = plans
    ens = family(parts)
    off = ens.offsets
    out = np.array([np.linalg.norm(ens.pos[off[s]:off[s + 1]] - ens.pos[off[s]], axis=1).max() for s in range(ens.n_sys)])
    P = dict(schedule=fb.SCHED_PERSISTENT)
    # about half of the systems stop; nearly all, so that compaction leaves a few wavefronts
    for r_eject, forms in ((float(np.median(out)), ({}, {"steps_per_quantum": 3}, {"steps_per_quantum": 3, "compact": True})),
                           (float(np.quantile(out, 0.05)), ({"steps_per_quantum": 2, "compact": True},))):
        for t_end in (None, 0.205):
            want = run(fb, ens, r_eject, t_end)
            assert np.any(want["status"] == fb.DONE) and np.any(want["status"] != fb.DONE)
            for o in forms:
                print("[case]", parts, r_eject, t_end, o, flush=True)
                got = run(fb, ens, r_eject, t_end, **P, **o)
                for k in ("pos", "vel", "acc", "jerk", "t", "status", "steps"):
                    assert np.array_equal(got[k], want[k]), k

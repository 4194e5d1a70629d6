"""Launches of a few steps, which run rolled where longer ones run with several
lanes a body or unrolled: runs cut into launches of one, two and four steps against
one launch, at sizes on both sides of every line of the choice.  All Hermite forms of
up to 16 bodies do the same arithmetic in the same order and the step is a power of
two, so every comparison is bitwise."""
import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu
SIMDS = 1024
KEYS = ("pos", "vel", "acc", "jerk", "t", "status", "steps", "dtn")


def counts(n):
    """Sizes around three eighths, a half and seven eighths of the SIMDs taken with
    two lanes a body, and half, three quarters and all of them with one."""
    S, S2 = 64 // n, 64 // (2 * n)
    out = [SIMDS * S // 2 + 1, SIMDS * S * 3 // 4 + 1, SIMDS * S, SIMDS * S + 1]
    return out if n == 4 else [SIMDS * S2 * 3 // 8 + S2, SIMDS * S2 // 2 + S2, SIMDS * S2 * 7 // 8 + S2] + out


def run(fb, ens, cuts, r_eject, adaptive, quantum):
    o = dict(steps_per_quantum=quantum, stop_rules=3 if r_eject else 0, r_eject=r_eject or 100.0)
    with fb.from_gen(ens) as E:
        if adaptive:
            E.integrate(0.15, 0.0, fb.Opts(adaptive=adaptive, eta=0.03, **o))
        else:
            for k in cuts:
                E.integrate_steps(k, 1 / 64, fb.Opts(**o))
        st = E.state()
        st["acc"], st["jerk"], st["dtn"] = E.hermite_state()
    return st


@pytest.mark.parametrize("n", range(4, 17))
def test_cut_runs_equal_whole_ones(plans, n):
    fb = plans
    fb.set_plan(n, fb.MAP_BPL, 1)
    for count in counts(n):
        ens = gen.ragged_hill(count, seed=500 + n, n_lo=n, n_hi=n, mlo=1e-5, mhi=1e-3, k_lo=2.5, k_hi=6.0, e_hi=0.2)
        x = ens.pos.reshape(count, n, 3)
        out = float(np.median(np.linalg.norm(x[:, -1] - x[:, 0], axis=1)))
        print("[case]", n, count, flush=True)
        for r_eject in (None, out):
            want = run(fb, ens, [12], r_eject, 0, 0)
            assert r_eject is None or len(set(want["status"])) > 1
            for cuts, quantum in (([1] * 12, 0), ([2] * 6, 0), ([4, 3, 5], 0), ([12], 1)):
                got = run(fb, ens, cuts, r_eject, 0, quantum)
                for k in KEYS:
                    assert np.array_equal(got[k], want[k]), (k, cuts, quantum, r_eject)
        for adaptive in (1, 2):
            want, got = (run(fb, ens, None, out, adaptive, q) for q in (0, 1))
            for k in KEYS:
                assert np.array_equal(got[k], want[k]), (k, adaptive)

"""Fused launches whose tiles all run at once, more than one a SIMD (1024 of
them): tile counts around the ends of that range, each tile taken exactly once
whatever the plan's resident wavefronts, against plain launches, bitwise."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1023, 1024, 1025, 1500, 2047, 2048, 2049])
def test_every_tile_once(plans, tiles):
    fb = plans
    n8, n4 = 500, tiles - 500   # tiles of 8 systems and of 16, the last of each not full
    parts = [gen.ragged_hill(8 * n8 - 3, 31, n_lo=8, n_hi=8), gen.ragged_hill(16 * n4 - 7, 32, n_lo=4, n_hi=4)]
    ens = gen.Ensemble(*(np.concatenate([getattr(p, f) for p in parts]) for f in ("n_body", "mass", "pos", "vel")))
    print("[case] placing", tiles, flush=True)

    def run(**kw):
        adaptive = kw.pop("adaptive", 0)
        E = fb.from_gen(ens)
        if adaptive:
            E.integrate(0.05 * 2 * math.pi, 0.0, fb.Opts(adaptive=adaptive, eta=0.02, stop_rules=3, **kw))
        else:
            E.integrate_steps(9, 0.002, fb.Opts(**kw))
        st = E.state()
        E.close()
        return st

    for adaptive in (0, 1):
        want = run(adaptive=adaptive)
        assert np.all(want["steps"] > 0)
        for groups in (8, 5):
            fb.set_plan(0, fb.MAP_AUTO, 2, groups)
            for kw in ({}, {"steps_per_quantum": 13, "compact": True}):
                got = run(adaptive=adaptive, schedule=fb.SCHED_PERSISTENT, **kw)
                for key in want:
                    assert np.array_equal(want[key], got[key]), (key, adaptive, groups, kw)

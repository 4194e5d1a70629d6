"""What the autotuner times and installs: a body-per-lane launch that does not
depend on the waves per workgroup once, and for the fused launch the automatic
class, which places tiles and runs thinned populations on, where an explicit
body-per-lane class is not clearly faster."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu
H = 2 * math.pi / 2000


def tune(fb, ens):
    with fb.from_gen(ens) as E:
        return E.autotune(40, H)


def test_automatic_class_stays(plans):
    fb = plans
    # too few systems for a system per lane, so the body-per-lane class is the faster
    entries = tune(fb, gen.ragged_hill(3000, seed=3, n_lo=4, n_hi=8))
    fused = [e for e in entries if e["n"] == 0]
    best = min((e for e in fused if e["mapping"] != fb.MAP_AUTO), key=lambda e: e["ms"])
    auto = [e for e in fused if e["mapping"] == fb.MAP_AUTO]
    chosen = [e for e in fused if e["chosen"]]
    assert best["mapping"] == fb.MAP_BPL and len(auto) == 1 and len(chosen) == 1
    assert (auto[0]["waves_per_group"], auto[0]["groups_per_cu"]) == (best["waves_per_group"], best["groups_per_cu"])
    assert chosen[0] == (auto[0] if auto[0]["ms"] <= 1.02 * best["ms"] else best)
    assert fb.get_plan(0) == (chosen[0]["mapping"], chosen[0]["waves_per_group"], chosen[0]["groups_per_cu"])


def test_waves_per_group_timed_where_they_matter(plans):
    fb = plans
    fb.set_plan(6, fb.MAP_AUTO, 3)
    entries = [e for e in tune(fb, gen.ragged_hill(3000, seed=4, n_lo=6, n_hi=6)) if e["n"] == 6]
    bpl = [e["waves_per_group"] for e in entries if e["mapping"] == fb.MAP_BPL]
    assert bpl == [3]
    assert sorted(e["waves_per_group"] for e in entries if e["mapping"] == fb.MAP_SPL) == [1, 2, 4]
    # rolled: 3 bodies with more wavefronts than SIMDs
    ens = gen.three_body(30000, 5)
    entries = [e for e in tune(fb, ens) if e["n"] == 3]
    assert sorted(e["waves_per_group"] for e in entries if e["mapping"] == fb.MAP_BPL) == [1, 2, 4]
    assert np.sum([e["chosen"] for e in entries]) == 1

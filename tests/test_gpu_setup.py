"""Set-up, start of a run and read-back of every bucket of an ensemble in one
launch: body counts that divide a wavefront and that do not, bucket sizes
around a tile and a workgroup, and more buckets than one launch takes."""
import math

import numpy as np
import pytest

from paper_1208_1157_amd import gen
from tests.helpers import per_system_rel_err, threads

pytestmark = pytest.mark.gpu
DT = 2 * math.pi / 1000


def ensemble(counts, seed):
    parts = [gen.planetesimal_disk(k, n, seed=seed + n) if n > 16 else gen.ragged_hill(k, seed + n, n_lo=n, n_hi=n)
             for n, k in counts]
    e = gen.Ensemble(*(np.concatenate([getattr(p, f) for p in parts]) for f in ("n_body", "mass", "pos", "vel")))
    return e.subset(np.random.default_rng(seed).permutation(e.n_sys))   # buckets gather scattered systems


@pytest.mark.parametrize("counts", [
    [(2, 1)], [(3, 21), (16, 4)], [(5, 12), (7, 9), (11, 5)], [(2, 129), (3, 85), (4, 64), (6, 41), (9, 257)],
    [(n, 3 + n) for n in range(2, 17)],
    [(n, 2) for n in range(2, 17)] + [(n, 1 + n % 3) for n in range(17, 52)],   # 50 buckets
], ids=lambda c: f"{len(c)}buckets-{sum(k for _, k in c)}")
def test_set_up_and_read_back(fb, ora, counts):
    ens = ensemble(counts, 700)
    t0 = np.random.default_rng(1).uniform(-3.0, 3.0, ens.n_sys)
    print("[case] setup", counts[:5], flush=True)
    E = fb.Ensemble(ens.n_body, ens.mass, ens.pos, ens.vel, t0=t0)
    st = E.state()
    assert np.array_equal(st["pos"], ens.pos) and np.array_equal(st["vel"], ens.vel)
    assert np.array_equal(st["t"], t0) and np.all(st["status"] == fb.DONE) and np.all(st["steps"] == 0)
    acc, jerk, dtn = E.hermite_state()
    assert np.all(dtn == 0)
    off = ens.offsets
    for s in range(ens.n_sys):
        a, j = ora.accjerk(*ens.system(s))
        sl = slice(off[s], off[s + 1])
        assert per_system_rel_err([ens.n_body[s]], acc[sl], a)[0] <= 1e-13, s
        assert per_system_rel_err([ens.n_body[s]], jerk[sl], j)[0] <= 1e-13, s
    energy, angmom = E.diagnostics()
    er, lr = ora.ensemble_energy(ens.n_body, ens.mass, ens.pos, ens.vel)
    assert np.all(np.abs(energy - er) <= 1e-12 * np.abs(er))
    assert np.all(np.linalg.norm(angmom - lr, axis=1) <= 1e-12 * np.linalg.norm(lr, axis=1))
    E.integrate_steps(7, DT)
    st = E.state()
    assert np.all(st["steps"] == 7) and np.allclose(st["t"], t0 + 7 * DT, rtol=0, atol=1e-14)
    x, v, _, _ = ora.ensemble_fixed(ens.n_body, ens.mass, ens.pos, ens.vel, DT, 7, nthreads=threads())
    assert per_system_rel_err(ens.n_body, st["pos"], x).max() <= 1e-12
    assert per_system_rel_err(ens.n_body, st["vel"], v).max() <= 1e-12
    # into the other form and back: the converted read-back is the state that the conversion in place leaves
    E.integrate_mvs(1, 1e-3)
    there = E.state()
    E.integrate_rkck_steps(1, 1e-12)
    back = E.state()
    E.close()
    assert per_system_rel_err(ens.n_body, there["pos"], back["pos"]).max() <= 1e-10
    assert per_system_rel_err(ens.n_body, there["vel"], back["vel"]).max() <= 1e-10


@pytest.mark.parametrize("what", ["mass", "pos", "vel", "t0"])
def test_invalid_device_inputs_are_refused(fb, what):
    ens = ensemble([(3, 30), (9, 30), (20, 3)], 710)
    bad = {"mass": ens.mass.copy(), "pos": ens.pos.copy(), "vel": ens.vel.copy(), "t0": np.zeros(ens.n_sys)}
    flat = bad[what].reshape(-1)
    for at in (0, len(flat) // 2, len(flat) - 1):
        keep, flat[at] = flat[at], math.nan
        with pytest.raises(fb.FewbodyError) as err:
            fb.Ensemble(ens.n_body, bad["mass"], bad["pos"], bad["vel"], t0=bad["t0"])
        assert err.value.code == fb.E_INVAL
        flat[at] = keep

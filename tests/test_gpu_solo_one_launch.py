"""Stateless batches that one launch sets up, steps and writes back, against
an ensemble of the same systems, bitwise: every body count, partial
wavefronts, sizes on either side of what takes the one launch, and a system
that turns non-finite."""
import math

import numpy as np
import pytest
import torch

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu
H = 2 * math.pi / 1000


@pytest.mark.parametrize("n", range(2, 17))
@pytest.mark.parametrize("count", [1, 5, 64, 1100, 17000])
def test_equals_ensemble(fb, n, count):
    ens = gen.ragged_hill(count, 400 + n, n_lo=n, n_hi=n)
    pos0 = ens.pos.copy()
    if count == 64 and n > 2:
        pos0[5 * n + 2] = pos0[5 * n + 1]   # system 5 turns non-finite
    print("[case] solo", n, count, flush=True)
    mass = torch.from_numpy(ens.mass).cuda()
    for steps in (1, 13):
        pos, vel = torch.from_numpy(pos0.copy()).cuda(), torch.from_numpy(ens.vel.copy()).cuda()
        status = torch.full((count,), 77, dtype=torch.int32, device="cuda")
        fb.hermite_steps_device(n, mass, pos, vel, steps, H, status=status)
        E = fb.Ensemble(ens.n_body, ens.mass, pos0, ens.vel)
        E.integrate_steps(steps, H)
        st = E.state()
        E.close()
        assert np.array_equal(pos.cpu().numpy(), st["pos"], equal_nan=True)
        assert np.array_equal(vel.cpu().numpy(), st["vel"], equal_nan=True)
        assert np.array_equal(status.cpu().numpy(), st["status"])
        assert (st["status"] == fb.NONFINITE).sum() == (1 if count == 64 and n > 2 else 0)
    pos, vel = torch.from_numpy(pos0.copy()).cuda(), torch.from_numpy(ens.vel.copy()).cuda()
    fb.hermite_steps_device(n, mass, pos, vel, 0, H)   # no steps, no status
    assert np.array_equal(pos.cpu().numpy(), pos0) and np.array_equal(vel.cpu().numpy(), ens.vel)

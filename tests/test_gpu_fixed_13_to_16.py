"""Fixed steps of 13..16 bodies, whose unrolled kernels read their partners in
parts: one, four and more wavefronts a SIMD (the last ones rolled in plain
launches), fused and plain, bitwise against the same systems in a small
ensemble (several lanes a body)."""
import numpy as np
import pytest

from paper_1208_1157_amd import gen

pytestmark = pytest.mark.gpu


def run(fb, ens, **o):
    with fb.from_gen(ens) as E:
        E.integrate_steps(14, 0.004, fb.Opts(**o))
        return E.state()


@pytest.mark.parametrize("count", [4 * 1024 + 3, 4 * 4096, 4 * 4096 + 1])
@pytest.mark.parametrize("n", [13, 14, 15, 16])
def test_equals_a_small_ensemble(fb, n, count):
    ens = gen.ragged_hill(count, seed=95 + n, n_lo=n, n_hi=n, mlo=1e-5, mhi=1e-3, k_lo=2.0, k_hi=6.0, e_hi=0.2)
    pick = np.concatenate([np.arange(8), count // 2 + np.arange(8), count - 8 + np.arange(8)])
    few = run(fb, ens.subset(pick))
    rows = (n * pick[:, None] + np.arange(n)).ravel()
    for o in ({}, {"schedule": fb.SCHED_PERSISTENT}):
        print("[case] fixed", n, count, o, flush=True)
        got = run(fb, ens, **o)
        for k in ("pos", "vel"):
            assert np.array_equal(got[k][rows], few[k]), k
        for k in ("t", "status", "steps"):
            assert np.array_equal(got[k][pick], few[k]), k

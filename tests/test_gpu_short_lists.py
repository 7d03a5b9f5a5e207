"""FP64 forces of dilute systems: the number of wavefronts that share a list
follows the expected length of the lists (12 and 54 entries) from 1280
wavefronts on.
Forces and energies against the oracle on either side, through a step and a
rebuild, and one step of a call against the fused ones."""
import numpy as np
import pytest

import oracle as O
from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


# 1250 wavefronts (four each, whatever the length), and 1594 with 2, 9, 17, 45 and 59 entries
@pytest.mark.parametrize("n,rho", [(80000, 0.1), (102000, 0.02), (102000, 0.1), (102000, 0.2), (102000, 0.53), (102000, 0.7)])
def test_fp64_forces_of_short_lists(n, rho):
    print(f"case short lists n={n} rho={rho}", flush=True)
    L = W.box_for(n, rho)
    na = W.n_a_for(n)
    pos, vel = W.lattice_config(n, L, 17, 0.05), W.gaussian_velocities(n, 1.0, 5)
    s = md.System([(n, na, L, 1.0, 3)], precision="fp64", positions=pos, velocities=vel, dt=0.002)
    t = md.System([(n, na, L, 1.0, 3)], precision="fp64", positions=pos, velocities=vel, dt=0.002)
    for steps in (0, 60, 300):  # (at 0.02 nothing is in reach at the start)
        s.step_nve(steps)
        for _ in range(steps):
            t.step_nve(1)
        obs = s.forces(energy=True)[0]
        a, b = s.numpy(), t.numpy()
        for k in ("x", "y", "z", "vx", "vy", "vz"):
            assert np.array_equal(a[k], b[k]), k
        fx, fy, fz, pe, w = O.forces(a["x"], a["y"], a["z"], na, L, "cell")
        num = sum(np.sum((a[k] - f) ** 2) for k, f in (("ax", fx), ("ay", fy), ("az", fz)))
        assert num <= 1e-24 * np.sum(fx ** 2 + fy ** 2 + fz ** 2)
        assert obs[0] == pytest.approx(pe, rel=1e-12, abs=1e-12 * n) and obs[1] == pytest.approx(w, rel=1e-12, abs=1e-12 * n)
    assert md.md_stats(s.ctx)["rebuilds"] > 1 and s.status() == 0
    s.close()
    t.close()

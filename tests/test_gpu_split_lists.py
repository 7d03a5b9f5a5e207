"""The shared-list force kernels on both sides of each size where the number
of wavefronts per list changes (512, 1024, 2048 and 8192 particle wavefronts),
and on a single wavefront per species.

MIXED and MIXED_FIXED: forces, energies and a few steps equal those of the
unsplit kernel, which the window variant runs, bit for bit.  FP64: forces
against the oracle; its sums are the same terms in another order, and 64 to 90
of them of either sign lose at most a few hundred units in the last place of
the largest, hence 1e-12."""
import numpy as np
import pytest

import oracle as O
from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


def make(n, prec):
    L = max(W.box_for(n, 1.2), 6.5)
    pos = W.lattice_config(n, L, 17, 0.08)
    return md.System([(n, W.n_a_for(n), L, 1.0, 3)], precision=prec, positions=pos,
                     velocities=W.gaussian_velocities(n, 1.0, 5)), pos, L


@pytest.mark.parametrize("prec", ["mixed", "mixed_fixed"])
@pytest.mark.parametrize("n", [70, 32700, 32900, 65400, 65800, 130900, 131300, 524100, 524900])
def test_split_equals_unsplit_bit_for_bit(n, prec):
    print(f"case split lists n={n} {prec}", flush=True)
    out = []
    for windows in (0, 1):
        s, _, _ = make(n, prec)
        md.md_set_force_kernel(s.ctx, windows, 256)
        s.build_cells()
        obs = s.forces(energy=True)
        s.step_nve(3)
        assert s.status() == 0
        out.append((obs, s.numpy()))
        s.close()
    assert np.array_equal(out[0][0], out[1][0])
    for k in out[0][1]:
        assert np.array_equal(out[0][1][k], out[1][1][k]), k


@pytest.mark.parametrize("n", [70, 32700, 32900])
def test_fp64_split_forces_match_oracle(n):
    print(f"case split lists n={n} fp64", flush=True)
    s, pos, L = make(n, "fp64")
    obs = s.forces(energy=True)[0]
    a = s.numpy(("ax", "ay", "az"))
    fx, fy, fz, pe, w = O.forces(*pos, W.n_a_for(n), L, "cell")
    num = sum(np.sum((a[k] - f) ** 2) for k, f in (("ax", fx), ("ay", fy), ("az", fz)))
    assert np.sqrt(num / np.sum(fx ** 2 + fy ** 2 + fz ** 2)) <= 1e-12
    assert obs[0] == pytest.approx(pe, rel=1e-12) and obs[1] == pytest.approx(w, rel=1e-12)
    s.close()

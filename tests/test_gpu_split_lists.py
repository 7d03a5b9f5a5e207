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


@pytest.mark.parametrize("n,prec,windows", [
    (70, "fp64", 0), (33000, "fp64", 0), (70, "mixed", 0), (70, "mixed_fixed", 0), (33000, "mixed_fixed", 0),
    (131300, "mixed", 0), (524900, "mixed", 0), (33000, "mixed", 1), (33000, "mixed_fixed", 1),
])
def test_the_force_kernel_closes_the_step(n, prec, windows):
    """The closing half kick of the force kernels that store the forces, in
    each of them: steps of one call each equal the fused ones bit for bit, the
    sampled kinetic energy is that of the velocities (sums in another order:
    1e-12), and a Nose-Hoover bath too heavy to act (xi ~ 1e-12) follows the
    NVE trajectory (a position on the fixed-point grid may round the other
    way: 2e-8 in a separation, 1e-7 in a velocity)."""
    print(f"case closing kick n={n} {prec} windows={windows}", flush=True)
    out = []
    for how in ("fused", "single", "sampled", "nose"):
        L = max(W.box_for(n, 1.2), 6.5)
        s = md.System([(n, W.n_a_for(n), L, 1.0, 3)], precision=prec, positions=W.lattice_config(n, L, 17, 0.08),
                      velocities=W.gaussian_velocities(n, 1.0, 5), sample_every=1 if how == "sampled" else 0,
                      sample_capacity=8)
        if prec != "fp64":
            md.md_set_force_kernel(s.ctx, windows, 256)
        s.build_cells()
        s.forces()
        if how == "fused":
            s.step_nve(3)
        elif how == "nose":
            s.step_nvt(3, md.NVT_NOSE_HOOVER, tau=1e6)
        else:
            for k in range(3):
                s.step_nve(1)
                if how == "sampled":
                    a = s.numpy(("vx", "vy", "vz"))
                    ke = 0.5 * sum(float(np.dot(u, u)) for u in a.values())
                    row = np.asarray(s.samples()).reshape(-1, 6)[k]
                    assert row[1] == pytest.approx(ke, rel=1e-12)
        assert s.status() == 0
        out.append(s.numpy())
        s.close()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k
        assert np.array_equal(out[0][k], out[2][k]), k
    for k in ("x", "y", "z", "vx", "vy", "vz"):
        assert np.abs(out[3][k] - out[0][k]).max() < 1e-6, k


@pytest.mark.parametrize("n", [81800, 82000])
def test_split_rule_of_mixed_fixed_at_1280_wavefronts(n):
    """Four and two wavefronts per list, on either side of the line: the sums
    are exact, so both equal the window variant's bit for bit."""
    test_split_equals_unsplit_bit_for_bit(n, "mixed_fixed")

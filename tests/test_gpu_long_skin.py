"""Skins longer than a small box can serve: the lists hold every pair within
the cutoff plus the skin in use (md_stats skin_min), so that no pair enters the
cutoff unlisted before a rebuild."""
import numpy as np
import pytest

from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed", "mixed_fixed"])
def test_a_pair_that_starts_beyond_0_707_box_edges_is_seen(prec):
    """Two particles close in from 0.84 box edges apart (list radius 0.96) to
    below the cutoff, without having moved half the skin: equal and opposite
    forces, that of the pair."""
    print(f"case long skin pair {prec}", flush=True)
    L, skin = 5.1, 2.4
    u = np.array([2.5, 2.5, 2.4])
    v = u / np.linalg.norm(u)
    s = md.System([(2, 2, L, 1.0, 1)], precision=prec, positions=([0.1, 0.1 + u[0]], [0.1, 0.1 + u[1]], [0.1, 0.1 + u[2]]),
                  velocities=([v[0], -v[0]], [v[1], -v[1]], [v[2], -v[2]]), skin=skin, dt=0.005)
    s.step_nve(225)  # 1.125 each
    a = s.numpy()
    d = np.array([a[k][0] - a[k][1] for k in "xyz"])
    r2 = float(d @ d)
    assert 1.9 < r2 ** 0.5 < 2.2 and s.status() == 0
    s6 = r2 ** -3
    f = 48.0 * s6 * (s6 - 0.5) / r2 * d
    got = np.array([a[k][0] for k in ("ax", "ay", "az")])
    assert np.abs(got - f).max() <= 1e-5 * np.abs(f).max()
    s.close()


@pytest.mark.parametrize("n,L,skin,dim,cell_div,windows", [
    (140, 5.3, 1.5, 3, 1, 0),
    (140, 5.3, 1.5, 3, 2, 0),
    (140, 5.3, 1.5, 3, 1, 1),
    (300, 6.5, 40.0, 3, 1, 0),
    (60, 7.1, 3.0, 2, 1, 0),
    (1000, 9.41, 4.5, 3, 1, 0),
])
def test_lists_hold_every_pair_within_the_skin_in_use(n, L, skin, dim, cell_div, windows):
    print(f"case long skin lists n={n} skin={skin} dim={dim} div={cell_div} windows={windows}", flush=True)
    na = W.n_a_for(n)
    if dim == 2:
        pos, v = W.planar_lattice_config(n, L, 5), W.gaussian_velocities(n, 0.1, 3)
        vel = (v[0], v[1], np.zeros(n))
    else:
        pos, vel = W.lattice_config(n, L, 5, 0.12), W.gaussian_velocities(n, 0.1, 3)
    s = md.System([(n, na, L, 1.0, 3)], precision="mixed", positions=pos, velocities=vel, skin=skin, dim=dim,
                  cell_div=cell_div)
    md.md_set_force_kernel(s.ctx, windows, 256)
    s.build_cells()
    st = md.md_stats(s.ctx)
    assert s.status() == 0
    d = np.stack([p[:, None] - p[None, :] for p in map(np.asarray, pos)])
    d -= L * np.rint(d / L)
    r = np.sqrt((d * d).sum(0))
    b = np.arange(n) >= na
    rc = 2.5 * np.array(md.KA_SIGMA)[b[:, None].astype(int) + b[None, :]]
    pairs = (r < rc + st["skin_min"]).sum(1) - 1
    assert st["mean_list_len"] * n >= pairs.sum()
    assert st["max_list_len"] >= pairs.max()
    s.close()

"""Which list builder a worklist gets: on either side of each line of the rule,
and the builders' corners that sizes alone do not reach, against the window
variant's builder.  The same entries in the same order, so the same MIXED
forces bit for bit."""
import numpy as np
import pytest

from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


def _config(n, L, dim, seed):
    if dim == 2:
        pos, v = W.planar_lattice_config(n, L, seed), W.gaussian_velocities(n, 0.5, 3)
        return pos, (v[0], v[1], np.zeros(n))
    return W.lattice_config(n, L, seed, 0.12), W.gaussian_velocities(n, 0.5, 3)


@pytest.mark.parametrize("reps,dim", [
    ([(48900, 34.4)], 3),                  # 765 wavefronts: by blocks
    ([(49300, 34.5)], 3),                  # 772: by masks
    ([(65300, 37.9), (60, 5.3)], 3),       # a batch of 1024, nearly 2^16 slots in one replica: by blocks
    ([(1000, 9.41)] * 75, 3),              # 1275: by blocks
    ([(1000, 9.41)] * 76, 3),              # 1292: by masks
    ([(20000, 128.9)] * 4, 2),             # planar, 1252: by blocks of three
    ([(20000, 128.9)] * 5, 2),             # planar, 1565: by masks
    ([(40, 5.8), (70, 8.5), (300, 15.8)] * 150, 2),  # planar, two (whole rows), three and five cells per edge: by masks
])
def test_builders_on_either_side_of_the_rule(reps, dim):
    print(f"case list rule {len(reps)} x {reps[0]} dim={dim}", flush=True)
    parts = [_config(n, L, dim, 5) for n, L in reps]
    pos = [np.concatenate([p[0][k] for p in parts]) for k in range(3)]
    vel = [np.concatenate([p[1][k] for p in parts]) for k in range(3)]
    out = []
    for windows in (0, 1):
        s = md.System([(n, W.n_a_for(n), L, 1.0, 3) for n, L in reps], precision="mixed", positions=pos, velocities=vel,
                      dim=dim, dt=0.001)
        md.md_set_force_kernel(s.ctx, windows, 256)
        s.build_cells()
        s.forces()
        st = md.md_stats(s.ctx)
        s.step_nve(3)
        assert s.status() == 0
        out.append((s.numpy(), st))
        s.close()
    for k in out[0][0]:
        assert np.array_equal(out[0][0][k], out[1][0][k]), k
    assert out[0][1]["mean_list_len"] == pytest.approx(out[1][1]["mean_list_len"], rel=0.006)

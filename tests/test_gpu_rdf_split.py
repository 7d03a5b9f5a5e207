"""The split histogram kernel at the edges of its ranges: counts equal the
oracle's O(N^2) ones exactly."""
import numpy as np
import pytest

import oracle as O
from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


def check(s, pos, reps, dr, nb, dim=3):
    h = s._host(s.rdf(dr, nb)).astype(np.uint64)
    o = 0
    for r, (n, na, L, _, _) in enumerate(reps):
        x, y, z = (p[o:o + n] for p in pos)
        ref = O.rdf_hist(x, y, z, na, L, dr, nb)
        assert np.array_equal(h[r], ref), (r, np.argwhere(h[r] != ref)[:5])
        o += n


@pytest.mark.parametrize("n,L,dr,nb", [
    (65, 9.0, 4.5, 1),            # one bin, one wavefront and a lane
    (300, 6.3, 3.1 / 5120, 5120), # more bins than the staging holds: atomics
    (513, 7.6, 4e-9, 40),         # bins about as wide as the fixed-point step
    (2049, 12.0, 6.0 / 200, 200), # half the box, 4 cells per edge
    (5003, 16.1, 3.3 / 77, 77),   # pruned stencils, several splits
])
def test_counts_at_the_edges_of_the_split(n, L, dr, nb):
    print(f"case rdf split n={n} nb={nb}", flush=True)
    pos = W.lattice_config(n, L, 7, 0.2)
    reps = [(n, W.n_a_for(n), L, 1.0, 1)]
    s = md.System(reps, precision="mixed", positions=pos, velocities=W.gaussian_velocities(n, 1.0, 2))
    check(s, pos, reps, dr, nb)
    s.close()


def test_pairs_on_bin_edges():
    """A perfect lattice of spacing 1 with bins of 1/4 and 1/8: every axis
    distance sits on an edge, where the definition alone decides."""
    m, L = 12, 12.0
    k = np.arange(m ** 3)
    pos = tuple(np.ascontiguousarray(v, np.float64) for v in (k % m + 0.25, (k // m) % m + 0.5, k // (m * m) + 0.0))
    reps = [(m ** 3, 1400, L, 1.0, 1)]
    print("case rdf lattice edges", flush=True)
    s = md.System(reps, precision="fp64", positions=pos, velocities=W.gaussian_velocities(m ** 3, 0.1, 2))
    for dr, nb in ((0.25, 24), (0.125, 40), (0.1, 60)):
        check(s, pos, reps, dr, nb)
    s.close()


def test_uneven_batch():
    ns = (250, 4097, 70, 1000, 511)
    reps = [(n, W.n_a_for(n), max(W.box_for(n, 1.2), 6.2), 1.0, 5 + n) for n in ns]
    parts = [W.lattice_config(n, L, 3 + n, 0.15) for n, _, L, _, _ in reps]
    pos = tuple(np.concatenate([p[k] for p in parts]) for k in range(3))
    n = sum(ns)
    print("case rdf uneven batch", flush=True)
    s = md.System(reps, precision="mixed_fixed", positions=pos, velocities=W.gaussian_velocities(n, 0.5, 2))
    check(s, pos, reps, 3.1 / 200, 200)
    check(s, pos, reps, 3.05 / 3000, 3000)
    s.close()

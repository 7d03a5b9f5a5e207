"""The result of a histogram measurement: two contexts that add to one tensor,
and bins as narrow as the positions' fixed-point step."""
import numpy as np
import pytest

import oracle as O
from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


def test_two_contexts_add_to_one_histogram():
    """Measurements of two contexts on their own streams accumulate into one
    tensor at the same time: no count is lost, of partial histograms (20 bins)
    or of blocks that add to the result themselves (600 bins of 200 particles)."""
    print("case rdf two contexts", flush=True)
    for n, nb in ((3000, 20), (200, 600)):
        L = max(W.box_for(n, 1.2), 6.2)
        reps = [(n, W.n_a_for(n), L, 1.0, 1)]
        pos = [W.lattice_config(n, L, 7 + k, 0.2) for k in range(2)]
        ss = [md.System(reps, precision="mixed", positions=p, velocities=W.gaussian_velocities(n, 1.0, 2)) for p in pos]
        hist = ss[0]._zeros((1, 3, nb), ss[0].torch.int64)
        ss[0].stream.synchronize()
        for _ in range(200):
            for s in ss:
                s.rdf(3.0 / nb, nb, hist)
        for s in ss:
            s.stream.synchronize()
        ref = sum(O.rdf_hist(*p, reps[0][1], L, 3.0 / nb, nb).astype(np.int64) for p in pos)
        assert np.array_equal(ss[0]._host(hist)[0], 200 * ref)
        for s in ss:
            s.close()


@pytest.mark.parametrize("dr,nb", [(1.4e-10, 5000), (6e-9, 60), (1e-60, 3)])
def test_bins_narrower_than_the_fixed_point_step(dr, nb):
    """Close pairs around the end of a histogram whose bins are narrower than
    the grid of the fixed-point positions (1.4e-9), or a few of its steps, and
    coincident ones: the definition's counts."""
    print(f"case rdf narrow bins dr={dr}", flush=True)
    L, m = 6.2, 8
    k = np.arange(m ** 3)
    site = np.stack([(k % m + 0.3) * L / m, (k // m % m + 0.3) * L / m, (k // (m * m) + 0.3) * L / m])
    rng = np.random.default_rng(4)
    u = rng.normal(size=(3, m ** 3))
    d = nb * dr * rng.uniform(0.97, 1.01, m ** 3) * u / np.sqrt((u * u).sum(0))
    d[:, :20] = 0.0
    pos = tuple(np.ascontiguousarray(np.concatenate([site[c], site[c] + d[c]])) for c in range(3))
    n = 2 * m ** 3
    na = 700
    s = md.System([(n, na, L, 1.0, 1)], precision="fp64", positions=pos, velocities=[np.zeros(n)] * 3)
    h = s._host(s.rdf(dr, nb))[0]
    s.close()
    i, j = np.triu_indices(n, 1)  # (the oracle's bins are 32-bit integers, which these distances exceed)
    dd = [p[i] - p[j] for p in pos]
    dd = [v - L * (v > 0.5 * L) + L * (v < -0.5 * L) for v in dd]
    q = np.sqrt(dd[0] * dd[0] + dd[1] * dd[1] + dd[2] * dd[2]) / dr
    near = q < nb
    kind = (i >= na).astype(int) + (j >= na)
    ref = np.stack([np.bincount(q[near & (kind == t)].astype(int), minlength=nb) * (1 if t == 1 else 2)
                    for t in range(3)])
    assert ref.sum() > 300
    assert np.array_equal(h, ref)

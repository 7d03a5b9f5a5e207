"""The self van Hove histogram of batches of small replicas: counts by the
definition on either side of the rule that picks its kernel (12 wavefronts per
segment in the mean), and the cost of a call where segments are a wavefront or
two."""
import time

import numpy as np
import pytest

from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


def _batch(sizes, species=None):
    reps, pos, vel = [], [[], [], []], [[], [], []]
    for k, n in enumerate(sizes):
        L = max(W.box_for(n, 1.1), 5.2)
        na = W.n_a_for(n) if species is None else {0: 0, 1: n, 2: W.n_a_for(n)}[species[k]]
        reps.append((n, na, L, 1.0, 3 + k))
        for i, a in enumerate(W.lattice_config(n, L, 5 + k, 0.08)):
            pos[i].append(a)
        for i, a in enumerate(W.gaussian_velocities(n, 1.0 + 0.1 * (k % 7), 9 + k)):
            vel[i].append(a)
    return md.System(reps, precision="fp64", positions=[np.concatenate(a) for a in pos],
                     velocities=[np.concatenate(a) for a in vel], msd_slots=2, dt=0.002), reps


@pytest.mark.parametrize("sizes,nb", [
    ([1, 2, 64, 65, 128, 129, 700] * 9, 60),      # small: segments of nothing, a wavefront and more than a block
    ([1, 2, 64, 65, 128, 129, 700] * 9, 1024),
    ([1500] * 3, 200),                            # 72 wavefronts in six segments: the most for that kernel
    ([1500, 1500, 1560], 200),                    # 73
])
def test_counts_by_the_definition(sizes, nb):
    print(f"case van Hove {len(sizes)} replicas, {nb} bins", flush=True)
    rng = np.random.default_rng(5)
    s, reps = _batch(sizes, rng.integers(0, 3, len(sizes)) if len(sizes) > 9 else None)
    a, im = s.numpy(("x", "y", "z")), s.images().astype(np.float64)
    box = np.concatenate([np.full(r[0], r[2]) for r in reps])
    u0 = [a[k] + im[c] * box for c, k in enumerate("xyz")]
    s.msd_set_origin(1)
    s.step_nve(100)
    a, im = s.numpy(("x", "y", "z")), s.images().astype(np.float64)
    d = [a[k] + im[c] * box - u0[c] for c, k in enumerate("xyz")]
    q = np.sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2])
    dr = 0.9 * q.max() / nb
    h = s._host(s.van_hove(1, dr, nb))
    off = 0
    for r, (n, na, *_) in enumerate(reps):
        for t, sl in ((0, slice(off, off + na)), (1, slice(off + na, off + n))):
            b = (q[sl] / dr).astype(np.int64)
            assert np.array_equal(h[r, t], np.bincount(b[b < nb], minlength=nb)), (r, t)
        off += n
    s.close()


def test_a_call_costs_no_more_than_a_mean_square_displacement():
    """4096 replicas of one wavefront per species: a histogram is one launch, a
    mean-square displacement three (one replica after the other, the histogram
    took twice its time)."""
    print("case van Hove time", flush=True)
    s, reps = _batch([70] * 4096)
    s.msd_set_origin(0)
    s.step_nve(3)
    h = s._zeros((len(reps), 2, 60), s.torch.int64)
    o = s._zeros((len(reps), 2), s.torch.float64)

    def us(f):
        best = 1e300
        for _ in range(5):
            s.stream.synchronize()
            t0 = time.perf_counter()
            for _ in range(50):
                f()
            s.stream.synchronize()
            best = min(best, (time.perf_counter() - t0) / 50)
        return 1e6 * best

    vh, msd = us(lambda: s.van_hove(0, 0.001, 60, h)), us(lambda: md.md_msd(s.ctx, 1, 0, o.data_ptr()))
    print(f"  van Hove {vh:.1f} us, MSD {msd:.1f} us", flush=True)
    assert vh <= 1.5 * msd
    s.close()

"""Batches of so many small replicas that the gate decides their rebuilds for
all blocks of the one-block sort (more than 384): the same trajectories as in
smaller batches, where every block decides for itself, and a step's time that
grows no faster than the number of replicas."""
import time

import numpy as np
import pytest

from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


def _run(sizes, temps, steps):
    reps, pos, vel = [], [[], [], []], [[], [], []]
    for n, T in zip(sizes, temps):
        L = max(W.box_for(n, 1.2), 5.2)
        reps.append((n, W.n_a_for(n), L, T, 3))
        for k, a in enumerate(W.lattice_config(n, L, 5 + n, 0.1)):
            pos[k].append(a)
        for k, a in enumerate(W.gaussian_velocities(n, T ** 0.5, 7 + n)):
            vel[k].append(a)
    s = md.System(reps, precision="mixed_fixed", positions=[np.concatenate(a) for a in pos],
                  velocities=[np.concatenate(a) for a in vel], msd_slots=1)
    s.step_nve(steps)
    assert s.status() == 0
    out, rebuilds = s.numpy(), md.md_stats(s.ctx)["rebuilds"]
    s.close()
    return out, rebuilds


@pytest.mark.parametrize("last", [100, 3200])  # the state moved by the sorting block, and by a kernel of its own
def test_gated_sort_equals_smaller_batches(last):
    print(f"case many replicas, largest {last}", flush=True)
    sizes = [70 + 3 * (k % 9) for k in range(399)] + [last]
    temps = [0.4 + 0.005 * k for k in range(400)]
    whole, rebuilds = _run(sizes, temps, 60)
    assert rebuilds > 2 * len(sizes)
    off = 0
    for a, b in ((0, 200), (200, 400)):
        part, _ = _run(sizes[a:b], temps[a:b], 60)
        n = sum(sizes[a:b])
        for k in part:
            assert np.array_equal(whole[k][off:off + n], part[k]), k
        off += n


def _step_us(count):
    n = 100
    L = 5.2
    pos, vel = W.lattice_config(n, L, 5, 0.1), W.gaussian_velocities(n, 0.7, 3)
    s = md.System([(n, W.n_a_for(n), L, 0.5, 3 + r) for r in range(count)], precision="mixed", dt=0.002,
                  positions=[np.tile(a, count) for a in pos], velocities=[np.tile(a, count) for a in vel], msd_slots=1)
    s.step_nve(20)
    s.capture(20)
    s.launch()
    s.stream.synchronize()
    best = 1e300
    for _ in range(5):
        t0 = time.perf_counter()
        for _ in range(3):
            s.launch()
        s.stream.synchronize()
        best = min(best, (time.perf_counter() - t0) / 60)
    assert s.status() == 0
    s.close()
    return 1e6 * best


def test_step_time_grows_no_faster_than_the_batch():
    """Eight times the replicas, at most eight times the time (quadratic work
    per step took thirteen)."""
    print("case many replicas, time", flush=True)
    a, b = _step_us(1024), _step_us(8192)
    print(f"  1024 replicas {a:.1f} us per step, 8192 {b:.1f}", flush=True)
    assert b <= 8.0 * a

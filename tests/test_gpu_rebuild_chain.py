"""The rebuild chain on replicas large enough that each type segment's cells
span several scan chunks (2048 cells each), with replicas that rebuild on
different steps (different temperatures), so that the chunked scan and the
per-particle sort-gather run with some replicas rebuilding and others not.
MIXED_FIXED forces do not depend on the order of the sums, and the replicas
of a batch do not interact, so each replica's trajectory in the batch must
equal, bit for bit, its trajectory run alone; the forces at the end are also
checked against the FP64 oracle (Eq. (KAFix))."""
import math
import sys

import numpy as np
import pytest

import oracle as O
from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu

KEYS = ("x", "y", "z", "vx", "vy", "vz", "ax", "ay", "az")


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# (n, rho, T, seed): at skin 0.3 each type segment has 13^3 = 2197 cells
# (two scan chunks, the second of 149 cells) in the first two replicas and
# 17^3 = 4913 (three chunks) in the third
REPS = [(60000, 1.2, 0.45, 51), (70000, 1.25, 2.0, 52), (150000, 1.2, 1.0, 53)]


def _reps(sel):
    out = []
    for n, rho, T, seed in sel:
        out.append((n, W.n_a_for(n), W.box_for(n, rho), T, seed))
    return out


def _start(sel):
    pos, vel = [[], [], []], [[], [], []]
    for n, rho, T, seed in sel:
        L = W.box_for(n, rho)
        for k, a in enumerate(W.lattice_config(n, L, seed, 0.1)):
            pos[k].append(a)
        for k, a in enumerate(W.gaussian_velocities(n, math.sqrt(T), seed + 7)):
            vel[k].append(a)
    return [np.concatenate(p) for p in pos], [np.concatenate(v) for v in vel]


def _run(sel, steps):
    pos, vel = _start(sel)
    s = md.System(_reps(sel), precision="mixed_fixed", positions=pos, velocities=vel, skin=0.3, auto_sync=False)
    s.step_nve(steps)
    s.sync()
    out = s.numpy(KEYS)
    img = s.images()
    st = md.md_stats(s.ctx)
    assert s.status() == 0
    s.close()
    return out, img, st


def test_batch_with_multi_chunk_segments_equals_replicas_alone():
    steps = 300
    log(f"case rebuild chain, batch {[r[0] for r in REPS]}, {steps} steps")
    ref, ref_img, st = _run(REPS, steps)
    log(f"  batch rebuilds {st['rebuilds']:.0f} (summed over replicas)")
    off, counts = 0, []
    for r in REPS:
        alone, img, st1 = _run([r], steps)
        counts.append(st1["rebuilds"])
        log(f"  n={r[0]} T={r[2]}: rebuilds alone {st1['rebuilds']:.0f}")
        sl = slice(off, off + r[0])
        for k in KEYS:
            assert np.array_equal(ref[k][sl], alone[k]), (r, k)
        assert np.array_equal(ref_img[:, sl], img), r
        off += r[0]
    # the replicas do not rebuild equally often alone, so some steps rebuilt
    # some replicas and not others; in the batch a replica also rebuilds
    # early, along with one that must, on steps where those that must leave
    # the device mostly idle (at most 4376 wavefronts here, against 4096)
    assert len(set(counts)) > 1
    assert sum(counts) <= st["rebuilds"] <= 1.5 * sum(counts)


def test_forces_after_partial_rebuilds_match_oracle():
    sel = REPS[:2]
    s_pos, s_vel = _start(sel)
    s = md.System(_reps(sel), precision="mixed_fixed", positions=s_pos, velocities=s_vel, skin=0.3,
                  auto_sync=False)
    s.step_nve(200)
    s.forces()
    s.sync()
    a = s.numpy(("x", "y", "z", "ax", "ay", "az"))
    assert s.status() == 0
    off = 0
    for n, rho, T, seed in sel:
        sl = slice(off, off + n)
        L = W.box_for(n, rho)
        fx, fy, fz, _, _ = O.forces(a["x"][sl], a["y"][sl], a["z"][sl], W.n_a_for(n), L, "cell")
        num = sum(np.sum((a[k][sl] - f) ** 2) for k, f in zip(("ax", "ay", "az"), (fx, fy, fz)))
        den = np.sum(fx ** 2 + fy ** 2 + fz ** 2)
        err = math.sqrt(num / den)
        log(f"  n={n}: normwise {err:.3e}")
        assert err <= 1e-5
        off += n
    s.close()


@pytest.mark.parametrize("n,L,skin,dim", [
    (140, 5.3, 0.2, 3),     # one cell per edge
    (330, 6.5, 0.3, 3),     # two cells per edge: every row is whole
    (1000, 9.41, 0.3, 3),   # three: every row wraps
    (4000, 14.94, 1.0, 3),  # lists longer than the image
    (9000, 19.2, 1.6, 3),   # rows of more chunks than masks
    (65300, 37.9, 0.3, 3),  # nearly 2^16 slots
    (1000, 28.82, 0.3, 2),  # planar
])
def test_wide_list_builder_equals_the_narrow_one(n, L, skin, dim):
    """The block-per-wave list builder against the wavefront-per-wave one, which
    the window variant uses: the same entries in the same order, so the same
    MIXED forces bit for bit, and the same list lengths up to the entries
    beyond the list radius that the coarse test lets in."""
    print(f"case wide list n={n} skin={skin} dim={dim}", flush=True)
    if dim == 2:
        pos = W.planar_lattice_config(n, L, 5)
        vel = W.gaussian_velocities(n, 0.5, 3)
        vel = (vel[0], vel[1], np.zeros(n))
    else:
        pos = W.lattice_config(n, L, 5, 0.12)
        vel = W.gaussian_velocities(n, 0.5, 3)
    out = []
    for windows in (0, 1):
        s = md.System([(n, W.n_a_for(n), L, 1.0, 3)], precision="mixed", positions=pos, velocities=vel, skin=skin, dim=dim)
        md.md_set_force_kernel(s.ctx, windows, 256)
        s.build_cells()
        s.forces()
        st = md.md_stats(s.ctx)
        assert s.status() == 0
        s.step_nve(4)
        out.append((s.numpy(), st))
        s.close()
    for k in out[0][0]:
        assert np.array_equal(out[0][0][k], out[1][0][k]), k
    assert out[0][1]["mean_list_len"] == pytest.approx(out[1][1]["mean_list_len"], rel=0.006)


@pytest.mark.parametrize("n,L", [
    (65, 6.5),       # one wavefront per species
    (2990, 13.6),    # 47 wavefronts: sorted and gathered by one block
    (3100, 13.7),    # 50: gathered by the whole device
    (8100, 18.9),    # just under 2^13 slots
    (8250, 19.0),    # just over
    (500, 30.0),     # 10 cells per edge: 8000 sub-cells
    (500, 31.0),     # 11: too many for one block
])
def test_one_block_sort_equals_the_chain(n, L):
    """A replica alone (sorted by one block where it is small enough) and the
    same replica beside a large one (always sorted by the kernel chain): one
    build from the same start gives the same slot order, so the same MIXED
    forces bit for bit, and through a few rebuilds the same MIXED_FIXED
    trajectory."""
    print(f"case one-block sort n={n} L={L}", flush=True)
    big = (9000, W.n_a_for(9000), W.box_for(9000, 1.2), 0.6, 9)
    small = (n, W.n_a_for(n), L, 1.5, 4)
    p0, p1 = W.lattice_config(n, L, 5, 0.1), W.lattice_config(9000, big[2], 6, 0.1)
    v0, v1 = W.gaussian_velocities(n, 1.2, 3), W.gaussian_velocities(9000, 0.7, 4)
    for prec, steps in (("mixed", 0), ("mixed_fixed", 30)):
        out = []
        for reps, pos, vel in (([small], p0, v0), ([small, big], [np.concatenate(q) for q in zip(p0, p1)],
                                                   [np.concatenate(q) for q in zip(v0, v1)])):
            s = md.System(reps, precision=prec, positions=pos, velocities=vel)
            if steps:
                s.step_nve(steps)
                assert md.md_stats(s.ctx)["rebuilds"] >= len(reps) + 1
            assert s.status() == 0
            a = s.numpy()
            out.append({k: a[k][:n] for k in a})
            s.close()
        for k in out[0]:
            assert np.array_equal(out[0][k], out[1][k]), (prec, k)


def test_explicit_build_is_not_repeated_by_the_next_call():
    """md_build_cells builds the lists once; md_forces on the same positions
    uses them, and a step after it rebuilds only once a particle has moved far
    enough."""
    n = 4000
    L = W.box_for(n, 1.2)
    s = md.System([(n, W.n_a_for(n), L, 0.8, 3)], precision="mixed_fixed", positions=W.lattice_config(n, L, 5, 0.1),
                  velocities=W.gaussian_velocities(n, 0.8, 3))
    s.forces()
    a = s.numpy(("ax", "ay", "az"))
    k = md.md_stats(s.ctx)["rebuilds"]
    s.build_cells()
    s.forces()
    s.step_nve(1)
    assert md.md_stats(s.ctx)["rebuilds"] == k + 1
    s.build_cells()
    assert md.md_stats(s.ctx)["rebuilds"] == k + 2
    b = md.System([(n, W.n_a_for(n), L, 0.8, 3)], precision="mixed_fixed", positions=W.lattice_config(n, L, 5, 0.1),
                  velocities=W.gaussian_velocities(n, 0.8, 3))
    b.build_cells()
    b.forces()
    c = b.numpy(("ax", "ay", "az"))
    for q in a:
        assert np.array_equal(a[q], c[q])
    s.close()
    b.close()


@pytest.mark.parametrize("count,n,L,skin,dim", [
    (500, 140, 5.3, 0.2, 3),    # one cell per edge
    (300, 330, 6.5, 0.3, 3),    # two: every row is whole
    (100, 1000, 9.41, 0.3, 3),  # three: every row wraps
    (1, 120000, 46.4, 1.3, 3),  # long rows: several masks per piece, pieces past the window
    (1, 90001, 273.4, 0.3, 2),  # planar, cells as 3-D ones but one layer
    (2, 70000, 38.8, 0.3, 3),   # replicas of more than 2^16 slots
])
def test_mask_list_builder_equals_the_window_builder(count, n, L, skin, dim):
    """Worklists too long for the block-per-wave builder: the mask builder
    against the window variant's, as above."""
    print(f"case mask lists {count} x {n} skin={skin} dim={dim}", flush=True)
    if dim == 2:
        pos, v = W.planar_lattice_config(n, L, 5), W.gaussian_velocities(n, 0.5, 3)
        vel = (v[0], v[1], np.zeros(n))
    else:
        pos, vel = W.lattice_config(n, L, 5, 0.12), W.gaussian_velocities(n, 0.5, 3)
    pos, vel = [np.tile(p, count) for p in pos], [np.tile(p, count) for p in vel]
    out = []
    for windows in (0, 1):
        s = md.System([(n, W.n_a_for(n), L, 1.0, 3)] * count, precision="mixed", positions=pos, velocities=vel,
                      skin=skin, dim=dim)
        md.md_set_force_kernel(s.ctx, windows, 256)
        s.build_cells()
        s.forces()
        st = md.md_stats(s.ctx)
        assert s.status() == 0
        s.step_nve(3)
        out.append((s.numpy(), st))
        s.close()
    for k in out[0][0]:
        assert np.array_equal(out[0][0][k], out[1][0][k]), k
    assert out[0][1]["mean_list_len"] == pytest.approx(out[1][1]["mean_list_len"], rel=0.006)


@pytest.mark.parametrize("n,L,dim", [
    (9000, 19.6, 3),      # the first sizes past the one-block sort
    (50000, 34.7, 3),     # eight scan chunks: each sums the ones before it
    (64000, 37.7, 3),     # nine: their totals come from a kernel of their own
    (140000, 341.0, 2),
])
def test_chain_of_a_single_replica_equals_the_gated_one(n, L, dim):
    """A single replica decides its rebuild in the assignment; beside a copy of
    itself it goes through the gate and its worklist.  The same rebuilds, order
    and lists: MIXED sums, which follow the list order, agree in every bit."""
    print(f"case chain {n} dim={dim}", flush=True)
    if dim == 2:
        pos, v = W.planar_lattice_config(n, L, 5), W.gaussian_velocities(n, 0.5, 3)
        vel = (v[0], v[1], np.zeros(n))
    else:
        pos, vel = W.lattice_config(n, L, 5, 0.12), W.gaussian_velocities(n, 0.5, 3)
    out = []
    for count in (1, 2):
        s = md.System([(n, W.n_a_for(n), L, 1.0, 3)] * count, precision="mixed", skin=0.1, dim=dim, dt=0.004,
                      positions=[np.tile(p, count) for p in pos], velocities=[np.tile(p, count) for p in vel])
        md.md_set_force_kernel(s.ctx, 0, 256)
        s.build_cells()
        s.forces()
        for _ in range(3):
            s.step_nve(8)
        assert s.status() == 0
        assert md.md_stats(s.ctx)["rebuilds"] >= 4 * count
        out.append({k: a[..., s.replica_slice(count - 1)] for k, a in s.numpy().items()})
        s.close()
    for k in out[0]:
        assert np.array_equal(out[0][k], out[1][k]), k


@pytest.mark.parametrize("prec", ["fp64", "mixed", "mixed_fixed"])
def test_mask_list_queues_of_uneven_lanes(prec):
    """A dense block in a dilute gas, long list radius: lanes whose queue of
    masks is full beside lanes that have nothing to write yet, whose lists get
    padding in their middle.  Padding adds zeros wherever it stands, so the
    mixed sums equal the window builder's bit for bit; FP64, which has no
    windows, against the lists of a smaller skin (sums in another order:
    1e-12 of the largest force)."""
    print(f"case uneven lanes {prec}", flush=True)
    side, L = 44.0, 66.0
    dense = np.stack(W.lattice_config(100000, side, 5, 0.12))
    g = np.arange(2.0, L - 2.0, 4.0)
    gas = np.stack(np.meshgrid(g, g, g, indexing="ij")).reshape(3, -1)
    gas = gas[:, (gas > side + 2.0).any(axis=0)]
    pos = np.concatenate([dense, gas], axis=1)
    n = pos.shape[1]
    pos = [np.ascontiguousarray(p) for p in pos[:, np.random.default_rng(3).permutation(n)]]
    vel = W.gaussian_velocities(n, 0.5, 3)
    out = []
    for skin, windows in ((1.3, 0), (0.3, 0) if prec == "fp64" else (1.3, 1)):
        s = md.System([(n, W.n_a_for(n), L, 1.0, 3)], precision=prec, positions=pos, velocities=vel, skin=skin,
                      list_capacity=6.0)
        if prec != "fp64":
            md.md_set_force_kernel(s.ctx, windows, 256)
        s.build_cells()
        s.forces()
        assert s.status() == 0
        out.append((s.numpy(("ax", "ay", "az")), md.md_stats(s.ctx)))
        s.close()
    top = max(np.abs(a).max() for a in out[1][0].values())
    for k in out[0][0]:
        if prec == "fp64":
            assert np.abs(out[0][0][k] - out[1][0][k]).max() <= 1e-12 * top, k
        else:
            assert np.array_equal(out[0][0][k], out[1][0][k]), k
    if prec != "fp64":
        assert out[0][1]["mean_list_len"] == pytest.approx(out[1][1]["mean_list_len"], rel=0.006)

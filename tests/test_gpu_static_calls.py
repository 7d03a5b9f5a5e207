"""md_init_static calls no allocating routine: the HIP runtime's own log of the
calls it makes, in a process that has made no other context before (so that
nothing was allocated for it earlier either)."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest

from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(md.__file__)))

CHILD = """
import sys
import numpy as np
import torch
from paper_2001_07089_amd import md, workload as W
n, stream = 1000, torch.cuda.Stream()
L = W.box_for(n, 1.2)
with torch.cuda.stream(stream):
    t = {k: torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda") for k, a in zip(
        ("x", "y", "z", "vx", "vy", "vz"), W.lattice_config(n, L, 5, 0.08) + W.gaussian_velocities(n, 0.8, 3))}
stream.synchronize()
st = md.State()
for k in t:
    setattr(st, k, t[k].data_ptr())
reps = md.make_replicas([(n, W.n_a_for(n), L, 0.8, 1)])
cfg = md.make_config("fp64", init_mode=md.INIT_GIVEN)
print("MARK-BEGIN", file=sys.stderr, flush=True)
ctx = md.md_init_static(cfg, reps, st, stream.cuda_stream)
print("MARK-END", file=sys.stderr, flush=True)
md.md_step_nve(ctx, 5)
assert md.md_status(ctx) == 0
md.md_destroy(ctx)
"""


def test_md_init_static_calls_no_allocating_routine():
    print("case calls of md_init_static", flush=True)
    env = dict(os.environ, AMD_LOG_LEVEL="3", AMD_LOG_MASK="1")
    r = subprocess.run([sys.executable, "-c", CHILD], capture_output=True, text=True, timeout=100, env=env, cwd=ROOT)
    assert r.returncode == 0, r.stderr[-2000:]
    log = r.stderr
    calls = re.findall(r"\b(hip[A-Z]\w+)\s*\(", log[log.index("MARK-BEGIN"):log.index("MARK-END")])
    assert "hipStreamSynchronize" in calls, "the runtime logged no calls"
    bad = sorted({c for c in calls if re.search(r"Malloc|HostAlloc|HostRegister|MemAlloc|MemPoolCreate|Array.*Create", c)})
    assert not bad, bad


def test_more_contexts_than_pinned_words():
    """64 contexts share one page of pinned words; the others do without.  All
    step alike, and the words that are given back serve later contexts."""
    print("case 70 contexts", flush=True)
    n = 100
    L = 5.5
    pos, vel = W.lattice_config(n, L, 5, 0.08), W.gaussian_velocities(n, 0.8, 3)
    for _ in range(2):
        all_ = [md.System([(n, W.n_a_for(n), L, 0.8, 1)], precision="fp64", positions=pos, velocities=vel, msd_slots=1)
                for _ in range(70)]
        for s in all_:
            s.step_nve(3)
            assert s.status() == 0
        ref = all_[0].numpy()
        for s in all_[1:]:
            a = s.numpy()
            assert all(np.array_equal(a[k], ref[k]) for k in ref)
        for s in all_:
            s.close()

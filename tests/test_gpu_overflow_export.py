"""A step call that fails because a list outgrew the caller's workspace leaves
the caller's arrays as they were and the state that of its start: repeated in a
larger workspace, it gives what a context with room for the list gives."""
import numpy as np
import pytest

from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


def _make(n, capacity):
    """A dilute lattice on its way to the centre of the box: over 300 steps it
    becomes more than twice as dense."""
    L = W.box_for(n, 0.3)
    pos = W.lattice_config(n, L, 5, 0.02)
    vel = [-0.16 * (p - 0.5 * L) for p in pos]
    return md.System([(n, W.n_a_for(n), L, 1.0, 3)], precision="mixed_fixed", positions=pos, velocities=vel,
                     list_capacity=capacity, msd_slots=1)


# exported in one pass and in two; rows that the start's lists just fit in
@pytest.mark.parametrize("n,capacity", [(4000, 0.01), (97000, 0.4)])
def test_a_refused_call_leaves_the_callers_arrays_alone(n, capacity):
    print(f"case overflow export n={n}", flush=True)
    s = _make(n, capacity)
    s.close()  # its workspace has room for longer lists; one that has not:
    need = md.md_workspace_size(s.cfg, s.reps)
    ws = s._zeros((need,), s.torch.uint8)
    s.stream.synchronize()
    s.ctx = md.md_init(s.cfg, s.reps, s.state, s.stream.cuda_stream, ws.data_ptr(), need)
    ref = _make(n, 3.0)
    # what the caller keeps in its arrays between calls is the caller's
    mark = s.torch.arange(n, dtype=s.torch.float64, device="cuda")
    with s.torch.cuda.stream(s.stream):
        for k in s.t:
            s.t[k].copy_(mark)
        s.img.fill_(7)
    with pytest.raises(md.KamdError) as e:
        md.md_step_nve(s.ctx, 300)
    assert e.value.code == md.KAMD_ENOMEM
    s.stream.synchronize()
    for k in s.t:
        assert s.torch.equal(s.t[k], mark), k
    assert bool((s.img == 7).all())
    for _ in range(3):  # in a workspace as large as the last refusal asked for
        try:
            s.step_nve(300)
            break
        except md.KamdError as e:
            assert e.code == md.KAMD_ENOMEM
    ref.step_nve(300)
    a, b = s.numpy(), ref.numpy()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    assert np.array_equal(s.images(), ref.images())
    assert ref.status() == 0  # (in s, bits that the abandoned attempts set stay set)
    s.close()
    ref.close()
    del ws

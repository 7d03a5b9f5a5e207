"""Lists of an uneven system take no more room with one builder than with
another: a captured graph cannot grow its lists, so it must not depend on how
many wavefronts rebuild at once."""
import numpy as np
import pytest

from paper_2001_07089_amd import md
from paper_2001_07089_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rot", [0, 1, 2])
def test_walked_entries_do_not_depend_on_the_builder(rot):
    """A dense block in a dilute gas, long list radius.  Alone (a worklist for
    the block-per-wave builder) and three times in a batch (one for the mask
    builder): the same wavefronts, so the same entries walked and the same rows
    needed.  The block lies at different places, for wavefronts across its
    faces in every direction of the walk."""
    print(f"case uneven lists {rot}", flush=True)
    side, L = 30.0, 48.0
    dense = np.stack(W.lattice_config(32000, side, 5, 0.12))
    g = np.arange(2.0, L - 2.0, 4.0)
    gas = np.stack(np.meshgrid(g, g, g, indexing="ij")).reshape(3, -1)
    gas = gas[:, (gas > side + 2.0).any(axis=0)]
    pos = np.concatenate([dense, gas], axis=1)
    pos = np.roll(np.mod(pos + 7.3 * rot, L), rot, axis=0)
    n = pos.shape[1]
    pos = [np.ascontiguousarray(p) for p in pos[:, np.random.default_rng(3).permutation(n)]]
    vel = W.gaussian_velocities(n, 0.5, 3)
    st = []
    for count in (1, 3):
        s = md.System([(n, W.n_a_for(n), L, 1.0, 3)] * count, precision="mixed", skin=1.3, list_capacity=8.0,
                      positions=[np.tile(p, count) for p in pos], velocities=[np.tile(p, count) for p in vel])
        s.build_cells()
        assert s.status() == 0
        st.append(md.md_stats(s.ctx))
        s.close()
    print(st[0]["mean_walked"], st[1]["mean_walked"], flush=True)
    assert st[0]["mean_list_len"] == st[1]["mean_list_len"]
    assert st[0]["mean_walked"] == st[1]["mean_walked"]

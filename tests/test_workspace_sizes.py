"""Workspace sizes of systems of a few particles (host call, no GPU)."""
import pytest

from paper_2001_07089_amd import md


@pytest.mark.parametrize("prec,rep,kw,count,limit", [
    ("mixed", (8, 6, 6.5, 1.0, 0), dict(cell_div=2), 1, 71424),
    ("fp64", (2, 1, 5.01, 1.0, 0), {}, 1, 71424),
    ("fp64", (1, 1, 9.0, 1.0, 0), dict(dim=2), 1, 41472),
    ("mixed", (8, 6, 6.5, 1.0, 0), dict(cell_div=2), 300, 19367680),
])
def test_tiny_workspaces_fit_the_sizes_they_had(prec, rep, kw, count, limit):
    """Callers may hold blocks of the sizes that md_workspace_size gave before
    eager calls kept their starting state in slot order."""
    assert md.md_workspace_size(md.make_config(prec, **kw), md.make_replicas([rep] * count)) <= limit

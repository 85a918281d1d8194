"""Workspaces that sufficed for a call go on sufficing: a program may have allocated one and kept it."""
import pytest

from paper_2311_10359_amd import binding


@pytest.mark.parametrize("records,tasks,most", [(0, 1, 2816), (32, 1, 5120), (1000, 4, 60416), (1024, 4, 60672), (10**6, 10, 56843776),
                                                (1 << 20, 64, 60416512)])
def test_profile_workspace_does_not_grow(records, tasks, most):
    assert 0 < binding.fikit_profile_workspace_bytes(records, tasks) <= most

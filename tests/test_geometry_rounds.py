"""CPU check of the scans' chunk counts in launches of many rounds (compiled
host-only from the library's own header)."""
import pytest

from test_geometry import test_launch_plans as launch_plans


@pytest.mark.parametrize("name", ["rounds_check"])
def test_many_rounds(tmp_path, name):
    launch_plans(tmp_path, name)

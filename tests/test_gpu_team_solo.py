"""Teams whose workgroups own every particle (up to 1024), which take the
smallest steps without an exchange: bitwise the separate calls' results, at the
edges of the slice counts and in each kernel variant.
"""
import pytest

from tests import test_gpu_team

pytestmark = pytest.mark.gpu

CASES = [(256, 0.0, 1, False), (512, 1e-4, 0, True), (513, 1e-4, 1, False), (768, 1e-4, 1, True),
         (769, 1e-4, 0, False), (1024, 0.0, 0, False), (1024, 1e-4, 0, True)]


@pytest.mark.parametrize("n,eps,flags,central", CASES)
def test_teams_of_whole_owners(n, eps, flags, central):
    test_gpu_team.test_team_steps_equal_separate_calls_bitwise(n, eps, flags, central)

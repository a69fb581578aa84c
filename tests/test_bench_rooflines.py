"""bench.py prices launches by what they hold: the check classes of an update may run
in one launch or in one each, a decode may change from one to the other, or run in
one launch altogether."""
import pytest

import bench
import paper_1711_01783_amd as met
from met_inputs import PROFILES

BYTES = {"k_check<3,1>": 900.0, "k_check<12,0>": 60.0, "k_check<2,1>": 40.0}


@pytest.mark.parametrize("kt,want", [
    ({"k_check<3,1>": (10, 5.0), "k_check<12,0>": (10, 1.0), "k_variable": (10, 2.0)}, ("k_check<3,1>", 900.0, 10, 5.0)),
    ({"k_check_set": (10, 6.0), "k_variable": (10, 2.0)}, ("k_check_set", 1000.0, 10, 6.0)),
    ({"k_check_set": (4, 2.0), "k_check<3,1>": (6, 3.0), "k_check<12,0>": (6, 0.5), "k_variable": (10, 2.0)},
     ("k_check<12,0>+k_check<3,1>+k_check_set", 1000.0, 16, 5.5)),
    ({"k_team": (1, 4.0), "k_test": (1, 9.0)}, ("k_team", 1500.0, 1, 4.0)),
    ({"k_team": (1, 4.0), "k_check_set": (5, 3.0), "k_variable": (5, 1.0)}, ("k_check_set+k_team+k_variable", 1500.0, 11, 8.0)),
    ({}, ("k_check<3,1>", 900.0, 0, 0.0))])
def test_check_launches(kt, want):
    assert bench.check_launches(kt, "k_check<3,1>", BYTES, 500.0) == want


def test_weighted_iterations_do_not_depend_on_merging():
    code = met.Code.build(PROFILES["r0.1"], 65536, 3)
    n = len(code.classes())
    assert n > 1
    apart = bench.wbp_rooflines(code, 32, {"k_check_weighted": (50 * n, 3.0), "k_variable": (50, 1.0)})
    merged = bench.wbp_rooflines(code, 32, {"k_check_weighted": (50, 3.0), "k_variable": (50, 1.0)})
    assert merged == apart
    assert merged["k_check_weighted"]["avg_launch_us"] == 60.0

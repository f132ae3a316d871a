"""Host check of which grids take their steps in pairs (no GPU), against gains
measured on the GPU."""
import pytest

from tests.test_report_rows_cpu import run


@pytest.mark.timeout(300)
def test_pairs_are_taken_where_they_are_faster():
    run("pair_rule_check.cpp")

"""Host check of the two-step kernel's addressing on the tile shapes that the
library launches (no GPU): 8 rows in FP32 with 34 and 54 populations, 5 rows in
FP64 with 34 and 25 (tests/twostep_shapes_check.cpp)."""
import pytest

from tests.test_report_rows_cpu import run


@pytest.mark.timeout(600)
def test_addressing_of_the_shipped_tiles():
    run("twostep_shapes_check.cpp")

"""Host check of the blocks that the row-tiled kernels take (no GPU)."""
import pytest

from tests.test_report_rows_cpu import run


@pytest.mark.timeout(300)
def test_blocks_of_row_tiles():
    run("tile_rule_check.cpp")

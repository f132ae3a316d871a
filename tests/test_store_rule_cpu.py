"""Host check of the rule by which a step's stores pass the caches (no GPU)."""
import pytest

from tests.test_report_rows_cpu import run


@pytest.mark.timeout(300)
def test_store_rule():
    run("store_rule_check.cpp")

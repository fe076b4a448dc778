"""The choice of the backward pass's groups (tests/sanitize/groups_driver.cpp), under AddressSanitizer and UndefinedBehaviorSanitizer, no GPU."""
import os

import pytest

from test_sanitizers import HIPCC, _run_driver


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_groups_of_the_backward_pass(tmp_path):
    _run_driver(tmp_path, "groups_driver")

"""The bench line's zone figures: the counters' key holds every source the measured kernel is made of.
No GPU."""
import os
import re

import pytest

from conftest import ROOT

import bench

CSRC = os.path.join(ROOT, "paper_1009_0457_amd", "csrc")


@pytest.mark.parametrize("sources", [bench.ZONE_H2_SOURCES, bench.STEP_SOURCES])
def test_counter_keys_hold_the_headers_of_their_kernels(sources):
    for name in sources:
        included = re.findall(r'#include "(hmc_\w+\.h)"', open(os.path.join(CSRC, name)).read())
        assert set(included) - {"hmc_internal.h"} <= set(sources), name   # the internal header holds declarations

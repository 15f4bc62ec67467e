"""The bench line's zone figures: the counters' key holds every source the measured kernel is made of, and a solve is
priced at heavy-ball steps only where the library takes those.  No GPU."""
import os
import re

import pytest

from conftest import ROOT

H = pytest.importorskip("paper_1009_0457_amd.hmc")
import bench  # noqa: E402

CSRC = os.path.join(ROOT, "paper_1009_0457_amd", "csrc")


@pytest.mark.parametrize("sources", [bench.ZONE_H2_SOURCES, bench.STEP_SOURCES])
def test_counter_keys_hold_the_headers_of_their_kernels(sources):
    for name in sources:
        included = re.findall(r'#include "(hmc_\w+\.h)"', open(os.path.join(CSRC, name)).read())
        assert set(included) - {"hmc_internal.h"} <= set(sources), name   # the internal header holds declarations


def test_price_of_a_solve():
    if not os.path.exists(H.LIB_PATH):
        pytest.skip("libhmc.so not built")
    for h, nr, variant, gradients in ((2, 200, 0, True), (2, 148, 0, False), (3, 231, 0, False), (3, 400, 0, True),
                                      (2, 200, 3, False), (2, 200, 4, False), (1, 400, 0, False)):
        p = H.hmc_default_params(128, 26, h)
        p.zone_steps, p.zone_variant = nr, variant
        method = bench.zone_flops_per_solve(h, nr)
        price = bench.zone_price(H.hmc_zone_by_gradients(p), None, method)[0]
        assert price == (None if gradients else method), (h, nr, variant)
        assert bench.zone_price(gradients, 1.0e6, method)[0] == 1.0e6

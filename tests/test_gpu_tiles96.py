"""Staged tiles of 96 columns: every second one starts in the middle of a 64-row group of scales, the last one ends inside
it; remainders of one row and one column. The same checks as for the other routes."""
import os

import pytest

from test_gpu_routes import test_product_is_the_same_on_every_route as check
from test_host_model_tiles96 import CASES

pytestmark = [pytest.mark.gpu, pytest.mark.skipif("MXFP8_HOSTMODEL_LIB" in os.environ, reason="sizes for the hardware")]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join([f"{c[1][1]}x{c[1][2]}"] + [str(v) for v in c[0]]))
def test_product(case):
    check(case)

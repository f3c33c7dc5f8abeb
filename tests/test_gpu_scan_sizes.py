"""The pattern build where the scans go from one launch to two: 4096 elements,
two rounds of a workgroup's loop (row pointers against numpy, exactly)."""
import pytest

import test_gpu_build_sizes as sizes
from test_gpu_build_sizes import gp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [1, 3, 4094, 4095, 4096, 4097, 4098, 6144, 6145])
def test_row_pointers_about_the_line(gp, V):  # noqa: F811
    sizes.test_row_pointers(gp, V)

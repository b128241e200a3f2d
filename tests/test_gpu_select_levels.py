"""The plan's list where its levels are shared out: groups of 64 sequences around a whole number of them, one and four
workgroups, sequences of more tiles than the sorted levels."""
import pytest

import test_gpu_select_routes as routes
from test_gpu_parity import tp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,most", [(2, 200000), (63, 3000), (64, 40000), (65, 40000), (128, 33000), (129, 33500), (192, 70000),
                                    (700, 6000), (1000, 40000)])
def test_levels(tp, B, most):
    routes.test_select_routes(tp, B, most)

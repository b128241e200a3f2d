"""The loss passes' grids of few workgroups: either side of the most they take, of the most sequences whose metadata is asked for at
once, and of the grids whose sums a part of one batch, one or two of the collecting workgroup's reads bring in."""
import numpy as np
import pytest

from test_gpu_parity import all_stages_against_oracle, tp  # noqa: F401

pytestmark = pytest.mark.gpu
FRAME = 1024


@pytest.mark.parametrize("win", [[512 * FRAME], [300 * FRAME, 211 * FRAME, 1023, 1], [512 * FRAME, 1], [1] * 3 + [512 * FRAME - 2],
                                 [9] * 256, [9] * 257, [3000] + [9] * 255, [3000] + [9] * 256, [0] * 200 + [9] * 56, [0] * 200 + [9] * 57,
                                 [500, 300, 100, 0, 700] * 51, [200] * 256, [500, 0, 1600] * 180,
                                 [4 * FRAME - 5] * 256, [4 * FRAME] * 256 + [3], [700 * FRAME, 324 * FRAME], [1025 * FRAME, 2]])
def test_few_workgroups(tp, win):
    rng = np.random.default_rng(sum(win) + len(win))
    all_stages_against_oracle(tp, rng, np.asarray(win, dtype=np.int64), len(win))

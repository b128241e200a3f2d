"""Frames of the loss passes with more sequences than their descriptor knows: as many as the workgroup fetches the metadata
of (256 behind the first two), one less, and more; and batches that end in empty windows, after a last frame that is not full."""
import numpy as np
import pytest

from test_gpu_parity import all_stages_against_oracle, tp  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("win", [[700, 1] + [1] * 2, [1, 1] + [2] * 255 + [600], [1, 1] + [2] * 256 + [600], [1, 1] + [2] * 257,
                                 [5, 0] + [1] * 254 + [0, 0, 3, 0, 900], [3] * 2000, [1] * 1500, [341, 341, 342, 1] * 5,
                                 [1023, 1, 0, 1, 1022, 2, 500, 500, 23],
                                 [700, 0], [700, 1, 0], [700, 0, 0], [1500, 3, 0, 0], [5, 3] + [0] * 300, [700] + [0] * 70,
                                 [2000, 5, 3] + [0] * 300, [1] * 400 + [3000],
                                 [4] * 299, [4] * 298 + [5]])       # ... and either side of the line between both kernels
def test_sequences_per_frame(tp, win):
    rng = np.random.default_rng(sum(win) + len(win))
    all_stages_against_oracle(tp, rng, np.asarray(win, dtype=np.int64), len(win))

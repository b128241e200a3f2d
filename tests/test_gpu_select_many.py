"""The token filter on batches of up to 1024 sequences whose kept tokens are more turns of all workers than the line between both ways
of dealing them out, and just fewer."""
import numpy as np
import pytest

from test_gpu_parity import check_select, tp  # noqa: F401

pytestmark = pytest.mark.gpu
TURN = 511 * 1024 * 4                                               # up to 128 sequences: all workgroups but one


@pytest.mark.parametrize("extra", [-3, 0, 1, 4096 * 300 + 2])
def test_many_turns(tp, extra):
    rng = np.random.default_rng(5)
    B, n = 7, 5 * TURN + extra
    win = np.diff(np.concatenate([[0], np.sort(rng.integers(0, n, size=B - 1)), [n]]))
    ctx = rng.integers(1, 9, size=B)
    cu = np.concatenate([[0], np.cumsum(win + ctx)]).astype(np.int32)
    check_select(tp, dict(cu_seqlens=cu, ctx_len=ctx.astype(np.int32), done=np.ones(B, np.int32), n_tok=int(cu[-1]),
                          input_ids=rng.integers(0, 1000, size=int(cu[-1])).astype(np.int32), tail_drop=0))

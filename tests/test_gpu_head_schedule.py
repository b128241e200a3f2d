"""The LM-head sweeps' schedule where it changes shape: few token tiles cut into
many vocabulary ranges, token tiles left over after whole rounds of workgroups,
and output tiles of the backward products whose contraction is cut into chunks."""
import numpy as np
import pytest

from test_gpu_parity import _bf16_case, assert_within_term_bound, check_logprob_grads, check_logprobs, dev, host, ofast, tp  # noqa: F401
from paper_2506_15050_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,V,H", [(5, 70000, 64),        # one token tile, as many vocabulary ranges as there may be
                                   (1030, 3000, 64),      # 5 token tiles against 12 vocabulary tiles
                                   (16500, 600, 64),      # 65 token tiles, 3 vocabulary tiles: whole rounds and a rest
                                   (33000, 300, 64),      # whole rounds of 2 columns, one token tile left
                                   (66000, 200, 64)])     # one vocabulary tile: rounds of 256 token tiles, 2 left
def test_logprobs_schedule_shapes(tp, M, V, H):
    rng = np.random.default_rng(M + V)
    hidden = synth.f32_to_bf16_bits(rng.normal(size=(999, H)).astype(np.float32))
    w = synth.f32_to_bf16_bits((rng.normal(size=(V, H)) / np.sqrt(H)).astype(np.float32))
    targets = rng.integers(0, V, size=M)
    targets[:3] = 0, V - 1, min(256, V - 1)
    check_logprobs(tp, hidden, w, rng.integers(0, 999, size=M), targets)


@pytest.mark.parametrize("M,V,H", [(300, 20000, 64),      # grad_hidden: 2 output tiles, 313 K steps in chunks
                                   (200, 9001, 320),      # ragged vocabulary and a second, short column of tiles
                                   (4500, 260, 64)])      # grad_w: 2 output tiles over 71 K steps of tokens
def test_logprob_grads_cut_contraction(tp, M, V, H):
    import torch
    hidden, w, rows, targets, g = _bf16_case(M, V, H, seed=M + V)
    dh, dw = check_logprob_grads(tp, hidden, w, rows, targets, g)
    _, lse = ofast.token_logprobs(hidden, w, rows, targets)
    args = (dev(hidden), dev(w), dev(rows.astype(np.int32)), dev(targets.astype(np.int32)),
            dev(lse.astype(np.float32)), dev(g.astype(np.float32)))
    acc = torch.full((V, H), 2.0, device="cuda")           # partial tiles added to what is there
    again, _ = tp.tppo_token_logprobs_backward(*args, grad_w=acc, accumulate_w=True)
    torch.cuda.synchronize()
    assert np.array_equal(host(again), dh)
    # one fp32 rounding of (2 + dw)
    assert np.abs(host(acc) - 2.0 - dw).max() <= 2.0 ** -23 * (2.0 + np.abs(dw).max())
